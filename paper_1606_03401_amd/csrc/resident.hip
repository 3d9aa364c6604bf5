// Resident launches: forward chains and sweeps, whose workgroups keep weights on the chip for many
// time steps (see the comments at each kernel).
#include "resident.h"

namespace mebptt {

// The bound every wait of a resident launch runs under, in ticks of the 100 MHz wall clock.  A
// host-side setting so that a test can make the waits give up at once -- every workgroup then leaves
// through the same path as after a real time-out -- without anything hanging.
constexpr long long RES_WAIT_TICKS = 50000000;   // 0.5 s
static long long g_wait_ticks = RES_WAIT_TICKS;
void set_resident_wait_ticks(long long ticks) { g_wait_ticks = ticks < 0 ? RES_WAIT_TICKS : ticks; }

// ---- which shapes have forward chains -------------------------------------------------------------------
// Sequences per XCD: as few as keep all of them on the chip at once, in whole halves of an MFMA tile, so
// that no group straddles tiles (a step takes the same time for 1 and for 8 sequences, so with B < 64
// fewer XCDs work rather than all of them on less).  Returns 0 for a batch that does not fit.
static int group_share(const Dims& d) { return d.B <= 64 ? 8 : (d.B <= 128 ? 16 : (d.B <= 256 ? 32 : 0)); }

struct ChainConfig {
  int nrt, nxw, nhw, ks, nbt;
  hipError_t (*launch[2])(const ResParams&, hipStream_t);   // by cell
};
#define CHAIN(T, NRT, NXW, NXL, NHW, KS, NBT) \
  {NRT, NXW, NHW, KS, NBT, {launch_chain_cell<T, NRT, NXW, NXL, NHW, KS, NBT, 0>, launch_chain_cell<T, NRT, NXW, NXL, NHW, KS, NBT, 1>}}
static const ChainConfig CHAIN_BF16[] = {
    CHAIN(__bf16, 8, 1, 1, 4, 8, 1),   // H = 1024, I <= 256
    CHAIN(__bf16, 4, 1, 0, 4, 4, 1), CHAIN(__bf16, 4, 1, 0, 4, 4, 2),   // H = 512, I <= 128
    CHAIN(__bf16, 2, 2, 0, 2, 4, 1), CHAIN(__bf16, 2, 2, 0, 2, 4, 2),   // H = 256, I <= 256
    CHAIN(__bf16, 1, 1, 0, 1, 4, 1), CHAIN(__bf16, 1, 1, 0, 1, 4, 2),   // H = 128, I <= 128
};

// The smallest instantiation the shape fits, or NULL.
static const ChainConfig* chain_config(const Dims& d) {
  if (!d.dtype || d.I < 8) return nullptr;
  const int kstep = 32, nsx = d.KX / kstep, nsh = d.KH / kstep, nrt = (d.KH + 127) / 128;
  const FwdConfig fc = forward_config<__bf16>(d);
  const int ks = (fc == FWD_TINY || fc == FWD_SMALLK) ? 4 : 8;   // the K split of the per-step kernels
  const int share = group_share(d), nbt = share > 16 ? 2 : 1;
  if (share == 0) return nullptr;
  for (const ChainConfig& c : CHAIN_BF16)
    if (c.nrt == nrt && c.ks == ks && c.nbt == nbt && c.nhw * ks >= nsh && c.nxw * ks >= nsx) return &c;
  return nullptr;
}

bool can_run_forward_chain(const Dims& d) { return chain_config(d) != nullptr; }
int forward_chain_max_steps() { return RES_MAX_STEPS; }
size_t forward_chain_ring_bytes(const Dims& d) { return (size_t)RES_RING * d.BP * d.KH * d.op_bytes(); }
size_t forward_chain_sync_bytes() { return (RES_SYNC_STATUS + 64) * sizeof(unsigned); }
size_t forward_chain_status_offset() { return RES_SYNC_STATUS * sizeof(unsigned); }
unsigned forward_chain_arrivals(int steps) { return steps > 1 ? (unsigned)(steps - 1) * RES_MEMBERS : 0u; }

hipError_t launch_forward_chain(const Dims& d, const void* Wp, const float* bp, const float* x_first, const float* src_unit,
                                const ChainStep* steps, int count, void* ring, unsigned* sync, unsigned published,
                                unsigned launch, hipStream_t st) {
  const ChainConfig* cfg = chain_config(d);
  if (!cfg || count < 1 || count > RES_MAX_STEPS) return hipErrorInvalidValue;
  ResParams p{};
  p.Wp = Wp;
  p.bp = bp;
  p.x0 = x_first;
  p.src = src_unit;
  p.ring = ring;
  p.sync = sync;
  p.published = published;
  p.launch = launch;
  p.wait_ticks = g_wait_ticks;
  p.count = count;
  p.B = d.B;
  p.I = d.I;
  p.H = d.H;
  p.HP = d.HP;
  p.KX = d.KX;
  p.KH = d.KH;
  p.BP = d.BP;
  p.nb = group_share(d);
  p.unit = d.unit;
  p.hplane = d.hplane;
  for (int j = 0; j < count; ++j) p.step[j] = ResStep{steps[j].out, steps[j].gates};
  return cfg->launch[d.cell](p, st);
}

// ---- backward sweep with resident weights ------------------------------------------------------
// Where a sub-sequence fits into memory the schedule alternates "forward operation of step s from
// the memorised h_{s-1}, keeping the internal state" and "backward operation of step s", s going
// down.  On shapes whose gate weights AND their transpose fit on the chip such a run of pairs goes
// out as one launch per chunk of steps, organised like the forward chain (batch split over the
// XCDs, hidden units over the 32 compute units of an XCD, weights in registers):
//   * the forward operation of a step needs nothing from other compute units (its input state was
//     memorised by an earlier launch), and its internal state never leaves the registers of the
//     thread that owns the (sequence, unit);
//   * the backward operation needs dG of the step after, all 4H columns of it, for the XCD's
//     sequences: the compute units publish their columns in the chunk's dG staging buffer (which
//     is already laid out as that GEMM's operand) and meet at the XCD's arrival counter;
//   * while the counter fills, every compute unit already runs the forward operation of the next
//     lower step, so the wait is mostly hidden.
// K splits and summation orders are those of forward_body and backward_body for the shape, the
// pointwise steps are the shared functions: bit-identical to the launch-per-step path.
static int group_tiles(const Dims& d, int nb) {
  int nbt = 1;
  for (int g = 0; g < RES_GROUPS; ++g) {
    const int lo = g * nb, hi = (lo + nb < d.B ? lo + nb : d.B);
    if (lo >= d.B) break;
    const int span = (hi - 1) / 16 - lo / 16 + 1;
    nbt = span > nbt ? span : nbt;
  }
  return nbt;
}
static int group_share(const Dims& d, int candidate) {
  const int even = (d.B + RES_GROUPS - 1) / RES_GROUPS;
  return candidate == 0 ? even : round_up(even, 16);
}
__device__ inline bf16x8 load_frag_l2(const void* base, unsigned byte_off) { return as_frag<bf16x8>(load_slot_16(base, byte_off, 0)); }

constexpr int SWEEP_MAX_STEPS = 32;
struct SweepParams {
  const void* Wp;
  const void* WTh;
  const float* bp;
  const float* x;        // x of step 1 (step s reads x + (s-1)*B*I)
  const float* dy;       // upstream gradients, first plane = step dy_first; NULL with dy_is_h
  int dy_first, dy_is_h;
  float* dc;             // running cell-state gradient plane
  float* y_out;          // outputs, plane of step 1 first, or NULL
  const void* dG_next;   // dG block of step s_hi + 1, or NULL when s_hi is the last step of the sequence
  void* dG_chunk[2];     // the two chunk buffers: step s lives in buffer ((s-1) / CH) & 1, its block at slot (s-1) % CH
  void* dGT[2];
  void* aT[2];
  unsigned* sync;
  unsigned base, launch;
  long long wait_ticks;  // bound of every wait, in ticks of the 100 MHz wall clock
  int s_hi, count;       // steps s_hi, s_hi - 1, ..., s_hi - count + 1 (in at most two consecutive chunks)
  int B, I, H, KX, KH, BP, nb, G4, NX, KC, CH;
  size_t unit;
  const float* src[SWEEP_MAX_STEPS];   // src[j]: unit holding the state before step s_hi - j
  const float* state[SWEEP_MAX_STEPS]; // FWD = false: unit holding the stored internal state of step s_hi - j
};

// FWD = false: the internal states are not recomputed but read from where an earlier launch
// stored them (internal-state slots): a run of backward operations only, W_hh^T alone resident.
template <bool FWD, int NRT, int NSWF, int KSF, int NSWB, int KSB, int NBT, int NSXW, int CELL = 0>
__global__ __launch_bounds__(512) void sweep_kernel(SweepParams p) {
  static_assert(!(FWD && CELL), "the launches that recompute internal states are built for the LSTM only");
  using T = __bf16;
  using M = Mma<T>;
  constexpr int VEC = 8, KSTEP = 32;
  constexpr int FT = 8 / KSF;                       // groups of waves that split the forward row tiles
  constexpr int NRTW = (NRT + FT - 1) / FT;         // forward row tiles per wave
  constexpr int UW = NRT * 4;                       // hidden units per workgroup
  constexpr int NTB = (UW + 15) / 16;               // 16-unit tiles of the dh GEMM that cover them
  constexpr int NTF = NRT * NBT, NTBT = NTB * NBT;
  constexpr int ITEMS = NRT * NBT * 64, IPT = (ITEMS + 511) / 512;
  constexpr int nstepsF = KSF * NSWF, nstepsB = KSB * NSWB;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* redF = reinterpret_cast<float*>(smem);                       // [KSF][NTF][4][64]
  float* redB = redF + (size_t)KSF * NTF * 4 * 64;                    // [KSB][NTBT][4][64]
  __shared__ int s_go, s_g, s_rank;
  // the wave index as a scalar: conditions on it become scalar branches (an MFMA under a lane mask
  // that is empty would still execute)
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int lrow = lane & 15, lq = lane >> 4;
  if (threadIdx.x == 0) {
    const unsigned xcc = xcc_id();
    int ok = xcc < (unsigned)RES_GROUPS;
    unsigned ticket = 0;
    if (ok) {
      ticket = __hip_atomic_fetch_add(p.sync + 512 + xcc * 64, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = ticket / RES_MEMBERS == p.launch;
    }
    if (!ok) __hip_atomic_store(p.sync + 1024, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_go = ok;
    s_g = ok ? (int)xcc : 0;
    s_rank = (int)(ticket % RES_MEMBERS);
  }
  __syncthreads();
  if (!s_go) return;
  const int g = s_g, rank = s_rank;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP;
  const size_t hhalf = (size_t)p.BP * p.KH, plane = (size_t)p.B * p.H;
  const int b_lo = g * p.nb, b_hi = min(p.B, b_lo + p.nb);
  const int nbt_all = p.BP / 16;
  const int ct0 = min(b_lo / 16, nbt_all - 1);
  unsigned* ctr = p.sync + g * 64;
  unsigned* status = p.sync + 1024;
  const int fk = wave % KSF, fg = wave / KSF;       // forward: K part and row-tile group of this wave
  const bool bwd_wave = wave < KSB;
  const int nt0 = (rank * UW) / 16;                 // first 16-unit tile of the dh GEMM

  // resident weights: forward rows of this workgroup's units, and the rows of W_hh^T for the same units
  typename M::Frag wf[FWD ? NRTW : 1][FWD ? NSWF : 1], wb[NTB][NSWB];
  if (FWD) {
#pragma unroll
    for (int i = 0; i < NRTW; ++i) {
      const int rt = min(fg * NRTW + i, NRT - 1);
#pragma unroll
      for (int k = 0; k < NSWF; ++k)
        wf[FWD ? i : 0][FWD ? k : 0] = M::load(reinterpret_cast<const T*>(p.Wp) +
                                               (((size_t)(rank * NRT + rt) * nstepsF + fk + KSF * k) * 64 + lane) * VEC);
    }
  }
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
    for (int k = 0; k < NSWB; ++k)
      wb[tb][k] = M::load(reinterpret_cast<const T*>(p.WTh) +
                          (((size_t)(nt0 + tb) * nstepsB + min(wave, KSB - 1) + KSB * k) * 64 + lane) * VEC);

  // items: (output tile, lane of the forward MFMA layout) = (sequence, unit)
  bool mine[IPT];
  int ib[IPT], iu[IPT], icellF[IPT], icellB[IPT];
  float4 bias[IPT];
  float dc_run[IPT];
  // internal state of the step whose backward operation comes next, and its input state
  float st_gate[IPT][4], st_c[IPT], st_h[IPT], st_cprev[IPT], st_hprev[IPT];
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const int item = (int)threadIdx.x + q * 512;
    const int tile = item >> 6, il = item & 63;
    const int rt = tile / NBT, bt = tile % NBT;
    const int b = (ct0 + bt) * 16 + (il & 15), u = rank * UW + rt * 4 + (il >> 4);
    mine[q] = item < ITEMS && b >= b_lo && b < b_hi;
    ib[q] = b;
    iu[q] = u;
    icellF[q] = tile * 4 * 64 + il;
    // dh of unit u: row u % 16 of tile u / 16 of the dh GEMM, i.e. lane (u%16/4)*16 + b%16, register u%4
    icellB[q] = (((u / 16 - nt0) * NBT + bt) * 4 + (u & 3)) * 64 + ((u & 15) >> 2) * 16 + (il & 15);
    bias[q] = float4{0.f, 0.f, 0.f, 0.f};
    dc_run[q] = 0.0f;
    if (mine[q]) {
      bias[q] = *reinterpret_cast<const float4*>(p.bp + 4 * u);
      dc_run[q] = p.dc[(size_t)b * p.H + u];
    }
  }
  // operands of a forward operation, requested a step ahead: raw x values, h fragments, c_{s-1}, h_{s-1}
  RawAct<VEC> xraw[FWD ? NSXW : 1][NBT];
  typename M::Frag hfr[FWD ? NSWF : 1][NBT];
  float pf_cprev[IPT], pf_hprev[IPT];
  float pf_gate[FWD ? 1 : IPT][4], pf_c[FWD ? 1 : IPT], pf_h[FWD ? 1 : IPT];   // FWD = false: the stored state, a step ahead
  const bool want_h = p.dy_is_h || p.y_out != nullptr;
  auto fetch_fwd = [&](int j) {
    if (!FWD) {
      const float* stp = p.state[j];
      const float* src = p.src[j];
#pragma unroll
      for (int q = 0; q < IPT; ++q) {
        pf_cprev[q] = pf_hprev[q] = 0.0f;
        pf_c[FWD ? 0 : q] = pf_h[FWD ? 0 : q] = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) pf_gate[FWD ? 0 : q][r] = 0.0f;
        if (mine[q]) {
          const size_t e = (size_t)ib[q] * p.H + iu[q];
          pf_gate[FWD ? 0 : q][0] = stp[p.unit + e];
          pf_gate[FWD ? 0 : q][1] = stp[p.unit + plane + e];
          pf_gate[FWD ? 0 : q][2] = stp[2 * p.unit + e];
          if (CELL == 0) pf_gate[FWD ? 0 : q][3] = stp[2 * p.unit + plane + e];   // the GRU has three gates
          pf_c[FWD ? 0 : q] = stp[hhalf + e];                                     // c_s, or the GRU's n_h
          if (want_h) pf_h[FWD ? 0 : q] = HPlane<T>::load(stp, ib[q], iu[q], nsh, p.H, hhalf);
          // what the pointwise step blends with: c_{s-1}, or the GRU's h_{s-1} in full precision
          pf_cprev[q] = CELL ? HPlane<T>::load(src, ib[q], iu[q], nsh, p.H, hhalf) : src[hhalf + e];
          pf_hprev[q] = (float)HPlane<T>::as_operand(src, ib[q], iu[q], nsh, p.H, hhalf);
        }
      }
      return;
    }
    const int s = p.s_hi - j;
    const float* x_s = p.x + (size_t)(s - 1) * p.B * p.I;
    const float* src = p.src[j];
#pragma unroll
    for (int k = 0; k < NSWF; ++k) {
      const int ms = fk + KSF * k;
#pragma unroll
      for (int bt = 0; bt < NBT; ++bt) {
        const int tile = min(ct0 + bt, nbt_all - 1);
        if (ms < nsx) {
          if (k < NSXW) xraw[(FWD && k < NSXW) ? k : 0][bt] = load_raw_whole<VEC>(x_s + (size_t)min(tile * 16 + lrow, p.B - 1) * p.I,
                                                                                  ms * KSTEP + VEC * lq, p.I);
        } else {
          hfr[FWD ? k : 0][bt] = M::load(reinterpret_cast<const T*>(src) + (((size_t)tile * nsh + (ms - nsx)) * 64 + lane) * VEC);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      pf_cprev[q] = pf_hprev[q] = 0.0f;
      if (mine[q]) {
        pf_cprev[q] = src[hhalf + (size_t)ib[q] * p.H + iu[q]];
        pf_hprev[q] = (float)HPlane<T>::as_operand(src, ib[q], iu[q], nsh, p.H, hhalf);
      }
    }
  };
  // The forward operation of step s_hi - j comes in two parts, so that the memory operations
  // between them overlap with neither's waits.  (Loads and stores share one in-order counter: once
  // both kinds are in flight, a wait for any load is a wait for everything, store acknowledgements
  // included.)  Part one runs right after an arrival, when nothing is outstanding: the GEMM slice
  // from the fetched operands, then the request for the operands of the step after.  Part two, after
  // the stores that only later launches read have been issued, reduces the slices and applies the
  // gate functions; it leaves the internal state in st_*.
  auto forward_gemm = [&](int j) {
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      st_cprev[q] = pf_cprev[q];
      st_hprev[q] = pf_hprev[q];
      if (!FWD) {   // nothing to compute: the fetched state becomes the current one
#pragma unroll
        for (int r = 0; r < 4; ++r) st_gate[q][r] = pf_gate[FWD ? 0 : q][r];
        st_c[q] = pf_c[FWD ? 0 : q];
        st_h[q] = pf_h[FWD ? 0 : q];
      }
    }
    if (FWD) {
      f32x4 acc[NRTW][NBT];
#pragma unroll
      for (int i = 0; i < NRTW; ++i)
#pragma unroll
        for (int bt = 0; bt < NBT; ++bt) acc[i][bt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < NSWF; ++k) {
        const int ms = fk + KSF * k;
#pragma unroll
        for (int bt = 0; bt < NBT; ++bt) {
          const typename M::Frag bfr = (k < NSXW && ms < nsx) ? M::from_f32(xraw[(FWD && k < NSXW) ? k : 0][bt].v) : hfr[FWD ? k : 0][bt];
#pragma unroll
          for (int i = 0; i < NRTW; ++i) acc[i][bt] = M::mma(wf[FWD ? i : 0][FWD ? k : 0], bfr, acc[i][bt]);
        }
      }
#pragma unroll
      for (int i = 0; i < NRTW; ++i) {
        const int rt = fg * NRTW + i;
        if (rt < NRT) {
#pragma unroll
          for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
            for (int r = 0; r < 4; ++r) redF[((fk * NTF + rt * NBT + bt) * 4 + r) * 64 + lane] = acc[i][bt][r];
        }
      }
    }
    if (j + 1 < p.count) fetch_fwd(j + 1);
  };
  auto forward_point = [&]() {
    if (!FWD) return;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      float G[4] = {0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < KSF; ++w)   // fixed order, as in forward_body
#pragma unroll
        for (int r = 0; r < 4; ++r) G[r] += redF[w * NTF * 4 * 64 + icellF[q] + r * 64];
      float second;
      st_h[q] = cell_forward<0>(G, bias[q], st_cprev[q], second, st_gate[q]);
      st_c[q] = second;
    }
  };

  fetch_fwd(0);
  forward_gemm(0);   // also requests the operands of the step after
  forward_point();

  for (int j = 0; j < p.count; ++j) {
    const int s = p.s_hi - j;                       // the step back-propagated now
    const int slot = (s - 1) % p.CH, buf = ((s - 1) / p.CH) & 1;   // where step s lives in the chunk buffers
    const size_t dG_step = (size_t)p.BP * p.G4;     // elements of one step's dG block
    const T* dG_next = (j == 0) ? reinterpret_cast<const T*>(p.dG_next)   // step s + 1: maybe in the other buffer
                                : reinterpret_cast<const T*>(p.dG_chunk[(s / p.CH) & 1]) + (size_t)(s % p.CH) * dG_step;
    if (j > 0) {
      // all 32 workgroups of this XCD have published their columns of dG of step s + 1?
      if (threadIdx.x == 0) {
        const unsigned target = p.base + (unsigned)j * RES_MEMBERS;
        int ok = 1, polls = 0;
        long long t0 = 0;
        while ((int)(__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
          if (p.wait_ticks == 0 || (++polls & 15) == 0) {   // a bound of 0: one look only
            const long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (now - t0 >= p.wait_ticks ||
                __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
              __hip_atomic_store(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              ok = 0;
              break;
            }
          }
        }
        s_go = ok;
      }
      __syncthreads();
      if (!s_go) return;
    }
    // dh = dG_{s+1} W_hh for this workgroup's units
    if (dG_next != nullptr) {
      if (bwd_wave) {
        f32x4 acc[NTB][NBT];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
          for (int bt = 0; bt < NBT; ++bt) acc[tb][bt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // The dG fragments come in rounds of GK macro steps: all fetches of a round go out before its
        // first MFMA (left to itself the scheduler pairs each fetch with the MFMA that needs it, one
        // L2 round trip after the other).  Two batch tiles beside resident forward weights leave
        // registers for half the fragments at a time only.
        constexpr int GK = (FWD && NBT > 1) ? NSWB / 2 : NSWB;
#pragma unroll
        for (int k0 = 0; k0 < NSWB; k0 += GK) {
          typename M::Frag gfr[GK][NBT];
#pragma unroll
          for (int k = 0; k < GK; ++k)
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) {
              const size_t fo = (((size_t)min(ct0 + bt, nbt_all - 1) * nstepsB + wave + KSB * (k0 + k)) * 64 + lane) * VEC;
              gfr[k][bt] = load_frag_l2(dG_next, (unsigned)(fo * sizeof(T)));
            }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < GK; ++k)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
              for (int bt = 0; bt < NBT; ++bt) acc[tb][bt] = M::mma(wb[tb][k0 + k], gfr[k][bt], acc[tb][bt]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
          for (int bt = 0; bt < NBT; ++bt)
#pragma unroll
            for (int r = 0; r < 4; ++r) redB[((wave * NTBT + tb * NBT + bt) * 4 + r) * 64 + lane] = acc[tb][bt][r];
      }
      __syncthreads();
    }
    // pointwise backward of step s on the internal state held in registers
    const bool publish = j + 1 < p.count;
    T* dG_cur = reinterpret_cast<T*>(p.dG_chunk[buf]) + (size_t)slot * dG_step;
    const int ncs = p.KC / KSTEP, col0 = slot * p.B;
    T gq[IPT][4];
    float keep_h[IPT], keep_hprev[IPT];
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      const int b = ib[q], n = iu[q];
      const size_t e = (size_t)b * p.H + n;
      float dh = 0.0f;
      if (dG_next != nullptr)
        for (int w = 0; w < KSB; ++w) dh += redB[w * NTBT * 4 * 64 + icellB[q]];   // fixed order, as in backward_body
      float dyv = 0.0f;
      if (p.dy_is_h)
        dyv = st_h[q];
      else if (p.dy != nullptr && s >= p.dy_first)
        dyv = p.dy[(size_t)(s - p.dy_first) * plane + e];
      dh += dyv;
      float dG[4], dc_out;
      if (CELL == 0)
        lstm_backward_point(dh, dc_run[q], st_gate[q][0], st_gate[q][1], st_gate[q][2], st_gate[q][3], st_c[q], st_cprev[q],
                            dG, dc_out);
      else   // the running plane carries dh_{s+1} * z_{s+1}, as in backward_body
        gru_backward_point(__fadd_rn(dh, dc_run[q]), st_gate[q][0], st_gate[q][1], st_gate[q][2], st_c[q], st_cprev[q], dG, dc_out);
      dc_run[q] = dc_out;
      // the four gates of a unit are consecutive in dG: one 8-byte store (what other compute units
      // fetch next must not be written in pieces smaller than a dword)
      union { T t[4]; unsigned long long v; } pk;
#pragma unroll
      for (int r = 0; r < 4; ++r) pk.t[r] = gq[q][r] = (T)dG[r];
      *reinterpret_cast<unsigned long long*>(dG_cur + ft_offset<T>(b, 4 * n, nstepsB)) = pk.v;
      keep_h[q] = st_h[q];
      keep_hprev[q] = st_hprev[q];
    }
    if (publish) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's columns of dG have reached the L2
      __syncthreads();
      if (threadIdx.x == 0) __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      forward_gemm(j + 1);
    }
    // What only later launches read -- the transposed copies for the weight gradient, the output --
    // is stored after the arrival: nobody in this launch waits for it.
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      const int b = ib[q], n = iu[q];
      const int col = col0 + b;
      T* dGT = reinterpret_cast<T*>(p.dGT[buf]);
#pragma unroll
      for (int r = 0; r < 4; ++r) dGT[ft_offset<T>(4 * n + r, col, ncs)] = gq[q][r];
      reinterpret_cast<T*>(p.aT[buf])[ft_offset<T>(p.NX + n, col, ncs)] = (T)keep_hprev[q];
      if (p.y_out) p.y_out[(size_t)(s - 1) * plane + (size_t)b * p.H + n] = keep_h[q];
    }
    // the pointwise part of the next lower step's forward operation runs while the others arrive
    if (publish) forward_point();
  }
#pragma unroll
  for (int q = 0; q < IPT; ++q)
    if (mine[q]) p.dc[(size_t)ib[q] * p.H + iu[q]] = dc_run[q];
}

struct SweepConfig {
  int nrt, nswf, ksf, nswb, ksb, nbt, nsxw;
};
static const SweepConfig SWEEP_CONFIGS[] = {
    {4, 5, 4, 8, 8, 1, 1}, {4, 5, 4, 8, 8, 2, 1},   // H = 512, I <= 128
    {2, 4, 4, 4, 8, 1, 2}, {2, 4, 4, 4, 8, 2, 2},   // H = 256, 128 < I <= 256
    {1, 2, 4, 4, 4, 1, 1}, {1, 2, 4, 4, 4, 2, 1},   // H = 128, I <= 128
    {8, 5, 8, 16, 8, 1, 1},                         // H = 1024, any I: backward operations only (W_hh^T fits, both do not)
};
constexpr int SWEEP_BACKWARD_ONLY_FROM = 6;   // configurations from this index on have no forward part

// backward_only: for a launch of backward operations on stored internal states, which never reads x
// or the gate weights -- only the backward part of a configuration has to fit the shape.
static int sweep_config(const Dims& d, int* nb_out = nullptr, bool backward_only = false) {
  if (!d.dtype || d.H % 128 != 0 || d.KH != d.H || d.HP != d.H) return -1;   // either cell; can_run_sweep() narrows
  const int nstepsF = d.KP / 32, nstepsB = d.G4 / 32;
  const FwdConfig fc = forward_config<__bf16>(d);
  const int ksf = (fc == FWD_TINY || fc == FWD_SMALLK) ? 4 : 8;
  const int ksb = backward_config<__bf16>(d) == BWD_SMALLK ? 4 : 8;
  if (nstepsB % ksb != 0) return -1;
  for (int cand = 0; cand < 2; ++cand) {
    const int nb = group_share(d, cand), nbt = group_tiles(d, nb);
    for (size_t i = 0; i < sizeof SWEEP_CONFIGS / sizeof SWEEP_CONFIGS[0]; ++i) {
      const SweepConfig& c = SWEEP_CONFIGS[i];
      if (c.nrt != d.H / 128 || c.ksb != ksb || c.nswb != nstepsB / ksb || c.nbt != nbt) continue;
      // the forward part fixes the width of x as well
      if (backward_only || (int)i >= SWEEP_BACKWARD_ONLY_FROM ||
          (d.I % 8 == 0 && nstepsF % ksf == 0 && c.ksf == ksf && c.nswf == nstepsF / ksf &&
           c.nsxw == (d.KX / 32 + ksf - 1) / ksf)) {
        if (nb_out) *nb_out = nb;
        return (int)i;
      }
    }
  }
  return -1;
}

bool can_run_sweep(const Dims& d) {   // with forward operations: LSTM only
  const int c = sweep_config(d);
  return d.cell == 0 && c >= 0 && c < SWEEP_BACKWARD_ONLY_FROM;
}
bool can_run_backward_sweep(const Dims& d) { return sweep_config(d, nullptr, true) >= 0; }
int sweep_max_steps() { return SWEEP_MAX_STEPS; }

template <bool FWD, int NRT, int NSWF, int KSF, int NSWB, int KSB, int NBT, int NSXW, int CELL = 0>
static hipError_t launch_sweep_cfg(const SweepParams& p, hipStream_t st) {
  constexpr int NTB = (NRT * 4 + 15) / 16;
  const size_t lds = ((size_t)KSF * NRT * NBT + (size_t)KSB * NTB * NBT) * 4 * 64 * sizeof(float);
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(sweep_kernel<FWD, NRT, NSWF, KSF, NSWB, KSB, NBT, NSXW, CELL>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    configured = true;
  }
  sweep_kernel<FWD, NRT, NSWF, KSF, NSWB, KSB, NBT, NSXW, CELL><<<dim3(RES_WGS), dim3(512), lds, st>>>(p);
  return hipGetLastError();
}

hipError_t launch_sweep(const Dims& d, const SweepArgs& a, hipStream_t st) {
  int nb = 0;
  const int cfg = sweep_config(d, &nb, a.state != nullptr);
  if (cfg < 0 || a.count < 1 || a.count > SWEEP_MAX_STEPS) return hipErrorInvalidValue;
  if ((a.s_hi - 1) / d.CH - (a.s_hi - a.count) / d.CH > 1) return hipErrorInvalidValue;   // two chunk buffers
  SweepParams p{};
  p.Wp = a.Wp;
  p.WTh = a.WTh;
  p.bp = a.bp;
  p.x = a.x;
  p.dy = a.dy;
  p.dy_first = a.dy_first;
  p.dy_is_h = a.dy_is_h;
  p.dc = a.dc;
  p.y_out = a.y_out;
  p.dG_next = a.dG_next;
  for (int i = 0; i < 2; ++i) {
    p.dG_chunk[i] = a.dG_chunk[i];
    p.dGT[i] = a.dGT[i];
    p.aT[i] = a.aT[i];
  }
  p.sync = a.sync;
  p.base = a.base;
  p.wait_ticks = g_wait_ticks;
  p.launch = a.launch;
  p.s_hi = a.s_hi;
  p.count = a.count;
  p.B = d.B;
  p.I = d.I;
  p.H = d.H;
  p.KX = d.KX;
  p.KH = d.KH;
  p.BP = d.BP;
  p.nb = nb;
  p.G4 = d.G4;
  p.NX = d.NX;
  p.KC = d.KC;
  p.CH = d.CH;
  p.unit = d.unit;
  for (int j = 0; j < a.count; ++j) {
    p.src[j] = a.src[j];
    p.state[j] = a.state ? a.state[j] : nullptr;
  }
  if (a.state) {   // backward operations through stored internal states
    if (d.cell)
      switch (cfg) {
        case 0: return launch_sweep_cfg<false, 4, 5, 4, 8, 8, 1, 1, 1>(p, st);
        case 1: return launch_sweep_cfg<false, 4, 5, 4, 8, 8, 2, 1, 1>(p, st);
        case 2: return launch_sweep_cfg<false, 2, 4, 4, 4, 8, 1, 2, 1>(p, st);
        case 3: return launch_sweep_cfg<false, 2, 4, 4, 4, 8, 2, 2, 1>(p, st);
        case 4: return launch_sweep_cfg<false, 1, 2, 4, 4, 4, 1, 1, 1>(p, st);
        case 5: return launch_sweep_cfg<false, 1, 2, 4, 4, 4, 2, 1, 1>(p, st);
        default: return launch_sweep_cfg<false, 8, 5, 8, 16, 8, 1, 1, 1>(p, st);
      }
    switch (cfg) {
      case 0: return launch_sweep_cfg<false, 4, 5, 4, 8, 8, 1, 1>(p, st);
      case 1: return launch_sweep_cfg<false, 4, 5, 4, 8, 8, 2, 1>(p, st);
      case 2: return launch_sweep_cfg<false, 2, 4, 4, 4, 8, 1, 2>(p, st);
      case 3: return launch_sweep_cfg<false, 2, 4, 4, 4, 8, 2, 2>(p, st);
      case 4: return launch_sweep_cfg<false, 1, 2, 4, 4, 4, 1, 1>(p, st);
      case 5: return launch_sweep_cfg<false, 1, 2, 4, 4, 4, 2, 1>(p, st);
      default: return launch_sweep_cfg<false, 8, 5, 8, 16, 8, 1, 1>(p, st);
    }
  }
  if (d.cell || cfg >= SWEEP_BACKWARD_ONLY_FROM) return hipErrorInvalidValue;
  switch (cfg) {
    case 0: return launch_sweep_cfg<true, 4, 5, 4, 8, 8, 1, 1>(p, st);
    case 1: return launch_sweep_cfg<true, 4, 5, 4, 8, 8, 2, 1>(p, st);
    case 2: return launch_sweep_cfg<true, 2, 4, 4, 4, 8, 1, 2>(p, st);
    case 3: return launch_sweep_cfg<true, 2, 4, 4, 4, 8, 2, 2>(p, st);
    case 4: return launch_sweep_cfg<true, 1, 2, 4, 4, 4, 1, 1>(p, st);
    case 5: return launch_sweep_cfg<true, 1, 2, 4, 4, 4, 2, 1>(p, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mebptt
