// The sweep kernel: a run of backward steps in one launch, with or without the forward operations that
// recompute their internal states.  Not part of the ABI.
#pragma once

#include "resident.h"

namespace mebptt {

constexpr int SWEEP_MAX_STEPS = 32;
struct SweepParams {
  static constexpr int RING = RES_RING;
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
  void* ring;            // RES_RING exchange slots [BP][G4] of dG, fragment-tiled
  unsigned* sync;
  unsigned published, launch;   // blocks published by this run's sweep launches before this one; resident launches before it
  long long wait_ticks;  // bound of every wait, in ticks of the 100 MHz wall clock
  long long patience;    // bound of the first one: then the launch may be given up
  int alone;             // only rank 0 of each XCD runs, and carries on alone
  int s_hi, count;       // steps s_hi, s_hi - 1, ..., s_hi - count + 1 (in at most two consecutive chunks)
  int B, I, H, HP, KX, KH, BP, nb, G4, NX, KC, CH;
  size_t unit, hplane;
  const float* src[SWEEP_MAX_STEPS];   // src[j]: unit holding the state before step s_hi - j
  const float* state[SWEEP_MAX_STEPS]; // FWD = false: unit holding the stored internal state of step s_hi - j
};
__device__ inline int units_of(const __attribute__((address_space(4))) SweepParams& p) { return p.HP; }

// All steps of a launch for units [u0, u1) of the XCD's sequences, by a workgroup that has stopped waiting (see
// chain_slowly).  Its waves deal the units out sixteen at a time: dh of a tile passes through LDS from the MFMA's layout (a lane has four
// consecutive units) to that of the gate sums (a lane has one unit of each four).
// HALVES: the odd macro steps of the KSB / 2 parts of K are the upper half of KSB (backward_in_halves).
template <class P, class T, bool FWD, int KSF, int KSB, int CELL, bool HALVES = false>
__device__ __forceinline__ void sweep_slowly(int b_lo, int b_hi, int u0, int u1, float* smem, int* s_fail) {
  const auto& p = *arguments_again<P>();
  const int waves = (int)(blockDim.x >> 6);
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, FRAG = 64 * VEC;
  constexpr bool SPLIT = HPlane<T>::SPLIT;
  typedef __attribute__((ext_vector_type(sizeof(T)))) unsigned int vec;   // the four gates of a unit
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int lrow = lane & 15, lq = lane >> 4;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP, nsteps = p.G4 / KSTEP, tiles = (u1 - u0 + 15) / 16, ncs = p.KC / KSTEP;
  const size_t hhalf = (size_t)p.BP * p.KH, dG_step = (size_t)p.BP * p.G4;
  const unsigned plane = (unsigned)(p.B * p.H);
  float* dhs = smem + wave * 256;   // [16 units][16 sequences]
  auto slot = [&](unsigned q) { return reinterpret_cast<T*>(p.ring) + (size_t)(q % P::RING) * dG_step; };
  auto off = [&](int t) {
    const int b = b_lo + t * 16 + lrow;
    return b < b_hi ? (unsigned)(((b >> 4) * nsteps * 64 + lq * 16 + (b & 15)) * 16) : RES_NO_LANE;
  };
  auto publish = [&](unsigned q, size_t o, vec v) {   // as in a sweep
    vec empty;
#pragma unroll
    for (int r = 0; r < (int)sizeof(T); ++r) empty[r] = RES_EMPTY;
    *reinterpret_cast<vec*>(slot(q) + o) = v;
    *reinterpret_cast<vec*>(slot(q + P::RING - 2) + o) = empty;
  };
  for (int tile = wave; tile < tiles; tile += waves)
    for (int c = b_lo; c < b_hi; c += 16) {
      const int b = c + lrow;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int u = u0 + 16 * tile + 4 * i + lq;
        if (b >= b_hi || u >= u1) continue;
        const size_t o = ft_offset<T>(b, 4 * u, nsteps);
        vec v{};
        if (u < p.H && p.dG_next) v = *reinterpret_cast<const vec*>(reinterpret_cast<const T*>(p.dG_next) + o);
#pragma unroll
        for (int r = 0; r < (int)sizeof(T); ++r) v[r] = not_empty(v[r]);
        publish(p.published, o, v);
      }
    }
  for (int j = 0; j < p.count; ++j) {
    const int s = p.s_hi - j, step_slot = (s - 1) % p.CH, buf = ((s - 1) / p.CH) & 1;
    const T* in = slot(p.published + (unsigned)j);
    if (!slot_is_there(in, nsteps, (b_hi - b_lo + 15) / 16, off, p.wait_ticks, p.sync + RES_SYNC_STATUS, s_fail)) return;
    T* dG_cur = reinterpret_cast<T*>(p.dG_chunk[buf]) + (size_t)step_slot * dG_step;
    T *dGT = reinterpret_cast<T*>(p.dGT[buf]), *aT = reinterpret_cast<T*>(p.aT[buf]);
    const float *src = p.src[j], *stp = FWD ? src : p.state[j];
    for (int tile = wave; tile < tiles; tile += waves)
      for (int c = b_lo; c < b_hi; c += 16) {
        const int b = c + lrow, row = b < b_hi ? b : b_lo;
        const bool own = b < b_hi;
        const unsigned goff = off((c - b_lo) / 16);
        const int n = min(u0 + 16 * tile + lrow, u1 - 1);   // this lane's row (a row past the units is never used)
        const T* base = reinterpret_cast<const T*>(p.WTh) + ((size_t)(n >> 4) * nsteps * 64 + lq * 16 + (n & 15)) * VEC;
        f32x4 acc[KSB], dh4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < KSB; ++w) acc[w] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < nsteps; s0 += KSB)
#pragma unroll
          for (int w0 = 0; w0 < KSB; w0 += 4) {
            typename M::Frag a[4], f[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const int m = min(s0 + w0 + w, nsteps - 1);
              a[w] = M::load(base + (size_t)m * FRAG);
              f[w] = as_frag<typename M::Frag>(load_slot_16(in, goff, m * 1024));
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              if (s0 + w0 + w >= nsteps) a[w] = f[w] = typename M::Frag{};
              acc[w0 + w] = M::mma(a[w], f[w], acc[w0 + w]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
        for (int r = 0; r < 4; ++r) {   // fixed order, as in backward_body
          if constexpr (HALVES) {
#pragma unroll
            for (int w = 0; w < KSB / 2; ++w) dh4[r] += acc[w][r] + acc[w + KSB / 2][r];
          } else if constexpr (KSB == WIDE_BACK_PARTS) {
            dh4[r] = sum_back_parts([&](int w) { return acc[w][r]; });
          } else {
#pragma unroll
            for (int w = 0; w < KSB; ++w) dh4[r] += acc[w][r];
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) dhs[(4 * lq + r) * 16 + lrow] = dh4[r];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's own part: no barrier
        __builtin_amdgcn_wave_barrier();
        const unsigned hsrc = SPLIT ? (unsigned)(((row >> 4) * nsh * 64 + lq * 16 + (row & 15)) * VEC) : (unsigned)(row * p.H);
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
          const int u4 = u0 + 16 * tile + 4 * i, u = u4 + lq;
          if (u4 >= u1) break;
          const bool real = own && u < p.H;
          const size_t e = real ? (size_t)b * p.H + u : 0, o = real ? ft_offset<T>(b, u, nsh) : 0;
          float gate[4], second = 0.0f, h = 0.0f;
          const float prev = CELL ? load_h<T>(src, (unsigned)e, (unsigned)o, hhalf) : (src + p.hplane)[e];
          if constexpr (FWD) {
            float G[4];
            gates_slowly<T, KSF>(p.Wp, u4 / 4, p.x + (size_t)(s - 1) * p.B * p.I, (unsigned)(row * p.I), p.I, nsx, nsh,
                                [&](int m) {
                                  if constexpr (SPLIT) {
                                    return M::load(reinterpret_cast<const T*>(src) + (size_t)m * FRAG + (size_t)hsrc);
                                  } else {
                                    RawAct<VEC> raw = load_window<VEC>(src, hsrc, m * KSTEP + VEC * lq, p.H);
                                    shift_tail<VEC>(raw, m * KSTEP + VEC * lq, p.H);
                                    return M::from_f32(raw.v);
                                  }
                                },
                                G);
            if (real) h = cell_forward<T, CELL>(G, *reinterpret_cast<const float4*>(p.bp + 4 * u), prev, second, gate);
          } else {
            gate[0] = (stp + p.unit)[e];
            gate[1] = (stp + p.unit + plane)[e];
            gate[2] = (stp + 2 * p.unit)[e];
            gate[3] = CELL == 0 ? (stp + 2 * p.unit + plane)[e] : 0.0f;
            second = (stp + p.hplane)[e];
            if (p.dy_is_h || p.y_out) h = load_h<T>(stp, (unsigned)e, (unsigned)o, hhalf);
          }
          union { T t[4]; unsigned w[sizeof(T)]; vec v; } dg;
          dg.v = vec{};
          if (real) {
            float dh = dhs[(4 * i + lq) * 16 + lrow], dG[4], dc_out;
            dh += p.dy_is_h ? h : (p.dy != nullptr && s >= p.dy_first ? (p.dy + (size_t)(s - p.dy_first) * plane)[e] : 0.0f);
            if (CELL == 0)
              lstm_backward_point<T>(dh, p.dc[e], gate[0], gate[1], gate[2], gate[3], second, prev, dG, dc_out);
            else
              gru_backward_point(__fadd_rn(dh, p.dc[e]), gate[0], gate[1], gate[2], second, prev, dG, dc_out);
            p.dc[e] = dc_out;
#pragma unroll
            for (int r = 0; r < 4; ++r) dg.t[r] = (T)dG[r];
#pragma unroll
            for (int r = 0; r < (int)sizeof(T); ++r) dg.w[r] = not_empty(dg.w[r]);
            if (p.y_out) (p.y_out + (size_t)(s - 1) * plane)[e] = h;
            const int col = step_slot * p.B + b;
#pragma unroll
            for (int r = 0; r < 4; ++r) dGT[ft_offset<T>(4 * u + r, col, ncs)] = dg.t[r];
            aT[ft_offset<T>(p.NX + u, col, ncs)] = (T)load_h_operand<T>(src, (unsigned)e, (unsigned)o);
          }
          if (own) {
            const size_t og = ft_offset<T>(b, 4 * u, nsteps);
            if (j + 1 < p.count) publish(p.published + (unsigned)j + 1, og, dg.v);
            if (real) *reinterpret_cast<vec*>(dG_cur + og) = dg.v;
          }
        }
      }
  }
}

// Where a sub-sequence fits into memory the schedule alternates "forward operation of step s from
// the memorised h_{s-1}, keeping the internal state" and "backward operation of step s", s going
// down.  On shapes whose gate weights AND their transpose fit on the chip such a run of pairs goes
// out as one launch (FWD), organised like the forward chain (batch split over the XCDs, hidden units over
// the 32 compute units of an XCD, weights in registers):
//   * the forward operation of a step needs nothing from other compute units (its input state was
//     memorised by an earlier launch), and its internal state never leaves the registers of the
//     thread that owns the (sequence, unit);
//   * the backward operation needs dG of the step after, all 4H columns of it, for the XCD's sequences:
//     the compute units exchange their columns the way the forward chain exchanges h; dG of the step
//     above the launch is published like any other, so all steps are alike;
//   * while the others' columns travel, every compute unit runs the forward operation of the next
//     lower step.
// FWD = false: the internal states are not recomputed but read from where an earlier launch stored them
// (internal-state slots, or the stage of a forward batch): backward operations only, W_hh^T alone resident.
// What only later launches read of a step (dG in the chunk buffer, its transposed copies, the outputs)
// is stored, and what the next step needs is fetched, right after the polls of the following
// exchange: memory operations complete in order, so in front of the polls they would hold them up.
// What bounds a step is that chain of latencies.  Measured per step, with counters and whole tiles before
// and so: without forward operations H = 1024, B = 64 5.3 -> 3.6 us; with them H = 512, B = 256 6.8 -> 5.0 us
// (4.1 - 4.4 with the GEMMs in order).
// K splits and summation orders are those of forward_body and backward_body for the shape, the
// pointwise steps are the shared functions: bit-identical to the launch-per-step path.
// Up to 64 sequences (half tiles), bf16, K split eight ways: the backward product takes two macro steps an instruction
// (Halves), half the matrix instructions and half the fetches of dG, whose every lane then carries data: H = 1024, B = 64 62.2 -> 57.9 us a
// launch of 18 steps on average.
// NXW, NHW, KSF: macro steps of x and h per wave and K split of the forward part; NBW, KSB: macro steps of
// dG per wave (the weights of the last NBL are parked in LDS: registers are what the two largest
// instantiations are short of) and K split of the backward part; NBT: batch tiles of the XCD's share.
template <class T, int KSB, int NBT>
constexpr bool sweep_in_halves = sizeof(T) == 2 && KSB == 8 && NBT == 0;
constexpr int SWEEP_KEPT = 320;   // values a wave turns over per step: 64 items' dG and h_{s-1}
template <class T, bool FWD, int NRT, int NXW, int NHW, int KSF, int NBW, int NBL, int KSB, int NBT, int CELL>
__global__ __launch_bounds__(512) void sweep_kernel(SweepParams p) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, FRAG = 64 * VEC;
  constexpr bool SPLIT = HPlane<T>::SPLIT;
  constexpr int UW = NRT * 4;                       // hidden units per workgroup
  constexpr int NTB = (UW + 15) / 16;               // 16-unit tiles of the dh GEMM that cover them
  constexpr int NB = NBT ? NBT : 1, COLS = NBT ? NBT * 16 : 8;
  // backward operations on stored states fetch whole planes: BLOCK order; with forward operations most of what
  // an item moves is fragment-tiled: the MFMA's order
  using It = Items<UW, COLS, !FWD>;
  constexpr int ITEMS = It::COUNT, IPT = (ITEMS + 511) / 512;
  constexpr int GF = 8 / KSF, FTB = (GF == 2 && NBT == 2) ? 2 : 1, FTR = GF / FTB;   // forward: groups of waves along batch, rows
  constexpr int NRTW = (NRT + FTR - 1) / FTR, BTWF = NB / FTB;
  constexpr int GB = 8 / KSB, BTB = (GB == 2 && NBT == 2) ? 2 : 1, BTWB = NB / BTB;   // backward: along the batch, or one group idles
  constexpr bool HALVES = sweep_in_halves<T, KSB, NBT>;
  static_assert(!HALVES || (NBW % 2 == 0 && NBL % 2 == 0), "macro steps in twos");
  constexpr int NBF = HALVES ? NBW / 2 : NBW, NBP = HALVES ? NBL / 2 : NBL;   // a wave's fetches of dG; weights of the last NBP parked
  using Weights = std::conditional_t<HALVES, bf16x16, typename M::Frag>;
  using SumF = Sums<NRTW, NBT == 0 ? 0 : BTWF>;
  using SumB = Sums<NTB, NBT == 0 ? 0 : BTWB>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f32x4* redB = reinterpret_cast<f32x4*>(smem);                       // [8 waves][SumB::BLOCKS][64]: dh of 4 units
  f32x4* redF = redB + 8 * SumB::BLOCKS * 64;                         // [8 waves][SumF::BLOCKS][64]: the gates of a unit
  T* wl = reinterpret_cast<T*>(redF + (FWD ? 8 * SumF::BLOCKS * 64 : 0));   // [8][NTB][NBL] fragments
  T* kept = wl + (size_t)8 * NTB * NBL * FRAG;                        // [8][IPT][SWEEP_KEPT]
  __shared__ int s_go, s_g, s_rank, s_fail;
  // the wave index as a scalar: conditions on it become scalar branches (an MFMA under a lane mask
  // that is empty would still execute)
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int lrow = lane & 15, lq = lane >> 4;
  if (threadIdx.x == 0) {
    int xg, xr;
    s_go = draw_rank(p.sync, p.launch, xg, xr);
    s_g = xg;
    s_rank = xr;
    s_fail = 0;
  }
  __syncthreads();
  if (!s_go) return;
  const int g = __builtin_amdgcn_readfirstlane(s_g), rank = __builtin_amdgcn_readfirstlane(s_rank);
  const int b_lo = g * p.nb, b_hi = min(p.B, b_lo + p.nb);
  // no sequences or no units here: nobody waits for this workgroup
  if (b_lo >= p.B || rank * UW >= p.HP || (p.alone && rank)) return;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP, nstepsF = nsx + nsh, nstepsB = p.G4 / KSTEP;
  const size_t hhalf = (size_t)p.BP * p.KH, dG_step = (size_t)p.BP * p.G4;
  const unsigned plane = (unsigned)(p.B * p.H);
  const int fk = wave % KSF, fg = wave / KSF, bk = wave % KSB, bg = wave / KSB;
  const int rt0 = (FTR > 1 ? fg : 0) * NRTW, btf0 = (FTB > 1 ? fg : 0) * BTWF, btb0 = (BTB > 1 ? bg : 0) * BTWB;
  const bool bwd_wave = bg < BTB;
  const int mh0 = (fk + KSF - nsx % KSF) % KSF;     // this wave's h macro steps: mh0, mh0 + KSF, ... (below nsh)

  // items: (sequence, unit).  A unit between H and the padded HP publishes zeros.
  bool mine[IPT], real[IPT];
  const f32x4* cellF[IPT];
  const float* cellB[IPT];
  unsigned ie[IPT], io[IPT], ig[IPT];   // b * H + u; places in the fragment-tiled h plane and (of gate 0) in a dG block
  float4 bias[IPT];
  float dc_run[IPT];
  // internal state of the step whose backward operation comes next, its input state, its loss gradient
  float st_gate[IPT][4], st_c[IPT], st_h[IPT], st_cprev[IPT], st_hprev[IPT], st_dy[IPT];
  unsigned dg[IPT][sizeof(T)];          // the four gates' dG of the last step, as published (8 or 16 bytes)
  float kp_h[IPT], kp_hprev[IPT];
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const int item = (int)threadIdx.x + q * 512;
    const int ul = It::unit(item), col = It::column(item), b = b_lo + col, u = rank * UW + ul;
    {   // the wave that holds its sums for K part 0 (row group, or batch group), then its block
      const int rt = ul >> 2, rw = FTR > 1 ? rt % NRTW : rt, wf = FTR > 1 ? rt / NRTW : (FTB > 1 ? (col >> 4) / BTWF : 0);
      cellF[q] = redF + (size_t)(wf * KSF * SumF::BLOCKS + SumF::block(rw, FTB > 1 ? col % (BTWF * 16) : col)) * 64 + SumF::lane(rw, ul & 3, col);
      const int tb = ul >> 4, wB = BTB > 1 ? (col >> 4) / BTWB : 0;
      if constexpr (HALVES)
        cellB[q] = reinterpret_cast<const float*>(redB + (tb >> 1) * 64 + Halves::lane_of(ul & 15, col)) + 2 * (tb & 1) + (col & 1);
      else
        cellB[q] = reinterpret_cast<const float*>(redB + (size_t)(wB * KSB * SumB::BLOCKS + SumB::block(tb, BTB > 1 ? col % (BTWB * 16) : col)) * 64 +
                                                  SumB::lane(tb, (ul & 15) >> 2, col)) + (ul & 3);
    }
    mine[q] = item < ITEMS && b < b_hi && u < p.HP;
    real[q] = mine[q] && u < p.H;
    ie[q] = real[q] ? (unsigned)(b * p.H + u) : 0u;     // element 0 is there for items without one to fetch
    io[q] = real[q] ? (unsigned)ft_offset<T>(b, u, nsh) : 0u;
    ig[q] = mine[q] ? (unsigned)ft_offset<T>(b, 4 * u, nstepsB) : 0u;
    bias[q] = real[q] ? *reinterpret_cast<const float4*>(p.bp + 4 * u) : float4{0.f, 0.f, 0.f, 0.f};
    dc_run[q] = real[q] ? p.dc[(size_t)ie[q]] : 0.0f;
    kp_h[q] = kp_hprev[q] = 0.0f;
#pragma unroll
    for (int i = 0; i < (int)sizeof(T); ++i) dg[q][i] = 0u;
    if (real[q] && p.dG_next) {
      const unsigned* src = reinterpret_cast<const unsigned*>(reinterpret_cast<const T*>(p.dG_next) + (size_t)ig[q]);
#pragma unroll
      for (int i = 0; i < (int)sizeof(T); ++i) dg[q][i] = not_empty(src[i]);
    }
  }
  // the four gates of a unit are consecutive in a dG block: one 8- or 16-byte store
  auto store_dg = [&](T* block, int q, bool empty) {
    typedef __attribute__((ext_vector_type(sizeof(T)))) unsigned int vec;
    vec v;
#pragma unroll
    for (int i = 0; i < (int)sizeof(T); ++i) v[i] = empty ? RES_EMPTY : dg[q][i];
    *reinterpret_cast<vec*>(block + (size_t)ig[q]) = v;
  };
  auto publish = [&](unsigned q_now) {
    T* slot_out = reinterpret_cast<T*>(p.ring) + (size_t)(q_now % RES_RING) * dG_step;
    T* slot_old = reinterpret_cast<T*>(p.ring) + (size_t)((q_now + 2) % RES_RING) * dG_step;   // two steps back
#pragma unroll
    for (int q = 0; q < IPT; ++q)
      if (mine[q]) {
        store_dg(slot_out, q, false);
        store_dg(slot_old, q, true);
      }
  };
  publish(p.published);   // travels while the weights are fetched

  // resident weights: the forward rows of this workgroup's units, and the rows of W_hh^T for the same units
  typename M::Frag wx[FWD ? NRTW : 1][FWD ? NXW : 1], wh[FWD ? NRTW : 1][FWD ? NHW : 1];
  Weights wb[NTB][NBF - NBP > 0 ? NBF - NBP : 1];
  if constexpr (FWD) {
#pragma unroll
    for (int rt = 0; rt < NRTW; ++rt) {
      const int row_tile = min(rank * NRT + min(rt0 + rt, NRT - 1), p.HP / 4 - 1);
      const T* base = reinterpret_cast<const T*>(p.Wp) + ((size_t)row_tile * nstepsF * 64 + lane) * VEC;
#pragma unroll
      for (int i = 0; i < NXW; ++i) {
        const int s = fk + KSF * i;
        wx[rt][i] = M::load(base + (size_t)min(s, nsx - 1) * FRAG);
        if (s >= nsx) wx[rt][i] = typename M::Frag{};
      }
#pragma unroll
      for (int i = 0; i < NHW; ++i) {
        const int m = mh0 + KSF * i;
        wh[rt][i] = M::load(base + (size_t)(nsx + min(m, nsh - 1)) * FRAG);
        if (m >= nsh) wh[rt][i] = typename M::Frag{};
      }
    }
  }
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) {
    const int n = min(rank * UW + min(tb * 16 + lrow, UW - 1), p.HP - 1);   // this lane's row (a row past the units is never used)
    const T* base = reinterpret_cast<const T*>(p.WTh) + ((size_t)(n >> 4) * nstepsB * 64 + lq * 16 + (n & 15)) * VEC;
#pragma unroll
    for (int k = 0; k < NBF; ++k) {
      if constexpr (HALVES) {
        const bf16x16 f = Halves::load(p.WTh, (unsigned)(((n >> 4) * nstepsB * 64 + (n & 15)) * 16), bk + 2 * KSB * k, bk + 2 * KSB * k + KSB, nstepsB, lq);
        if (k < NBF - NBP) {
          wb[tb][k < NBF - NBP ? k : 0] = f;
        } else {
          typename M::Frag* to = reinterpret_cast<typename M::Frag*>(wl) + ((size_t)(wave * NTB + tb) * NBP + (k - (NBF - NBP))) * 128 + lane;
          to[0] = __builtin_shufflevector(f, f, 0, 1, 2, 3, 4, 5, 6, 7);
          to[64] = __builtin_shufflevector(f, f, 8, 9, 10, 11, 12, 13, 14, 15);
        }
      } else {
        const int m = bk + KSB * k;
        typename M::Frag f = M::load(base + (size_t)min(m, nstepsB - 1) * FRAG);
        if (m >= nstepsB) f = typename M::Frag{};
        if (k < NBW - NBL)
          wb[tb][k < NBW - NBL ? k : 0] = f;
        else
          *reinterpret_cast<typename M::Frag*>(&wl[((size_t)(wave * NTB + tb) * NBL + (k - (NBW - NBL))) * FRAG + lane * VEC]) = f;
      }
    }
  }

  // where this lane's operands come from.  Columns of a tile that belong to no sequence of this XCD read
  // the first one's rows and fetch no dG.
  unsigned xrow[BTWF], hsrc[BTWF], goff[BTWB];
#pragma unroll
  for (int t = 0; t < BTWF; ++t) {
    const int b = b_lo + (btf0 + t) * 16 + lrow, row = b < b_hi ? b : b_lo;
    xrow[t] = (unsigned)(row * p.I);
    hsrc[t] = SPLIT ? (unsigned)(((row >> 4) * nsh * 64 + lq * 16 + (row & 15)) * VEC) : (unsigned)(row * p.H);
  }
#pragma unroll
  for (int t = 0; t < BTWB; ++t) {
    const int b = b_lo + (btb0 + t) * 16 + (HALVES ? lrow & 7 : lrow);
    goff[t] = b < b_hi ? (unsigned)(((b >> 4) * nstepsB * 64 + lq * 16 + (b & 15)) * 16) : RES_NO_LANE;
  }

  // what the next lower step needs, fetched a step ahead: raw x values and h fragments, or the stored
  // internal state; c_{s-1}, h_{s-1}, the loss gradient
  RawAct<VEC> xraw[FWD ? NXW : 1][BTWF];
  typename M::Frag hfr[(FWD && SPLIT) ? NHW : 1][BTWF];
  RawAct<VEC> hraw[(FWD && !SPLIT) ? NHW : 1][BTWF];
  float pf_gate[IPT][4], pf_c[IPT], pf_h[IPT], pf_cprev[IPT], pf_hprev[IPT], pf_dy[IPT];
  const bool want_h = p.dy_is_h || p.y_out != nullptr;
  // Half tiles leave the upper waves without items: those skip the items' fetches and stores, which
  // still took their issue slots with every lane masked (sweep of H = 512, B = 64 store all, a whole
  // run 1.243 -> 1.194 ms; H = 1024 10.92 -> 10.64 ms). With forward operations a branch between the
  // operands' loads and the items' costs more than it saves (H = 256 2.00 -> 2.18 ms, H = 512 of
  // 10000 steps 109.6 -> 115.5 ms), so not there.
  const bool has_items = FWD || wave * 64 < ITEMS;
  auto fetch = [&](int j) {
    const int s = p.s_hi - j;
    const float* src = p.src[j];
    if constexpr (FWD) {
      const float* x_s = p.x + (size_t)(s - 1) * p.B * p.I;
#pragma unroll
      for (int t = 0; t < BTWF; ++t) {
#pragma unroll
        for (int i = 0; i < NXW; ++i) xraw[i][t] = load_window<VEC>(x_s, xrow[t], (fk + KSF * i) * KSTEP + VEC * lq, p.I);
#pragma unroll
        for (int i = 0; i < NHW; ++i) {
          const int m = mh0 + KSF * i;
          if constexpr (SPLIT)
            hfr[i][t] = M::load(reinterpret_cast<const T*>(src) + (size_t)min(m, nsh - 1) * FRAG + (size_t)hsrc[t]);
          else
            hraw[i][t] = load_window<VEC>(src, hsrc[t], m * KSTEP + VEC * lq, p.H);
        }
      }
    }
    const float* stp = FWD ? src : p.state[j];
    if (!has_items) return;
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if constexpr (!FWD) {
        pf_gate[q][0] = (stp + p.unit)[(size_t)ie[q]];
        pf_gate[q][1] = (stp + p.unit + plane)[(size_t)ie[q]];
        pf_gate[q][2] = (stp + 2 * p.unit)[(size_t)ie[q]];
        if (CELL == 0) pf_gate[q][3] = (stp + 2 * p.unit + plane)[(size_t)ie[q]];   // the GRU has three gates
        pf_c[q] = (stp + p.hplane)[(size_t)ie[q]];                                 // c_s, or the GRU's n_h
        if (want_h) pf_h[q] = load_h<T>(stp, ie[q], io[q], hhalf);
      }
      // what the pointwise step blends with: c_{s-1}, or the GRU's h_{s-1} in full precision
      pf_cprev[q] = CELL ? load_h<T>(src, ie[q], io[q], hhalf) : (src + p.hplane)[(size_t)ie[q]];
      pf_hprev[q] = load_h_operand<T>(src, ie[q], io[q]);
      pf_dy[q] = 0.0f;
    }
    if (p.dy != nullptr && s >= p.dy_first) {
      const float* dy_s = p.dy + (size_t)(s - p.dy_first) * plane;
#pragma unroll
      for (int q = 0; q < IPT; ++q) pf_dy[q] = dy_s[(size_t)ie[q]];
    }
  };
  // Makes the fetched step the current one: its forward operation (FWD; a barrier inside), or its stored state.
  auto advance = [&]() {
    if constexpr (FWD) {
      f32x4 acc[NRTW][BTWF];
#pragma unroll
      for (int rt = 0; rt < NRTW; ++rt)
#pragma unroll
        for (int t = 0; t < BTWF; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NXW; ++i) {
        const int s = fk + KSF * i;
        if ((s + 1) * KSTEP > p.I) {
#pragma unroll
          for (int t = 0; t < BTWF; ++t) shift_tail<VEC>(xraw[i][t], s * KSTEP + VEC * lq, p.I);
        }
#pragma unroll
        for (int t = 0; t < BTWF; ++t) {
          const typename M::Frag f = M::from_f32(xraw[i][t].v);
#pragma unroll
          for (int rt = 0; rt < NRTW; ++rt) acc[rt][t] = M::mma(wx[rt][i], f, acc[rt][t]);
        }
      }
#pragma unroll
      for (int i = 0; i < NHW; ++i) {
        const int m = mh0 + KSF * i;
#pragma unroll
        for (int t = 0; t < BTWF; ++t) {
          typename M::Frag f;
          if constexpr (SPLIT) {
            f = hfr[i][t];
            if (m >= nsh) f = typename M::Frag{};
          } else {
            if ((m + 1) * KSTEP > p.H) shift_tail<VEC>(hraw[i][t], m * KSTEP + VEC * lq, p.H);
            f = M::from_f32(hraw[i][t].v);
          }
#pragma unroll
          for (int rt = 0; rt < NRTW; ++rt) acc[rt][t] = M::mma(wh[rt][i], f, acc[rt][t]);
        }
      }
      SumF::write(redF + (size_t)wave * SumF::BLOCKS * 64, lane, acc);
      lds_barrier();
    }
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      st_cprev[q] = pf_cprev[q];
      st_hprev[q] = pf_hprev[q];
      st_dy[q] = pf_dy[q];
      if constexpr (FWD) {
        if (!mine[q]) continue;
        float G[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (parts_in_pairs<T, KSF>) {   // fixed order, as in forward_body
          add_pairs<KSF>(G, [&](int w) { return cellF[q][w * SumF::BLOCKS * 64]; });
        } else {
#pragma unroll
          for (int w = 0; w < KSF; ++w) {
            const f32x4 v = cellF[q][w * SumF::BLOCKS * 64];
#pragma unroll
            for (int r = 0; r < 4; ++r) G[r] += v[r];
          }
        }
        st_h[q] = cell_forward<T, CELL>(G, bias[q], st_cprev[q], st_c[q], st_gate[q]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) st_gate[q][r] = pf_gate[q][r];
        st_c[q] = pf_c[q];
        st_h[q] = pf_h[q];
      }
    }
  };
  // What only later launches read of step s: dG in the chunk buffer, the transposed copies for the weight
  // gradient, the output.  A block of items holds whole 16-byte slots of the transposed operands when the
  // batch is a multiple of the sequences in a slot: the wave then turns its block over in LDS (keep_transposed,
  // right after the step; each wave its own part, so no barrier) and stores them slot by slot.  Not beside
  // forward operations, which have no time to spare on LDS where the stored states' loads would have been
  // (H = 512, B = 256: 79 instead of 70 us a launch).
  const bool slots_whole = !FWD && p.B % VEC == 0;
  T* kept_w = kept + (size_t)wave * IPT * SWEEP_KEPT;
  auto keep_transposed = [&]() {
    if (!slots_whole || !has_items) return;
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      union { unsigned u[sizeof(T)]; T t[4]; } pk;
#pragma unroll
      for (int i = 0; i < (int)sizeof(T); ++i) pk.u[i] = dg[q][i];
      const int ul = It::unit_in(lane), bl = It::row_in(lane);
      T* k = kept_w + q * SWEEP_KEPT;
#pragma unroll
      for (int r = 0; r < 4; ++r) k[(ul * 4 + r) * It::WB + bl] = pk.t[r];   // [row 4u + gate][sequence]
      k[256 + ul * It::WB + bl] = (T)kp_hprev[q];                            // [unit][sequence]
    }
  };
  auto store_kept = [&](int s) {
    if (!has_items) return;
    const int slot = (s - 1) % p.CH, buf = ((s - 1) / p.CH) & 1;   // where step s lives in the chunk buffers
    T* dG_cur = reinterpret_cast<T*>(p.dG_chunk[buf]) + (size_t)slot * dG_step;
    T* dGT = reinterpret_cast<T*>(p.dGT[buf]);
    T* aT = reinterpret_cast<T*>(p.aT[buf]);
    float* y_s = p.y_out ? p.y_out + (size_t)(s - 1) * plane : nullptr;
    const int ncs = p.KC / KSTEP;
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (real[q]) {
        store_dg(dG_cur, q, false);
        if (y_s) y_s[(size_t)ie[q]] = kp_h[q];
      }
      const int item = (int)threadIdx.x + q * 512, first = item & ~63;   // the block's first item
      if (slots_whole) {
        // chunk c of the block: VEC sequences of one row; rows of dG first, then rows of h_{s-1}
        constexpr int CR = It::WB / VEC, NDG = 4 * It::WU * CR, NALL = NDG + It::WU * CR;
        const int u0 = rank * UW + It::unit(first), b0 = b_lo + It::column(first);
#pragma unroll
        for (int c0 = 0; c0 < NALL; c0 += 64) {
          const int c = c0 + lane, row = c / CR, b = b0 + c % CR * VEC;
          const bool is_dg = c < NDG;
          const int n = u0 + (is_dg ? row >> 2 : row - 4 * It::WU);
          if (c < NALL && first < ITEMS && b < b_hi && n < p.H) {
            T* dst = is_dg ? dGT + (size_t)ft_offset<T>(4 * n + (row & 3), slot * p.B + b, ncs)
                           : aT + (size_t)ft_offset<T>(p.NX + n, slot * p.B + b, ncs);
            *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(kept_w + q * SWEEP_KEPT + c * VEC);
          }
        }
      } else if (real[q]) {
        const int b = b_lo + It::column(item), n = rank * UW + It::unit(item);
        const int col = slot * p.B + b;
        union { unsigned u[sizeof(T)]; T t[4]; } pk;
#pragma unroll
        for (int i = 0; i < (int)sizeof(T); ++i) pk.u[i] = dg[q][i];
        // rows 4n .. 4n + 3 of one column lie VEC elements apart (they share a 16-row tile)
        const unsigned o = (unsigned)ft_offset<T>(4 * n, col, ncs);
#pragma unroll
        for (int r = 0; r < 4; ++r) dGT[(size_t)(o + r * VEC)] = pk.t[r];
        aT[(size_t)ft_offset<T>(p.NX + n, col, ncs)] = (T)kp_hprev[q];
      }
    }
  };

  const int picks = Halves::picks(lane);
  fetch(0);
  advance();

  for (int j = 0; j < p.count; ++j) {
    const int s = p.s_hi - j;                       // the step back-propagated now
    // dG of step s + 1, all columns of the XCD's sequences
    typename M::Frag gfr[NBF][BTWB];
    if (bwd_wave) {
      const T* slot = reinterpret_cast<const T*>(p.ring) + (size_t)((p.published + (unsigned)j) % RES_RING) * dG_step;
      WaitBound bound{j == 0 ? p.patience : p.wait_ticks, p.sync + RES_SYNC_STATUS};
      while (true) {
        u32x4 raw[NBF][BTWB];
        unsigned top = 0;
#pragma unroll
        for (int k = 0; k < NBF; ++k) {
          const int m = bk + (HALVES ? KSB * (2 * k + (lrow >> 3)) : KSB * k);
#pragma unroll
          for (int t = 0; t < BTWB; ++t)
            raw[k][t] = HALVES ? load_slot_16(slot, m < nstepsB ? goff[t] + KSB * 1024u * (unsigned)(lrow >> 3) : RES_NO_LANE, (bk + 2 * KSB * k) * 1024)
                               : load_slot_16(slot, m < nstepsB ? goff[t] : RES_NO_LANE, m * 1024);
        }
#pragma unroll
        for (int k = 0; k < NBF; ++k)
#pragma unroll
          for (int t = 0; t < BTWB; ++t) {
            top = max(top, largest_dword(raw[k][t]));
            gfr[k][t] = as_frag<typename M::Frag>(raw[k][t]);
          }
        if (__builtin_amdgcn_ballot_w64(top == RES_EMPTY) == 0) break;
        if (bound.expired()) {
          s_fail = 1 + j;
          break;
        }
        asm volatile("" ::: "memory");   // the next look is another load
      }
    }
    if (j > 0) store_kept(s + 1);
    fetch(min(j + 1, p.count - 1));
    __builtin_amdgcn_sched_barrier(0);
    // dh = dG_{s+1} W_hh for this workgroup's units
    if (bwd_wave) {
      f32x4* sums = redB + (size_t)wave * SumB::BLOCKS * 64;
      f32x4 acc[NTB][BTWB];
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int t = 0; t < BTWB; ++t) acc[tb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < NBF; ++k)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
          Weights a;
          if (k < NBF - NBP) {
            a = wb[tb][k < NBF - NBP ? k : 0];
          } else if constexpr (HALVES) {
            const typename M::Frag* from = reinterpret_cast<const typename M::Frag*>(wl) + ((size_t)(wave * NTB + tb) * NBP + (k - (NBF - NBP))) * 128 + lane;
            a = __builtin_shufflevector(from[0], from[64], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
          } else {
            a = M::load(&wl[((size_t)(wave * NTB + tb) * NBL + (k - (NBW - NBL))) * FRAG + lane * VEC]);
          }
#pragma unroll
          for (int t = 0; t < BTWB; ++t) {
            if constexpr (HALVES)
              acc[tb][t] = Halves::mma(gfr[k][t], a, acc[tb][t], picks);
            else
              acc[tb][t] = M::mma(a, gfr[k][t], acc[tb][t]);
          }
        }
      if constexpr (HALVES) {
#pragma unroll
        for (int tb = 0; tb < NTB; tb += 2) {
          const Halves::Sum lo = Halves::fold(acc[tb][0]), hi = tb + 1 < NTB ? Halves::fold(acc[tb + 1 < NTB ? tb + 1 : tb][0]) : Halves::Sum{};
          sums[tb / 2 * 64 + lane] = f32x4{lo.v[0], lo.v[1], hi.v[0], hi.v[1]};
        }
      } else {
        SumB::write(sums, lane, acc);
      }
    }
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(s_fail))   // a wave has stopped waiting: written before the barrier, so all see it
      stop_waiting<SweepParams, UW>(&s_g, &s_rank, &s_fail, [&](int b_lo, int b_hi, int u0, int u1) {
        sweep_slowly<SweepParams, T, FWD, KSF, HALVES ? 2 * KSB : KSB, CELL, HALVES>(b_lo, b_hi, u0, u1, reinterpret_cast<float*>(smem), &s_fail);
      });
    // pointwise backward of step s on the internal state held in registers
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      float dh = 0.0f;
#pragma unroll
      for (int w = 0; w < KSB; ++w) dh += cellB[q][w * SumB::BLOCKS * 64 * 4];   // fixed order, as in backward_body
      dh += p.dy_is_h ? st_h[q] : st_dy[q];
      float dG[4], dc_out;
      if (CELL == 0)
        lstm_backward_point<T>(dh, dc_run[q], st_gate[q][0], st_gate[q][1], st_gate[q][2], st_gate[q][3], st_c[q], st_cprev[q],
                            dG, dc_out);
      else   // the running plane carries dh_{s+1} * z_{s+1}, as in backward_body
        gru_backward_point(__fadd_rn(dh, dc_run[q]), st_gate[q][0], st_gate[q][1], st_gate[q][2], st_c[q], st_cprev[q], dG, dc_out);
      dc_run[q] = dc_out;
      union { T t[4]; unsigned u[sizeof(T)]; } pk;
#pragma unroll
      for (int r = 0; r < 4; ++r) pk.t[r] = (T)dG[r];
#pragma unroll
      for (int i = 0; i < (int)sizeof(T); ++i) dg[q][i] = real[q] ? not_empty(pk.u[i]) : 0u;
      kp_h[q] = st_h[q];
      kp_hprev[q] = st_hprev[q];
    }
    if (j + 1 < p.count) {
      publish(p.published + (unsigned)j + 1);
      keep_transposed();
      // The partial sums have been read: the next step may overwrite them (FWD: advance() meets).  Two buffers in turn without this
      // barrier are slower, here and in chains: the waves that have no items ask for the next step sooner, and ask in vain (a gradient
      // step of H = 1024, B = 64 10.0 -> 10.5 ms, of H = 512, B = 256 104.6 -> 108.9).
      if constexpr (!FWD) lds_barrier();
      advance();
    }
  }
  keep_transposed();
  store_kept(p.s_hi - p.count + 1);
#pragma unroll
  for (int q = 0; q < IPT; ++q)
    if (real[q]) p.dc[(size_t)ie[q]] = dc_run[q];
}

template <class T, bool FWD, int NRT, int NXW, int NHW, int KSF, int NBW, int NBL, int KSB, int NBT, int CELL>
hipError_t launch_sweep_cell(const SweepParams& p, hipStream_t st) {
  constexpr int NTB = (NRT * 4 + 15) / 16, NB = NBT ? NBT : 1, IPT = (Items<NRT * 4, NBT ? NBT * 16 : 8, !FWD>::COUNT + 511) / 512;
  constexpr int GF = 8 / KSF, FTB = (GF == 2 && NBT == 2) ? 2 : 1, FTR = GF / FTB, BTB = (KSB == 4 && NBT == 2) ? 2 : 1;
  constexpr int blocksB = Sums<NTB, NBT == 0 ? 0 : NB / BTB>::BLOCKS, blocksF = Sums<(NRT + FTR - 1) / FTR, NBT == 0 ? 0 : NB / FTB>::BLOCKS;
  constexpr size_t lds = (size_t)8 * (blocksB + (FWD ? blocksF : 0) + NTB * NBL) * 1024 + (size_t)8 * IPT * SWEEP_KEPT * sizeof(T);
  static_assert(lds >= 8 * 1024 && lds <= 160 * 1024 - 64, "8 KiB for a workgroup that carries on slowly; LDS of a compute unit");
  hipError_t e = allow_dynamic_lds<sweep_kernel<T, FWD, NRT, NXW, NHW, KSF, NBW, NBL, KSB, NBT, CELL>>(lds);
  if (e != hipSuccess) return e;
  sweep_kernel<T, FWD, NRT, NXW, NHW, KSF, NBW, NBL, KSB, NBT, CELL><<<dim3(RES_WGS), dim3(512), lds, st>>>(p);
  return hipGetLastError();
}

struct SweepConfig {   // with forward operations: LSTM only
  int nrt, nxw, nhw, ksf, nbw, ksb, nbt;
  hipError_t (*launch)(const SweepParams&, hipStream_t);
};
#define MEBPTT_SWEEP(T, NRT, NXW, NHW, KSF, NBW, NBL, KSB, NBT) \
  SweepConfig{NRT, NXW, NHW, KSF, NBW, KSB, NBT, launch_sweep_cell<T, true, NRT, NXW, NHW, KSF, NBW, NBL, KSB, NBT, 0>}
struct BackSweepConfig {
  int nrt, nbw, ksb, nbt;
  hipError_t (*launch[2])(const SweepParams&, hipStream_t);   // by cell
};
#define MEBPTT_BACK_SWEEP(T, NRT, NBW, NBL, KSB, NBT)                                                     \
  BackSweepConfig{NRT, NBW, KSB, NBT, {launch_sweep_cell<T, false, NRT, 1, 1, 8, NBW, NBL, KSB, NBT, 0>, \
                                       launch_sweep_cell<T, false, NRT, 1, 1, 8, NBW, NBL, KSB, NBT, 1>}}
Table<SweepConfig> sweep_table_bf16();
Table<SweepConfig> sweep_table_fp32();
Table<BackSweepConfig> back_sweep_table_bf16();
Table<BackSweepConfig> back_sweep_table_fp32();

}  // namespace mebptt
