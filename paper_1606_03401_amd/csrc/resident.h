// Shared parts of the resident launches (forward chains and sweeps): placement of the workgroups, the
// exchange through an XCD's L2, and the kernel of the forward chain.  Not part of the ABI.
#pragma once

#include "device.h"
#include "dynamic_lds.h"

namespace mebptt {

// ---- where a resident workgroup runs ---------------------------------------------------------------
// The batch is split over the 8 XCDs, each with its own L2: XCD g takes the sequences [g*nb, (g+1)*nb)
// and never needs anything from another XCD.  Inside an XCD the 32 workgroups (one per compute unit)
// split the hidden units.  Which XCD a workgroup runs on is read from the hardware (register XCC_ID),
// not inferred from its id: workgroups are dealt round-robin to the XCDs, but where the deal starts
// depends on the launches before.  A workgroup takes the next free rank of its XCD from a counter; the
// launch relies on no XCD receiving more than 32 of the 256 workgroups, checks it (a rank counter that
// runs past 32 raises the status word) and gives up rather than compute on an assumption that does
// not hold.
//
// The workgroups of an XCD wait for each other, so all that have units (`producers`: the first ranks) have to
// be on the chip at once.  Work of somebody else -- another stream, a replayed graph, another process -- can keep
// some of them off it, and two resident launches can keep each other off for good.  A workgroup whose first
// exchange does not come within `patience` therefore gives the launch up for its XCD, in one atomic step on the
// rank word that only succeeds while producers are missing (then nobody can have got past the first exchange, and
// nothing a launch leaves behind has been written).  The others see it and leave, late ones leave at once, and
// the one that gave up runs all steps for the XCD's sequences alone: slow, but it waits for nobody, and its
// sums are formed in the same order.
constexpr int RES_WGS = 256, RES_GROUPS = 8, RES_MEMBERS = RES_WGS / RES_GROUPS;
constexpr int RES_RING = 4;   // exchange slots
// sync words of XCD g from [g * 64] on: the rank word (the counter in its low half, in its high half the launch given
// up last, + 1), the workgroups that have left that launch; the same two of group g of wide chains and of wide sweeps;
// status at [512]
constexpr int RES_SYNC_RANK = 0, RES_SYNC_LEFT = 2, RES_SYNC_CHAIN_GROUP = 4, RES_SYNC_SWEEP_GROUP = 8, RES_SYNC_STATUS = 512;

__device__ inline unsigned xcc_id() {
  unsigned v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & 0xf;
}

__device__ inline unsigned long long* rank_word(unsigned* sync, int g) {
  return reinterpret_cast<unsigned long long*>(sync + RES_SYNC_RANK + g * 64);
}

// One thread of a workgroup: draws the workgroup's rank on its XCD.  False: nothing to do here; the workgroups
// were not dealt 32 per XCD (the status word says so), or the XCD has given this launch up.
__device__ inline bool draw_rank(unsigned* sync, unsigned launch, int& g, int& rank) {
  const unsigned xcc = xcc_id();
  bool ok = xcc < (unsigned)RES_GROUPS;
  unsigned long long word = 0;
  if (ok) {
    word = __hip_atomic_fetch_add(rank_word(sync, (int)xcc), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ok = (unsigned)word / RES_MEMBERS == launch;   // more than 32 workgroups on this XCD: ranks would collide
  }
  if (!ok) __hip_atomic_store(sync + RES_SYNC_STATUS, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  g = ok ? (int)xcc : 0;
  rank = (int)((unsigned)word % RES_MEMBERS);
  return ok && (unsigned)(word >> 32) != launch + 1;
}

// ---- the exchange ------------------------------------------------------------------------------------
// What a step publishes goes into one of RES_RING slots that hold the consumer's operand layout.  There
// is no counter: a slot starts out filled with the bit pattern EMPTY, and a wave that needs operand
// fragments fetches them until none of the dwords it got is EMPTY.  (A bf16 pair or an fp32 value of
// that pattern is a NaN with all payload bits set; a producer publishes it as the NaN next to it.)  A
// step thus costs one store and one load through the L2 the XCD's compute units share, where a counter
// costs the store, its acknowledgement, a barrier, an atomic, a load of the counter, a barrier and the
// fetch one after the other.  A wave waits for the producers of its own part of K only.  Measured, this
// exchange against the counters, whole gradient steps: H = 1024, B = 64 chains 14.8 -> 12.9 ms, sweeps
// 12.9 -> 12.1 ms; H = 512, B = 256 163.5 -> 126.9 -> 109.5 ms; H = 256, B = 64 3.61 -> 2.86 -> 2.03 ms.
//
// Slots are recycled in order: step q goes to slot q mod 4.  Whoever publishes step q has fetched all
// of step q - 1, whose producers had fetched all of step q - 2: nobody reads q - 2 any more, and the
// publisher resets its own part of that slot to EMPTY right after publishing q.  The next use of the slot
// is step q + 2; a reader polls it only after it has seen the publisher's q + 1, which the publisher
// stores after it waited for loads issued behind the reset (memory operations of a wave complete in
// order), so the reset is visible before anyone can look.  Step numbers run on from launch to launch
// of a run, so the slots a launch starts with are the ones the launch before left reset.
constexpr unsigned RES_EMPTY = 0xffffffffu;

// A wave's 16 bytes per lane of an exchange slot: past the compute unit's vector cache (sc1), from the
// XCD's L2.  byte_off at or above 2^31 lies outside the buffer: such a lane gets zeros and moves no data.
constexpr unsigned RES_NO_LANE = 0x80000000u;
__device__ inline u32x4 load_slot_16(const void* slot, unsigned byte_off, int uniform_off) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(slot), 0, 0x7fffffff, 0x00020000);
  return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte_off, uniform_off, 16 /* sc1: agent scope */);
}
__device__ inline unsigned largest_dword(u32x4 v) { return max(max(v.x, v.y), max(v.z, v.w)); }
__device__ inline unsigned not_empty(unsigned v) { return min(v, RES_EMPTY - 1u); }   // for a value about to be published

// The bound of a wait: true when it is time to stop waiting, or a launch of the run has failed.
struct WaitBound {
  long long ticks;      // of the 100 MHz wall clock; 0: stop after one look
  unsigned* status;
  int polls = 0;
  long long t0 = 0;
  __device__ bool expired() {
    if (ticks != 0 && (++polls & 15) != 0) return false;
    const long long now = wall_clock64();
    if (t0 == 0) t0 = now;
    return now - t0 >= ticks || __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
  }
};

// The kernel's arguments (it has one, a struct) once more, by an address the compiler cannot see through: what only
// a workgroup that has stopped waiting reads is not fetched ahead, and kept in registers, for the others.
template <class P>
__device__ __forceinline__ const __attribute__((address_space(4))) P* arguments_again() {
  auto* p = (const __attribute__((address_space(4))) P*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// Where a workgroup's waves go, all of them, when one has stopped waiting (*s_fail: 1 + the step).  There is no way
// back into the loop over the steps, and none to the kernel's end: an exit that rejoined either had the
// compiler copy what the loop carries and wait for the step's stores, in every step (H = 512, B = 256
// 3 - 9 % slower); for the same reason it takes nothing along but LDS.  carry_on: all steps once more, slowly -- for
// all units of the XCD's sequences where this workgroup has given the launch up, for its own UW where all
// producers have turned out to be here after all.
template <class P, int UW, class CarryOn>
__device__ __forceinline__ void stop_waiting(const int* s_g, const int* s_rank, int* s_fail, CarryOn&& carry_on) {
  const auto& p = *arguments_again<P>();
  const int g = __builtin_amdgcn_readfirstlane(*s_g), rank = __builtin_amdgcn_readfirstlane(*s_rank);
  const int units = units_of(p), producers = (units + UW - 1) / UW;
  unsigned* sync = p.sync;
  unsigned* left = sync + RES_SYNC_LEFT + g * 64;
  __threadfence();   // the workgroup's own stores are done when it says that it leaves
  __syncthreads();
  if (threadIdx.x == 0) {
    enum { LEAVE, ALONE, TOGETHER };
    int role = LEAVE;
    bool ok = *s_fail == 1 && p.wait_ticks != 0 && __hip_atomic_load(sync + RES_SYNC_STATUS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u;
    if (ok && p.alone) {
      role = ALONE;
    } else if (ok) {
      unsigned long long* word = rank_word(sync, g);
      unsigned long long v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned here = 0;
      while (role == LEAVE && (unsigned)(v >> 32) != p.launch + 1) {
        here = (unsigned)v - p.launch * RES_MEMBERS;
        if ((int)here >= producers)
          role = TOGETHER;
        else if (__hip_atomic_compare_exchange_strong(word, &v, (unsigned long long)(p.launch + 1) << 32 | (unsigned)v, __ATOMIC_RELAXED,
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
          role = ALONE;
      }
      if (role == LEAVE) __hip_atomic_fetch_add(left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (role == ALONE) {   // those who are here see it, and leave
        WaitBound bound{p.wait_ticks, sync + RES_SYNC_STATUS};
        while (ok && __hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != here - 1) ok = !bound.expired();
        __hip_atomic_store(left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
      }
    }
    if (!ok) __hip_atomic_store(sync + RES_SYNC_STATUS, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_fail = ok ? role : (int)LEAVE;
  }
  __threadfence();
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(*s_fail);
  __syncthreads();
  if (role != 0) {
    if (threadIdx.x == 0) *s_fail = 0;
    carry_on(g * p.nb, min(p.B, (g + 1) * p.nb), role == 1 ? 0 : rank * UW, role == 1 ? units : min((rank + 1) * UW, units));
  }
  __builtin_amdgcn_endpgm();
}
// For carry_on, all threads, before a step: waits until the exchange slot is there, `pieces` fragments of each of the
// XCD's batch tiles, off: this lane's offset in a tile.  False: it does not come (the status word says so).
template <class Off>
__device__ __forceinline__ bool slot_is_there(const void* slot, int pieces, int tiles, Off&& off, long long wait_ticks, unsigned* status,
                                              int* s_fail) {
  __threadfence();   // what this workgroup's waves have stored for the step can be fetched
  __syncthreads();
  WaitBound bound{wait_ticks, status};
  for (int m = (int)(threadIdx.x >> 6); m < pieces; m += (int)(blockDim.x >> 6))
    for (int t = 0; t < tiles; ++t)
      while (__builtin_amdgcn_ballot_w64(largest_dword(load_slot_16(slot, off(t), m * 1024)) == RES_EMPTY) != 0) {
        if (bound.expired()) {
          __hip_atomic_store(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          *s_fail = 1;
          break;
        }
        asm volatile("" ::: "memory");   // the next look is another load
      }
  __syncthreads();
  return *s_fail == 0;
}

// h of one element in full precision, and as the GEMM operand: `e` = b * H + u (plain plane), `o` its place
// in a split plane of `half` elements per 16-bit plane.
template <class T>
__device__ inline float load_h(const float* plane, unsigned e, unsigned o, size_t half) {
  if constexpr (HPlane<T>::SPLIT) {
    const unsigned short* hi = reinterpret_cast<const unsigned short*>(plane);
    const unsigned lo = (hi + half)[(size_t)o];
    return __uint_as_float((((unsigned)hi[(size_t)o] - (lo >> 15)) << 16) | lo);
  } else {
    return plane[(size_t)e];
  }
}
template <class T>
__device__ inline float load_h_operand(const float* plane, unsigned e, unsigned o) {
  if constexpr (HPlane<T>::SPLIT)
    return (float)reinterpret_cast<const T*>(plane)[(size_t)o];
  else
    return plane[(size_t)e];
}

// ---- columns, items, partial sums ----------------------------------------------------------------------
// Column c of the MFMA tiles is sequence b_lo + c of the XCD's share.  NBT is the number of 16-column tiles of
// the share; NBT = 0 stands for half a tile, 8 sequences.
//
// The pointwise work of a workgroup -- UW units x the XCD's sequences -- is dealt to its threads in blocks
// of 64.  BLOCK order: WU units x 64/WU sequences (WU = 8, or 4 where UW is no multiple of 8), unit fastest: every
// array a wave touches falls into runs of at least 32 bytes, and the fragment-tiled ones into whole cache lines.
// Otherwise the MFMA's own order, sequence fastest: 4 units x 16 sequences (8 x 8 on half a tile).  The difference is in plain planes: 16 rows of
// 16 bytes per instruction keep a compute unit's address path busy so long that the twenty such
// loads and stores of a backward step took three times as long as the MFMAs beside them.
// Either way the blocks of one group of units follow each other (columns outermost: a chain launch of H = 1024, B = 64
// 85.5 -> 90.6 us).  BLOCK order for every plane, split ones too, was 2 % slower on H = 512, B = 256.
template <int UW, int COLUMNS, bool BLOCK>
struct Items {
  static constexpr int WU = (BLOCK || COLUMNS == 8) && UW % 8 == 0 ? 8 : 4, WB = 64 / WU;   // units, sequences of a block
  static constexpr int DOWN = (COLUMNS + WB - 1) / WB, COUNT = UW / WU * DOWN * 64;   // blocks of one group of units; items
  __device__ static int unit_in(int item) { return BLOCK ? item & (WU - 1) : (item & 63) / WB; }
  __device__ static int row_in(int item) { return BLOCK ? (item & 63) / WU : item & (WB - 1); }
  // unit (of the workgroup) and column of an item
  __device__ static int unit(int item) { return (item >> 6) / DOWN * WU + unit_in(item); }
  __device__ static int column(int item) { return (item >> 6) % DOWN * WB + row_in(item); }
};

// Partial sums meet in LDS as the MFMA leaves them: blocks of 64 lanes x 4 consecutive rows.  Writing one costs a
// compute unit 31 cycles whatever its lanes hold (reading one 17), which at 64 blocks a step was more than
// the MFMAs; with half a tile of sequences, two row tiles share a block: the second one's sums take the
// place of the first one's empty columns (with the items dense, H = 1024, B = 64 12.14 -> 11.04 ms a gradient
// step; H = 650, B = 20 2.50 -> 2.13 ms).  Rows permuted against bank conflicts lost 5 % on H = 512, B = 256.
__device__ inline f32x4 join_halves(f32x4 a, f32x4 b) {
  f32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i)   // lanes 8-15 of every 16 take b from lanes 0-7
    r[i] = __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(a[i]), __float_as_uint(b[i]), 0x128 /* row_ror:8 */, 0xf, 0xc, false));
  return r;
}
// Two row tiles of Halves products, whose rows are the gates 0 and 1 of eight units (lanes j: gate j / 8, unit j % 8), and the
// gates 2 and 3: lane (j, lq) gets all four gates of unit j % 8 for sequence 4 (lq & 1) + 2 (lq >> 1) + j / 8.
__device__ inline f32x4 join_gates(const Halves::Sum& a, const Halves::Sum& b) {
  auto dpp = [](float own, float other, auto banks) {   // lanes of these banks of four take the value eight lanes on
    return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(own), __float_as_uint(other), 0x128 /* row_ror:8 */, 0xf, decltype(banks)::value, false));
  };
  using upper = std::integral_constant<int, 0xc>;
  using lower = std::integral_constant<int, 0x3>;
  return f32x4{dpp(a.v[0], a.v[1], upper{}), dpp(a.v[1], a.v[0], lower{}), dpp(b.v[0], b.v[1], upper{}), dpp(b.v[1], b.v[0], lower{})};
}
// Blocks a wave writes for its NR row tiles x NB batch tiles, and the block and lane of (row tile, row group lq, column).
template <int NR, int NBT>
struct Sums {
  static constexpr bool HALF = NBT == 0;
  static constexpr int NB = HALF ? 1 : NBT, BLOCKS = HALF ? (NR + 1) / 2 : NR * NB;
  __device__ static int block(int tile, int column) { return HALF ? tile >> 1 : tile * NB + (column >> 4); }
  __device__ static int lane(int tile, int lq, int column) { return lq * 16 + (HALF ? ((tile & 1) << 3) + column : column & 15); }
  template <class Acc>
  __device__ static void write(f32x4* red, int lane, const Acc& acc) {
    if constexpr (HALF) {
#pragma unroll
      for (int t = 0; t < NR; t += 2) red[(t / 2) * 64 + lane] = t + 1 < NR ? join_halves(acc[t][0], acc[t + 1 < NR ? t + 1 : t][0]) : acc[t][0];
    } else {
#pragma unroll
      for (int t = 0; t < NR; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b) red[(t * NB + b) * 64 + lane] = acc[t][b];
    }
  }
};

// ---- forward chain -------------------------------------------------------------------------------------
struct ResStep {
  float* out;     // unit that receives (h, c) of this step, or NULL
  float* gates;   // two units that receive (i, f), (g, o), or NULL
};
constexpr int RES_MAX_STEPS = 192;  // steps of one launch: their destinations travel as kernel arguments (3 KiB of the 4 KiB there are)
struct ResParams {
  static constexpr int RING = RES_RING;
  const void* Wp;
  const float* bp;
  const float* x0;     // x of the first step of this launch
  const float* src;    // unit holding the input state of the first step
  void* ring;          // RES_RING slots [BP][KH] of GEMM operands, fragment-tiled
  float* spare;        // [B][H]: the state that stays in registers, where a workgroup carries on slowly
  unsigned* sync;
  unsigned published;  // states published by this run's chain launches before this one
  unsigned launch;     // resident launches of this run before this one (every rank counter stands at 32 * launch)
  long long wait_ticks;   // bound of every wait, in ticks of the 100 MHz wall clock
  long long patience;     // bound of the first one: then the launch may be given up
  int alone;              // only rank 0 of each XCD runs, and carries on alone
  int count;
  int B, I, H, HP, KX, KH, BP, nb;
  size_t unit, hplane; // floats per unit, floats of its h part
  ResStep step[RES_MAX_STEPS];
};
__device__ inline int units_of(const __attribute__((address_space(4))) ResParams& p) { return p.KH; }   // dealt out among an XCD's workgroups

// Gate sums of 16 packed rows (units 4 * tile .. + 3) and 16 sequences, by one wave on its own, for workgroups
// that carry on slowly: the KS partial sums of the cooperating waves one beside the other, added in their order.
// load_h(m): this lane's h fragment of macro step m.  Two loops over K, four macro steps in flight (eight would
// set the register count of the smaller instantiations, and two launches of those fit the chip together); steps
// outside a loop's range run on zeros.
template <class T, int KS, class LoadH>
__device__ __forceinline__ void gates_slowly(const void* Wp, int tile, const float* x, unsigned xrow, int I, int nsx, int nsh, LoadH&& load_h,
                                   float (&G)[4]) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, FRAG = 64 * VEC;
  const int lane = threadIdx.x & 63, lq = lane >> 4, nsteps = nsx + nsh;
  const T* base = reinterpret_cast<const T*>(Wp) + ((size_t)tile * nsteps * 64 + lane) * VEC;
  f32x4 acc[KS];
#pragma unroll
  for (int w = 0; w < KS; ++w) acc[w] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < nsx; s0 += KS) {
#pragma unroll
    for (int w0 = 0; w0 < KS; w0 += 4) {
      typename M::Frag a[4];
      RawAct<VEC> raw[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        a[w] = M::load(base + (size_t)min(s0 + w0 + w, nsx - 1) * FRAG);
        raw[w] = load_window<VEC>(x, xrow, (s0 + w0 + w) * KSTEP + VEC * lq, I);
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (s0 + w0 + w >= nsx) a[w] = typename M::Frag{};
        shift_tail<VEC>(raw[w], (s0 + w0 + w) * KSTEP + VEC * lq, I);
        acc[w0 + w] = M::mma(a[w], M::from_f32(raw[w].v), acc[w0 + w]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  for (int s0 = nsx / KS * KS; s0 < nsteps; s0 += KS) {
#pragma unroll
    for (int w0 = 0; w0 < KS; w0 += 4) {
      typename M::Frag a[4], f[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int s = min(max(s0 + w0 + w, nsx), nsteps - 1);
        a[w] = M::load(base + (size_t)s * FRAG);
        f[w] = load_h(s - nsx);
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (s0 + w0 + w < nsx || s0 + w0 + w >= nsteps) a[w] = f[w] = typename M::Frag{};
        acc[w0 + w] = M::mma(a[w], f[w], acc[w0 + w]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) G[r] = 0.0f;
  if constexpr (parts_in_pairs<T, KS>) {
    add_pairs<KS>(G, [&](int w) { return acc[w]; });
  } else {
#pragma unroll
    for (int w = 0; w < KS; ++w)
#pragma unroll
      for (int r = 0; r < 4; ++r) G[r] += acc[w][r];
  }
}

// All steps of a launch for units [u0, u1) of the XCD's sequences, by a workgroup that has stopped waiting.  Its waves
// deal the units out four at a time; the state that stays in registers in a chain goes through `spare`, and the
// weights are fetched again in every step.
template <class P, class T, int KS, int CELL>
__device__ __forceinline__ void chain_slowly(int b_lo, int b_hi, int u0, int u1, int* s_fail) {
  const auto& p = *arguments_again<P>();
  const int deal = (int)(blockDim.x >> 6) * 4;   // units the workgroup's waves take at a time
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC;
  constexpr bool SPLIT = HPlane<T>::SPLIT;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int lrow = lane & 15, lq = lane >> 4;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP;
  const size_t hhalf = (size_t)p.BP * p.KH;
  const unsigned plane = (unsigned)(p.B * p.H);
  auto slot = [&](unsigned q) { return reinterpret_cast<T*>(p.ring) + (size_t)(q % P::RING) * hhalf; };
  auto off = [&](int t) {
    const int b = b_lo + t * 16 + lrow;
    return b < b_hi ? (unsigned)(((b >> 4) * nsh * 64 + lq * 16 + (b & 15)) * 16) : RES_NO_LANE;
  };
  auto publish = [&](unsigned q, int b, int u, float h) {   // as in a chain; all lanes
    const size_t o = ft_offset<T>(b, u, nsh);
    unsigned *to = reinterpret_cast<unsigned*>(slot(q)), *old = reinterpret_cast<unsigned*>(slot(q + P::RING - 2));
    if constexpr (SPLIT) {
      const unsigned hi16 = (__float_as_uint(h) + 0x8000u) >> 16;
      const auto rows = __builtin_amdgcn_permlane16_swap(hi16, hi16, false, false);
      if (b < b_hi && (lq & 1) == 0) {
        to[o >> 1] = not_empty(rows[0] | (rows[1] << 16));
        old[o >> 1] = RES_EMPTY;
      }
    } else if (b < b_hi) {
      to[o] = not_empty(__float_as_uint(h));
      old[o] = RES_EMPTY;
    }
  };
  for (int u4 = u0 + 4 * wave; u4 < u1; u4 += deal)
    for (int c = b_lo; c < b_hi; c += 16) {
      const int b = c + lrow, u = u4 + lq;
      float h = 0.0f;
      if (b < b_hi && u < p.H) {
        h = HPlane<T>::load(p.src, b, u, p.KH / 32, p.H, hhalf);
        p.spare[(size_t)b * p.H + u] = CELL ? h : (p.src + p.hplane)[(size_t)b * p.H + u];
      }
      publish(p.published, b, u, h);
    }
  for (int j = 0; j < p.count; ++j) {
    const T* in = slot(p.published + (unsigned)j);
    if (!slot_is_there(in, nsh, (b_hi - b_lo + 15) / 16, off, p.wait_ticks, p.sync + RES_SYNC_STATUS, s_fail)) return;
    float *dst = p.step[j].out, *gates = p.step[j].gates;
    for (int u4 = u0 + 4 * wave; u4 < u1; u4 += deal)
      for (int c = b_lo; c < b_hi; c += 16) {
        const int b = c + lrow, u = u4 + lq;
        const bool own = b < b_hi, real = own && u < p.H;
        const unsigned hoff = off((c - b_lo) / 16);
        float G[4] = {0.f, 0.f, 0.f, 0.f}, second = 0.0f, gate[4], h = 0.0f;
        if (u4 < p.HP)
          gates_slowly<T, KS>(p.Wp, u4 / 4, p.x0 + (size_t)j * p.B * p.I, (unsigned)((own ? b : b_lo) * p.I), p.I, nsx, nsh,
                              [&](int m) { return as_frag<typename M::Frag>(load_slot_16(in, hoff, m * 1024)); }, G);
        const size_t e = (size_t)b * p.H + u, o = ft_offset<T>(b, u, nsh);
        if (real) {
          h = cell_forward<T, CELL>(G, *reinterpret_cast<const float4*>(p.bp + 4 * u), p.spare[e], second, gate);
          p.spare[e] = CELL ? h : second;
          if (dst) (dst + p.hplane)[e] = second;
          if (gates) {
            gates[e] = gate[0];
            (gates + plane)[e] = gate[1];
            (gates + p.unit)[e] = gate[2];
            if (CELL == 0) (gates + p.unit + plane)[e] = gate[3];
          }
        }
        if (j + 1 < p.count) publish(p.published + (unsigned)j + 1, b, u, h);
        if (dst && own) {
          if constexpr (SPLIT) {
            unsigned short* hi = reinterpret_cast<unsigned short*>(dst);
            hi[o] = (unsigned short)((__float_as_uint(h) + 0x8000u) >> 16);
            (hi + hhalf)[o] = (unsigned short)(__float_as_uint(h) & 0xffffu);
          } else if (real) {
            dst[e] = h;
          }
        }
      }
  }
}

// Consecutive forward operations (Algorithm 2's forward loop; also the single-step pushes that
// follow each other when memory is plentiful) depend on each other only through h, so a chain of
// them can run inside ONE launch if the gate weights stay on the chip and only h travels.
// Workgroup `rank` of an XCD owns the NRT * 4 units from rank * NRT * 4 on and keeps their packed weight
// rows in registers (and a part in LDS) for the whole launch.  Its 8 waves split K KS ways; where
// KS = 4 the two halves of the workgroup take a batch tile each, or half of the row tiles.  The input
// state of the first step is published like any other, so all steps are alike:
//   1. the x part of the gate GEMM (fetched a step ahead), which needs nothing from other workgroups;
//   2. fetch h_{s-1} of the XCD's sequences from the exchange slot until all of it is there;
//   3. store what the step before has to keep, and fetch the next x: issued here they complete behind
//      the MFMAs.  Memory operations complete in order, so anything issued in front of the polls
//      would hold them up;
//   4. the h part of the GEMM, partial sums through LDS, the pointwise step (c, or the GRU's h, stays in a
//      register), publish h_s.
// What bounds a step is this chain of latencies, not bytes or flops: no weight moves.  Measured per step,
// with counters and whole tiles before and so: H = 1024, B = 64 3.3 -> 2.27 us, H = 512, B = 256 3.6 -> 1.98 us.
// Of those 2.27 us (whole tiles' products and gate functions with divisions; now see halves_from), in cycles of 2.2 GHz: x part 560, polls 620 - 820 (1.0 - 1.4 of them), h part with the
// stores and the next x 1280, barrier 250 - 520, pointwise step 1050, publishing 170.
// Sums are formed exactly as forward_body forms them (KS partial sums over the macro steps
// w, w+KS, ..., added in order, or as add_pairs adds them), so a step gives the same bits either way.  A wave whose part of
// x or h is shorter than the others' runs its surplus macro steps on zeros.
// Up to 64 sequences (half tiles), bf16, K split eight ways: each instruction does two of the eight parts (Halves), so four waves
// split K and the two halves of the workgroup take half of the units each, in pairs of row tiles that hold eight units.  Against
// eight waves with a part and all rows each: half the matrix instructions, half the partial sums through LDS (a 1 KiB block
// costs a compute unit 30 cycles to write and 17 to read, and there were 32; the matrix unit was busy for 1024 of the h part's 1280 cycles):
// H = 1024, B = 64 85.7 -> 79.4 us a launch of 41 steps on average.  Fetching the weights takes longer that way (a load takes 32
// bytes of each line for 128), see halves_from.
// NXW, NHW: macro steps of x and of h per wave (Halves: per part); the weights of the last NXL of x are parked in LDS (they are
// read while the wave would wait anyway); NBT: batch tiles of the XCD's share (0: half a tile).
template <int NRT, int KS, int NBT, bool HALVES>   // row tiles of a wave
constexpr int chain_row_tiles = HALVES || (KS == 4 && NBT != 2) ? (NRT + 1) / 2 : NRT;
template <class T, int NRT, int NXW, int NXL, int NHW, int KS, int NBT, int CELL, bool HALVES>
__global__ __launch_bounds__(512) void forward_chain_kernel(ResParams p) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, FRAG = 64 * VEC;
  constexpr int KW = HALVES ? KS / 2 : KS;         // waves that split K
  constexpr int GROUPS = 8 / KW, FTB = (GROUPS == 2 && NBT == 2) ? 2 : 1, FTR = GROUPS / FTB;
  constexpr int NRTW = chain_row_tiles<NRT, KS, NBT, HALVES>, BTW = (NBT ? NBT : 1) / FTB;   // row and batch tiles of one wave
  using Weights = std::conditional_t<HALVES, bf16x16, typename M::Frag>;
  constexpr int NXR = NXW - NXL, COLS = NBT ? NBT * 16 : 8;
  constexpr int UW = NRT * 4;
  using It = Items<UW, COLS, NBT == 0>;
  constexpr int ITEMS = It::COUNT, IPT = (ITEMS + 511) / 512;
  using Sum = Sums<NRTW, NBT == 0 ? 0 : BTW>;
  constexpr bool SPLIT = HPlane<T>::SPLIT;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f32x4* red = reinterpret_cast<f32x4*>(smem);                                     // [8 waves][Sum::BLOCKS][64]
  T* wl = reinterpret_cast<T*>(red + 8 * Sum::BLOCKS * 64);                        // [8][NRTW][NXL] fragments (Halves: of two macro steps)
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
  if (b_lo >= p.B || rank * UW >= p.KH || (p.alone && rank)) return;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP, nsteps = nsx + nsh;
  const size_t hhalf = (size_t)p.BP * p.KH;
  const int ks = wave % KW, grp = wave / KW;
  const int rt0 = (FTR > 1 ? grp : 0) * NRTW, bt0 = (FTB > 1 ? grp : 0) * BTW;   // wave = group * KW + K part
  const int ngroups = p.HP / 4;                    // 16-row tiles of the packed weights
  // this wave's part of K (Halves: this lane's of the two); its h macro steps: mh0, mh0 + KS, ... (below nsh)
  const int kpart = HALVES ? 2 * ks + (lrow >> 3) : ks;
  const int mh0 = (kpart + KS - nsx % KS) % KS;

  // Pointwise items of this thread; c stays in registers.  A unit between H and the padded KH has no
  // weights: its h is zero, and is published as such.
  bool mine[IPT], real[IPT];
  unsigned ie[IPT], io[IPT];   // b * H + u; the element's place in a fragment-tiled plane
  const f32x4* cell[IPT];      // its gate sums of K part 0
  float4 bias[IPT];
  float c_state[IPT], keep_h[IPT], keep_second[IPT], keep_gate[IPT][4];
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const int item = (int)threadIdx.x + q * 512;
    const int ul = It::unit(item), col = It::column(item), b = b_lo + col, u = rank * UW + ul, rt = ul >> 2;
    // the wave that holds it: row group (or batch group) of the workgroup, then its block
    const int w0 = FTR > 1 ? rt / NRTW : (FTB > 1 ? (col >> 4) / BTW : 0);
    if constexpr (HALVES)
      cell[q] = red + (size_t)(w0 * KW * Sum::BLOCKS + rt % NRTW / 2) * 64 + Halves::lane_of((ul & 7) + 8 * (col & 1), col);
    else
      cell[q] = red + (size_t)(w0 * KS * Sum::BLOCKS + Sum::block(FTR > 1 ? rt % NRTW : rt, FTB > 1 ? col % (BTW * 16) : col)) * 64 +
                Sum::lane(FTR > 1 ? rt % NRTW : rt, ul & 3, col);
    mine[q] = item < ITEMS && b < b_hi && u < p.KH;
    real[q] = u < p.H;
    ie[q] = (unsigned)(b * p.H + u);
    io[q] = (unsigned)ft_offset<T>(b, u, nsh);
    bias[q] = float4{0.f, 0.f, 0.f, 0.f};
    c_state[q] = keep_h[q] = 0.0f;
    if (mine[q] && real[q]) {
      bias[q] = *reinterpret_cast<const float4*>(p.bp + 4 * u);
      keep_h[q] = HPlane<T>::load(p.src, b, u, p.KH / 32, p.H, hhalf);
      // the state the pointwise step blends with, kept in this register from step to step:
      // c_{s-1} (LSTM) or h_{s-1} in full precision (GRU)
      c_state[q] = CELL ? keep_h[q] : (p.src + p.hplane)[(size_t)ie[q]];
    }
  }
  // publishes keep_h as step number `q_now` and resets this thread's part of the slot two steps back
  auto publish = [&](unsigned q_now) {
    unsigned* slot_out = reinterpret_cast<unsigned*>(reinterpret_cast<T*>(p.ring) + (size_t)(q_now % RES_RING) * hhalf);
    unsigned* slot_old = reinterpret_cast<unsigned*>(reinterpret_cast<T*>(p.ring) + (size_t)((q_now + 2) % RES_RING) * hhalf);
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      if constexpr (SPLIT) {
        // the lane of an even unit stores it and the next one as one dword: its neighbour's, or 16 lanes on
        const unsigned hi16 = (__float_as_uint(keep_h[q]) + 0x8000u) >> 16;
        unsigned pair;
        if constexpr (NBT == 0) {
          pair = hi16 | (__builtin_amdgcn_update_dpp(hi16, hi16, 0xb1 /* quad_perm 1,0,3,2 */, 0xf, 0xf, false) << 16);
        } else {
          const auto rows = __builtin_amdgcn_permlane16_swap(hi16, hi16, false, false);   // even rows of 16 lanes, odd rows
          pair = rows[0] | (rows[1] << 16);
        }
        if ((io[q] & 1) == 0) {
          slot_out[(size_t)(io[q] >> 1)] = not_empty(pair);
          slot_old[(size_t)(io[q] >> 1)] = RES_EMPTY;
        }
      } else {
        slot_out[(size_t)io[q]] = not_empty(__float_as_uint(keep_h[q]));
        slot_old[(size_t)io[q]] = RES_EMPTY;
      }
    }
  };
  publish(p.published);   // travels while the weights are fetched

  // this wave's packed weight rows; the last NXL macro steps of x are parked in LDS (read back by this wave only)
  Weights wx[NRTW][NXR > 0 ? NXR : 1], wh[NRTW][NHW];
  if constexpr (HALVES) {
    const int me = (2 * ks + KS - nsx % KS) % KS, mo = (2 * ks + 1 + KS - nsx % KS) % KS;   // the two parts' first macro steps of h
#pragma unroll
    for (int rt = 0; rt < NRTW; ++rt) {
      // lane j of tile rt: unit j % 8 of the pair of tiles, gate 2 * (rt % 2) + j / 8; packed row 4 * unit + gate
      const int row = 4 * (lrow & 7) + 2 * (rt & 1) + (lrow >> 3);
      const int row_tile = min(rank * NRT + min(rt0 + (rt & ~1) + (row >> 4), NRT - 1), ngroups - 1);
      const unsigned at = (unsigned)((row_tile * nsteps * 64 + (row & 15)) * 16);
#pragma unroll
      for (int i = 0; i < NXW; ++i) {
        const bf16x16 f = Halves::load(p.Wp, at, 2 * ks + KS * i, 2 * ks + 1 + KS * i, nsx, lq);
        if (i < NXR) {
          wx[rt][i < NXR ? i : 0] = f;
        } else {
          typename M::Frag* to = reinterpret_cast<typename M::Frag*>(wl) + ((size_t)(wave * NRTW + rt) * NXL + (i - NXR)) * 128 + lane;
          to[0] = __builtin_shufflevector(f, f, 0, 1, 2, 3, 4, 5, 6, 7);
          to[64] = __builtin_shufflevector(f, f, 8, 9, 10, 11, 12, 13, 14, 15);
        }
      }
#pragma unroll
      for (int i = 0; i < NHW; ++i) wh[rt][i] = Halves::load(p.Wp, at, nsx + me + KS * i, nsx + mo + KS * i, nsteps, lq);
    }
  } else {
#pragma unroll
    for (int rt = 0; rt < NRTW; ++rt) {
      const int row_tile = min(rank * NRT + min(rt0 + rt, NRT - 1), ngroups - 1);
      const T* base = reinterpret_cast<const T*>(p.Wp) + ((size_t)row_tile * nsteps * 64 + lane) * VEC;
#pragma unroll
      for (int i = 0; i < NXW; ++i) {
        const int s = ks + KS * i;
        typename M::Frag f = M::load(base + (size_t)min(s, nsx - 1) * FRAG);
        if (s >= nsx) f = typename M::Frag{};
        if (i < NXR)
          wx[rt][i < NXR ? i : 0] = f;
        else
          *reinterpret_cast<typename M::Frag*>(&wl[((size_t)(wave * NRTW + rt) * NXL + (i - NXR)) * FRAG + lane * VEC]) = f;
      }
#pragma unroll
      for (int i = 0; i < NHW; ++i) {
        const int m = mh0 + KS * i;
        wh[rt][i] = M::load(base + (size_t)(nsx + min(m, nsh - 1)) * FRAG);
        if (m >= nsh) wh[rt][i] = typename M::Frag{};
      }
    }
  }

  // where this lane's operands come from: x rows, exchange-slot offsets (fragment 0 of each batch tile).
  // Columns of a tile that belong to no sequence of this XCD read the first one's x and fetch no h.
  unsigned xrow[BTW], hoff[BTW];
#pragma unroll
  for (int t = 0; t < BTW; ++t) {
    const int b = b_lo + (bt0 + t) * 16 + (HALVES ? lrow & 7 : lrow);
    const bool own = b < b_hi;
    xrow[t] = (unsigned)((own ? b : b_lo) * p.I);
    hoff[t] = own ? (unsigned)(((b >> 4) * nsh * 64 + lq * 16 + (b & 15)) * 16) : RES_NO_LANE;
  }
  RawAct<VEC> xraw[NXW][BTW];   // x of the step about to run
  auto fetch_x = [&](int j) {
    const float* x_j = p.x0 + (size_t)j * p.B * p.I;
#pragma unroll
    for (int i = 0; i < NXW; ++i)
#pragma unroll
      for (int t = 0; t < BTW; ++t) xraw[i][t] = load_window<VEC>(x_j, xrow[t], (kpart + KS * i) * KSTEP + VEC * lq, p.I);
  };
  fetch_x(0);

  auto store_kept = [&](int j) {   // what the schedule wants of step j
    const ResStep dst = p.step[j];
    if (!dst.out && !dst.gates) return;
    const unsigned plane = (unsigned)(p.B * p.H);
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      if (dst.out) {
        if constexpr (SPLIT) {   // padding columns of a split h plane are part of the operand other launches fetch: zero
          unsigned short* hi = reinterpret_cast<unsigned short*>(dst.out);
          const unsigned bits = __float_as_uint(keep_h[q]);
          hi[(size_t)io[q]] = (unsigned short)((bits + 0x8000u) >> 16);
          (hi + hhalf)[(size_t)io[q]] = (unsigned short)(bits & 0xffffu);
        } else if (real[q]) {
          dst.out[(size_t)ie[q]] = keep_h[q];
        }
        if (real[q]) (dst.out + p.hplane)[(size_t)ie[q]] = keep_second[q];
      }
      if (dst.gates && real[q]) {
        dst.gates[(size_t)ie[q]] = keep_gate[q][0];
        (dst.gates + plane)[(size_t)ie[q]] = keep_gate[q][1];
        (dst.gates + p.unit)[(size_t)ie[q]] = keep_gate[q][2];
        if (CELL == 0) (dst.gates + p.unit + plane)[(size_t)ie[q]] = keep_gate[q][3];
      }
    }
  };

  const int picks = Halves::picks(lane);
  auto mma = [&](const Weights& w, const typename M::Frag& f, f32x4 c) {
    if constexpr (HALVES)
      return Halves::mma(f, w, c, picks);
    else
      return M::mma(w, f, c);
  };
  for (int j = 0; j < p.count; ++j) {
    f32x4 acc[NRTW][BTW];
#pragma unroll
    for (int rt = 0; rt < NRTW; ++rt)
#pragma unroll
      for (int t = 0; t < BTW; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the x part (a wave's x macro steps precede its h macro steps, so the order of the additions is
    // that of forward_body)
#pragma unroll
    for (int i = 0; i < NXW; ++i) {
      const int s = kpart + KS * i;
      if (((HALVES ? 2 * ks + 1 + KS * i : s) + 1) * KSTEP > p.I) {   // over the end of the row, or a surplus step
#pragma unroll
        for (int t = 0; t < BTW; ++t) shift_tail<VEC>(xraw[i][t], s * KSTEP + VEC * lq, p.I);
      }
      typename M::Frag xf[BTW];
#pragma unroll
      for (int t = 0; t < BTW; ++t) xf[t] = M::from_f32(xraw[i][t].v);
#pragma unroll
      for (int rt = 0; rt < NRTW; ++rt) {
        Weights a;
        if (i < NXR) {
          a = wx[rt][i < NXR ? i : 0];
        } else if constexpr (HALVES) {
          const typename M::Frag* from = reinterpret_cast<const typename M::Frag*>(wl) + ((size_t)(wave * NRTW + rt) * NXL + (i - NXR)) * 128 + lane;
          a = __builtin_shufflevector(from[0], from[64], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
        } else {
          a = M::load(&wl[((size_t)(wave * NRTW + rt) * NXL + (i - NXR)) * FRAG + lane * VEC]);
        }
#pragma unroll
        for (int t = 0; t < BTW; ++t) acc[rt][t] = mma(a, xf[t], acc[rt][t]);
      }
    }
    // h fragments of the step before
    typename M::Frag hf[NHW][BTW];
    {
      const T* slot = reinterpret_cast<const T*>(p.ring) + (size_t)((p.published + (unsigned)j) % RES_RING) * hhalf;
      WaitBound bound{j == 0 ? p.patience : p.wait_ticks, p.sync + RES_SYNC_STATUS};
      while (true) {
        u32x4 raw[NHW][BTW];
        unsigned top = 0;
#pragma unroll
        for (int i = 0; i < NHW; ++i) {
          const int m = mh0 + KS * i;
#pragma unroll
          for (int t = 0; t < BTW; ++t)
            raw[i][t] = HALVES ? load_slot_16(slot, m < nsh ? hoff[t] + (unsigned)mh0 * 1024 : RES_NO_LANE, KS * i * 1024)
                               : load_slot_16(slot, m < nsh ? hoff[t] : RES_NO_LANE, m * 1024);
        }
#pragma unroll
        for (int i = 0; i < NHW; ++i)
#pragma unroll
          for (int t = 0; t < BTW; ++t) {
            top = max(top, largest_dword(raw[i][t]));
            hf[i][t] = as_frag<typename M::Frag>(raw[i][t]);
          }
        if (__builtin_amdgcn_ballot_w64(top == RES_EMPTY) == 0) break;
        if (bound.expired()) {
          s_fail = 1 + j;
          break;
        }
        asm volatile("" ::: "memory");   // the next look is another load
      }
    }
    if (j > 0) store_kept(j - 1);
    fetch_x(min(j + 1, p.count - 1));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NHW; ++i)
#pragma unroll
      for (int rt = 0; rt < NRTW; ++rt)
#pragma unroll
        for (int t = 0; t < BTW; ++t) acc[rt][t] = mma(wh[rt][i], hf[i][t], acc[rt][t]);
    f32x4* sums = red + (size_t)wave * Sum::BLOCKS * 64;
    if constexpr (HALVES) {
#pragma unroll
      for (int rt = 0; rt < NRTW; rt += 2) sums[rt / 2 * 64 + lane] = join_gates(Halves::fold(acc[rt][0]), Halves::fold(acc[rt + 1][0]));
    } else {
      Sum::write(sums, lane, acc);
    }
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(s_fail))   // a wave has stopped waiting: written before the barrier, so all see it
      stop_waiting<ResParams, UW>(&s_g, &s_rank, &s_fail, [&](int b_lo, int b_hi, int u0, int u1) { chain_slowly<ResParams, T, KS, CELL>(b_lo, b_hi, u0, u1, &s_fail); });
#pragma unroll
    for (int q = 0; q < IPT; ++q) {
      if (!mine[q]) continue;
      float G[4] = {0.f, 0.f, 0.f, 0.f};   // fixed order, as in forward_body; a sum of Halves is that of two parts
      if constexpr (parts_in_pairs<T, KW>) {
        add_pairs<KW>(G, [&](int w) { return cell[q][w * Sum::BLOCKS * 64]; });
      } else {
#pragma unroll
        for (int w = 0; w < KW; ++w) {
          const f32x4 v = cell[q][w * Sum::BLOCKS * 64];
#pragma unroll
          for (int r = 0; r < 4; ++r) G[r] += v[r];
        }
      }
      const float h = cell_forward<T, CELL>(G, bias[q], c_state[q], keep_second[q], keep_gate[q]);
      keep_h[q] = real[q] ? h : 0.0f;
      c_state[q] = CELL ? keep_h[q] : keep_second[q];
    }
    if (j + 1 < p.count) publish(p.published + (unsigned)j + 1);
    lds_barrier();   // the partial sums have been read: the next step may overwrite them
  }
  store_kept(p.count - 1);
}

// Steps from which on a launch takes two macro steps per instruction (0: never); the bits are the same.  us a launch's start and a step,
// one macro step and two: H = 1024, I = 256 20.1 + 1.40, 23.7 + 1.16; H = 1024, I = 64 18.7 + 1.41, 20.4 + 1.25; H = 896, I = 256
// 17.4 + 1.51, 20.0 + 1.25: even at 9 to 15 steps.  Not with more columns of x than one macro step a part (H = 896, I = 512 19.6 + 1.60,
// 25.1 + 1.43, launches of 8 to 12 steps 9 - 14 % slower), and not where a wave has two row tiles, whose sums are small either way (H = 500
// I = 256 9.8 + 1.15, 9.7 + 1.42, I = 768 12.2 + 1.86, 11.4 + 2.38, I = 64 even).  Up to two tiles half of the waves would have none, and of five
// or six one half has twice the other's (H = 640, I = 502, B = 5 2.4 % slower a gradient step, H = 650, I = 650 7 %).
template <class T, int NRT, int NXW, int KS, int NBT>
constexpr int halves_from = sizeof(T) == 2 && KS == 8 && NBT == 0 && NRT > 6 && NXW == 1 ? 16 : 0;
template <class T, int NRT, int NXW, int NXL, int NHW, int KS, int NBT, int CELL, bool HALVES>
hipError_t launch_chain_kernel(const ResParams& p, hipStream_t st) {
  constexpr int FTB = (KS == 4 && NBT == 2) ? 2 : 1, NRTW = chain_row_tiles<NRT, KS, NBT, HALVES>;
  constexpr int BLOCKS = Sums<NRTW, NBT == 0 ? 0 : NBT / FTB>::BLOCKS;
  constexpr size_t lds = (size_t)8 * BLOCKS * 1024 + (size_t)8 * NRTW * NXL * (HALVES ? 2048 : 1024);
  static_assert(lds <= 160 * 1024 - 64, "LDS of a compute unit");
  hipError_t e = allow_dynamic_lds<forward_chain_kernel<T, NRT, NXW, NXL, NHW, KS, NBT, CELL, HALVES>>(lds);
  if (e != hipSuccess) return e;
  forward_chain_kernel<T, NRT, NXW, NXL, NHW, KS, NBT, CELL, HALVES><<<dim3(RES_WGS), dim3(512), lds, st>>>(p);
  return hipGetLastError();
}
template <class T, int NRT, int NXW, int NXL, int NHW, int KS, int NBT, int CELL>
hipError_t launch_chain_cell(const ResParams& p, hipStream_t st) {
  constexpr int from = halves_from<T, NRT, NXW, KS, NBT>;
  if constexpr (from > 0) {
    if (p.count >= from) return launch_chain_kernel<T, NRT, NXW, NXL, NHW, KS, NBT, CELL, true>(p, st);
  }
  return launch_chain_kernel<T, NRT, NXW, NXL, NHW, KS, NBT, CELL, false>(p, st);
}

// An instantiation: what it covers (see the kernel) and its launchers by cell.  The tables are split over
// several sources so that they compile side by side.
struct ChainConfig {
  int nrt, nxw, nhw, ks, nbt;
  hipError_t (*launch[2])(const ResParams&, hipStream_t);
};
#define MEBPTT_CHAIN(T, NRT, NXW, NXL, NHW, KS, NBT) \
  ChainConfig{NRT, NXW, NHW, KS, NBT, {launch_chain_cell<T, NRT, NXW, NXL, NHW, KS, NBT, 0>, launch_chain_cell<T, NRT, NXW, NXL, NHW, KS, NBT, 1>}}
template <class C>
struct Table {
  const C* at;
  int n;
};
Table<ChainConfig> chain_table_bf16_k4();   // K split 4 ways
Table<ChainConfig> chain_table_bf16_k8();
Table<ChainConfig> chain_table_fp32_k4();
Table<ChainConfig> chain_table_fp32_k8();

}  // namespace mebptt
