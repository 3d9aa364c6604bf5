// Wide resident launches: forward chains and backward sweeps whose weights are spread once over the whole device (or
// over a half or a quarter of it) instead of once per XCD, for shapes a copy per XCD does not fit (wide_shape in
// device.h).  Not part of the ABI.
#pragma once

#include "resident_sweep.h"

namespace mebptt {

// ---- who is where, and what a wide launch waits for ------------------------------------------------------
// The batch is split over `groups` parts of the device, 8 / groups XCDs each; a workgroup finds its XCD and its rank
// there as in the other resident launches.  The workgroups of a group exchange every step's result through memory, past
// the L2s (loads and stores with the sc1 bit, coherent across XCDs): the polled exchange of resident.h, whose argument for
// reusing slots holds alike -- whoever publishes step q knows that all of step q - 1 has been published, by workgroups
// that had read all of q - 2 (in a sweep: through the three workgroups it adds up dh with) -- with eight slots instead of
// four, so that a reset is half a dozen steps old when the slot is used again.  Measured alone, 256 workgroups: 1.6 us a step
// for a small exchange, where a meeting by counter takes 7.4; 256 KiB from an L2 into every compute unit at once take
// 2.1 us (32 TB/s).
//
// All workgroups of a group that have work (`producers`) have to be on the chip together.  They count themselves in on
// one word per group and go on once all are there, which the fetch of the weights hides.  A workgroup that sees some
// missing for longer than `patience` marks the word, in one atomic step that only succeeds while some are; everybody who
// sees the mark leaves, and the last to arrive, when all others have left, runs all steps for the group's sequences alone:
// slow, but it waits for nobody, and its sums are formed in the same order.
constexpr int WIDE_THREADS = 256, WIDE_WAVES = 4, WIDE_RING = 8, WIDE_PART_RING = 4;

struct WideChainParams : ResParams {
  static constexpr int RING = WIDE_RING, GROUP_WORD = RES_SYNC_CHAIN_GROUP;
  int groups;
  unsigned arrived;   // workgroups of a group that the run's chain launches before this one have counted in
  const void* xs;     // x of this launch's steps as GEMM operands, fragment-tiled: [step][BP][KX]
};
struct WideSweepParams : SweepParams {
  static constexpr int RING = WIDE_RING, GROUP_WORD = RES_SYNC_SWEEP_GROUP;
  int groups;
  unsigned arrived;   // the same, sweep launches
  void* parts;   // WIDE_PART_RING slots of partial sums of dh: [group][block of units][receiver][sender][item]
};

enum WideRole { WIDE_LEAVE, WIDE_GO, WIDE_ALONE };

// Where the workgroups of a group count themselves in: the word (the count in its low half, in its high half the launch
// given up last, + 1) and, two dwords on, those that have left that launch.
struct WideGroup {
  unsigned* word;
  unsigned* status;
  unsigned launch, arrived, producers;
  __device__ unsigned long long* count() const { return reinterpret_cast<unsigned long long*>(word); }
  // One thread of a workgroup that has work.
  __device__ int arrive(long long wait_ticks) const {
    const unsigned long long v = __hip_atomic_fetch_add(count(), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((unsigned)(v >> 32) != launch + 1) return WIDE_GO;
    unsigned* left = word + 2;
    if ((unsigned)v - arrived != producers - 1) {
      __hip_atomic_fetch_add(left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return WIDE_LEAVE;
    }
    WaitBound bound{wait_ticks, status};
    bool ok = wait_ticks != 0;
    while (ok && __hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != producers - 1) ok = !bound.expired();
    __hip_atomic_store(left, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    if (!ok) __hip_atomic_store(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return ok ? WIDE_ALONE : WIDE_LEAVE;
  }
  // One thread of a workgroup that has arrived: waits for the others.  False: the launch is given up, or has failed.
  __device__ bool all_here(long long patience) const {
    WaitBound bound{patience, status};
    unsigned long long v = __hip_atomic_load(count(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while ((unsigned)(v >> 32) != launch + 1 && (unsigned)v - arrived < producers) {
      if (bound.expired()) {
        if (__hip_atomic_compare_exchange_strong(count(), &v, (unsigned long long)(launch + 1) << 32 | (unsigned)v, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
          return false;
      } else {
        v = __hip_atomic_load(count(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    return (unsigned)(v >> 32) != launch + 1;
  }
  // All threads of a workgroup for which all_here was false.
  __device__ void leave() const {
    __threadfence();   // its own stores are done when it says that it leaves
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(word + 2, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};
// All threads of a workgroup in which a wait has run into its bound; the program ends here (a way out that rejoined the
// kernel's end would have the compiler wait for the step's stores in every step).
template <class P>
__device__ __forceinline__ void wide_fail() {
  const auto& p = *arguments_again<P>();
  if (threadIdx.x == 0) __hip_atomic_store(p.sync + RES_SYNC_STATUS, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __builtin_amdgcn_endpgm();
}

// Stores past the L2s, visible to every XCD (sc1).
template <int DW>
__device__ __forceinline__ void store_slot(void* slot, unsigned byte_off, const unsigned (&v)[DW]) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(slot, 0, 0x7fffffff, 0x00020000);
  typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
  if constexpr (DW == 1)
    __builtin_amdgcn_raw_buffer_store_b32(v[0], rsrc, (int)byte_off, 0, 16);
  else if constexpr (DW == 2)
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, rsrc, (int)byte_off, 0, 16);
  else {
    static_assert(DW == 4, "1, 2 or 4 dwords");
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{v[0], v[1], v[2], v[3]}, rsrc, (int)byte_off, 0, 16);
  }
}
template <int DW>
__device__ __forceinline__ void load_slot(const void* slot, unsigned byte_off, unsigned (&v)[DW]) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(slot), 0, 0x7fffffff, 0x00020000);
  if constexpr (DW == 1) {
    v[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)byte_off, 0, 16);
  } else if constexpr (DW == 2) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)byte_off, 0, 16);
    v[0] = q[0];
    v[1] = q[1];
  } else {
    static_assert(DW == 4, "1, 2 or 4 dwords");
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte_off, 0, 16);
    for (int i = 0; i < 4; ++i) v[i] = q[i];
  }
}

// What an item touches in planes of memory, by a 32-bit offset that is the same in every step: with one wave per SIMD each
// address calculation shows.  RES_NO_LANE: nothing to touch (loads give zeros, stores are dropped).
template <int DW>
__device__ __forceinline__ void load_dwords(const void* base, unsigned byte_off, unsigned (&v)[DW]) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
  if constexpr (DW == 1) {
    v[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)byte_off, 0, 0);
  } else if constexpr (DW == 2) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)byte_off, 0, 0);
    v[0] = q[0];
    v[1] = q[1];
  } else {
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte_off, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = q[i];
  }
}
template <int DW>
__device__ __forceinline__ void store_dwords(void* base, unsigned byte_off, const unsigned (&v)[DW]) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000);
  typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
  if constexpr (DW == 1)
    __builtin_amdgcn_raw_buffer_store_b32(v[0], rsrc, (int)byte_off, 0, 0);
  else if constexpr (DW == 2)
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, rsrc, (int)byte_off, 0, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{v[0], v[1], v[2], v[3]}, rsrc, (int)byte_off, 0, 0);
}
// N consecutive values of a row, of units u .. u + N - 1.  Where a row ends inside them they are fetched as the window that
// ends there (byte_off says where it begins), see load_window; `ragged` shapes only.
template <int N>
struct Run {
  unsigned v[N];
  __device__ float operator[](int i) const { return __uint_as_float(v[i]); }
};
template <int N>
__device__ __forceinline__ void shift_run(Run<N>& r, int d) {   // d: how far the window was moved back
#pragma unroll
  for (int bit = 1; bit < N; bit *= 2)
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const unsigned from = i + bit < N ? r.v[i + bit] : 0u;
      r.v[i] = (d & bit) ? from : r.v[i];
    }
}
template <int N>
__device__ __forceinline__ void store_run(float* plane, unsigned byte_off, bool ragged, int real, const float (&f)[N]) {   // the first `real` values
  unsigned v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = __float_as_uint(f[i]);
  if (!ragged) {
    store_dwords<N>(plane, byte_off, v);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const unsigned one[1] = {v[i]};
      store_dwords<1>(plane, i < real ? byte_off + 4 * i : RES_NO_LANE, one);
    }
  }
}
// N 16-bit values, packed
template <int N>
__device__ __forceinline__ void load_half(const void* plane, unsigned byte_off, unsigned (&v)[(N + 1) / 2]) {
  if constexpr (N == 1) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(plane), 0, 0x7fffffff, 0x00020000);
    v[0] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)byte_off, 0, 0);
  } else {
    load_dwords<N / 2>(plane, byte_off, v);
  }
}
template <int N>
__device__ __forceinline__ void store_half(void* plane, unsigned byte_off, const unsigned (&v)[(N + 1) / 2]) {
  if constexpr (N == 1) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(plane, 0, 0x7fffffff, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v[0], rsrc, (int)byte_off, 0, 0);
  } else {
    store_dwords<N / 2>(plane, byte_off, v);
  }
}
template <int N>
__device__ __forceinline__ void pack_half(const unsigned (&v)[N], unsigned (&d)[(N + 1) / 2]) {
#pragma unroll
  for (int i = 0; i < (N + 1) / 2; ++i) d[i] = 2 * i + 1 < N ? v[2 * i] | v[2 * i + 1 < N ? 2 * i + 1 : 0] << 16 : v[2 * i];
}

// ---- the shared product ---------------------------------------------------------------------------------
// Both kernels multiply 16 * NR resident rows with the operand that was exchanged, 16 * NB sequences of it, over nsh macro
// steps: a forward workgroup its units' gate rows with all of h, a backward workgroup a block of units of W_hh^T with a
// quarter of dG's columns (four consecutive macro steps of every sixteen), which is as long.  Four waves share the macro steps: wave w has w,
// w + 4, ...; with one wave per SIMD a lane has 512 registers.  A wave's weights are NHW macro steps: the first in
// registers, NHL in LDS, the last NHS fetched again in every step.
//
// Items: an item is QU consecutive units of one sequence, so that planes are touched 4 * QU bytes at a time; the
// units of a workgroup are fastest.  QU grows with the batch so that there are 64 * NR items for any NB.
template <int NR, int NB>
struct WideTile {
  static constexpr int UW = 4 * NR, COLS = 16 * NB, QU = NB, UG = UW / QU, ITEMS = UG * COLS;
  static_assert((NB == 1 || NB == 2 || NB == 4) && ITEMS <= WIDE_THREADS, "");
  static constexpr int BLOCK = 64 + 4;   // of partial sums, in 16-byte vectors: items of different blocks hit different banks
};

template <int NR, int NB>
__device__ __forceinline__ void wide_write_sums(f32x4* red, int wave, int lane, const f32x4 (&acc)[NR][NB]) {
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int b = 0; b < NB; ++b) red[((wave * NR + r) * NB + b) * WideTile<NR, NB>::BLOCK + lane] = acc[r][b];
}

// Fragments of a weight operand, 16 bytes a lane, by scalar offsets: rows of `nsteps` macro steps.  A lane that asks past 2^31
// gets zeros: so does a macro step past a wave's last one, without a select (which would need the fragments in VGPRs).
struct WideOperand {
  __amdgpu_buffer_rsrc_t rsrc;
  int nsteps;
  __device__ WideOperand(const void* w, int nsteps_)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(w), 0, 0x7fffffff, 0x00020000)), nsteps(nsteps_) {}
  __device__ __forceinline__ bf16x8 load(int tile, int step, bool there) const {
    const int lane = (int)(threadIdx.x & 63);
    return as_frag<bf16x8>(__builtin_amdgcn_raw_buffer_load_b128(rsrc, there ? lane * 16 : (int)RES_NO_LANE, (tile * nsteps + step) * 1024, 0));
  }
};

// This wave's resident weights: rows of the tiles tile0 .. tile0 + NR - 1, macro steps step(0), step(1), ... n of them.
template <int NR, int NHW, int NHL, int NHS, int NB>
struct WideWeights {
  static constexpr int FRAG = 512, NHR = NHW - NHL - NHS;
  static constexpr int NMIN = NHW * (NR - 1) / NR;   // macro steps a wave has at least: below, fewer row tiles would do
  static __device__ __forceinline__ bool there(int i, int n) { return i < NMIN || i < n; }
  // The first NHA macro steps are held to the accumulation registers, where the matrix instructions read them in place (on its
  // own the compiler keeps them there too, but copies each fragment back before every use); the rest and whatever
  // else a lane holds share the other 256.
  // (The sums, 4 * NR * NB, are there too.)
  static constexpr int ACC = NB == 4 ? 192 : 208, NHA = NHR * NR * 4 <= ACC ? NHR : ACC / (NR * 4);
  u32x4 reg[NR][NHR];
  WideOperand w;
  int tile0, ntiles;
  __bf16* lds;
  __device__ WideWeights(const WideOperand& w_, int tile0_, int ntiles_, __bf16* lds_wave)
      : w(w_), tile0(tile0_), ntiles(ntiles_), lds(lds_wave + (threadIdx.x & 63) * 8) {}
  __device__ __forceinline__ int tile(int r) const { return min(tile0 + r, ntiles - 1); }
  template <class Step>
  __device__ __forceinline__ void load(int n, Step&& step) {
#pragma unroll
    for (int i = NHR; i < NHR + NHL; ++i)
#pragma unroll
      for (int r = 0; r < NR; ++r)
        *reinterpret_cast<bf16x8*>(lds + (r * NHL + (i - NHR)) * FRAG) = w.load(tile(r), step(there(i, n) ? i : 0), there(i, n));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NHR; ++i)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        union { bf16x8 f; u32x4 u; } cv;
        cv.f = w.load(tile(r), step(there(i, n) ? i : 0), there(i, n));
        reg[r][i] = cv.u;
      }
#pragma unroll
    for (int i = 0; i < NHA; ++i)
#pragma unroll
      for (int r = 0; r < NR; ++r) asm volatile("" : "+a"(reg[r][i]));
  }
};

// acc += weights x exchanged operand.  off: this lane's place in the batch tiles of the slot (RES_NO_LANE: no sequence);
// step(i): macro step i of this wave, n of them.  The operand's fragments are polled macro step by macro step, U in flight, the
// first U from begin() on: what is not there yet is fetched again, what came stays.
template <int NR, int NHW, int NHL, int NHS, int NB, int U>
struct WideProduct {
  using W = WideWeights<NR, NHW, NHL, NHS, NB>;
  static constexpr int G = 2;                                     // macro steps looked at together
  static_assert(U % G == 0 && U > G, "the next ones are in flight");
  static constexpr int US = NHS > 0 ? (NHS < 2 ? NHS : 2) : 1;   // macro steps of streamed weights in flight
  u32x4 raw[U][NB];
  template <class Step>
  __device__ __forceinline__ void fetch(int i, const void* slot, const unsigned (&at)[NB], int n, Step&& step) {
    const int m = step(W::there(i, n) ? i : 0);
#pragma unroll
    for (int b = 0; b < NB; ++b) raw[i % U][b] = load_slot_16(slot, W::there(i, n) ? at[b] : RES_NO_LANE, m * 1024);
  }
  template <class Step>
  __device__ __forceinline__ void begin(const void* slot, const unsigned (&off)[NB], int n, Step&& step) {
#pragma unroll
    for (int i = 0; i < U; ++i) fetch(i, slot, off, n, step);
  }
  // w_step: macro steps of a weight row before those of the operand
  template <class Step>
  __device__ __forceinline__ void run(const W& w, int w_step, const void* slot, const unsigned (&off)[NB], int n, Step&& step, f32x4 (&acc)[NR][NB],
                                      WaitBound& bound, int* s_fail) {
    // opaque, or the compiler keeps the places of all macro steps in registers across the steps of the launch
    unsigned at[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      at[b] = off[b];
      asm volatile("" : "+v"(at[b]));
    }
    asm volatile("" : "+s"(n));
    bf16x8 ws[US][NR];
    auto stream = [&](int i) {
      if (NHS > 0 && i >= NHW - NHS && i < NHW)
#pragma unroll
        for (int r = 0; r < NR; ++r) ws[(i - (NHW - NHS)) % US][r] = w.w.load(w.tile(r), step(W::there(i, n) ? i : 0) + w_step, W::there(i, n));
    };
    // macro steps are looked at G at a time, while the matrix pipe works on the G before: with one wave per SIMD
    // whatever is not issued between two MFMAs is added to them
    auto largest = [&](int g) {
      unsigned top = 0;
#pragma unroll
      for (int i = g * G; i < (g + 1) * G && i < NHW; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) top = max(top, largest_dword(raw[i % U][b]));
      return top;
    };
    unsigned top = largest(0);
#pragma unroll
    for (int g = 0; g < (NHW + G - 1) / G; ++g) {
      if (__builtin_amdgcn_ballot_w64(top == RES_EMPTY) != 0) {   // a loop of its own: the look above waits for its own loads only
        do {
          if (bound.expired()) {
            *s_fail = 1;
            break;
          }
          asm volatile("" ::: "memory");   // the next look is another load
#pragma unroll
          for (int i = g * G; i < (g + 1) * G && i < NHW; ++i) fetch(i, slot, at, n, step);
        } while (__builtin_amdgcn_ballot_w64(largest(g) == RES_EMPTY) != 0);
      }
#pragma unroll
      for (int i = g * G; i < (g + 1) * G && i < NHW; ++i) {
        if (i == NHW - NHS - US)
#pragma unroll
          for (int k = 0; k < US; ++k) stream(NHW - NHS + k);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          bf16x8 a;
          if (i < W::NHR)
            a = as_frag<bf16x8>(w.reg[r][i < W::NHR ? i : 0]);
          else if (i < NHW - NHS)
            a = *reinterpret_cast<const bf16x8*>(w.lds + (r * NHL + (i - W::NHR)) * W::FRAG);
          else
            a = ws[(i - (NHW - NHS)) % US][r];
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[r][b] = Mma<__bf16>::mma(a, as_frag<bf16x8>(raw[i % U][b]), acc[r][b]);
        }
        if (i >= NHW - NHS) stream(i + US);
        if (i + U < NHW) fetch(i + U, slot, at, n, step);
      }
      top = largest(g + 1);
      constexpr int MF = G * NR * NB, VA = G * NB * 2 + 4;
#pragma unroll
      for (int k = 0; k < MF; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);              // an MFMA,
        if (k >= MF / 2) __builtin_amdgcn_sched_group_barrier(0x002, (VA + MF / 2 - 1) / (MF / 2), 0);   // some of the look ahead
      }
      __builtin_amdgcn_sched_barrier(0);   // what a macro step needs is not fetched from LDS, or kept, earlier
    }
  }
};

// ---- forward chain -----------------------------------------------------------------------------------------
// Consecutive forward operations in one launch, see forward_chain_kernel.  A step:
//   1. while h of the step before travels, the x part of the gate product: x as operands, laid out by a kernel before the
//      launch and fetched a step ahead; its weights in registers, NX macro steps a wave of them, or in LDS (NXL); what goes
//      beyond is fetched again in every step;
//   2. the h part on the exchanged fragments, macro step by macro step as they come;
//   3. partial sums through LDS, the pointwise step;
//   4. h published, and stored where the schedule keeps it.
// X_EARLY: the next x is requested in front of the pointwise step instead of behind the published h, where it is waited for as
// long as that takes to reach the memory (operations of a wave complete in order).  Worth 2 - 3 % where a lane has the registers
// (64 sequences, H up to 1024: a run of H = 1024, B = 200 1858 -> 1818 us), and -2 % at H = 2048, which spills.
// H_EARLY: the first fragments of h are requested in the middle of the x part, 1 - 2 % with up to 32 sequences; with 64 they hold
// registers the x part needs (H = 2048 3 % slower), and where weights are streamed the x part is long enough for the exchange.
// Two halves of the batch that take turns, so that one travels while the other is worked on, were 1 - 18 % slower than all
// at once: a step's fixed costs come twice.
template <int NR, int NX, int NXL, int NHW, int NHL, int NHS, int NB, int CELL>
__global__ __launch_bounds__(WIDE_THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void wide_chain_kernel(WideChainParams p) {
  using T = __bf16;
  using M = Mma<T>;
  using Tile = WideTile<NR, NB>;
  constexpr int KSTEP = 32, FRAG = 512, UW = Tile::UW, QU = Tile::QU, UG = Tile::UG;
  constexpr int U = NB == 4 ? 4 : 6;   // macro steps of h in flight
  constexpr bool H_EARLY = NHS == 0 && NB <= 2;
  constexpr bool X_EARLY = NB == 4 && NHW <= 8;
  constexpr int RED = WIDE_WAVES * NR * NB * Tile::BLOCK;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f32x4* red = reinterpret_cast<f32x4*>(smem);                     // [4 waves][NR][NB] blocks
  T* wl = reinterpret_cast<T*>(red + RED);                    // [4][NR][NHL] fragments of W_hh, [4][NR][NXL] of W_ih
  __shared__ int s_role, s_xcd, s_rank, s_fail, s_here;   // s_here: not s_role again, which late waves may still read
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int lrow = lane & 15;
  const int per = RES_GROUPS / p.groups;   // XCDs of a group
  auto at = [&](int g) {
    return WideGroup{p.sync + RES_SYNC_CHAIN_GROUP + g * 64, p.sync + RES_SYNC_STATUS, p.launch, p.arrived, (unsigned)((p.KH + UW - 1) / UW)};
  };
  if (threadIdx.x == 0) {
    int xg, xr, role = draw_rank(p.sync, p.launch, xg, xr) ? WIDE_GO : WIDE_LEAVE;
    const int g = xg / per, m = xr * per + xg % per;
    if (g * p.nb >= p.B || m * UW >= p.KH) role = WIDE_LEAVE;   // no sequences or no units: nobody waits for this workgroup
    if (role == WIDE_GO) role = p.alone ? (m == 0 ? WIDE_ALONE : WIDE_LEAVE) : at(g).arrive(p.wait_ticks);
    s_role = role;
    s_xcd = xg;
    s_rank = xr;
    s_fail = 0;
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role), xcd = __builtin_amdgcn_readfirstlane(s_xcd);
  if (role == WIDE_LEAVE) return;
  const int group = xcd / per, member = __builtin_amdgcn_readfirstlane(s_rank) * per + xcd % per;
  const int b_lo = group * p.nb, b_hi = min(p.B, b_lo + p.nb);
  if (role == WIDE_ALONE) {
    chain_slowly<WideChainParams, T, WIDE_FWD_KS, CELL>(b_lo, b_hi, 0, p.KH, &s_fail);
    return;
  }
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP, nsteps = nsx + nsh;
  const size_t hhalf = (size_t)p.BP * p.KH;
  // this wave's macro steps of a gate row: wave, wave + 4, ...; nx of x, then nh of h, from mh0 on
  const int nx = (nsx - wave + 3) / 4, mh0 = wave + 4 * nx - nsx, nh = (nsh - mh0 + 3) / 4;

  const int ug = (int)threadIdx.x % UG, col = (int)threadIdx.x / UG, b = b_lo + col, u0 = member * UW + ug * QU;
  const bool item = (int)threadIdx.x < Tile::ITEMS && b < b_hi && u0 < p.KH;
  const unsigned at_h = item ? (unsigned)ft_offset<T>(b, u0, nsh) * 2 : RES_NO_LANE;
  const f32x4* cell = red + (((ug * QU) >> 2) * NB + (col >> 4)) * Tile::BLOCK + ((ug * QU) & 3) * 16 + (col & 15);
  float4 bias[QU];
  float c_state[QU], keep_h[QU], keep_second[QU], keep_gate[4][QU];
  // publishes keep_h as step number q and resets this thread's part of the slot two steps back
  auto publish = [&](unsigned q) {
    T* now = reinterpret_cast<T*>(p.ring) + (size_t)(q % WIDE_RING) * hhalf;
    T* old = reinterpret_cast<T*>(p.ring) + (size_t)((q + WIDE_RING - 2) % WIDE_RING) * hhalf;
    unsigned hi[QU];
#pragma unroll
    for (int i = 0; i < QU; ++i) hi[i] = (__float_as_uint(keep_h[i]) + 0x8000u) >> 16;
    constexpr int DW = QU == 4 ? 2 : 1;
    unsigned v[DW], empty[DW];
    if constexpr (QU == 1) {   // the lane of an even unit stores its neighbour's too
      v[0] = hi[0] | (__builtin_amdgcn_update_dpp(hi[0], hi[0], 0xb1 /* quad_perm 1,0,3,2 */, 0xf, 0xf, false) << 16);
    } else {
#pragma unroll
      for (int i = 0; i < DW; ++i) v[i] = hi[2 * i] | hi[2 * i + 1] << 16;
    }
#pragma unroll
    for (int i = 0; i < DW; ++i) {
      v[i] = not_empty(v[i]);
      empty[i] = RES_EMPTY;
    }
    const unsigned to = QU > 1 || (ug & 1) == 0 ? at_h : RES_NO_LANE;
    store_slot<DW>(now, to, v);
    store_slot<DW>(old, to, empty);
  };
#pragma unroll
  for (int i = 0; i < QU; ++i) {
    bias[i] = float4{0.f, 0.f, 0.f, 0.f};
    c_state[i] = keep_h[i] = keep_second[i] = 0.0f;
    if (item && u0 + i < p.H) {
      bias[i] = *reinterpret_cast<const float4*>(p.bp + 4 * (u0 + i));
      keep_h[i] = HPlane<T>::load(p.src, b, u0 + i, p.KH / 32, p.H, hhalf);
      c_state[i] = CELL ? keep_h[i] : (p.src + p.hplane)[(size_t)b * p.H + u0 + i];
    }
  }
  publish(p.published);   // travels while the weights are fetched

  WideWeights<NR, NHW, NHL, NHS, NB> w(WideOperand(p.Wp, nsteps), member * NR, p.HP / 4, wl + (size_t)wave * NR * NHL * FRAG);
  auto h_step = [&](int i) { return mh0 + 4 * i; };
  T* wxl = wl + (size_t)WIDE_WAVES * NR * NHL * FRAG + (size_t)wave * NR * NXL * FRAG + lane * 8;
  constexpr int NXH = NX + NXL;   // macro steps of x held, one way or the other
#pragma unroll
  for (int i = 0; i < NXL; ++i)
#pragma unroll
    for (int r = 0; r < NR; ++r)
      *reinterpret_cast<bf16x8*>(wxl + (r * NXL + i) * FRAG) = w.w.load(w.tile(r), NX + i < nx ? wave + 4 * (NX + i) : 0, NX + i < nx);
  bf16x8 wx[NX > 0 ? NX : 1][NR];
#pragma unroll
  for (int i = 0; i < NX; ++i)
#pragma unroll
    for (int r = 0; r < NR; ++r) wx[i][r] = w.w.load(w.tile(r), i < nx ? wave + 4 * i : 0, i < nx);
  w.load(nh, [&](int i) { return nsx + h_step(i); });
  if (threadIdx.x == 0) s_here = at(group).all_here(p.patience);
  __syncthreads();
  if (!__builtin_amdgcn_readfirstlane(s_here)) {
    at(group).leave();
    return;
  }

  // where this lane's operands come from; columns that belong to no sequence of the group fetch no h
  unsigned off[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t)
    off[t] = b_lo + t * 16 + lrow < b_hi ? (unsigned)((((b_lo >> 4) + t) * nsh * 64 + lane) * 16) : RES_NO_LANE;
  auto slot = [&](int j) { return reinterpret_cast<const T*>(p.ring) + (size_t)((p.published + (unsigned)j) % WIDE_RING) * hhalf; };
  const WideOperand xw(p.xs, nsx);
  const int xtiles = p.count * p.BP / 16;
  auto x_load = [&](int j, int t, int i) {   // x of macro step i of this wave
    return xw.load(min((j * p.BP + b_lo) / 16 + t, xtiles - 1), i < nx ? wave + 4 * i : 0, i < nx);
  };
  f32x4 acc[NR][NB];
  bf16x8 xf[NXH > 0 ? NXH : 1][NB];
  auto fetch_x = [&](int j) {
#pragma unroll
    for (int i = 0; i < NXH; ++i)
#pragma unroll
      for (int t = 0; t < NB; ++t) xf[i][t] = x_load(j, t, i);
  };
  WideProduct<NR, NHW, NHL, NHS, NB, U> product;
  auto x_part = [&](int j) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int t = 0; t < NB; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto held = [&](int i0, int i1) {
#pragma unroll
      for (int i = i0; i < i1 && i < NXH; ++i)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const bf16x8 a = i < NX ? wx[i < NX ? i : 0][r] : *reinterpret_cast<const bf16x8*>(wxl + (r * NXL + (i < NX ? 0 : i - NX)) * FRAG);
#pragma unroll
          for (int t = 0; t < NB; ++t) acc[r][t] = M::mma(a, xf[i][t], acc[r][t]);
        }
    };
    held(0, 2);   // macro steps past nx are zeros; few branches: each costs more than two macro steps' MFMAs
    if (H_EARLY) product.begin(slot(j), off, nh, h_step);
    if (nx > 2) held(2, 4);
    if (nx > 4) held(4, NXH);
    if (nx > NXH) {   // wider inputs: UX macro steps in flight
      constexpr int UX = NB == 4 ? 2 : 3;
      bf16x8 a[UX][NR], f[UX][NB];
      auto fetch = [&](int e, int i) {
#pragma unroll
        for (int r = 0; r < NR; ++r) a[e][r] = w.w.load(w.tile(r), i < nx ? wave + 4 * i : 0, i < nx);
#pragma unroll
        for (int t = 0; t < NB; ++t) f[e][t] = x_load(j, t, i);
      };
#pragma unroll
      for (int e = 0; e < UX; ++e) fetch(e, NXH + e);
      for (int i = NXH; i < nx; i += UX) {
#pragma unroll
        for (int e = 0; e < UX; ++e) {
#pragma unroll
          for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int t = 0; t < NB; ++t) acc[r][t] = M::mma(a[e][r], f[e][t], acc[r][t]);
          fetch(e, i + e + UX);
        }
      }
    }
  };
  const bool ragged = p.H % QU != 0;
  const int real = p.H - u0;   // units of an item that exist: QU or more, but for the last of a row
  const size_t plane = (size_t)p.B * p.H;
  const unsigned at_plane = item && real > 0 ? (unsigned)(b * p.H + u0) * 4 : RES_NO_LANE;
  auto store_kept = [&](int j) {   // what the schedule wants of step j
    const ResStep dst = p.step[j];
    if (!dst.out && !dst.gates) return;
    if (dst.out) {   // padding columns of the split h plane are part of the operand other launches fetch: zero
      unsigned hi[QU], lo[QU], d[(QU + 1) / 2];
#pragma unroll
      for (int i = 0; i < QU; ++i) {
        hi[i] = (__float_as_uint(keep_h[i]) + 0x8000u) >> 16;
        lo[i] = __float_as_uint(keep_h[i]) & 0xffffu;
      }
      pack_half<QU>(hi, d);
      store_half<QU>(dst.out, at_h, d);
      pack_half<QU>(lo, d);
      store_half<QU>(reinterpret_cast<unsigned short*>(dst.out) + hhalf, at_h, d);
      store_run<QU>(dst.out + p.hplane, at_plane, ragged, real, keep_second);
    }
    if (dst.gates) {
      store_run<QU>(dst.gates, at_plane, ragged, real, keep_gate[0]);
      store_run<QU>(dst.gates + plane, at_plane, ragged, real, keep_gate[1]);
      store_run<QU>(dst.gates + p.unit, at_plane, ragged, real, keep_gate[2]);
      if (CELL == 0) store_run<QU>(dst.gates + p.unit + plane, at_plane, ragged, real, keep_gate[3]);
    }
  };

  fetch_x(0);
#pragma unroll 1
  for (int j = 0; j < p.count; ++j) {
    x_part(j);
    if (!H_EARLY) product.begin(slot(j), off, nh, h_step);
    WaitBound bound{p.wait_ticks, p.sync + RES_SYNC_STATUS};
    product.run(w, nsx, slot(j), off, nh, h_step, acc, bound, &s_fail);
    if (X_EARLY) fetch_x(min(j + 1, p.count - 1));
    wide_write_sums<NR, NB>(red, wave, lane, acc);
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(s_fail)) wide_fail<WideChainParams>();
#pragma unroll
    for (int i = 0; i < QU; ++i) {
      float G[4] = {0.f, 0.f, 0.f, 0.f}, gate[4];
#pragma unroll
      for (int v = 0; v < WIDE_WAVES; ++v) {   // fixed order, as in forward_body
        const f32x4 q = item ? cell[v * NR * NB * Tile::BLOCK + i * 16] : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) G[r] += q[r];
      }
      const float h = cell_forward<T, CELL>(G, bias[i], c_state[i], keep_second[i], gate);
      keep_h[i] = u0 + i < p.H ? h : 0.0f;
      c_state[i] = CELL ? keep_h[i] : keep_second[i];
#pragma unroll
      for (int r = 0; r < 4; ++r) keep_gate[r][i] = gate[r];
    }
    if (j + 1 < p.count) publish(p.published + (unsigned)j + 1);
    lds_barrier();   // the partial sums have been read: the next step may overwrite them
    if (!X_EARLY) fetch_x(min(j + 1, p.count - 1));
    store_kept(j);
  }
}

// ---- backward sweep on stored internal states --------------------------------------------------------------
// Consecutive backward operations in one launch, see sweep_kernel.  A workgroup holds 16 * NR rows (units) of W_hh^T and
// four consecutive macro steps of every sixteen of their K = 4 H columns (4 KiB at a time: 128 KB into every compute unit in
// 4.75 us, every fourth macro step 5.26): with whole rows it would have to fetch all of dG, 1 MiB a step for 64
// sequences of H = 2048 where a quarter takes 2.1 us.  The four workgroups of a block of units sit on one XCD; each adds up dh
// for a quarter of the block's units, to which the others send their sums through that XCD's L2 (the polled
// exchange once more, fp32).  A step:
//   1. this workgroup's part of dh = dG W_hh on the exchanged fragments as they come;
//   2. partial sums through LDS, the others' quarters sent, the own one completed; the pointwise step;
//   3. dG published; while it travels, the stored state of the next step is fetched, and what only later launches read
//      is stored (transposed copies turned over in LDS).
template <int NR, int NHW, int NHL, int NHS, int NB, int CELL>
__global__ __launch_bounds__(WIDE_THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void wide_sweep_kernel(WideSweepParams p) {
  using T = __bf16;
  using M = Mma<T>;
  using Tile = WideTile<NR, NB>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, FRAG = 64 * VEC, UW = Tile::UW, QU = Tile::QU, UG = Tile::UG, COLS = Tile::COLS;
  constexpr int UB = 16 * NR;          // units of a block
  constexpr int U = NB == 4 || NHS > 0 ? 4 : 6;   // macro steps of dG in flight
  constexpr int KROW = COLS + 8;       // row of the kept values in LDS
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int RED = WIDE_WAVES * NR * NB * Tile::BLOCK;
  f32x4* red = reinterpret_cast<f32x4*>(smem);               // [4 waves][NR][NB] blocks
  T* wl = reinterpret_cast<T*>(red + RED);              // [4][NR][NHL] fragments
  T* kept = wl + (size_t)WIDE_WAVES * NR * NHL * FRAG;       // [5 UW][KROW]: rows 4 u + gate, then h_{s-1}
  __shared__ int s_role, s_xcd, s_rank, s_fail, s_here;   // s_here: not s_role again, which late waves may still read
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int lrow = lane & 15;
  const int per = RES_GROUPS / p.groups, blocks = (p.HP + UB - 1) / UB;
  auto at = [&](int g) {
    return WideGroup{p.sync + RES_SYNC_SWEEP_GROUP + g * 64, p.sync + RES_SYNC_STATUS, p.launch, p.arrived, 4u * (unsigned)blocks};
  };
  if (threadIdx.x == 0) {
    int xg, xr, role = draw_rank(p.sync, p.launch, xg, xr) ? WIDE_GO : WIDE_LEAVE;
    const int g = xg / per, ub = (xr >> 2) * per + xg % per;
    if (g * p.nb >= p.B || ub >= blocks) role = WIDE_LEAVE;   // no sequences or no units: nobody waits for this workgroup
    if (role == WIDE_GO) role = p.alone ? (ub == 0 && (xr & 3) == 0 ? WIDE_ALONE : WIDE_LEAVE) : at(g).arrive(p.wait_ticks);
    s_role = role;
    s_xcd = xg;
    s_rank = xr;
    s_fail = 0;
  }
  __syncthreads();
  const int role = __builtin_amdgcn_readfirstlane(s_role), xcd = __builtin_amdgcn_readfirstlane(s_xcd), rank = __builtin_amdgcn_readfirstlane(s_rank);
  if (role == WIDE_LEAVE) return;
  const int group = xcd / per, ub = (rank >> 2) * per + xcd % per, kq = rank & 3;
  const int b_lo = group * p.nb, b_hi = min(p.B, b_lo + p.nb);
  constexpr int SEND = Tile::ITEMS * QU;   // values one workgroup sends another
  const size_t part_slot = (size_t)p.groups * blocks * 16 * SEND;
  float* parts = reinterpret_cast<float*>(p.parts) + ((size_t)group * blocks + ub) * 16 * SEND;   // of this block, slot 0: [receiver][sender][item]
  if (role == WIDE_ALONE) {
    sweep_slowly<WideSweepParams, T, false, 8, WIDE_BACK_PARTS, CELL>(b_lo, b_hi, 0, p.HP, reinterpret_cast<float*>(smem), &s_fail);
    // nothing was sent: what the launch before left in its last slots is cleared for the next one
    for (int s = 0; s < WIDE_PART_RING; ++s)
      for (size_t i = threadIdx.x; i < (size_t)blocks * 16 * SEND; i += WIDE_THREADS)
        reinterpret_cast<unsigned*>(p.parts)[s * part_slot + (size_t)group * blocks * 16 * SEND + i] = RES_EMPTY;
    return;
  }
  const int nsh = p.KH / KSTEP, nsteps = p.G4 / KSTEP;   // nsteps = 4 nsh
  const size_t hhalf = (size_t)p.BP * p.KH, dG_step = (size_t)p.BP * p.G4, plane = (size_t)p.B * p.H;

  // items: QU units u0 .. (of the quarter kq of the block's units) of one sequence
  const int ug = (int)threadIdx.x % UG, col = (int)threadIdx.x / UG, u0 = ub * UB + kq * UW + ug * QU;
  const int b = b_lo + col;
  const bool in = (int)threadIdx.x < Tile::ITEMS, ragged = p.H % QU != 0;
  const bool has = in && b < b_hi && u0 < p.HP, real = has && u0 < p.H;      // something to publish; at least one real unit
  const int units = p.H - u0, back = max(0, QU - units);   // units of an item that exist; how far the window on them is moved back
  // places of an item in a plane (and of the window on it), a split h plane, a dG block
  const unsigned at_plane = real ? (unsigned)(b * p.H + u0) * 4 : RES_NO_LANE, at_window = real ? at_plane - 4 * back : RES_NO_LANE;
  const unsigned at_h = has ? (unsigned)ft_offset<T>(b, u0, nsh) * 2 : RES_NO_LANE, at_g = has ? (unsigned)ft_offset<T>(b, 4 * u0, nsteps) * 2 : RES_NO_LANE;
  const unsigned at_dg = real ? at_g : RES_NO_LANE;
  constexpr int NV = QU == 4 ? 2 : 1, DW = QU == 1 ? 2 : 4;   // stores of an item's dG, dwords each; 16-byte slots lie 256 bytes apart
  unsigned dg[NV][DW];
  float dc_run[QU], kp_h[QU];
  unsigned short kp_hprev[QU];   // as operands
  auto publish = [&](unsigned q) {
    T* now = reinterpret_cast<T*>(p.ring) + (size_t)(q % WIDE_RING) * dG_step;
    T* old = reinterpret_cast<T*>(p.ring) + (size_t)((q + WIDE_RING - 2) % WIDE_RING) * dG_step;   // two steps back
    unsigned empty[DW];
#pragma unroll
    for (int i = 0; i < DW; ++i) empty[i] = RES_EMPTY;
#pragma unroll
    for (int k = 0; k < NV; ++k) store_slot<DW>(now, at_g + k * 256, dg[k]);
#pragma unroll
    for (int k = 0; k < NV; ++k) store_slot<DW>(old, at_g + k * 256, empty);
  };
#pragma unroll
  for (int i = 0; i < QU; ++i) {
    dc_run[i] = real && i < units ? p.dc[(size_t)b * p.H + u0 + i] : 0.0f;
    kp_h[i] = 0.0f;
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
#pragma unroll
    for (int i = 0; i < DW; ++i) dg[k][i] = 0u;
    if (p.dG_next) {
      load_dwords<DW>(p.dG_next, at_dg + k * 256, dg[k]);
#pragma unroll
      for (int i = 0; i < DW; ++i) dg[k][i] = not_empty(dg[k][i]);
    }
  }
  publish(p.published);   // travels while the weights are fetched

  WideWeights<NR, NHW, NHL, NHS, NB> w(WideOperand(p.WTh, nsteps), ub * NR, p.HP / 16, wl + (size_t)wave * NR * NHL * FRAG);
  const int part = 4 * kq + wave, n = (nsteps - part + WIDE_BACK_PARTS - 1) / WIDE_BACK_PARTS;   // this wave's macro steps: part, part + 16, ...
  auto g_step = [&](int i) { return part + WIDE_BACK_PARTS * i; };
  w.load(n, g_step);
  if (threadIdx.x == 0) s_here = at(group).all_here(p.patience);
  __syncthreads();
  if (!__builtin_amdgcn_readfirstlane(s_here)) {
    at(group).leave();
    return;
  }
  unsigned off[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t)
    off[t] = b_lo + t * 16 + lrow < b_hi ? (unsigned)((((b_lo >> 4) + t) * nsteps * 64 + lane) * 16) : RES_NO_LANE;
  auto slot = [&](int j) { return reinterpret_cast<const T*>(p.ring) + (size_t)((p.published + (unsigned)j) % WIDE_RING) * dG_step; };

  // the stored internal state of the step about to run, its input state, its loss gradient, as fetched
  Run<QU> gate[4], c_s, c_prev, dy;
  constexpr int HD = (QU + 1) / 2;                       // dwords of QU 16-bit values
  unsigned hs_hi[HD], hs_lo[HD], hp_hi[HD], hp_lo[HD];   // h_s and h_{s-1}, split
  const bool want_h = p.dy_is_h || p.y_out != nullptr;
  auto half_of = [](const unsigned (&v)[HD], int i) { return i % 2 ? v[i / 2] >> 16 : v[i / 2] & 0xffffu; };
  auto whole = [&](const unsigned (&hi)[HD], const unsigned (&lo)[HD], int i) {   // h in full precision
    return __uint_as_float(((half_of(hi, i) - (half_of(lo, i) >> 15)) << 16) | half_of(lo, i));
  };
  auto fetch = [&](int j) {
    const int s = p.s_hi - j;
    const float *src = p.src[j], *stp = p.state[j];
    load_dwords<QU>(stp + p.unit, at_window, gate[0].v);
    load_dwords<QU>(stp + p.unit + plane, at_window, gate[1].v);
    load_dwords<QU>(stp + 2 * p.unit, at_window, gate[2].v);
    if (CELL == 0) load_dwords<QU>(stp + 2 * p.unit + plane, at_window, gate[3].v);   // the GRU has three gates
    load_dwords<QU>(stp + p.hplane, at_window, c_s.v);                               // c_s, or the GRU's n_h
    if (CELL == 0) load_dwords<QU>(src + p.hplane, at_window, c_prev.v);
    if (want_h) {
      load_half<QU>(stp, at_h, hs_hi);
      load_half<QU>(reinterpret_cast<const unsigned short*>(stp) + hhalf, at_h, hs_lo);
    }
    load_half<QU>(src, at_h, hp_hi);
    if (CELL != 0) load_half<QU>(reinterpret_cast<const unsigned short*>(src) + hhalf, at_h, hp_lo);   // the GRU blends with h_{s-1}
    // no loss gradient at this step: nothing is fetched, zeros
    const bool injected = p.dy != nullptr && s >= p.dy_first;
    load_dwords<QU>(injected ? p.dy + (size_t)(s - p.dy_first) * plane : stp, injected ? at_window : RES_NO_LANE, dy.v);
  };
  auto settle = [&]() {   // rows that end inside an item
    if (!ragged) return;
#pragma unroll
    for (int r = 0; r < (CELL == 0 ? 4 : 3); ++r) shift_run(gate[r], back);
    shift_run(c_s, back);
    if (CELL == 0) shift_run(c_prev, back);
    shift_run(dy, back);
  };
  const bool slots_whole = p.B % VEC == 0;   // a 16-byte slot of the transposed operands holds sequences of one step only
  auto keep_transposed = [&]() {
    if (!slots_whole || !in || b >= b_hi) return;
#pragma unroll
    for (int i = 0; i < QU; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const unsigned v = dg[i / 2][(i % 2) * 2 + r / 2];
        reinterpret_cast<unsigned short*>(kept)[((ug * QU + i) * 4 + r) * KROW + col] = (unsigned short)(r % 2 ? v >> 16 : v & 0xffffu);
      }
      reinterpret_cast<unsigned short*>(kept)[(4 * UW + ug * QU + i) * KROW + col] = kp_hprev[i];
    }
  };
  const unsigned tid = threadIdx.x;
  const int ncs = p.KC / KSTEP;
  constexpr unsigned CG = 4 * UW, CH_G = CG * (COLS / VEC), CH_H = UW * (COLS / VEC);   // rows of dG; chunks of VEC sequences of one row
  auto chunk_row = [&](int rowid) { return (unsigned)(((rowid >> 4) * ncs * 64 + (rowid & 15)) * VEC) * 2; };   // bytes, column 0
  const int uq = ub * UB + kq * UW;
  auto store_kept = [&](int s) {
    const int cslot = (s - 1) % p.CH, buf = ((s - 1) / p.CH) & 1;   // where step s lives in the chunk buffers
    T* dG_cur = reinterpret_cast<T*>(p.dG_chunk[buf]) + (size_t)cslot * dG_step;
    T* dGT = reinterpret_cast<T*>(p.dGT[buf]);
    T* aT = reinterpret_cast<T*>(p.aT[buf]);
#pragma unroll
    for (int k = 0; k < NV; ++k) store_dwords<DW>(dG_cur, at_dg + k * 256, dg[k]);
    if (p.y_out) store_run<QU>(p.y_out + (size_t)(s - 1) * plane, at_plane, ragged, units, kp_h);
    if (slots_whole) {
      // chunks of VEC sequences of one row; rows fastest: 16 of them lie side by side
      const unsigned c8 = (unsigned)(cslot * p.B + b_lo) / VEC;
      auto move = [&](T* base, unsigned c, unsigned rows, int row0, int first) {   // row0: in `kept`; first: in the operand
        const unsigned r = c % rows, cb = c / rows, at = c8 + cb;
        const unsigned to = chunk_row(first + (int)r) + ((at >> 2) * 64 + (at & 3) * 16) * VEC * 2;
        const bool there = b_lo + (int)cb * VEC < b_hi && (rows == CG ? (int)(r >> 2) : (int)r) < p.H - uq;
        union { u32x4 q; unsigned v[4]; } cv;
        cv.q = *reinterpret_cast<const u32x4*>(kept + (row0 + r) * KROW + cb * VEC);
        store_dwords<4>(base, there ? to : RES_NO_LANE, cv.v);
      };
#pragma unroll
      for (unsigned c0 = 0; c0 < CH_G; c0 += WIDE_THREADS)
        if (c0 + WIDE_THREADS <= CH_G || c0 + tid < CH_G) move(dGT, c0 + tid, CG, 0, 4 * uq);
#pragma unroll
      for (unsigned c0 = 0; c0 < CH_H; c0 += WIDE_THREADS)
        if (c0 + WIDE_THREADS <= CH_H || c0 + tid < CH_H) move(aT, c0 + tid, UW, CG, p.NX + uq);
    } else if (real) {
      const int cc = cslot * p.B + b;
#pragma unroll
      for (int i = 0; i < QU; ++i)
        if (i < units) {
          const size_t o = ft_offset<T>(4 * (u0 + i), cc, ncs);   // rows 4n .. 4n + 3 of one column lie VEC elements apart
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const unsigned v = dg[i / 2][(i % 2) * 2 + r / 2];
            reinterpret_cast<unsigned short*>(dGT)[o + r * VEC] = (unsigned short)(r % 2 ? v >> 16 : v & 0xffffu);
          }
          reinterpret_cast<unsigned short*>(aT)[ft_offset<T>(p.NX + u0 + i, cc, ncs)] = kp_hprev[i];
        }
    }
  };
  // this thread's value i of quarter q of the block: row q * UW + ug * QU + i
  auto sum_at = [&](int q, float (&v)[QU]) {
    const int n0 = q * UW + ug * QU;
    const int c = in ? col : 0;
    const f32x4* at = red + ((n0 >> 4) * NB + (c >> 4)) * Tile::BLOCK + ((n0 & 15) >> 2) * 16 + (c & 15);
#pragma unroll
    for (int i = 0; i < QU; ++i) v[i] = 0.0f;
#pragma unroll
    for (int wv = 0; wv < WIDE_WAVES; ++wv) {
      const float* f = reinterpret_cast<const float*>(at + wv * NR * NB * Tile::BLOCK) + (n0 & 3);
      if constexpr (QU == 4) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(f);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += x[i];
      } else if constexpr (QU == 2) {
        const float2 x = *reinterpret_cast<const float2*>(f);
        v[0] += x.x;
        v[1] += x.y;
      } else {
        v[0] += f[0];
      }
    }
  };

  WideProduct<NR, NHW, NHL, NHS, NB, U> product;
  fetch(0);
#pragma unroll 1
  for (int j = 0; j < p.count; ++j) {
    product.begin(slot(j), off, n, g_step);
    WaitBound bound{p.wait_ticks, p.sync + RES_SYNC_STATUS};
    f32x4 acc[NR][NB];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int t = 0; t < NB; ++t) acc[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    product.run(w, 0, slot(j), off, n, g_step, acc, bound, &s_fail);
    wide_write_sums<NR, NB>(red, wave, lane, acc);
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(s_fail)) wide_fail<WideSweepParams>();
    // the other quarters' sums, for the workgroups that complete them
    float* now = parts + ((p.published + (unsigned)j) % WIDE_PART_RING) * part_slot;
    float* old = parts + ((p.published + (unsigned)j + WIDE_PART_RING - 2) % WIDE_PART_RING) * part_slot;
    if (in) {
      typedef float vec __attribute__((ext_vector_type(QU)));
      vec empty;
#pragma unroll
      for (int i = 0; i < QU; ++i) empty[i] = __uint_as_float(RES_EMPTY);
#pragma unroll
      for (int k = 1; k < 4; ++k) {
        const int q = (kq + k) & 3;
        float v[QU];
        sum_at(q, v);
        vec o;
#pragma unroll
        for (int i = 0; i < QU; ++i) o[i] = __uint_as_float(not_empty(__float_as_uint(v[i])));
        *reinterpret_cast<vec*>(now + (size_t)(q * 4 + kq) * SEND + threadIdx.x * QU) = o;
        *reinterpret_cast<vec*>(old + (size_t)(q * 4 + kq) * SEND + threadIdx.x * QU) = empty;
      }
    }
    float own[QU], dh[QU];
    sum_at(kq, own);
    unsigned got[3][QU];
    auto look = [&]() {
#pragma unroll
      for (int k = 0; k < 3; ++k) load_slot<QU>(now + (size_t)(kq * 4 + ((kq + k + 1) & 3)) * SEND, in ? threadIdx.x * QU * 4 : RES_NO_LANE, got[k]);
    };
    auto missing = [&]() {
      unsigned top = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < QU; ++i) top = max(top, got[k][i]);
      return __builtin_amdgcn_ballot_w64(top == RES_EMPTY) != 0;
    };
    look();
    while (missing()) {
      if (bound.expired()) {
        s_fail = 1;
        break;
      }
      asm volatile("" ::: "memory");   // the next look is another load
      look();
    }
#pragma unroll
    for (int i = 0; i < QU; ++i) {   // fixed order, see sum_back_parts
      dh[i] = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v = own[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) v = ((kq + k + 1) & 3) == q ? __uint_as_float(got[k][i]) : v;
        dh[i] += v;
      }
    }
    settle();
#pragma unroll
    for (int i = 0; i < QU; ++i) {
      const float h_s = want_h ? whole(hs_hi, hs_lo, i) : 0.0f;
      const float before = CELL ? whole(hp_hi, hp_lo, i) : c_prev[i];
      float d = dh[i] + (p.dy_is_h ? h_s : dy[i]), dG[4], dc_out;
      if (CELL == 0)
        lstm_backward_point<T>(d, dc_run[i], gate[0][i], gate[1][i], gate[2][i], gate[3][i], c_s[i], before, dG, dc_out);
      else   // the running plane carries dh_{s+1} * z_{s+1}, as in backward_body
        gru_backward_point(__fadd_rn(d, dc_run[i]), gate[0][i], gate[1][i], gate[2][i], c_s[i], before, dG, dc_out);
      dc_run[i] = dc_out;
      union { T t[4]; unsigned u[2]; } pk;
#pragma unroll
      for (int r = 0; r < 4; ++r) pk.t[r] = (T)dG[r];
#pragma unroll
      for (int r = 0; r < 2; ++r) dg[i / 2][(i % 2) * 2 + r] = i < units ? not_empty(pk.u[r]) : 0u;
      kp_h[i] = h_s;
      kp_hprev[i] = (unsigned short)half_of(hp_hi, i);
    }
    if (j + 1 < p.count) publish(p.published + (unsigned)j + 1);
    fetch(min(j + 1, p.count - 1));
    keep_transposed();
    lds_barrier();   // the partial sums have been read, the kept values are there
    if (__builtin_amdgcn_readfirstlane(s_fail)) wide_fail<WideSweepParams>();
    store_kept(p.s_hi - j);
  }
#pragma unroll
  for (int i = 0; i < QU; ++i)
    if (real && i < units) p.dc[(size_t)b * p.H + u0 + i] = dc_run[i];
}

// ---- launchers -------------------------------------------------------------------------------------------------
// What a shape's two kernels keep where, see WideWeights and wide_chain_kernel.
template <int NR_, int NHW_, int NHL_, int NHS_, int NX_, int NXL_, int GHL_, int GHS_, int NB_>
struct WideKind {
  static constexpr int NR = NR_, NHW = NHW_, NHL = NHL_, NHS = NHS_, NX = NX_, NXL = NXL_, NB = NB_; // the chain's
  static constexpr int GHL = GHL_, GHS = GHS_;                                                       // the sweep's NHL, NHS
  using Tile = WideTile<NR, NB>;
  static constexpr size_t RED = (size_t)WIDE_WAVES * NR * NB * Tile::BLOCK * 16;
};
template <class K, int CELL>
hipError_t launch_wide_chain_cell(const WideChainParams& p, hipStream_t st) {
  constexpr size_t lds = K::RED + (size_t)WIDE_WAVES * K::NR * (K::NHL + K::NXL) * 1024;
  static_assert(lds <= 160 * 1024 - 64, "LDS of a compute unit");
  constexpr auto kernel = wide_chain_kernel<K::NR, K::NX, K::NXL, K::NHW, K::NHL, K::NHS, K::NB, CELL>;
  hipError_t e = allow_dynamic_lds<kernel>(lds);
  if (e != hipSuccess) return e;
  kernel<<<dim3(RES_WGS), dim3(WIDE_THREADS), lds, st>>>(p);
  return hipGetLastError();
}
template <class K, int CELL>
hipError_t launch_wide_sweep_cell(const WideSweepParams& p, hipStream_t st) {
  constexpr size_t lds = K::RED + (size_t)WIDE_WAVES * K::NR * K::GHL * 1024 + (size_t)5 * K::Tile::UW * (K::Tile::COLS + 8) * 2;
  static_assert(lds >= 4 * 1024 && lds <= 160 * 1024 - 64, "4 KiB for a workgroup that runs alone; LDS of a compute unit");
  constexpr auto kernel = wide_sweep_kernel<K::NR, K::NHW, K::GHL, K::GHS, K::NB, CELL>;
  hipError_t e = allow_dynamic_lds<kernel>(lds);
  if (e != hipSuccess) return e;
  kernel<<<dim3(RES_WGS), dim3(WIDE_THREADS), lds, st>>>(p);
  return hipGetLastError();
}
struct WideConfig {
  int nr, nhw, nb;
  hipError_t (*chain[2])(const WideChainParams&, hipStream_t);   // by cell
  hipError_t (*sweep[2])(const WideSweepParams&, hipStream_t);
};
template <class K>
WideConfig wide_config_of() {
  return WideConfig{K::NR, K::NHW, K::NB, {launch_wide_chain_cell<K, 0>, launch_wide_chain_cell<K, 1>},
                    {launch_wide_sweep_cell<K, 0>, launch_wide_sweep_cell<K, 1>}};
}
Table<WideConfig> wide_table_1(), wide_table_2(), wide_table_3();

}  // namespace mebptt
