// Executor for a chain of non-homogeneous layers (appendix "Generalizing to deep feed-forward
// networks"): runs the schedule of a mebptt_chain_plan_t on a stack of dense tanh layers
//     y_i = tanh(y_{i-1} W_i^T + b_i),   W_i [d_i, d_{i-1}],   i = 1 .. n
// of differing widths, so that forward cost u_i = d_{i-1} d_i and state size s_i = B d_i differ from
// layer to layer.  Memorised outputs live in the caller's pool at the unit offsets the plan
// assigned; everything else (the two most recent activations of a forward run, the dz of the layer being
// back-propagated and of the one below) is working memory in the caller's workspace, outside the budget.
//
// All three products of a layer run in one kernel body on fp32 MFMA tiles (v_mfma_f32_16x16x4_f32, fp32
// accumulate), operands read in place whichever way they are stored:
//   forward         y    [B, d_i]       = y_{i-1} [B, d_{i-1}] . W_i^T              then + b, tanh
//   backward data   dz'  [B, d_{i-1}]   = dz [B, d_i] . W_i                         then * (1 - y_{i-1}^2)
//   backward weight dW   [d_i, d_{i-1}] = dz^T . y_{i-1}                            (K = B), db = column sums of dz
// The epilogue of the data product turns the gradient with respect to y_{i-1} into dz of the layer below at
// once; only the last layer's dz has a launch of its own.  The two backward products of a layer need
// nothing from each other and share a launch, except where dx0 is to be written over x0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "common.h"
#include "dynamic_lds.h"

using namespace mebptt;

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// D[i][j] = sum_k A(i,k) B(j,k).  An operand is stored along k (element (i, k) at i * ld + k) or across it
// (at k * ld + i); ld in floats, rows need a float's alignment only.
struct Product {
  const float *A, *Bm;
  long lda, ldb;
  float *C, *C2;          // C2: a second copy of the result, or NULL
  long ldc;
  int M, N, K;
  const float* bias;      // BIAS_TANH: added to column j, or NULL
  const float* y;         // TIMES_DTANH: [M][ldc] values v of a tanh, the result is multiplied by 1 - v^2; NULL: stored as is
  float* db;              // A's sums over k, or NULL
  int gx;                 // workgroups along j
};
enum { BIAS_TANH, TIMES_DTANH, STORE_AND_DB };
constexpr int KS = 8;     // waves of a workgroup, which split K

// 4 values of k (4*lq .. +3 of the macro step at k0) for T tiles of 16 rows.  Operands stored along k: tile t's
// row lrow is row r0 + 16 t + lrow, one 16-byte load per tile.  Stored across k: the rows are dealt so that a
// lane's T rows are neighbours, row r0 + T * lrow + t, one T-wide load per k.  Rows past the end repeat rows
// before it (moved as a window in the second case): their results are the same values, stored twice or
// not at all.  TAIL: the macro step runs over K; surplus values are zero.  NARROW: fewer rows (or fewer k)
// than a vector: value by value.
template <bool ACROSS, int T, bool TAIL, bool NARROW>
__device__ inline void fetch_tiles(float (&v)[T][4], const float* __restrict__ base, long ld, int r0, int rows, int k0, int K, int lrow,
                                   int lq) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
  if constexpr (!ACROSS) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float* row = base + (long)min(r0 + 16 * t + lrow, rows - 1) * ld;
      if constexpr (TAIL || NARROW) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = k0 + 4 * lq + e;
          const float x = row[min(k, K - 1)];
          v[t][e] = k < K ? x : 0.0f;
        }
      } else {
        const f4u x = *reinterpret_cast<const f4u*>(row + k0 + 4 * lq);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[t][e] = x[e];
      }
    }
  } else {
    const int c = min(r0 + T * lrow, rows - T);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + 4 * lq + e;
      const float* p = base + (long)(TAIL ? min(k, K - 1) : k) * ld;
      if constexpr (NARROW) {
#pragma unroll
        for (int t = 0; t < T; ++t) v[t][e] = p[max(min(c + t, rows - 1), 0)];
      } else if constexpr (T == 4) {
        const f4u x = *reinterpret_cast<const f4u*>(p + c);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t][e] = x[t];
      } else if constexpr (T == 2) {
        const f2u x = *reinterpret_cast<const f2u*>(p + c);
        v[0][e] = x[0];
        v[1][e] = x[1];
      } else {
        v[0][e] = p[c];
      }
      if constexpr (TAIL) {
#pragma unroll
        for (int t = 0; t < T; ++t) v[t][e] = k < K ? v[t][e] : 0.0f;
      }
    }
  }
}
// The row of an operand that tile t's row x stands for.
template <bool ACROSS, int T>
__device__ inline int tile_row(int r0, int rows, int t, int x) {
  return ACROSS ? max(min(r0 + T * x, rows - T), 0) + t : r0 + 16 * t + x;
}

// One workgroup of 8 waves = TM x TN tiles of 16 x 16 outputs.  The waves split K in macro steps of 16, every
// wave covering all outputs: no operand byte is fetched twice by a workgroup, and there is no barrier inside the
// loop.  Partial sums meet in LDS and are added in a fixed order.  What bounds a product is the delivery of its
// panels through the L2s: the next macro step is requested when the MFMAs of this one have been issued, and more
// steps in flight are slower (twelve layers of 256 to 2048 units, batch 256: 455 us a gradient step at one
// step ahead, 468 and 494 us at two and three; 438 with forward products staged), as are workgroups for 512 or 128 places instead of 256 (514 and
// 488 us), and macro steps of a whole cache line per row (474 us).  The kernel before this one (a tile per wave, strided scalar
// loads, separate launches for dz, db and the copy of y) took 3543 us.
// STAGED (both operands stored along k): they pass through LDS, each wave's own part of it (no barrier).  A fragment straight from memory
// takes 16 bytes of each of 16 rows in neighbouring lanes, which the address path takes one by one; eight lanes
// that fetch a row's 128 bytes straight into LDS take it a line at a time.  A step is then 32 of k; slot c of row r holds the row's
// 16 bytes c ^ (r % 8), so that the reads of 16 rows fall into different banks.  The next step's fetches go out when the fragments
// of this one are in registers, and arrive behind its MFMAs.
constexpr int STEP = 32;   // of k, staged
template <int TM, int TN, bool STAGED>
constexpr size_t product_lds = std::max((size_t)KS * TM * TN * 256 * sizeof(float), STAGED ? (size_t)KS * 16 * (TM + TN) * STEP * sizeof(float) : 0);
template <bool A_ACROSS, bool B_ACROSS, int TM, int TN, int EPI, bool NARROW, bool STAGED>
__device__ inline void product_body(const Product& p, int id, float* red) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: conditions on it are scalar branches
  const int lrow = lane & 15, lq = lane >> 4;
  const int bx = id % p.gx, by = id / p.gx;
  const int i0 = by * TM * 16, j0 = bx * TN * 16;
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float rowsum[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) rowsum[i] = 0.0f;
  const bool sums = EPI == STORE_AND_DB && p.db != nullptr && bx == 0;
  auto use = [&](const float (&a)[TM][4], const float (&b)[TN][4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
    if (sums) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) rowsum[i] += a[i][e];
    }
  };
  if constexpr (STAGED) {
    static_assert(!A_ACROSS && !B_ACROSS, "both operands along k");
    typedef __attribute__((address_space(1))) const void global_void;
    typedef __attribute__((address_space(3))) void lds_void;
    constexpr int R = 16 * (TM + TN), NQ = R / 8;
    float* stage = red + wave * R * STEP;
    const int full = p.K / STEP, nw = (full - wave + KS - 1) / KS;   // steps wholly inside K; this wave's: wave, wave + KS, ...
    const float* src[NQ];   // this lane's 16 bytes of row 8 q + lane / 8, step 0 of the wave
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int r = 8 * q + (lane >> 3);
      const float* row = 8 * q < 16 * TM ? p.A + (long)min(i0 + r, p.M - 1) * p.lda : p.Bm + (long)min(j0 + r - 16 * TM, p.N - 1) * p.ldb;
      src[q] = row + wave * STEP + 4 * ((lane & 7) ^ (r & 7));
    }
    auto issue = [&](int n) {
#pragma unroll
      for (int q = 0; q < NQ; ++q)
        __builtin_amdgcn_global_load_lds((global_void*)(src[q] + n * (KS * STEP)), (lds_void*)(stage + q * 256), 16, 0, 0);
    };
    auto staged = [&](float (&v)[4], int r, int h) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(stage + r * STEP + 4 * ((4 * h + lq) ^ (r & 7)));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = x[e];
    };
    if (nw > 0) issue(0);
    for (int n = 0; n < nw; ++n) {
      float a[2][TM][4], b[2][TN][4];
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the step is here
      asm volatile("" ::: "memory");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < TM; ++i) staged(a[h][i], 16 * i + lrow, h);
#pragma unroll
        for (int j = 0; j < TN; ++j) staged(b[h][j], 16 * (TM + j) + lrow, h);
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): read, the stage may be filled again
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (n + 1 < nw) issue(n + 1);
      __builtin_amdgcn_sched_barrier(0);
      use(a[0], b[0]);
      use(a[1], b[1]);
    }
    if (wave == full % KS)
      for (int k0 = full * STEP; k0 < p.K; k0 += 16) {
        float a[TM][4], b[TN][4];
        fetch_tiles<A_ACROSS, TM, true, NARROW>(a, p.A, p.lda, i0, p.M, k0, p.K, lrow, lq);
        fetch_tiles<B_ACROSS, TN, true, NARROW>(b, p.Bm, p.ldb, j0, p.N, k0, p.K, lrow, lq);
        use(a, b);
      }
    __syncthreads();   // the sums take the place of the stages
  } else {
    const int full = p.K / 16;   // macro steps wholly inside K
    const int nw = (full - wave + KS - 1) / KS;   // this wave's macro steps: wave, wave + KS, ...
    float a[TM][4], b[TN][4];
    auto fetch = [&](int n) {
      const int k0 = (wave + n * KS) * 16;
      fetch_tiles<A_ACROSS, TM, false, NARROW>(a, p.A, p.lda, i0, p.M, k0, p.K, lrow, lq);
      fetch_tiles<B_ACROSS, TN, false, NARROW>(b, p.Bm, p.ldb, j0, p.N, k0, p.K, lrow, lq);
    };
    if (nw > 0) {
      fetch(0);
      for (int n = 0; n + 1 < nw; ++n) {
        use(a, b);
        fetch(n + 1);
      }
      use(a, b);
    }
    if (p.K % 16 != 0 && wave == full % KS) {
      fetch_tiles<A_ACROSS, TM, true, NARROW>(a, p.A, p.lda, i0, p.M, full * 16, p.K, lrow, lq);
      fetch_tiles<B_ACROSS, TN, true, NARROW>(b, p.Bm, p.ldb, j0, p.N, full * 16, p.K, lrow, lq);
      use(a, b);
    }
  }
  // red[wave][tile][r][lane]
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((wave * TM * TN + i * TN + j) * 4 + r) * 64 + lane] = acc[i][j][r];
  __syncthreads();
  // A thread finishes the TN values of one row that sit in one lane: neighbours in the row where B is stored across k.
#pragma unroll
  for (int item = threadIdx.x; item < TM * 4 * 64; item += KS * 64) {
    const int l = item & 63, r = (item >> 6) & 3, ti = item >> 8;
    const int i = tile_row<A_ACROSS, TM>(i0, p.M, ti, 4 * (l >> 4) + r);
    float v[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      v[j] = 0.0f;
#pragma unroll
      for (int w = 0; w < KS; ++w) v[j] += red[((w * TM * TN + ti * TN + j) * 4 + r) * 64 + l];   // fixed order
    }
    if (i >= p.M) continue;
    const int c0 = tile_row<B_ACROSS, TN>(j0, p.N, 0, l & 15);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int c = B_ACROSS ? c0 + j : c0 + 16 * j;
      if (c >= p.N) continue;
      const long e = (long)i * p.ldc + c;
      float x = v[j];
      if constexpr (EPI == BIAS_TANH) {
        x = tanhf(x + (p.bias ? p.bias[c] : 0.0f));
        if (p.C2) p.C2[e] = x;
      } else if constexpr (EPI == TIMES_DTANH) {
        if (p.y) x = x * (1.0f - p.y[e] * p.y[e]);
      }
      p.C[e] = x;
    }
  }
  if constexpr (EPI == STORE_AND_DB) {
    if (sums) {   // uniform over the workgroup
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TM; ++i) red[(wave * TM + i) * 64 + lane] = rowsum[i];
      __syncthreads();
      if ((int)threadIdx.x < TM * 16) {
        const int ti = threadIdx.x >> 4, x = threadIdx.x & 15, i = tile_row<A_ACROSS, TM>(i0, p.M, ti, x);
        float s = 0.0f;
        for (int w = 0; w < KS; ++w)
          for (int q = 0; q < 4; ++q) s += red[(w * TM + ti) * 64 + q * 16 + x];   // fixed order
        if (i < p.M) p.db[i] = s;
      }
    }
  }
}

template <int TM, int TN, bool NARROW, bool STAGED>
__global__ __launch_bounds__(KS * 64) void chain_forward_kernel(Product p) {
  extern __shared__ __attribute__((aligned(16))) float chain_smem[];
  product_body<false, false, TM, TN, BIAS_TANH, NARROW, STAGED>(p, blockIdx.x, chain_smem);
}
// The first nd workgroups compute the data product (none: nd = 0), the others, if any, the weight product.
template <int DTM, int DTN, int WTM, int WTN, bool NARROW>
__global__ __launch_bounds__(KS * 64) void chain_backward_kernel(Product data, int nd, Product weight) {
  extern __shared__ __attribute__((aligned(16))) float chain_smem[];
  if ((int)blockIdx.x < nd)
    product_body<false, true, DTM, DTN, TIMES_DTANH, NARROW, false>(data, blockIdx.x, chain_smem);
  else
    product_body<true, true, WTM, WTN, STORE_AND_DB, NARROW, false>(weight, blockIdx.x - nd, chain_smem);
}

// dz = g * (1 - y^2), elementwise over B * d values.
__global__ void chain_dz_kernel(const float* __restrict__ g, const float* __restrict__ y, float* __restrict__ dz, size_t n) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dz[i] = g[i] * (1.0f - y[i] * y[i]);
}

int blocks_of(int rows, int tiles) { return (rows + 16 * tiles - 1) / (16 * tiles); }
constexpr int FILL = 256;   // workgroups that give every compute unit one

template <int TM, int TN, bool NARROW, bool STAGED>
hipError_t launch_forward_tiles(Product& p, hipStream_t st) {
  constexpr size_t lds = product_lds<TM, TN, STAGED>;
  hipError_t e = allow_dynamic_lds<chain_forward_kernel<TM, TN, NARROW, STAGED>>(lds);
  if (e != hipSuccess) return e;
  p.gx = blocks_of(p.N, TN);
  chain_forward_kernel<TM, TN, NARROW, STAGED><<<dim3(p.gx * blocks_of(p.M, TM)), dim3(KS * 64), lds, st>>>(p);
  return hipGetLastError();
}

// The largest output block per workgroup that still gives every compute unit one.  Vectors of four along
// k (or along a row, for operands stored across k) need dimensions of at least four.
// Operands pass through LDS (product_body) where all rows are whole 16-byte slots -- `slots`, which for a layer has to be the same wherever
// its input sits, or a recomputed activation would not have the first one's bits -- and every wave has a step of 32.  us a launch, direct and staged,
// batch 256: 1024 -> 1024 (2 x 2 tiles) 11.0 and 10.2, 1024 -> 832 (1 x 2) 13.3 and 10.8, 1536 -> 512 (1 x 2) 10.6 and 8.7, 1024 -> 256 (1 x 1)
// 6.3 and 4.7.  Where it does not pay:
//   K % 32 != 0: what is left over is fetched by one wave alone when its steps are done.  1 x 1 tiles, batch 16, 284 -> 1024 3.3 and 3.8 us;
//   even at about K = 700 (less than 16 left over: 600), 0.71 - 0.98 of the time from 1024 (896) on.  1 x 2 tiles 1.05 - 1.2 of the
//   time up to K = 1000, 0.9 - 1.08 from there to 2040; 2 x 2 tiles up to 1.35 (batch 192, 2044 -> 2048 26.6 and 36.2);
//   2 x 2 tiles that give some compute units a second workgroup: batch 461, 832 -> 832 15.0 and 16.5, batch 256, 1536 -> 1536 25.0 and 27.7.  With
//   one each 0.84 - 1.04 of the time, 0.96 on average;
//   2 x 4 tiles, 11.6 and 15.7: there the stages leave a compute unit one workgroup.
// Two stages a wave, two steps in flight, were slower: 13.3 us on 2 x 2 tiles, 12.4 for 10.1 on 1 x 2.
hipError_t launch_chain_forward(Product p, bool slots, hipStream_t st) {
  if (p.K < 4) return launch_forward_tiles<1, 1, true, false>(p, st);
  if (blocks_of(p.N, 4) * blocks_of(p.M, 4) >= FILL) return launch_forward_tiles<4, 4, false, false>(p, st);
  if (blocks_of(p.N, 4) * blocks_of(p.M, 2) >= FILL) return launch_forward_tiles<2, 4, false, false>(p, st);
  const int rest = p.K % STEP;
  const bool staged = slots && p.K >= KS * STEP && rest == 0;
  const int wgs = blocks_of(p.N, 2) * blocks_of(p.M, 2);
  if (wgs >= FILL) return staged && wgs == FILL ? launch_forward_tiles<2, 2, false, true>(p, st) : launch_forward_tiles<2, 2, false, false>(p, st);
  if (blocks_of(p.N, 2) * blocks_of(p.M, 1) >= FILL) return staged ? launch_forward_tiles<1, 2, false, true>(p, st) : launch_forward_tiles<1, 2, false, false>(p, st);
  const bool long_k = slots && p.K >= (rest < 16 ? 896 : 1024);
  return staged || long_k ? launch_forward_tiles<1, 1, false, true>(p, st) : launch_forward_tiles<1, 1, false, false>(p, st);
}

template <int DTM, int DTN, int WTM, int WTN, bool NARROW>
hipError_t launch_backward_tiles(Product& data, Product& weight, hipStream_t st) {
  constexpr int tiles = DTM * DTN > WTM * WTN ? DTM * DTN : WTM * WTN;
  constexpr size_t lds = (size_t)KS * tiles * 256 * sizeof(float);
  hipError_t e = allow_dynamic_lds<chain_backward_kernel<DTM, DTN, WTM, WTN, NARROW>>(lds);
  if (e != hipSuccess) return e;
  data.gx = blocks_of(data.N, DTN);
  weight.gx = blocks_of(weight.N, WTN);
  const int nd = data.C ? data.gx * blocks_of(data.M, DTM) : 0, nw = weight.C ? weight.gx * blocks_of(weight.M, WTM) : 0;
  chain_backward_kernel<DTM, DTN, WTM, WTN, NARROW><<<dim3(nd + nw), dim3(KS * 64), lds, st>>>(data, nd, weight);
  return hipGetLastError();
}

hipError_t launch_chain_backward(Product data, Product weight, hipStream_t st) {
  const int d_in = weight.N, d_out = weight.M, B = data.M;
  if (d_in < 4 || d_out < 4) return launch_backward_tiles<1, 1, 1, 1, true>(data, weight, st);
  if (blocks_of(d_in, 4) * blocks_of(d_out, 4) >= FILL) {
    if (blocks_of(d_in, 4) * blocks_of(B, 2) >= FILL) return launch_backward_tiles<2, 4, 4, 4, false>(data, weight, st);
    return launch_backward_tiles<1, 4, 4, 4, false>(data, weight, st);
  }
  if (blocks_of(d_in, 2) * blocks_of(d_out, 2) >= FILL) return launch_backward_tiles<1, 2, 2, 2, false>(data, weight, st);
  return launch_backward_tiles<1, 1, 1, 1, false>(data, weight, st);
}

unsigned blocks_for(size_t n) { return (unsigned)std::min<size_t>((n + 255) / 256, 2048); }

bool overlap(const float* a, const float* b, size_t n) { return a < b + n && b < a + n; }

constexpr size_t ALIGN = 256;
size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

int check_chain_desc(const mebptt_chain_desc* d) {
  if (!d) return set_error(MEBPTT_EINVAL, "desc is NULL");
  if (d->n < 1 || d->B < 1 || !d->widths) return set_error(MEBPTT_EINVAL, "a chain needs n >= 1 layers, B >= 1 and widths");
  for (int i = 0; i <= d->n; ++i)
    if (d->widths[i] < 1 || d->widths[i] > (1 << 20)) return set_error(MEBPTT_EINVAL, "width %d is out of range", i);
  if (d->unit_bytes < 4 || d->unit_bytes % 4) return set_error(MEBPTT_EINVAL, "unit_bytes must be a positive multiple of 4");
  return MEBPTT_OK;
}

size_t max_width(const mebptt_chain_desc* d) {
  int w = 0;
  for (int i = 0; i <= d->n; ++i) w = std::max(w, d->widths[i]);
  return (size_t)w;
}

#define HIP_TRY(expr)                                                                                 \
  do {                                                                                                \
    hipError_t e_ = (expr);                                                                           \
    if (e_ != hipSuccess) return set_error(MEBPTT_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

}  // namespace


extern "C" {

int mebptt_chain_layers(const mebptt_chain_desc* desc, mebptt_layer* out) {
  int rc = check_chain_desc(desc);
  if (rc) return rc;
  if (!out) return set_error(MEBPTT_EINVAL, "out is NULL");
  for (int i = 1; i <= desc->n; ++i) {
    out[i - 1].cost = (int64_t)desc->widths[i - 1] * desc->widths[i];
    const size_t bytes = (size_t)desc->B * desc->widths[i] * sizeof(float);
    out[i - 1].state_units = (int32_t)((bytes + desc->unit_bytes - 1) / desc->unit_bytes);
    out[i - 1].work_units = 0;   // working memory is the caller's workspace, outside the budget
  }
  return MEBPTT_OK;
}

size_t mebptt_chain_workspace_bytes(const mebptt_chain_desc* desc) {
  if (check_chain_desc(desc) != MEBPTT_OK) return 0;
  // two activations, the dz of a layer and of the layer below it, each of the widest layer
  return 4 * align_up((size_t)desc->B * max_width(desc) * sizeof(float));
}

int mebptt_chain_run(const mebptt_chain_desc* desc, const mebptt_chain_plan_t* plan, const float* const* W,
                     const float* const* b, const float* x0, const float* dy, void* pool, size_t pool_bytes,
                     void* workspace, size_t workspace_bytes, float* const* dW, float* const* db, float* dx0,
                     float* y_out, mebptt_chain_stats* stats, void* stream) {
  int rc = check_chain_desc(desc);
  if (rc) return rc;
  if (!plan) return set_error(MEBPTT_EINVAL, "plan is NULL");
  if (!W || !b || !x0 || !dy || !dW || !db) return set_error(MEBPTT_EINVAL, "a required pointer is NULL");
  const int n = desc->n, B = desc->B;
  for (int i = 0; i < n; ++i)
    if (!W[i] || !dW[i] || !db[i]) return set_error(MEBPTT_EINVAL, "layer %d: W, dW and db are required", i + 1);
  if (!workspace) return set_error(MEBPTT_EWORKSPACE, "workspace is NULL");
  if (workspace_bytes < mebptt_chain_workspace_bytes(desc))
    return set_error(MEBPTT_EWORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes,
                     mebptt_chain_workspace_bytes(desc));
  if ((reinterpret_cast<uintptr_t>(workspace) | reinterpret_cast<uintptr_t>(pool)) & (ALIGN - 1))
    return set_error(MEBPTT_EWORKSPACE, "pool and workspace must be 256-byte aligned");
  size_t nops = 0;
  const mebptt_chain_op* ops = mebptt_chain_plan_schedule(plan, &nops);
  if (!ops || nops == 0) return set_error(MEBPTT_EINVAL, "the plan carries no schedule");

  // the plan must have been made for this chain: same layer count, state sizes that match the widths
  std::vector<mebptt_layer> layers(n);
  rc = mebptt_chain_layers(desc, layers.data());
  if (rc) return rc;
  {
    int32_t pn = 0;
    const mebptt_layer* pl = mebptt_chain_plan_layers(plan, &pn);
    if (pn != n) return set_error(MEBPTT_ESHAPE, "the plan is for %d layers, the descriptor has %d", pn, n);
    for (int i = 0; i < n; ++i)
      if (pl[i].cost != layers[i].cost || pl[i].state_units != layers[i].state_units || pl[i].work_units != layers[i].work_units)
        return set_error(MEBPTT_ESHAPE, "layer %d of the plan does not match the descriptor (see mebptt_chain_layers)", i + 1);
  }
  const size_t unit = desc->unit_bytes;
  // Host-side check of every location before anything is enqueued.
  int64_t high_water = 0;
  int backward_seen = 0;
  for (size_t k = 0; k < nops; ++k) {
    const mebptt_chain_op& o = ops[k];
    if (o.layer < 1 || o.count < 1 || o.layer + o.count - 1 > n) return set_error(MEBPTT_ESHAPE, "schedule names a layer outside the chain");
    if (o.op == MEBPTT_CHAIN_FORWARD) {
      if (o.src >= 0) {
        if (o.layer < 2) return set_error(MEBPTT_ESHAPE, "schedule reads a memorised state below the first layer");
        high_water = std::max<int64_t>(high_water, (int64_t)o.src + layers[o.layer - 2].state_units);
      } else if (o.src != MEBPTT_CHAIN_INPUT) {
        return set_error(MEBPTT_ESHAPE, "a forward run must start from the input or a memorised state");
      } else if (o.layer != 1) {
        return set_error(MEBPTT_ESHAPE, "only the first layer reads the network input");
      }
      if (o.dst >= 0)
        high_water = std::max<int64_t>(high_water, (int64_t)o.dst + layers[o.layer + o.count - 2].state_units);
      else if (o.dst != MEBPTT_CHAIN_WORKING)
        return set_error(MEBPTT_ESHAPE, "unknown destination %d", o.dst);
    } else if (o.op == MEBPTT_CHAIN_BACKWARD) {
      if (o.layer != n - backward_seen) return set_error(MEBPTT_ESHAPE, "backward operations out of order");
      ++backward_seen;
      if (o.src >= 0) {
        if (o.layer < 2) return set_error(MEBPTT_ESHAPE, "schedule reads a memorised state below the first layer");
        high_water = std::max<int64_t>(high_water, (int64_t)o.src + layers[o.layer - 2].state_units);
      } else if (o.src == MEBPTT_CHAIN_INPUT ? o.layer != 1 : o.src != MEBPTT_CHAIN_WORKING) {
        return set_error(MEBPTT_ESHAPE, "unknown source %d", o.src);
      }
    } else {
      return set_error(MEBPTT_EINVAL, "unknown schedule entry %d", o.op);
    }
  }
  if (backward_seen != n) return set_error(MEBPTT_ESHAPE, "the plan is for another number of layers");
  if (high_water > 0 && !pool) return set_error(MEBPTT_ENOMEM_SLOTS, "pool is NULL");
  if ((size_t)high_water * unit > pool_bytes)
    return set_error(MEBPTT_ENOMEM_SLOTS, "pool has %zu bytes, the schedule reaches %zu", pool_bytes, (size_t)high_water * unit);

  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* ws = reinterpret_cast<char*>(workspace);
  const size_t slab = align_up((size_t)B * max_width(desc) * sizeof(float));
  float* act[2] = {reinterpret_cast<float*>(ws), reinterpret_cast<float*>(ws + slab)};
  float* dzs[2] = {reinterpret_cast<float*>(ws + 2 * slab), reinterpret_cast<float*>(ws + 3 * slab)};
  auto pool_at = [&](int32_t off) { return reinterpret_cast<float*>(reinterpret_cast<char*>(pool) + (size_t)off * unit); };

  // working memory after a forward run: `wk_out` = its last output, `wk_in` = the activation before it
  const float* wk_in = nullptr;
  const float* wk_out = nullptr;
  int flip = 0, zflip = 0;   // dzs[zflip]: dz of the layer back-propagated next (filled by the layer above)
  int64_t forward_cost = 0, backward_ops = 0;

  for (size_t k = 0; k < nops; ++k) {
    const mebptt_chain_op& o = ops[k];
    if (o.op == MEBPTT_CHAIN_FORWARD) {
      const float* a = o.src == MEBPTT_CHAIN_INPUT ? x0 : pool_at(o.src);
      const float* before = nullptr;
      for (int i = 0; i < o.count; ++i) {
        const int L = o.layer + i;                         // 1-based layer
        const int din = desc->widths[L - 1], dout = desc->widths[L];
        const bool last = i == o.count - 1;
        float* out = (last && o.dst >= 0) ? pool_at(o.dst) : act[flip];
        if (!(last && o.dst >= 0)) flip ^= 1;
        Product p{};
        p.A = a;
        p.lda = din;
        p.Bm = W[L - 1];
        p.ldb = din;
        p.C = out;
        p.C2 = L == n ? y_out : nullptr;
        p.ldc = dout;
        p.M = B;
        p.N = dout;
        p.K = din;
        p.bias = b[L - 1];
        // the input sits in x0, in the pool (256-byte aligned, units apart) or in the workspace
        auto aligned = [](const float* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; };
        const bool slots = din % 4 == 0 && aligned(W[L - 1]) && (L == 1 ? aligned(x0) : unit % 16 == 0);
        HIP_TRY(launch_chain_forward(p, slots, st));
        forward_cost += layers[L - 1].cost;
        before = a;
        a = out;
      }
      wk_in = before;
      wk_out = a;
    } else {
      const int L = o.layer, din = desc->widths[L - 1], dout = desc->widths[L];
      const float* xin = o.src == MEBPTT_CHAIN_INPUT ? x0 : (o.src == MEBPTT_CHAIN_WORKING ? wk_in : pool_at(o.src));
      if (!wk_out || !xin) return set_error(MEBPTT_ESHAPE, "backward operation without a forward operation before it");
      if (L == n) {
        const size_t ne = (size_t)B * dout;
        chain_dz_kernel<<<blocks_for(ne), 256, 0, st>>>(dy, wk_out, dzs[zflip], ne);
        HIP_TRY(hipGetLastError());
      }
      const float* dz = dzs[zflip];
      Product data{}, weight{};
      data.A = dz;
      data.lda = dout;
      data.Bm = W[L - 1];
      data.ldb = din;
      data.C = L == 1 ? dx0 : dzs[zflip ^ 1];   // NULL: nobody wants dx0
      data.ldc = din;
      data.M = B;
      data.N = din;
      data.K = dout;
      data.y = L == 1 ? nullptr : xin;          // y_{L-1}: dz of the layer below at once
      weight.A = dz;
      weight.lda = dout;
      weight.Bm = xin;
      weight.ldb = din;
      weight.C = dW[L - 1];
      weight.ldc = din;
      weight.M = dout;
      weight.N = din;
      weight.K = B;
      weight.db = db[L - 1];
      if (L == 1 && dx0 && overlap(dx0, x0, (size_t)B * din)) {   // dx0 takes the place of x0: after its last reader
        Product no_data = data, no_weight = weight;
        no_data.C = nullptr;
        no_weight.C = nullptr;
        HIP_TRY(launch_chain_backward(no_data, weight, st));
        HIP_TRY(launch_chain_backward(data, no_weight, st));
      } else {
        HIP_TRY(launch_chain_backward(data, weight, st));
      }
      zflip ^= 1;
      ++backward_ops;
      wk_out = nullptr;   // consumed: the next backward operation needs its own forward operation
    }
  }
  if (stats) {
    stats->forward_cost = forward_cost;
    stats->backward_ops = backward_ops;
    stats->peak_units = (int32_t)high_water;
    stats->reserved = 0;
  }
  return MEBPTT_OK;
}

}  // extern "C"
