// Device-side building blocks shared by the kernel files: MFMA operand traits, the fragment-tiled
// layout, the h plane of a state unit, the pointwise steps, and the shape rules that fix how a
// shape's sums are split.  Not part of the ABI.
#pragma once

#include <type_traits>

#include "kernels.h"

namespace mebptt {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) __bf16 bf16x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// ---- operand traits ------------------------------------------------------------------------

template <class T>
struct Mma;

template <>
struct Mma<__bf16> {
  static constexpr int VEC = 8;
  using Frag = bf16x8;
  __device__ static Frag load(const __bf16* p) { return *reinterpret_cast<const Frag*>(p); }
  __device__ static Frag from_f32(const float (&v)[8]) {
    Frag f;
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = (__bf16)v[e];
    return f;
  }
  __device__ static f32x4 mma(Frag a, Frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Mma<float> {
  static constexpr int VEC = 4;
  using Frag = f32x4;
  __device__ static Frag load(const float* p) { return *reinterpret_cast<const Frag*>(p); }
  __device__ static Frag from_f32(const float (&v)[4]) { return Frag{v[0], v[1], v[2], v[3]}; }
  __device__ static f32x4 mma(Frag a, Frag b, f32x4 c) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
    return c;
  }
};

// Pointwise activations on the hardware exp2 / reciprocal units (a few ulp; the absolute error of
// tanh stays below 1e-7, far inside the fp32 gradient tolerance).  The reciprocals with one Newton step are as good as a
// division (within an ulp of 2^-24 either way) at a third of its instructions, and a step of a resident launch has little
// else to do between two exchanges: a gradient step of H = 1024, B = 64 10.67 -> 10.49 ms, of H = 512, B = 256 107.0 -> 104.5.
// With fp32 operands both keep the division: tanh alone with it is worth -1 - +1 % over eleven shapes (H = 100, B = 24, t = 150
// 1322 -> 1335 us), neither makes the launches with forward operations of H = 256, B = 32 5 % slower (1705 -> 1795 us a gradient
// step; unexplained).
__device__ inline float reciprocal(float d) {   // of d >= 1, infinity included
  const float r = __builtin_amdgcn_rcpf(d);
  return d < 3e38f ? __fmaf_rn(__fmaf_rn(-d, r, 1.0f), r, r) : r;
}
template <class T>
__device__ inline float sigmoidf_(float z) {
  const float d = 1.0f + __expf(-z);
  return sizeof(T) == 2 ? reciprocal(d) : __frcp_rn(d);
}
template <class T>
__device__ inline float tanhf_(float z) {
  const float e = __expf(-2.0f * fabsf(z));            // in (0, 1]: no overflow
  const float d = 1.0f + e;
  float r;
  if constexpr (sizeof(T) == 2) {
    r = __builtin_amdgcn_rcpf(d);
    r = __fmaf_rn(__fmaf_rn(-d, r, 1.0f), r, r);
  } else {
    r = __frcp_rn(d);
  }
  return copysignf(__fmul_rn(1.0f - e, r), z);
}

// ---- the h plane of a hidden-state unit ----------------------------------------------------------
// (layout described in kernels.h).  HPlane<T>::store/load hide whether h is a plain fp32 plane or
// the split, fragment-tiled pair of 16-bit planes.
template <class T>
struct HPlane;

template <>
struct HPlane<float> {
  static constexpr bool SPLIT = false;
  __device__ static void store(float* plane, int b, int u, float v, int, int H, size_t) { plane[(size_t)b * H + u] = v; }
  __device__ static float load(const float* plane, int b, int u, int, int H, size_t) { return plane[(size_t)b * H + u]; }
  __device__ static float as_operand(const float* plane, int b, int u, int, int H, size_t) {
    return plane[(size_t)b * H + u];
  }
};

template <class T>
__device__ inline size_t ft_offset(int row, int k, int nsteps);

template <>
struct HPlane<__bf16> {
  static constexpr bool SPLIT = true;
  // nsh = KH / 32 macro steps per batch tile; half = BP * KH elements per 16-bit plane
  __device__ static void store(float* plane, int b, int u, float v, int nsh, int, size_t half) {
    unsigned short* hi = reinterpret_cast<unsigned short*>(plane);
    const unsigned bits = __float_as_uint(v);
    const size_t o = ft_offset<__bf16>(b, u, nsh);
    hi[o] = (unsigned short)((bits + 0x8000u) >> 16);
    hi[half + o] = (unsigned short)(bits & 0xffffu);
  }
  __device__ static float load(const float* plane, int b, int u, int nsh, int, size_t half) {
    const unsigned short* hi = reinterpret_cast<const unsigned short*>(plane);
    const size_t o = ft_offset<__bf16>(b, u, nsh);
    const unsigned lo = hi[half + o];
    return __uint_as_float((((unsigned)hi[o] - (lo >> 15)) << 16) | lo);
  }
  __device__ static __bf16 as_operand(const float* plane, int b, int u, int nsh, int, size_t) {
    const __bf16* hi = reinterpret_cast<const __bf16*>(plane);
    return hi[ft_offset<__bf16>(b, u, nsh)];
  }
};

// Operand arrays the library builds itself are stored "fragment-tiled": for a logical matrix
// M[rows][K] the element (row, k) lives at
//     (((row/16) * (K/KSTEP) + k/KSTEP) * 64 + ((k%KSTEP)/VEC)*16 + row%16) * VEC + k%VEC
// so that the 64 lanes of a wave fetch the fragment of one 16-row tile and one macro step as one
// contiguous, fully coalesced block of 64*VEC elements (1 KiB).
template <class T>
__device__ inline void ft_decode(size_t idx, int nsteps, int& row, int& k) {
  constexpr int VEC = Mma<T>::VEC, KSTEP = 4 * VEC;
  const int e = (int)(idx % VEC);
  const int lane = (int)((idx / VEC) % 64);
  const size_t blk = idx / (VEC * 64);
  const int kstep = (int)(blk % nsteps);
  const int tile = (int)(blk / nsteps);
  row = tile * 16 + (lane & 15);
  k = kstep * KSTEP + (lane >> 4) * VEC + e;
}

template <class T>
__device__ inline size_t ft_offset(int row, int k, int nsteps) {
  constexpr int VEC = Mma<T>::VEC, KSTEP = 4 * VEC;
  return ((((size_t)(row >> 4) * nsteps + k / KSTEP) * 64 + ((k % KSTEP) / VEC) * 16 + (row & 15)) * VEC) + k % VEC;
}

// The four packed rows 4u .. 4u+3 of hidden unit u, and which gate block of the caller's W_ih / W_hh
// feeds each of them (-1: that half of the row is zero).
//   LSTM: rows i, f, g, o, both halves from the same gate block.
//   GRU:  rows r, z, n_x, n_h.  The candidate's input part and recurrent part are kept as two rows
//         (n = tanh(n_x + r * n_h)), so one GEMM with the same 4-rows-per-unit shape serves both cells.
__host__ __device__ inline int packed_gate_x(int cell, int row) { return cell == 0 ? row : (row < 3 ? row : -1); }
__host__ __device__ inline int packed_gate_h(int cell, int row) { return cell == 0 ? row : (row == 2 ? -1 : (row == 3 ? 2 : row)); }

// ---- pointwise forward step of one (sequence, hidden unit) -------------------------------------
// G: the four gate-GEMM results of the unit (packed rows), bias: their biases, state_prev: c_{s-1}
// (LSTM) or h_{s-1} in full precision (GRU).  Returns h_s; `second` is what the second plane of
// the state unit keeps (LSTM: c_s; GRU: the recurrent part n_h of the candidate), `gate` the
// values the backward step needs (LSTM: i, f, g, o; GRU: r, z, n).  Every kernel that computes a
// forward step calls this one function, with the multiply-adds spelled out, so that a step gives
// the same bits whichever kernel ran it.
template <class T, int CELL>
__device__ inline float cell_forward(const float (&G)[4], const float4& bias, float state_prev, float& second,
                                     float (&gate)[4]) {
  if (CELL == 0) {
    const float gi = sigmoidf_<T>(G[0] + bias.x);
    const float gf = sigmoidf_<T>(G[1] + bias.y);
    const float gg = tanhf_<T>(G[2] + bias.z);
    const float go = sigmoidf_<T>(G[3] + bias.w);
    const float c = __fmaf_rn(gf, state_prev, __fmul_rn(gi, gg));
    gate[0] = gi;
    gate[1] = gf;
    gate[2] = gg;
    gate[3] = go;
    second = c;
    return __fmul_rn(go, tanhf_<T>(c));
  } else {
    // rows r, z, n_x, n_h: n = tanh(n_x + r * n_h), h = (1 - z) n + z h_prev
    const float r = sigmoidf_<T>(G[0] + bias.x);
    const float z = sigmoidf_<T>(G[1] + bias.y);
    const float nh = G[3] + bias.w;
    const float n = tanhf_<T>(__fmaf_rn(r, nh, G[2] + bias.z));
    gate[0] = r;
    gate[1] = z;
    gate[2] = n;
    gate[3] = 0.0f;
    second = nh;
    return __fmaf_rn(1.0f - z, n, __fmul_rn(z, state_prev));
  }
}

// Pointwise backward step of one (sequence, hidden unit) of the LSTM: from dh_s (recurrent part
// plus injected loss gradient), the running dc, the internal state (i, f, g, o, c_s) and c_{s-1}
// to the four gate pre-activation gradients and dc_{s-1}.  One function, multiply-adds spelled
// out, for every kernel that runs a backward step: the same bits whichever kernel ran it.
template <class T>
__device__ inline void lstm_backward_point(float dh, float dc_in, float gi, float gf, float gg, float go, float c_s,
                                           float c_prev, float (&dG)[4], float& dc_out) {
  const float tc = tanhf_<T>(c_s);
  const float d_o = __fmul_rn(dh, tc);
  const float dct = __fmaf_rn(__fmul_rn(dh, go), __fmaf_rn(-tc, tc, 1.0f), dc_in);
  dG[0] = __fmul_rn(__fmul_rn(__fmul_rn(dct, gg), gi), __fsub_rn(1.0f, gi));
  dG[1] = __fmul_rn(__fmul_rn(__fmul_rn(dct, c_prev), gf), __fsub_rn(1.0f, gf));
  dG[2] = __fmul_rn(__fmul_rn(dct, gi), __fmaf_rn(-gg, gg, 1.0f));
  dG[3] = __fmul_rn(__fmul_rn(d_o, go), __fsub_rn(1.0f, go));
  dc_out = __fmul_rn(dct, gf);
}

// The same for the GRU: r, z, n the gates, nh the recurrent part of the candidate (n = tanh(n_x + r * nh)),
// h_prev = h_{s-1} in full precision.  dh is the whole dL/dh_s: the GEMM part, the injected loss
// gradient and the part that bypasses the GEMM (dh_{s+1} * z_{s+1}, carried in the running plane).
// dG: gradients of the packed rows r, z, n_x, n_h; carry: what step s - 1 adds to its dh.
__device__ inline void gru_backward_point(float dh, float r, float z, float n, float nh, float h_prev, float (&dG)[4],
                                          float& carry) {
  const float da_n = __fmul_rn(__fmul_rn(dh, __fsub_rn(1.0f, z)), __fmaf_rn(-n, n, 1.0f));
  dG[0] = __fmul_rn(__fmul_rn(__fmul_rn(da_n, nh), r), __fsub_rn(1.0f, r));
  dG[1] = __fmul_rn(__fmul_rn(__fmul_rn(dh, __fsub_rn(h_prev, n)), z), __fsub_rn(1.0f, z));
  dG[2] = da_n;
  dG[3] = __fmul_rn(da_n, r);
  carry = __fmul_rn(dh, z);
}

// Raw (unconverted) activation fragment: VEC fp32 values, zero beyond `limit`.
template <int VEC>
struct RawAct {
  float v[VEC];
};
template <int VEC>
__device__ inline RawAct<VEC> load_raw(const float* __restrict__ row, int k, int limit, bool vec_ok) {
  RawAct<VEC> r;
  if (vec_ok && k + VEC <= limit) {
#pragma unroll
    for (int e = 0; e < VEC; e += 4) {
      float4 q = *reinterpret_cast<const float4*>(row + k + e);
      r.v[e] = q.x;
      r.v[e + 1] = q.y;
      r.v[e + 2] = q.z;
      r.v[e + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < VEC; ++e) r.v[e] = (k + e < limit) ? row[k + e] : 0.0f;
  }
  return r;
}

// As load_raw for rows whose length is a multiple of VEC (k is one too): a fragment lies wholly
// inside the row or wholly outside, so one address clamp and one select replace the branches.
// (Branches that load into the same registers make the compiler wait for every outstanding memory
// operation between them.)
template <int VEC>
__device__ inline RawAct<VEC> load_raw_whole(const float* __restrict__ row, int k, int limit) {
  RawAct<VEC> r;
  const bool inside = k < limit;
  const float* src = row + (inside ? k : 0);
#pragma unroll
  for (int e = 0; e < VEC; e += 4) {
    const float4 q = *reinterpret_cast<const float4*>(src + e);
    r.v[e] = inside ? q.x : 0.0f;
    r.v[e + 1] = inside ? q.y : 0.0f;
    r.v[e + 2] = inside ? q.z : 0.0f;
    r.v[e + 3] = inside ? q.w : 0.0f;
  }
  return r;
}

// A barrier that orders LDS only: stores to memory stay in flight across it.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <class F>
__device__ inline F as_frag(u32x4 v) {
  union { u32x4 u; F f; } cv;
  cv.u = v;
  return cv.f;
}

// Fragments of fp32 rows of any length.  A lane's VEC values start at k; where they would run over the end
// of the row (`limit` values, at least VEC) the VEC last values of the row are fetched instead, and
// shift_tail puts them where they belong when they are used: fetching has no branches (loads under
// branches make the compiler wait for everything outstanding), and needs only a float's alignment.
template <int VEC>
__device__ inline RawAct<VEC> load_window(const float* __restrict__ base, unsigned row, int k, int limit) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  RawAct<VEC> r;
  const unsigned off = row + (unsigned)min(k, limit - VEC);
#pragma unroll
  for (int e = 0; e < VEC; e += 4) {
    const f4u q = *reinterpret_cast<const f4u*>(base + (size_t)off + e);
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[e + i] = q[i];
  }
  return r;
}
template <int VEC>
__device__ inline void shift_tail(RawAct<VEC>& r, int k, int limit) {
  const int d = k + VEC - limit;   // how far the window was moved back: <= 0 not at all, >= VEC all of it lies outside
#pragma unroll
  for (int bit = 1; bit < VEC; bit *= 2)
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float from = e + bit < VEC ? r.v[e + bit] : 0.0f;
      r.v[e] = (d > 0 && (d & bit)) ? from : r.v[e];
    }
#pragma unroll
  for (int e = 0; e < VEC; ++e) r.v[e] = d >= VEC ? 0.0f : r.v[e];
}

// Products with at most eight columns (sequences), bf16.  A 16 x 16 tile would be half empty and the matrix unit take as
// long, so the idle half takes another part of K: in the structured-sparse instruction every row of the first operand picks two of
// each four k of the dense one.  The dense operand holds two macro steps of 16 weight rows side by side, k in twos; rows 0 - 7
// of the other are the sequences' fragments of the first macro step, picking those twos, rows 8 - 15 their fragments of the
// second.  One instruction in the time of a dense one (16 cycles) thus does two macro steps, every lane of a fetched fragment
// carries data, and each of the two sums has the bits the dense instruction gives (measured on random operands of several
// magnitudes, all 51 200 values alike).
// D: lane (column j = weight row, group lq) holds sequences 4 lq .. 4 lq + 3 of the first macro step's sums (lq < 2), then of the second's.
struct Halves {
  __device__ static int picks(int lane) { return lane & 8 ? 0xeeee : 0x4444; }   // of each four k, the last or the first two
  // The dense operand, loaded: `row` is the byte offset of row j of the tile's fragment of macro step 0, e and o the two macro steps;
  // zeros from `end` on.  A lane fetches two whole slots, of e where lq is even, of o where it is odd (lane groups lq / 2 and
  // 2 + lq / 2 of the fragment), and neighbouring groups swap the halves they need.  (Fetching 8 bytes of each of four fragments
  // instead: launches of few steps 2 - 4 % slower, H = 832, B = 15, t = 22 292 against 303 us a gradient step.)
  __device__ static bf16x16 load(const void* weights, unsigned row, int e, int o, int end, int lq) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(weights), 0, 0x7fffffff, 0x00020000);
    const int mine = lq & 1 ? o : e;
    const unsigned at = mine < end ? row + 1024u * (unsigned)mine + 256u * (unsigned)(lq >> 1) : 0x80000000u;
    union { unsigned u[8]; bf16x16 f; } r;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 512 * k, 0);
      const auto a = __builtin_amdgcn_permlane16_swap(v.x, v.z, false, false), b = __builtin_amdgcn_permlane16_swap(v.y, v.w, false, false);
      r.u[4 * k] = a[0];
      r.u[4 * k + 1] = a[1];
      r.u[4 * k + 2] = b[0];
      r.u[4 * k + 3] = b[1];
    }
    return r.f;
  }
  __device__ static f32x4 mma(bf16x8 h, bf16x16 w, f32x4 c, int picks) {
    return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(h, w, c, picks, 0, 0);
  }
  // Both sums added: of lane (j, lq), element r: sequence 4 (lq & 1) + 2 (lq >> 1) + r.
  struct Sum {
    float v[2];
  };
  __device__ static Sum fold(f32x4 a) {
    Sum s;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[r]), __float_as_uint(a[r + 2]), false, false);
      s.v[r] = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    }
    return s;
  }
  __device__ static int lane_of(int j, int seq) { return j + 16 * (seq >> 2) + 32 * ((seq >> 1) & 1); }
};

// Kernel configurations by shape.  Tiles per workgroup grow with the problem so that the grid
// stays near one workgroup per compute unit while every operand byte is reused as often as
// possible; the choice depends on the shape only, never on the schedule.
enum FwdConfig { FWD_TINY, FWD_SMALLK, FWD_B1, FWD_42, FWD_82 };
enum BwdConfig { BWD_SMALLK, BWD_11, BWD_12, BWD_21, BWD_22 };
constexpr int TARGET_WGS = 256;

template <class T>
inline FwdConfig forward_config(const Dims& d) {
  const int nsteps = d.KP / (4 * Mma<T>::VEC);
  if (nsteps <= 8) return FWD_TINY;
  if (nsteps <= 20) return FWD_SMALLK;
  const int ngroups = d.HP / 4, bt = d.BP / 16;
  if (bt >= 2 && ((ngroups + 7) / 8) * ((bt + 1) / 2) >= TARGET_WGS) return FWD_82;
  if (bt >= 2 && ((ngroups + 3) / 4) * ((bt + 1) / 2) >= TARGET_WGS) return FWD_42;
  return FWD_B1;
}

template <class T>
inline BwdConfig backward_config(const Dims& d) {
  const int nsteps = d.G4 / (4 * Mma<T>::VEC);
  if (nsteps <= 16) return BWD_SMALLK;
  const int nt = d.HP / 16, bt = d.BP / 16;
  if (nt >= 2 && bt >= 2 && ((nt + 1) / 2) * ((bt + 1) / 2) >= TARGET_WGS) return BWD_22;
  if (bt >= 2 && nt * ((bt + 1) / 2) >= TARGET_WGS) return BWD_12;
  return BWD_11;
}

// Shapes whose resident launches spread one copy of the weights over `groups` equal parts of the device (see
// resident_wide.h): bf16 operands too wide, or batches too large, for a copy per XCD.  groups parts of 256 / groups
// compute units each take `share` sequences; a compute unit has nr 16-row tiles of a product's rows.  groups 0: not such
// a shape.  Against a launch per step with eight-way split sums, a gradient step of 121 calls in these ranges takes 0.48 - 0.99 of the
// time (H = 2048, B = 128, t = 1000 54.5 -> 32.3 ms; H = 4096, B = 32 103.8 -> 50.9 ms; B = 1 and 16, which leave one of two groups
// without sequences, t = 40 0.48 - 0.80).  The sums of more sequences do not fit beside the weights; up
// to H = 1024 and B = 128 a copy per XCD fits, whose steps take 2 - 2.5 us for a wide one's 5 - 7.
// The K splits of every kernel that runs a step of such a shape follow from what a compute unit's four
// waves can add up: see WIDE_FWD_KS and sum_back_parts.
struct WideShape {
  int groups, share, nr;
};
constexpr size_t WIDE_X_BYTES = (size_t)32 << 20;   // x of a chain launch's steps as operands: as many steps as this holds
inline WideShape wide_shape(const Dims& d) {
  WideShape w{};
  if (d.dtype == 0 || d.I < 8 || d.KP / 32 <= 20) return w;   // (20: the forward kernels that split K four ways)
  int groups = 0;
  if (d.KH > 512 && d.KH <= 1024 && d.B > 128 && d.B <= 256) groups = 4;
  if (d.KH > 1024 && d.KH <= 2048 && d.B <= 128) groups = 2;
  if (d.KH > 2048 && d.KH <= 4096 && d.B <= 32) groups = 1;
  if (!groups) return w;
  // The resident launches address these operands by 32-bit byte offsets, and offsets from 2^31 on mean that there is nothing to
  // fetch: inputs of more than 61 000 columns (H = 4096) go out a launch per step, whose kernels have 64-bit offsets.
  constexpr size_t LIMIT = (size_t)1 << 31;
  if ((size_t)d.G4 * d.KP * 2 >= LIMIT || (size_t)d.G4 * d.KC * 2 >= LIMIT || (size_t)d.NA * d.KC * 2 >= LIMIT) return w;
  if ((size_t)d.BP * d.KX * 2 > WIDE_X_BYTES) return w;   // not one step's x fits the staging
  // Weights of x beyond what stays on the chip are streamed in every step, by one wave per SIMD with three macro steps in flight;
  // where a batch is small and half of the device streams them all, launches per step with eight waves a compute unit
  // are as fast from I = 4096 on.  A gradient step of t = 40, wide against per step: B = 1, H = 2048, I = 4096 0.95, 5000 1.03, 10000
  // 1.14; B = 1, I = 10000, H = 1792 1.11, H = 1536 1.04, H = 1280 0.98; B = 32, H = 2048, I = 4096 0.93, 6000 1.04, 10000 1.10, H = 1536
  // 0.96.  (With two batch tiles only if both tiles of a row land on one XCD, or the launches per step fetch the weights
  // twice: H = 1600, 1856, 1984 0.82 - 0.83.  More sequences, wider states, more groups: 0.55 - 0.97 at any I measured, to 24576.)
  if (groups == 2 && d.KX > 4096 && (d.BP == 16 ? d.KH > 1280 : d.BP == 32 && d.KH > 1536 && d.HP % 128 == 0)) return w;
  w.groups = groups;
  w.share = round_up((d.B + groups - 1) / groups, 16);
  w.nr = (d.KH * groups + 1023) / 1024;
  return w;
}

// Gate sums of a forward step whose K is split eight ways, bf16 operands: neighbouring parts are added first, then the four pairs
// in order.  (One instruction gives both parts of a pair in the launches of up to 64 sequences, see Halves.)  Other splits add
// one part after the other, in loops of their own: with both orders behind one function that took the array of sums, the compiler
// laid all chain kernels out differently, and K split four ways (H = 64, I = 128, B = 192) took 84 us a launch for 81, fp32 0.9 % more.
template <class T, int KS>
constexpr bool parts_in_pairs = sizeof(T) == 2 && KS == 8;
template <int KS, class Part>
__device__ __forceinline__ void add_pairs(float (&G)[4], Part&& part) {
#pragma unroll
  for (int w = 0; w < KS; w += 2) {
    const f32x4 v = part(w) + part(w + 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) G[r] += v[r];
  }
}
// Backward steps of up to 64 sequences, bf16 operands, K split eight ways: each of the eight keeps its even and its odd macro
// steps apart and adds the two sums before the eight are added in order.
inline bool backward_in_halves(const Dims& d) {
  return d.dtype && d.B <= 64 && d.KH <= 1024 && !wide_shape(d).groups && backward_config<__bf16>(d) == BWD_11;
}

constexpr int WIDE_FWD_KS = 4;   // K split of a forward step of a wide shape
// Tiles of a wide shape's launch-per-step kernels, which run it where resident launches do not (switched off, or fewer than 256
// compute units), with the resident launches' K splits and so their bits.  unit groups x batch tiles of a workgroup, macro steps in
// flight.  Four waves a workgroup instead of the other shapes' eight, so small tiles pay longer: 2 x 2 (a batch tile: 2 x 1) up to
// half a workgroup per compute unit (us a launch, 4 x 2 against it: B = 8, H = 1100 5.5 / 4.5; B = 32, I = 512, H = 2048 12.7 / 10.4;
// at B = 64, H = 1280, 160 workgroups, 7.1 / 9.6).  Four macro steps in flight instead of two where a workgroup has the compute
// unit to itself and the x part of a wave is at least four long (it is fetched in whole fours): B = 64, I = 512, H = 2048
// 13.0 -> 11.9, B = 32, I = 1024, H = 4096 30.2 -> 28.0; at B = 64, I = 128, H = 1280 7.1 -> 8.1.  8 x 2 where that still gives every
// compute unit one: B = 128, I = 512, H = 2048 17.9 -> 16.4.  Against eight waves and an eight-way split, as other shapes have, 40 of 48
// gradient steps take 0.70 - 1.00 of the time, the others 1.01 - 1.05 (where a launch has exactly 256 large tiles: B = 128, H = 2048 2752
// -> 2867 us) and 1.07 (B = 16, I = 700, H = 1536: rows of x that are no whole fragments).
enum WideFwdConfig { WIDE_FWD_21, WIDE_FWD_22, WIDE_FWD_42_2, WIDE_FWD_42_4, WIDE_FWD_82 };
inline WideFwdConfig wide_forward_config(const Dims& d) {
  const int ngroups = d.HP / 4, bt = d.BP / 16, wgs = ((ngroups + 3) / 4) * ((bt + 1) / 2);
  if (wgs <= TARGET_WGS / 2) return bt == 1 ? WIDE_FWD_21 : WIDE_FWD_22;
  if (d.KX < 512) return WIDE_FWD_42_2;
  if (((ngroups + 7) / 8) * ((bt + 1) / 2) >= TARGET_WGS) return WIDE_FWD_82;
  return wgs <= TARGET_WGS ? WIDE_FWD_42_4 : WIDE_FWD_42_2;
}
// Backward: row tiles x batch tiles, the smallest of 1 x 1, 2 x 1, 2 x 2 that gives no compute unit two workgroups (us a launch, against
// the other shapes' rule: B = 64, H = 1280 11.4 -> 10.4; B = 128, H = 1280 19.4 -> 15.0; B = 32, H = 4096 25.9 -> 25.2).
inline BwdConfig wide_backward_config(const Dims& d) {
  const int nt = d.HP / 16, bt = d.BP / 16;
  if (nt * bt <= TARGET_WGS) return BWD_11;
  return (nt + 1) / 2 * bt <= TARGET_WGS ? BWD_21 : BWD_22;
}
// Of a backward step of a wide shape: part p has the macro steps p, p + 16, ...; the parts 4q .. 4q + 3 are
// the waves of one workgroup of a resident launch and are added first, then the four workgroups' sums.
constexpr int WIDE_BACK_PARTS = 16;
template <class Part>
__device__ __forceinline__ float sum_back_parts(Part&& part) {
  float dh = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += part(4 * q + w);
    dh += v;
  }
  return dh;
}

}  // namespace mebptt
