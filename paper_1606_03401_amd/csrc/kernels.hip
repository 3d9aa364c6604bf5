// HIP kernels for gfx950 (CDNA4, 64-wide wavefronts, MFMA matrix cores).
//
// Every contraction is written as D[i][j] = sum_k A[i][k] * B[j][k] with both operands
// k-contiguous in memory, and executed with 16x16 MFMA tiles:
//   bf16 operands: v_mfma_f32_16x16x32_bf16, each lane supplies 8 consecutive k of row lane%16
//   fp32 operands: v_mfma_f32_16x16x4_f32 issued 4 times over 4 consecutive k per lane
// so one "macro step" covers 4*VEC values of k (VEC = 8 or 4), lane group lane/16 owning the
// VEC-wide slice number lane/16.  (Which k a lane feeds is irrelevant as long as A and B agree.)
// The accumulator of lane l holds D[4*(l/16) + r][l%16], r = 0..3.
//
// The weights always play A (rows = gate rows or hidden units) and the batch plays B (columns),
// so a lane ends up with FOUR CONSECUTIVE ROWS of one batch column.  The forward operand is
// row-permuted so that those four rows are the gates i, f, g, o of one hidden unit: the LSTM
// pointwise step then runs on the GEMM result without leaving the workgroup (gate GEMM and
// pointwise forward fused).  In the backward step the four rows are four consecutive hidden
// units of dh, and loss-gradient injection and the pointwise backward again run on the GEMM
// result (the dh = dG W_hh product of step s+1 fused with the pointwise backward of step s).
#include <algorithm>

#include "common.h"
#include "device.h"
#include "dynamic_lds.h"

namespace mebptt {

Dims make_dims(int B, int I, int H, int dtype, int cell) {
  Dims d{};
  d.cell = cell;
  d.B = B;
  d.I = I;
  d.H = H;
  d.dtype = dtype;
  d.HP = round_up(H, dtype ? 32 : 16);   // bf16: HP == KH, so every column of a split h plane belongs to a tile
  d.KX = round_up(I, 32);
  d.KH = round_up(H, 32);
  d.KP = d.KX + d.KH;
  d.NX = round_up(I, 16);
  d.BP = round_up(B, 16);
  d.G4 = 4 * d.HP;
  d.NA = d.NX + d.HP + 16;
  // Steps per weight-gradient chunk: as many as keep one dG chunk buffer within 64 MiB (the
  // staging is t-independent workspace), at least 2 and at most 32.  Every chunk costs one
  // read-modify-write of the whole dW accumulator, so longer chunks are cheaper per step.
  // Small batches get up to 64 steps (K = CH*B of at least 2048 where 64 MiB allow it): the dW
  // accumulator pass of a chunk otherwise outweighs its GEMM.
  const size_t step_bytes = (size_t)d.BP * d.G4 * (dtype ? 2 : 4);
  size_t ch = ((size_t)64 << 20) / step_bytes;
  d.CH = ch < 2 ? 2 : (ch > 32 ? 32 : (int)ch);
  if (d.CH == 32 && B <= 32 && ((size_t)64 << 20) / step_bytes >= 64) d.CH = 64;
  d.hplane = dtype ? (size_t)d.BP * d.KH : (size_t)B * H;
  d.unit = (d.hplane + (size_t)B * H + 63) / 64 * 64;
  d.KC = round_up(d.CH * B, 32);
  return d;
}

// ---- small utility kernels -------------------------------------------------------------------

// The parts of setup_kernel: what threads first, first + stride, ... of each have to do.
__device__ inline void fill_part(uint4* p, size_t n16, uint4* empty, size_t ne16, size_t first, size_t stride) {
  for (size_t i = first; i < n16 + ne16; i += stride) {
    if (i < n16)
      p[i] = uint4{0, 0, 0, 0};
    else
      empty[i - n16] = uint4{~0u, ~0u, ~0u, ~0u};
  }
}
template <class T>
__device__ inline void prep_weights_part(const Dims& d, const float* __restrict__ W_ih, const float* __restrict__ W_hh,
                                         const float* __restrict__ b, T* __restrict__ Wp, float* __restrict__ bp,
                                         T* __restrict__ WTh, T* __restrict__ WTx, size_t first, size_t stride) {
  constexpr int KSTEP = 4 * Mma<T>::VEC;
  const size_t nWp = (size_t)d.G4 * d.KP, nWTh = (size_t)d.HP * d.G4, nWTx = (size_t)d.NX * d.G4;
  const size_t total = nWp + nWTh + nWTx + (size_t)d.G4;
  for (size_t idx = first; idx < total; idx += stride) {
    if (idx < nWp) {   // Wp: logical [G4][KP], row' = 4u + gate
      int rowp, k;
      ft_decode<T>(idx, d.KP / KSTEP, rowp, k);
      int u = rowp >> 2, gate = rowp & 3;
      float v = 0.0f;
      if (u < d.H) {
        if (k < d.KX) {
          const int gx = packed_gate_x(d.cell, gate);
          if (k < d.I && gx >= 0) v = W_ih[((size_t)gx * d.H + u) * d.I + k];
        } else if (k - d.KX < d.H) {
          const int gh = packed_gate_h(d.cell, gate);
          if (gh >= 0) v = W_hh[((size_t)gh * d.H + u) * d.H + (k - d.KX)];
        }
      }
      Wp[idx] = (T)v;
    } else if (idx < nWp + nWTh + nWTx) {   // WTh: logical [HP][G4]; WTx: logical [NX][G4]; k' = 4u + gate
      size_t j = idx - nWp;
      bool is_h = j < nWTh;
      if (!is_h) j -= nWTh;
      int n, kp;
      ft_decode<T>(j, d.G4 / KSTEP, n, kp);
      int u = kp >> 2, gate = kp & 3;
      float v = 0.0f;
      if (u < d.H) {
        const int g = is_h ? packed_gate_h(d.cell, gate) : packed_gate_x(d.cell, gate);
        if (g >= 0) {
          const size_t row = (size_t)g * d.H + u;
          if (is_h) {
            if (n < d.H) v = W_hh[row * d.H + n];
          } else {
            if (n < d.I) v = W_ih[row * d.I + n];
          }
        }
      }
      (is_h ? WTh : WTx)[j] = (T)v;
    } else {
      int kp = (int)(idx - nWp - nWTh - nWTx);
      int u = kp >> 2, gate = kp & 3;
      float v = 0.0f;
      if (b != nullptr && u < d.H) {
        if (d.cell == 0) {
          v = b[(size_t)gate * d.H + u];
        } else {   // b = [b_ih (r, z, n) | b_hh (r, z, n)]
          const int gx = packed_gate_x(1, gate), gh = packed_gate_h(1, gate);
          if (gx >= 0) v += b[(size_t)gx * d.H + u];
          if (gh >= 0) v += b[(size_t)(3 + gh) * d.H + u];
        }
      }
      bp[kp] = v;
    }
  }
}

// One thread per 16 bytes of a fragment.
__global__ void x_operands_kernel(const float* __restrict__ x, int B, int I, int nsx, size_t n, bf16x8* __restrict__ xs, int btiles) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int lane = (int)(i & 63), s = (int)((i >> 6) % nsx);
    const size_t tile = (i >> 6) / nsx;
    const int b = (int)(tile % btiles) * 16 + (lane & 15), k = s * 32 + (lane >> 4) * 8;
    const float* row = x + (tile / btiles * B + b) * I;
    const RawAct<8> v = load_raw<8>(row, k, b < B ? I : 0, (I & 3) == 0);
    xs[i] = Mma<__bf16>::from_f32(v.v);
  }
}
hipError_t launch_x_operands(const Dims& d, const float* x_first, int steps, void* xs, hipStream_t st) {
  const size_t n = (size_t)steps * d.BP * d.KX / 8;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 2048);
  x_operands_kernel<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(x_first, d.B, d.I, d.KX / 32, n, reinterpret_cast<bf16x8*>(xs), d.BP / 16);
  return hipGetLastError();
}

template <class T>
__device__ inline void init_state_part(const Dims& d, const float* __restrict__ h0, const float* __restrict__ c0, float* __restrict__ dst,
                                       size_t first, size_t stride) {
  const int W = HPlane<T>::SPLIT ? d.KH : d.H;   // split layout: padding columns are written as zero
  const size_t n = (size_t)d.B * W;
  for (size_t i = first; i < n; i += stride) {
    const int b = (int)(i / W), u = (int)(i % W);
    const size_t e = (size_t)b * d.H + u;
    HPlane<T>::store(dst, b, u, (u < d.H && h0) ? h0[e] : 0.0f, d.KH / 32, d.H, (size_t)d.BP * d.KH);
    if (u < d.H) dst[d.hplane + e] = c0 ? c0[e] : 0.0f;
  }
}

// All of a run's preparations in one launch, which for a toy model are as long as a sweep: blocks [0, nprep) the operand
// copies of the weights, the next nfill the cleared staging and the exchange rings, the rest the start state; none reads
// what another writes.  Three launches before; with dc_0 written by wgrad_finish_kernel a gradient step of
// H = 32, t = 20 164 -> 159 us, others 6 - 12 us less.
// Large weights go ahead alone: with the fills behind them in one launch they take longer than in turn (H = 3000, I = 128: 303 us, apart
// 247 + 37).  A gradient step of a single time step, together / apart: H = 1600, I = 512 196 / 213 us, H = 2048, I = 512 387 / 395 (42 million
// elements), H = 3000, I = 128 587 / 569 (75 million), H = 4096, I = 1024 1249 / 1235.
constexpr size_t SETUP_APART = (size_t)1 << 26;   // elements of the operand copies
struct SetupParams {
  Dims d;
  const float *W_ih, *W_hh, *b;
  void *Wp, *WTh, *WTx;
  float* bp;
  uint4 *zero, *empty;
  size_t n_zero, n_empty;
  const float *h0, *c0;
  float* state;
  int nprep, nfill;
};
template <class T>
__global__ void setup_kernel(SetupParams p) {
  const int blk = (int)blockIdx.x, ninit = (int)gridDim.x - p.nprep - p.nfill;
  if (blk < p.nprep)
    prep_weights_part<T>(p.d, p.W_ih, p.W_hh, p.b, (T*)p.Wp, p.bp, (T*)p.WTh, (T*)p.WTx, (size_t)blk * blockDim.x + threadIdx.x,
                         (size_t)p.nprep * blockDim.x);
  else if (blk < p.nprep + p.nfill)
    fill_part(p.zero, p.n_zero, p.empty, p.n_empty, (size_t)(blk - p.nprep) * blockDim.x + threadIdx.x, (size_t)p.nfill * blockDim.x);
  else
    init_state_part<T>(p.d, p.h0, p.c0, p.state, (size_t)(blk - p.nprep - p.nfill) * blockDim.x + threadIdx.x, (size_t)ninit * blockDim.x);
}

hipError_t launch_setup(const Dims& d, const SetupArgs& a, hipStream_t st) {
  SetupParams p{};
  p.d = d;
  p.W_ih = a.W_ih;
  p.W_hh = a.W_hh;
  p.b = a.b;
  p.Wp = a.Wp;
  p.bp = a.bp;
  p.WTh = a.WTh;
  p.WTx = a.WTx;
  p.zero = reinterpret_cast<uint4*>(a.zero);
  p.n_zero = a.zero_bytes / 16;   // callers keep every buffer a multiple of 16 bytes
  p.empty = reinterpret_cast<uint4*>(a.empty);
  p.n_empty = a.empty_bytes / 16;
  p.h0 = a.h0;
  p.c0 = a.c0;
  p.state = a.state;
  auto blocks = [](size_t n, size_t most) { return (int)std::min<size_t>((n + 255) / 256, most); };
  const size_t nweights = (size_t)d.G4 * d.KP + (size_t)d.HP * d.G4 + (size_t)d.NX * d.G4 + d.G4;
  const int nprep = a.W_ih ? blocks(nweights, 2048) : 0, nfill = blocks(p.n_zero + p.n_empty, 4096);
  const int ninit = a.state ? blocks((size_t)d.B * d.KH, 2048) : 0;
  auto launch = [&](int prep, int fill, int init) {
    p.nprep = prep;
    p.nfill = fill;
    if (prep + fill + init == 0) return hipSuccess;
    if (d.dtype)
      setup_kernel<__bf16><<<dim3(prep + fill + init), dim3(256), 0, st>>>(p);
    else
      setup_kernel<float><<<dim3(prep + fill + init), dim3(256), 0, st>>>(p);
    return hipGetLastError();
  };
  if (nprep && nweights >= SETUP_APART) {
    const hipError_t e = launch(nprep, 0, 0);
    return e == hipSuccess ? launch(0, nfill, ninit) : e;
  }
  return launch(nprep, nfill, ninit);
}

// ---- forward step: gate GEMM + LSTM pointwise -------------------------------------------------

struct FwdParams {
  const void* Wp;
  const float* bp;
  const float* x_s;
  const float* src_h;   // h plane of the input state (layout: HPlane)
  const float* src_c;
  float* dst_h;         // h plane of the output state
  float* dst_c;
  float* g_i;   // NULL: do not keep the gates
  float* g_f;
  float* g_g;
  float* g_o;
  int B, I, H, HP, KX, KH, KP, BP;
};

// One workgroup of 64*KS threads = BT batch tiles (16 sequences each) x NG unit groups (4 hidden
// units = 16 gate rows each).  Its KS waves split the K axis; every wave covers all NG x BT output
// tiles (each weight fragment is reused for BT batch tiles, each activation fragment for NG unit
// groups) and issues all loads of U macro steps before the first MFMA, so that several KiB per
// wave are in flight.  Partial sums meet in LDS (`red`, forward_red_floats(NG, BT, KS) floats) and
// are added in a fixed order by the thread that then does the LSTM pointwise step of that
// (sequence, unit).  (bx, by) = (unit-group tile, batch-tile group).
template <class T, int NG, int BT, int KS, int U, int CELL>
__device__ inline void forward_body(const FwdParams& p, int bx, int by, float* red) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC;
  // wave_index note: the wave index is read into a scalar register.  Conditions on it then compile
  // to scalar branches; as a vector value they become lane masks, and an MFMA under a lane mask that
  // is empty still executes (short masked blocks get no branch around them).
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: see wave_index note
  if (wave >= KS) return;   // surplus waves of a wider (fused) workgroup leave before any barrier
  const int lrow = lane & 15, lq = lane >> 4;
  const int group0 = bx * NG;
  const int ngroups = p.HP >> 2;
  const int b0 = by * BT * 16;
  using HP_ = HPlane<T>;
  const bool x_vec = (p.I & 3) == 0, h_vec = (p.H & 3) == 0;
  const int nsteps = p.KP / KSTEP;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP;   // macro steps of the x and the h segment
  const size_t hhalf = (size_t)p.BP * p.KH;           // elements of one 16-bit plane (split layout)
  const float* xrow[BT];
  const float* hrow[BT];   // plain layout: row pointer
  const T* hfrag[BT];      // split layout: this lane's slot in the batch tile's first fragment
#pragma unroll
  for (int t = 0; t < BT; ++t) {
    const int b_ld = min(b0 + t * 16 + lrow, p.B - 1);
    xrow[t] = p.x_s + (size_t)b_ld * p.I;
    hrow[t] = p.src_h + (size_t)b_ld * p.H;
    const int btile = min(by * BT + t, p.BP / 16 - 1);
    hfrag[t] = reinterpret_cast<const T*>(p.src_h) + ((size_t)btile * nsh * 64 + lane) * VEC;
  }
  const T* wbase[NG];   // fragment-tiled: tile (group) stride = nsteps * 64 * VEC
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    int grp = min(group0 + g, ngroups - 1);
    wbase[g] = reinterpret_cast<const T*>(p.Wp) + ((size_t)grp * nsteps * 64 + lane) * VEC;
  }
  f32x4 acc[NG][BT];
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int t = 0; t < BT; ++t) acc[g][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Epilogue work is dealt out by memory layout, not by MFMA layout: item i of the workgroup's
  // BT*16 rows x UW units is (row, unit) with the unit index fastest, so that consecutive lanes
  // own consecutive units of one sequence and every pointwise load and store of a wave falls
  // into runs of UW*4 bytes (plain planes) or 16 bytes (the 16-bit h planes) instead of one
  // element per row.  The operands are fetched now, so that their latency hides behind the K loop.
  constexpr int UW = NG * 4, RS = UW + 1;          // units per workgroup; padded row stride in `red`
  constexpr int ITEMS = BT * 16 * UW, NTHR = 64 * KS, IPT = (ITEMS + NTHR - 1) / NTHR;
  bool epi[IPT];
  size_t eidx[IPT];
  int eb[IPT], eu[IPT];
  float4 bias[IPT];
  float c_prev[IPT];
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const int item = (int)threadIdx.x + q * NTHR;
    const int b = b0 + (item / UW) % (BT * 16);     // rows of batch tile t follow those of t-1
    const int u = group0 * 4 + item % UW;
    epi[q] = item < ITEMS && b < p.B && u < p.H;
    eidx[q] = (size_t)b * p.H + u;
    eb[q] = item < ITEMS ? b : p.B;
    eu[q] = u;
    bias[q] = float4{0.f, 0.f, 0.f, 0.f};
    c_prev[q] = 0.0f;
    if (epi[q]) {
      bias[q] = *reinterpret_cast<const float4*>(p.bp + 4 * u);
      // the state the pointwise step blends with: c_{s-1} (LSTM) or h_{s-1} in full precision (GRU)
      c_prev[q] = CELL ? HP_::load(p.src_h, b, u, nsh, p.H, hhalf) : p.src_c[eidx[q]];
    }
  }

  // This wave's macro steps wave, wave + KS, ... in rising order: first those of the x segment
  // (and, in the plain layout, all of them), U at a time: all loads, then all MFMAs.  When every
  // row length is a multiple of the fragment width the loads are the branch-free ones (a loader
  // with branches makes the compiler wait for all outstanding loads between fragments); the
  // choice is made once, outside the loop.
  const int n_batch = HP_::SPLIT ? nsx : nsteps;   // macro steps handled by the batched loop
  auto batched = [&](auto whole_tag) {
    constexpr bool WHOLE = decltype(whole_tag)::value;
    for (int s0 = wave; s0 < n_batch; s0 += KS * U) {
      RawAct<VEC> rb[U][BT];          // fp32 activations still to be converted (x; h in the plain layout)
      typename M::Frag af[U][NG];
#pragma unroll
      for (int uu = 0; uu < U; ++uu) {
        const int s = min(s0 + uu * KS, n_batch - 1);   // clamped: the surplus fragment is discarded
        const int k = s * KSTEP + VEC * lq;
#pragma unroll
        for (int t = 0; t < BT; ++t) {
          if (WHOLE)
            rb[uu][t] = s < nsx ? load_raw_whole<VEC>(xrow[t], k, p.I) : load_raw_whole<VEC>(hrow[t], k - p.KX, p.H);
          else if (s < nsx)
            rb[uu][t] = load_raw<VEC>(xrow[t], k, p.I, x_vec);
          else
            rb[uu][t] = load_raw<VEC>(hrow[t], k - p.KX, p.H, h_vec);
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) af[uu][g] = M::load(wbase[g] + (size_t)s * 64 * VEC);
      }
#pragma unroll
      for (int uu = 0; uu < U; ++uu) {
        const int s = s0 + uu * KS;
        if (s < n_batch) {
#pragma unroll
          for (int t = 0; t < BT; ++t) {
            typename M::Frag bf = M::from_f32(rb[uu][t].v);
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g][t] = M::mma(af[uu][g], bf, acc[g][t]);
          }
        }
      }
    }
  };
  if (p.I % VEC == 0 && (HP_::SPLIT || p.H % VEC == 0))
    batched(std::true_type{});
  else
    batched(std::false_type{});
  if (HP_::SPLIT) {
    // The h segment (ready-made fragments: every load is 16 bytes per lane, no branches) runs
    // through a ring of U register slots: a slot is refilled with the step U ahead as soon as its
    // MFMAs are issued, so U steps' loads stay in flight while the matrix pipe works, instead of
    // the pipe idling through every batch of loads.  The main loop has no conditions (the compiler
    // can then wait for exactly the loads a step needs); the last steps are peeled.
    const int sh0 = wave >= nsx ? wave : wave + KS * ((nsx - wave + KS - 1) / KS);   // this wave's first h step
    typename M::Frag af[U][NG], hb[U][BT];
    auto load_slot = [&](int u, int step) {
      const int sc = min(step, nsteps - 1);   // clamped: a surplus fragment is discarded
#pragma unroll
      for (int t = 0; t < BT; ++t) hb[u][t] = M::load(hfrag[t] + (size_t)(sc - nsx) * 64 * VEC);
#pragma unroll
      for (int g = 0; g < NG; ++g) af[u][g] = M::load(wbase[g] + (size_t)sc * 64 * VEC);
    };
    auto mma_slot = [&](int u) {
#pragma unroll
      for (int t = 0; t < BT; ++t)
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g][t] = M::mma(af[u][g], hb[u][t], acc[g][t]);
    };
    if (sh0 < nsteps) {
#pragma unroll
      for (int u = 0; u < U; ++u) load_slot(u, sh0 + u * KS);
      int s = sh0;
      for (; s + KS * (2 * U - 1) < nsteps; s += KS * U) {   // every refill target is a real step
#pragma unroll
        for (int u = 0; u < U; ++u) {
          mma_slot(u);
          load_slot(u, s + (u + U) * KS);
        }
      }
      // what the slots hold now, then at most U - 1 further steps, fetched as a batch
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s + u * KS < nsteps) mma_slot(u);
      s += KS * U;
      if (s < nsteps) {
#pragma unroll
        for (int u = 0; u < U; ++u) load_slot(u, s + u * KS);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (s + u * KS < nsteps) mma_slot(u);
      }
    }
  }

  // partial sums -> red[wave][row][unit], four gates each: one 16-byte write and read where four of 4 bytes
  // took twice the LDS time on the way back (row stride padded against bank conflicts)
  f32x4* red4 = reinterpret_cast<f32x4*>(red);
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int t = 0; t < BT; ++t) red4[(wave * BT * 16 + t * 16 + lrow) * RS + g * 4 + lq] = acc[g][t];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const int item = (int)threadIdx.x + q * NTHR;
    if (item >= ITEMS) break;
    const int cell = ((item / UW) % (BT * 16)) * RS + item % UW;
    float G[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (parts_in_pairs<T, KS>) {   // fixed order: results do not depend on scheduling
      add_pairs<KS>(G, [&](int w) { return red4[w * BT * 16 * RS + cell]; });
    } else {
#pragma unroll
      for (int w = 0; w < KS; ++w) {
        const f32x4 v = red4[w * BT * 16 * RS + cell];
#pragma unroll
        for (int r = 0; r < 4; ++r) G[r] += v[r];
      }
    }
    if (!epi[q]) {
      // split layout: the padding columns H..KH of a valid row are part of the operand other
      // launches fetch, so they are (re)written as zero with every state
      if (HP_::SPLIT && eb[q] < p.B && eu[q] < p.KH) HP_::store(p.dst_h, eb[q], eu[q], 0.0f, nsh, p.H, hhalf);
      continue;
    }
    const size_t e = eidx[q];
    float second, gate[4];
    const float h = cell_forward<T, CELL>(G, bias[q], c_prev[q], second, gate);
    HP_::store(p.dst_h, eb[q], eu[q], h, nsh, p.H, hhalf);
    p.dst_c[e] = second;
    if (p.g_i) {
      p.g_i[e] = gate[0];
      p.g_f[e] = gate[1];
      p.g_g[e] = gate[2];
      if (CELL == 0) p.g_o[e] = gate[3];
    }
  }
}

// Floats of LDS a forward workgroup needs for its partial sums.
constexpr int forward_red_floats(int NG, int BT, int KS) { return KS * 4 * BT * 16 * (NG * 4 + 1); }

template <class T, int NG, int BT, int KS, int U, int CELL>
__global__ __launch_bounds__(64 * KS) void forward_kernel(FwdParams p) {
  __shared__ __attribute__((aligned(16))) float red[forward_red_floats(NG, BT, KS)];
  forward_body<T, NG, BT, KS, U, CELL>(p, blockIdx.x, blockIdx.y, red);
}

// ---- backward step: dh GEMM + loss-gradient injection + LSTM pointwise backward --------------

struct BwdParams {
  const void* WTh;
  const void* dG_next;
  const float *h, *c, *g_i, *g_f, *g_g, *g_o, *h_prev, *c_prev, *dy_s;
  int dy_is_h;
  float* dc;
  void* dG_cur;
  void* dGT;
  void* aT;
  int col0;
  float* y_out_s;
  int B, H, HP, KH, G4, NX, KC, BP;
  int cell;     // 0 LSTM, 1 GRU
};

// One workgroup of 64*KS threads = NT hidden-unit tiles x BT batch tiles (16 x 16 outputs each);
// its KS waves split K = 4*HP, every wave covering all NT x BT tiles and issuing the loads of U
// macro steps before the first MFMA.  Partial sums meet in LDS (`red`, KS*NT*BT*256 floats).  The
// pointwise backward has NT*BT*4 pieces of work (tile x which of the lane's four hidden units),
// dealt round-robin to the waves.  (bx, by) = (hidden-unit tile group, batch-tile group).
// PARTS = 2: a wave keeps its even and its odd macro steps apart; wide shapes see sum_back_parts, HALVES: the two are added here
// (backward_in_halves).
template <class T, int NT, int BT, int KS, int U, int PARTS = 1, bool HALVES = false>
__device__ inline void backward_body(const BwdParams& p, int bx, int by, float* red) {
  using M = Mma<T>;
  static_assert(PARTS == 1 || (U % 2 == 0 && KS * PARTS == WIDE_BACK_PARTS), "a slot of the ring always holds the same part");
  constexpr int OUT = HALVES ? 1 : PARTS;   // sums of a wave that go through LDS
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC;
  constexpr int NTILE = NT * BT, NPIECE = NTILE * 4, PPW = (NPIECE + KS - 1) / KS;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: see wave_index note
  if (wave >= KS) return;   // surplus waves of a wider (fused) workgroup leave before any barrier
  const int lrow = lane & 15, lq = lane >> 4;
  const int ntiles_n = p.HP / 16, ntiles_b = p.BP / 16;
  // Epilogue pieces of this wave: piece id = tile * 4 + r, tile = tn * BT + tb.  Their pointwise
  // operands are fetched before the K loop so that the latency overlaps with it.
  bool epi[PPW];
  size_t eidx[PPW];
  int en[PPW], eb[PPW];
  float h[PPW], dy[PPW], gi[PPW], gf[PPW], gg[PPW], go[PPW], c_s[PPW], c_prev[PPW], dc_in[PPW], h_prev[PPW];
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    const int piece = wave + q * KS;
    const int tile = piece >> 2, r = piece & 3;
    const int tn = tile / BT, tb = tile % BT;
    const int b = (by * BT + tb) * 16 + lrow;
    const int n = (bx * NT + tn) * 16 + 4 * lq + r;
    epi[q] = piece < NPIECE && b < p.B && n < p.H;
    eidx[q] = (size_t)b * p.H + n;
    en[q] = n;
    eb[q] = b;
    h[q] = dy[q] = gi[q] = gf[q] = gg[q] = go[q] = c_s[q] = c_prev[q] = dc_in[q] = h_prev[q] = 0.f;
    if (epi[q]) {
      const size_t e = eidx[q];
      if (p.dy_is_h || p.y_out_s) h[q] = HPlane<T>::load(p.h, b, n, p.KH / 32, p.H, (size_t)p.BP * p.KH);
      if (!p.dy_is_h && p.dy_s) dy[q] = p.dy_s[e];
      gi[q] = p.g_i[e];
      gf[q] = p.g_f[e];
      gg[q] = p.g_g[e];
      c_s[q] = p.c[e];
      dc_in[q] = p.dc[e];
      h_prev[q] = (float)HPlane<T>::as_operand(p.h_prev, b, n, p.KH / 32, p.H, (size_t)p.BP * p.KH);
      if (p.cell == 0) {
        go[q] = p.g_o[e];
        c_prev[q] = p.c_prev[e];
      } else {   // GRU blends with h_{s-1} itself: its full-precision value takes c_prev's place
        c_prev[q] = HPlane<T>::load(p.h_prev, b, n, p.KH / 32, p.H, (size_t)p.BP * p.KH);
      }
    }
  }
  if (p.dG_next) {
    f32x4 acc[PARTS][NT][BT];
#pragma unroll
    for (int e = 0; e < PARTS; ++e)
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < BT; ++j) acc[e][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nsteps = p.G4 / KSTEP;
    const T* abase[NT];
    const T* bbase[BT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
      abase[i] = reinterpret_cast<const T*>(p.WTh) + ((size_t)min(bx * NT + i, ntiles_n - 1) * nsteps * 64 + lane) * VEC;
#pragma unroll
    for (int j = 0; j < BT; ++j)
      bbase[j] = reinterpret_cast<const T*>(p.dG_next) + ((size_t)min(by * BT + j, ntiles_b - 1) * nsteps * 64 + lane) * VEC;
    // This wave's macro steps are wave, wave + KS, ...: nw of them.  A ring of U fragment slots
    // keeps U steps in flight from the first load to the last: slot u is refilled with the step U
    // places further on as soon as its MFMAs are issued.  Steps are consumed in the same order
    // as a plain loop would, so the sums are unchanged.  The main loop covers whole groups of U
    // steps that all have a refill, so its body has no branches and the number of loads
    // outstanding at every wait is known at compile time; the tail (at most two groups) is
    // conditional.
    const int nw = (nsteps - wave + KS - 1) / KS;
    typename M::Frag af[U][NT], bf[U][BT];
    auto load_slot = [&](int u, int j) {   // j: index into this wave's steps (always < nw here or clamped)
      const size_t off = (size_t)min(wave + j * KS, nsteps - 1) * 64 * VEC;
#pragma unroll
      for (int i = 0; i < NT; ++i) af[u][i] = M::load(abase[i] + off);
#pragma unroll
      for (int jj = 0; jj < BT; ++jj) bf[u][jj] = M::load(bbase[jj] + off);
    };
    auto mma_slot = [&](int u) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int jj = 0; jj < BT; ++jj) acc[u % PARTS][i][jj] = M::mma(af[u][i], bf[u][jj], acc[u % PARTS][i][jj]);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load_slot(u, u);   // surplus slots (u >= nw) hold a clamped copy and are never used
    int j0 = 0;
    for (; j0 + 2 * U <= nw; j0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        mma_slot(u);
        load_slot(u, j0 + u + U);
      }
    }
    for (; j0 < nw; j0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (j0 + u < nw) mma_slot(u);
        if (j0 + u + U < nw) load_slot(u, j0 + u + U);
      }
    }
    if constexpr (HALVES) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < BT; ++j) acc[0][i][j] += acc[PARTS - 1][i][j];
    }
#pragma unroll
    for (int e = 0; e < OUT; ++e)
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < BT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) red[(((wave + e * KS) * NTILE + i * BT + j) * 4 + r) * 64 + lane] = acc[e][i][j][r];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    const int piece = wave + q * KS;
    if (piece >= NPIECE) break;
    float dh = 0.0f;
    if (p.dG_next) {   // fixed order
      if constexpr (OUT == 1)
        for (int w = 0; w < KS; ++w) dh += red[(w * NPIECE + piece) * 64 + lane];
      else
        dh = sum_back_parts([&](int w) { return red[(w * NPIECE + piece) * 64 + lane]; });
    }
    if (!epi[q]) continue;
    const size_t e = eidx[q];
    const int n = en[q], b = eb[q];
    dh += p.dy_is_h ? h[q] : dy[q];
    if (p.y_out_s) p.y_out_s[e] = h[q];
    float dGi, dGf, dGg, dGo;
    if (p.cell == 0) {
      float dG[4], dc_out;
      lstm_backward_point<T>(dh, dc_in[q], gi[q], gf[q], gg[q], go[q], c_s[q], c_prev[q], dG, dc_out);
      dGi = dG[0];
      dGf = dG[1];
      dGg = dG[2];
      dGo = dG[3];
      p.dc[e] = dc_out;
    } else {
      // GRU: r = gi, z = gf, n = gg, n_h = c_s, h_{s-1} = c_prev.  The running plane `dc` carries
      // the part of dL/dh_{s-1} that bypasses the GEMM: dh_s * z_s.
      float dG[4], carry;
      gru_backward_point(__fadd_rn(dh, dc_in[q]), gi[q], gf[q], gg[q], c_s[q], c_prev[q], dG, carry);
      dGi = dG[0];
      dGf = dG[1];
      dGg = dG[2];
      dGo = dG[3];
      p.dc[e] = carry;
    }
    const T q0 = (T)dGi, q1 = (T)dGf, q2 = (T)dGg, q3 = (T)dGo;
    // dG of this step, fragment-tiled [b][4n + gate]: the four gates are consecutive in one lane slot
    T* dG4 = reinterpret_cast<T*>(p.dG_cur) + ft_offset<T>(b, 4 * n, p.G4 / KSTEP);
    dG4[0] = q0;
    dG4[1] = q1;
    dG4[2] = q2;
    dG4[3] = q3;
    // transposed copies for the weight gradient, fragment-tiled [4n + gate][col] and [NX + n][col]
    const int col = p.col0 + b, ncs = p.KC / KSTEP;
    T* dGT = reinterpret_cast<T*>(p.dGT);
    dGT[ft_offset<T>(4 * n + 0, col, ncs)] = q0;
    dGT[ft_offset<T>(4 * n + 1, col, ncs)] = q1;
    dGT[ft_offset<T>(4 * n + 2, col, ncs)] = q2;
    dGT[ft_offset<T>(4 * n + 3, col, ncs)] = q3;
    reinterpret_cast<T*>(p.aT)[ft_offset<T>(p.NX + n, col, ncs)] = (T)h_prev[q];
  }
}

template <class T, int NT, int BT, int KS, int U, int PARTS, bool HALVES>
__global__ __launch_bounds__(64 * KS) void backward_kernel(BwdParams p) {
  __shared__ float red[KS * (HALVES ? 1 : PARTS) * NT * BT * 4 * 64];
  backward_body<T, NT, BT, KS, U, PARTS, HALVES>(p, blockIdx.x, blockIdx.y, red);
}

// ---- fused launch: a backward step and an independent forward step ---------------------------
// The recomputation chain (forward operations) never depends on the backward chain, so the
// forward operation that follows a backward step in the schedule can share its launch whenever
// it does not overwrite a state that backward step still reads.  Workgroups [0, nf) play the
// forward role, the rest the backward role; 512 threads each, and the launch bounds hold the kernel
// to 128 registers (4 waves per SIMD), so that two workgroups are resident on a compute unit at
// the same time and the 2 x 256 workgroups of a launch run as one wave of work, not two.  Each role splits K over the
// same number of waves as its stand-alone kernel, so sums are formed in the same order and results
// do not depend on whether a step was fused.
constexpr int PAIR_FKS = 8, PAIR_NG = 4, PAIR_FU = 1, PAIR_BKS = 8, PAIR_BU = 4;

// Roles of one fused launch: forward tile FNG x 1 split over FKS waves, backward tile BNT x BBT over
// BKS waves (the K splits of the stand-alone kernels of the same shape class).  FU and BU, the
// macro steps a wave keeps in flight, are smaller than the stand-alone kernels': two resident
// workgroups share a compute unit's load path, and measured launch times fall as the queues get
// shorter (large-K class: 9.98 us at FU, BU = 2, 8; 9.47 us at 1, 4; small-K class 12.2 -> 10.8 us).
template <class T, int CELL, int FNG, int FKS, int FU, int BNT, int BBT, int BKS, int BU, int PARTS = 1, bool HALVES = false>
__global__ __launch_bounds__(64 * (FKS > BKS ? FKS : BKS), 4) void pair_kernel(FwdParams f, BwdParams b, int nfx, int nf,
                                                                             int nbx) {
  constexpr int FRED = forward_red_floats(FNG, 1, FKS), BRED = BKS * (HALVES ? 1 : PARTS) * BNT * BBT * 4 * 64;
  __shared__ __attribute__((aligned(16))) float red[FRED > BRED ? FRED : BRED];
  const int id = blockIdx.x;
  if (id < nf)
    forward_body<T, FNG, 1, FKS, FU, CELL>(f, id % nfx, id / nfx, red);
  else
    backward_body<T, BNT, BBT, BKS, BU, PARTS, HALVES>(b, (id - nf) % nbx, (id - nf) / nbx, red);
}

template <class T, int NG, int BT, int KS, int U>
static hipError_t launch_forward_cfg(const Dims& d, const FwdParams& p, hipStream_t st) {
  dim3 grid((d.HP / 4 + NG - 1) / NG, (d.BP / 16 + BT - 1) / BT), block(64 * KS);
  if (d.cell)
    forward_kernel<T, NG, BT, KS, U, 1><<<grid, block, 0, st>>>(p);
  else
    forward_kernel<T, NG, BT, KS, U, 0><<<grid, block, 0, st>>>(p);
  return hipGetLastError();
}

template <class T>
static hipError_t launch_forward_t(const Dims& d, const FwdParams& p, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    if (wide_shape(d).groups) switch (wide_forward_config(d)) {
      case WIDE_FWD_21: return launch_forward_cfg<T, 2, 1, WIDE_FWD_KS, 5>(d, p, st);
      case WIDE_FWD_22: return launch_forward_cfg<T, 2, 2, WIDE_FWD_KS, 4>(d, p, st);
      case WIDE_FWD_42_2: return launch_forward_cfg<T, 4, 2, WIDE_FWD_KS, 2>(d, p, st);
      case WIDE_FWD_42_4: return launch_forward_cfg<T, 4, 2, WIDE_FWD_KS, 4>(d, p, st);
      case WIDE_FWD_82: return launch_forward_cfg<T, 8, 2, WIDE_FWD_KS, 4>(d, p, st);
    }
  }
  switch (forward_config<T>(d)) {
    case FWD_TINY: return launch_forward_cfg<T, 1, 1, 4, 2>(d, p, st);   // tiny K: one small workgroup per tile
    case FWD_SMALLK: return launch_forward_cfg<T, 4, 1, 4, 5>(d, p, st);
    case FWD_82: return launch_forward_cfg<T, 8, 2, 8, 1>(d, p, st);
    // bf16: two macro steps in flight, 26.6 us on H = 4096, B = 32; three 27.3, four waves 27.9.  fp32, whose macro
    // steps are half as long: three; a gradient step of H = 1024, B = 128 (t = 60) takes 5.12 ms so, 5.57 with two, of
    // H = 4096, B = 32 (t = 20) 6.75 against 8.07
    case FWD_42: return launch_forward_cfg<T, 4, 2, 8, sizeof(T) == 2 ? 2 : 3>(d, p, st);
    default: return launch_forward_cfg<T, PAIR_NG, 1, PAIR_FKS, 5>(d, p, st);
  }
}

static FwdParams make_fwd_params(const Dims& d, const void* Wp, const float* bp, const float* x_s,
                                 const float* src_unit, float* dst_unit, float* gates_units) {
  const size_t plane = (size_t)d.B * d.H;
  FwdParams p{};
  p.Wp = Wp;
  p.bp = bp;
  p.x_s = x_s;
  p.src_h = src_unit;
  p.src_c = src_unit + d.hplane;
  p.dst_h = dst_unit;
  p.dst_c = dst_unit + d.hplane;
  if (gates_units) {   // two units: (i, f) and (g, o)
    p.g_i = gates_units;
    p.g_f = gates_units + plane;
    p.g_g = gates_units + d.unit;
    p.g_o = gates_units + d.unit + plane;
  }
  p.B = d.B;
  p.I = d.I;
  p.H = d.H;
  p.HP = d.HP;
  p.KX = d.KX;
  p.KH = d.KH;
  p.KP = d.KP;
  p.BP = d.BP;
  return p;
}

hipError_t launch_forward(const Dims& d, const void* Wp, const float* bp, const float* x_s, const float* src_unit,
                          float* dst_unit, float* gates_units, hipStream_t st) {
  FwdParams p = make_fwd_params(d, Wp, bp, x_s, src_unit, dst_unit, gates_units);
  return d.dtype ? launch_forward_t<__bf16>(d, p, st) : launch_forward_t<float>(d, p, st);
}

// ---- independent forward operations in one launch ----------------------------------------------
// Where every step of a stretch has its input hidden state in memory, the forward operations that
// recompute the steps' internal states do not depend on each other: they go out as one launch,
// grid.z = the operation.  A workgroup is a forward workgroup of its step (forward_body, with the K
// split of the shape's stand-alone kernel, so a step gives the same bits whichever launch ran it).
constexpr int FWD_BATCH_MAX_STEPS = 32;
struct FwdBatchSteps {
  const float* x[FWD_BATCH_MAX_STEPS];     // x_s [B, I]
  const float* src[FWD_BATCH_MAX_STEPS];   // unit (h_{s-1}, c_{s-1})
  float* dst[FWD_BATCH_MAX_STEPS];         // three units: (h_s, c_s), (i, f), (g, o)
};

template <class T, int NG, int BT, int KS, int U, int CELL>
__global__ __launch_bounds__(64 * KS) void forward_batch_kernel(FwdParams p, FwdBatchSteps steps, size_t hplane, size_t unit,
                                                                size_t plane) {
  __shared__ __attribute__((aligned(16))) float red[forward_red_floats(NG, BT, KS)];
  const int j = blockIdx.z;
  float* dst = steps.dst[j];
  p.x_s = steps.x[j];
  p.src_h = steps.src[j];
  p.src_c = steps.src[j] + hplane;
  p.dst_h = dst;
  p.dst_c = dst + hplane;
  p.g_i = dst + unit;
  p.g_f = dst + unit + plane;
  p.g_g = dst + 2 * unit;
  p.g_o = dst + 2 * unit + plane;
  forward_body<T, NG, BT, KS, U, CELL>(p, blockIdx.x, blockIdx.y, red);
}

// The same on larger tiles, bf16: a workgroup of four waves computes 64 NR packed rows x NC batch tiles, which may be of several
// operations.  A wave owns NR row tiles and covers all columns: its weight fragments go straight into the MFMA registers, those
// of the activations (x converted on the way) through LDS, where the four waves share them.  Macro steps are taken in the order
// of the K parts of the shape's stand-alone kernel -- w, w + KS, ... for each part w in turn -- and a part's sums are added to the
// total when it ends (of an eight-way split, those of two parts: add_pairs), so a step gives the same bits here too.
// What bounds it: delivery of the panels to the compute units (128 x 64 tiles half the bytes of 64 x 32; H = 1024, B = 64, 31 operations
// 55.3 -> 49.9 us), with few workgroups the rounds in turn: LDS, MFMAs, a barrier. Sixty-four more columns a workgroup, or 256 rows, leave
// compute units idle (52 - 82 us), three or four rounds in flight instead of two gain nothing. Two waves per SIMD are asked for because
// with all 512 registers to use the compiler keeps the sums in accumulation registers and copies them in and out in every macro step (63 us).
constexpr int ORDER_MAX = 128, ORDER_ENDS = 0x8000, ORDER_WAITS = 0x4000;
struct MacroStepOrder {   // two macro steps a round, the first in the low half; ORDER_ENDS: its K part ends with it (and ORDER_WAITS for the next)
  unsigned at[ORDER_MAX];
};
static bool macro_step_order(int nsteps, int ks, MacroStepOrder& o) {
  if (nsteps > 2 * ORDER_MAX) return false;
  int i = 0;
  o = MacroStepOrder{};
  for (int w = 0; w < ks; ++w)
    for (int s = w; s < nsteps; s += ks, ++i) o.at[i / 2] |= (unsigned)(s | (s + ks >= nsteps ? (ks == 8 && w % 2 == 0 ? ORDER_ENDS | ORDER_WAITS : ORDER_ENDS) : 0)) << 16 * (i % 2);
  return true;
}
template <int NR, int NC, int CELL>
__global__ __launch_bounds__(256, 2) void forward_batch_tiles_kernel(FwdParams p, FwdBatchSteps steps, MacroStepOrder order, int n, int row_blocks,
                                                                     size_t hplane, size_t unit, size_t plane) {
  using T = __bf16;
  using M = Mma<T>;
  using HP_ = HPlane<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, FRAG = 64 * VEC;
  constexpr int UW = 16 * NR, SEQ = 16 * NC, RS = UW + 1, NQ = NC / 2;   // NQ: activation fragments a wave stages per round
  constexpr int STAGE = 2 * NC * FRAG;                                   // elements: two macro steps
  constexpr size_t LDS = (size_t)2 * STAGE * sizeof(T) > (size_t)SEQ * RS * 16 ? (size_t)2 * STAGE * sizeof(T) : (size_t)SEQ * RS * 16;
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];
  T* lds = reinterpret_cast<T*>(smem);
  f32x4* red = reinterpret_cast<f32x4*>(smem);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: see wave_index note
  const int lrow = lane & 15, lq = lane >> 4;
  // ids equal modulo 8 share an XCD: each works through a contiguous range of row blocks, whose weights its L2 then holds
  const int id = (int)blockIdx.x, total_wgs = (int)gridDim.x, xcd = id & 7;
  const int work = xcd * (total_wgs >> 3) + min(xcd, total_wgs & 7) + (id >> 3), col_blocks = total_wgs / row_blocks;
  const int by = work % col_blocks, bx = work / col_blocks;
  const int btiles = p.BP / 16;
  const int nsx = p.KX / KSTEP, nsh = p.KH / KSTEP, nsteps = nsx + nsh;
  const size_t hhalf = (size_t)p.BP * p.KH;

  // the workgroup's batch tiles: operation and tile of it (scalars; one division)
  int op[NC], bt[NC];
  op[0] = by * NC / btiles;
  bt[0] = by * NC - op[0] * btiles;
#pragma unroll
  for (int t = 1; t < NC; ++t) {
    const bool over = bt[t - 1] + 1 == btiles;
    op[t] = op[t - 1] + (over ? 1 : 0);
    bt[t] = over ? 0 : bt[t - 1] + 1;
  }
  auto op_in = [&](int t) { return min(op[t], n - 1); };   // for fetches: tiles past the last operation read it again

  // epilogue items: unit fastest; a thread's items are of one unit, item q of a sequence of batch tile q * ROWS / 16
  constexpr int ROWS = 256 / UW, IPT = SEQ / ROWS;
  static_assert(ROWS <= 16, "items of one q are of one batch tile");
  const int u = bx * UW + (int)threadIdx.x % UW;
  auto row_of = [&](int q) { return bt[q * ROWS / 16] * 16 + q * ROWS % 16 + (int)threadIdx.x / UW; };
  const int uc = min(u, p.H - 1);   // an item without a unit or sequence fetches a neighbour's values
  const float4 bias = *reinterpret_cast<const float4*>(p.bp + 4 * uc);
  float c_prev[IPT];
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const float* src = steps.src[op_in(q * ROWS / 16)];
    const int b = min(row_of(q), p.B - 1);
    c_prev[q] = CELL ? HP_::load(src, b, uc, nsh, p.H, hhalf) : (src + hplane)[(size_t)b * p.H + uc];
  }

  const int FB = FRAG * (int)sizeof(T);
  int wrow[NR];   // of each row tile, the first fragment (bytes)
#pragma unroll
  for (int r = 0; r < NR; ++r) wrow[r] = min((bx * 4 + wave) * NR + r, (p.HP >> 2) - 1) * nsteps * FB;
  const __amdgpu_buffer_rsrc_t weights = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.Wp), 0, 0x7fffffff, 0x00020000);
  // the batch tile whose activations this wave stages
  int my_op = op_in(0), my_bt = bt[0];
#pragma unroll
  for (int t = 1; t < NC; ++t)
    if (wave % NC == t) {
      my_op = op_in(t);
      my_bt = bt[t];
    }
  const float *x_op = steps.x[my_op], *h_op = steps.src[my_op];
  const unsigned xrow = (unsigned)(min(my_bt * 16 + lrow, p.B - 1) * p.I) * 4, hoff = (unsigned)((my_bt * nsh * 64 + lane) * 16);

  typename M::Frag a[2][2][NR];
  u32x4 raw[NQ][2];
  int raw_s[NQ];
  auto step_of = [&](int q) { return (wave + 4 * q) / NC; };   // of the round's two macro steps, the one fragment q belongs to
  auto first = [](unsigned o) { return (int)(o & 0x3fff); };
  auto second = [](unsigned o) { return (int)(o >> 16 & 0x3fff); };
  auto fetch_a = [&](int set, unsigned o) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      a[set][0][r] = as_frag<typename M::Frag>(__builtin_amdgcn_raw_buffer_load_b128(weights, lane * 16, wrow[r] + first(o) * FB, 0));
      a[set][1][r] = as_frag<typename M::Frag>(__builtin_amdgcn_raw_buffer_load_b128(weights, lane * 16, wrow[r] + second(o) * FB, 0));
    }
  };
  // Without branches: a fragment of x is 32 bytes of a row (a window that ends inside it, see load_window), one of h 16 bytes,
  // whose second load lies outside the buffer and moves nothing.
  const unsigned xlane = xrow + 32u * (unsigned)lq;
  const int over = p.I - VEC - VEC * lq;
  auto fetch_b = [&](unsigned o) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int s = step_of(q) ? second(o) : first(o);
      const bool is_x = s < nsx;
      const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(is_x ? x_op : h_op), 0, 0x7fffffff, 0x00020000);
      const unsigned xo = xlane + 4u * (unsigned)min(s * KSTEP, over);
      const int so = is_x ? 0 : 1024 * (s - nsx);
      raw[q][0] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(is_x ? xo : hoff), so, 0);
      raw[q][1] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(is_x ? xo + 16u : 0x80000000u), 0, 0);
      raw_s[q] = s;
    }
  };
  auto stash = [&](int stage) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int s = raw_s[q];
      typename M::Frag f = as_frag<typename M::Frag>(raw[q][0]);
      if (s < nsx) {
        RawAct<VEC> v;
#pragma unroll
        for (int e = 0; e < VEC; ++e) v.v[e] = __uint_as_float(raw[q][e / 4][e % 4]);
        if ((s + 1) * KSTEP > p.I) shift_tail<VEC>(v, s * KSTEP + VEC * lq, p.I);
        f = M::from_f32(v.v);
      }
      *reinterpret_cast<typename M::Frag*>(&lds[(size_t)stage * STAGE + (size_t)(wave + 4 * q) * FRAG + lane * VEC]) = f;
    }
  };
  f32x4 part[NR][NC], waits[NR][NC], sum[NR][NC];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int t = 0; t < NC; ++t) part[r][t] = waits[r][t] = sum[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto read_b = [&](int stage, int e, typename M::Frag (&bf)[NC]) {
#pragma unroll
    for (int t = 0; t < NC; ++t) bf[t] = M::load(&lds[(size_t)stage * STAGE + (size_t)(e * NC + t) * FRAG + lane * VEC]);
  };
  auto compute = [&](const typename M::Frag (&af)[NR], const typename M::Frag (&bf)[NC], unsigned o) {
#pragma unroll
    for (int t = 0; t < NC; ++t)
#pragma unroll
      for (int r = 0; r < NR; ++r) part[r][t] = M::mma(af[r], bf[t], part[r][t]);
    if (o & ORDER_ENDS) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int t = 0; t < NC; ++t) {
          if (o & ORDER_WAITS)
            waits[r][t] = part[r][t];
          else
            sum[r][t] += waits[r][t] + part[r][t];
          part[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
  };
  // Round r: two macro steps.  Its weights sit in register set r & 1, its activations in LDS stage r & 1; those of the next round
  // are on their way.  One barrier per round.
  const int rounds = (nsteps + 1) / 2;
  unsigned o_now = order.at[0], o_next = order.at[min(1, rounds - 1)];
  fetch_b(o_now);
  fetch_a(0, o_now);
  stash(0);
  fetch_b(o_next);
  fetch_a(1, o_next);
  lds_barrier();
  auto round = [&](int r, int set) {
    typename M::Frag b0[NC], b1[NC];
    read_b(set, 0, b0);
    read_b(set, 1, b1);
    stash(set ^ 1);   // past the last round: what nobody reads
    const unsigned o_then = order.at[min(r + 2, rounds - 1)];
    fetch_b(o_then);
    compute(a[set][0], b0, o_now);
    if (2 * r + 1 < nsteps) compute(a[set][1], b1, o_now >> 16);
    fetch_a(set, o_then);
    o_now = o_next;
    o_next = o_then;
    lds_barrier();
  };
  for (int r = 0; r < rounds; r += 2) {
    round(r, 0);
    if (r + 1 < rounds) round(r + 1, 1);
  }

  // sums -> red[sequence][unit], four gates each
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int t = 0; t < NC; ++t) red[(t * 16 + lrow) * RS + (wave * NR + r) * 4 + lq] = sum[r][t];
  lds_barrier();
#pragma unroll
  for (int q = 0; q < IPT; ++q) {
    const int b = row_of(q);
    if (op[q * ROWS / 16] >= n || b >= p.B) continue;
    float* dst = steps.dst[op[q * ROWS / 16]];
    if (u >= p.H) {   // padding columns are part of the operand other launches fetch: zero
      if (u < p.KH) HP_::store(dst, b, u, 0.0f, nsh, p.H, hhalf);
      continue;
    }
    const f32x4 v = red[(q * ROWS + (int)threadIdx.x / UW) * RS + (int)threadIdx.x % UW];
    const float G[4] = {v[0], v[1], v[2], v[3]};
    float second, gate[4];
    const float h = cell_forward<T, CELL>(G, bias, c_prev[q], second, gate);
    const size_t e = (size_t)b * p.H + u;
    HP_::store(dst, b, u, h, nsh, p.H, hhalf);
    (dst + hplane)[e] = second;
    (dst + unit)[e] = gate[0];
    (dst + unit + plane)[e] = gate[1];
    (dst + 2 * unit)[e] = gate[2];
    if (CELL == 0) (dst + 2 * unit + plane)[e] = gate[3];
  }
}

template <int NR, int NC>
static void launch_forward_batch_tiles(const Dims& d, const FwdParams& p, const FwdBatchSteps& steps, const MacroStepOrder& order, int n, hipStream_t st) {
  const int rows = (d.HP / 4 + 4 * NR - 1) / (4 * NR), cols = (n * (d.BP / 16) + NC - 1) / NC;
  const dim3 grid(rows * cols), block(256);
  const size_t plane = (size_t)d.B * d.H;
  if (d.cell)
    forward_batch_tiles_kernel<NR, NC, 1><<<grid, block, 0, st>>>(p, steps, order, n, rows, d.hplane, d.unit, plane);
  else
    forward_batch_tiles_kernel<NR, NC, 0><<<grid, block, 0, st>>>(p, steps, order, n, rows, d.hplane, d.unit, plane);
}

int forward_batch_max_steps() { return FWD_BATCH_MAX_STEPS; }

// What a launch of n operations takes (us, bf16) on 64 x 32, 128 x 32 and 128 x 64 tiles, from 17 000 launches timed on all three: B of 4 to 256, H of 200 to
// 4096, I of 8 to 1024, LSTM and GRU.  Two thirds of the small tiles' estimates lie within 10 % of the time (whole 16-byte rows of x: 15 %), of the larger ones' within 7 %.
// * Small tiles: rounds of workgroups, one on every compute unit, each with its K.  Rows of x that are no whole 16 bytes are fetched value by value, for as many sequences
//   as a tile holds: H = I = 650, B = 20, 8 operations 17.7 us, on 128 x 32 tiles 13.8.  Workgroups go to the XCDs in turn; where their number per operation is no
//   multiple of eight an XCD gets other rows of the weights each time, and what does not stay in its L2 (6 MB of a copy still do) is fetched anew
//   for every operation: H = 1816, I = 416, B = 95, 7 operations 105 us (53 on 128 x 32), H = 1898, I = 20, B = 67, whose XCDs see an eighth each, 51 (46).
// * Larger tiles: a compute unit holds two of them (128 x 32 with K split four ways: three), and up to there their number costs little.
// With a workgroup each small tiles are up to 1.7 times as fast (H = 600, I = 193, B = 20, 5 operations 6.5 us for 10.1 and 13.9).  Of the launches timed, choosing larger
// ones for 5 % takes 0.76 of the small ones' time in the mean (the best of the three 0.75), more than 1.05 of it for one in 150, 1.26 at worst.
struct ForwardBatchTimes {
  float small, narrow, wide;
};
static ForwardBatchTimes forward_batch_us(const Dims& d, int n, int ks) {
  const float K = d.KP / 1024.f, X = d.KX / 1024.f, Hk = d.KH / 1024.f;
  const int gx = (d.HP / 4 + 3) / 4, gy = (d.BP / 16 + 1) / 2, rows = d.HP / 32, tiles = n * (d.BP / 16);
  const float rounds = (float)((gx * gy * n + TARGET_WGS - 1) / TARGET_WGS), filled = (float)d.B / (32 * gy);
  int same = 8;   // an XCD sees one of this many neighbouring row groups of the weights
  while ((gx * gy) % same != 0 || (gy > 1 && gx % same != 0)) same /= 2;
  const float weights = (float)d.HP * 4 * d.KP * 2e-6f;   // MB
  const bool ragged = d.I % 4 != 0;
  ForwardBatchTimes t;
  t.small = 3 + (ragged ? std::min(1.f, 4 * X) : 0) + rounds * (0.6f + 2.1f * Hk + (0.4f + (ragged ? 11.f : 4.f) * filled) * X) + (weights / same > 6 ? 0.045f * n * weights : 0);
  const int narrow = rows * ((tiles + 1) / 2), wide = rows * ((tiles + 3) / 4);
  t.narrow = narrow <= 256 ? 5 + 7 * K : narrow <= 512 ? 7 + 7.5f * K : narrow <= 768 ? (ks == 8 ? 6.5f + 13 * K : 8.5f + 10.3f * K) :
             (ks == 8 ? 8.5f + 17 * K : 10.5f + 16.5f * K) * std::max(1.f, narrow / 1024.f);
  t.wide = wide <= 256 ? 8 + 8.7f * K : wide <= 512 ? (ks == 8 ? 9 + 12.2f * K : 10.5f + 9.9f * K) : (14 + 19 * K) * std::max(1.f, wide / 768.f);
  return t;
}

template <class T>
static void launch_forward_batch_t(const Dims& d, const FwdParams& p, const FwdBatchSteps& steps, int n, hipStream_t st) {
  // 64 gate rows x 32 sequences per workgroup, two macro steps in flight per wave: two workgroups
  // fit a compute unit.  Measured on H = 1024, B = 64, partial sums as single floats: 2.7 us per operation;
  // 64 x 64 tiles 3.1 us, three or four macro steps in flight 4.4 - 5.1 us.  With the sums as 16-byte
  // vectors a launch of 17 operations takes 43.8 us instead of 45.4.  fp32 as the stand-alone kernel: three (whole
  // gradient steps 1 % faster than with two, which needs scratch memory).
  constexpr int NG = 4, BT = 2, FU = sizeof(T) == 2 ? 2 : 3;
  const dim3 grid((d.HP / 4 + NG - 1) / NG, (d.BP / 16 + BT - 1) / BT, n);
  const size_t plane = (size_t)d.B * d.H;
  const FwdConfig cfg = forward_config<T>(d);
  // the K split of the shape's stand-alone forward kernel
  const bool small_k = cfg == FWD_TINY || cfg == FWD_SMALLK || wide_shape(d).groups;
  if constexpr (sizeof(T) == 2) {
    // Larger tiles (forward_batch_tiles_kernel) where forward_batch_us expects 5 % of them.  Rows of x that are whole 16 bytes keep the small ones
    // while GEMMs run beside: a gradient step of H = 1024, B = 64 takes 10 539 us with larger ones for 10 489.
    MacroStepOrder order;
    constexpr size_t LIMIT = (size_t)1 << 31;   // 32-bit byte offsets
    if (d.I >= 8 && (size_t)d.G4 * d.KP * 2 < LIMIT && (size_t)d.B * d.I * 4 < LIMIT && macro_step_order(d.KP / 32, small_k ? 4 : 8, order)) {
      const ForwardBatchTimes us = forward_batch_us(d, n, small_k ? 4 : 8);
      const bool larger = std::min(us.narrow, us.wide) < 0.95f * us.small && (d.I % 4 != 0 || !gemms_beside(d));
      const bool use_wide = larger && us.wide < us.narrow, use_narrow = larger && !use_wide;
      if (use_wide) return launch_forward_batch_tiles<2, 4>(d, p, steps, order, n, st);
      if (use_narrow) return launch_forward_batch_tiles<2, 2>(d, p, steps, order, n, st);
    }
  }
  if (small_k && d.cell)
    forward_batch_kernel<T, NG, BT, 4, FU, 1><<<grid, dim3(64 * 4), 0, st>>>(p, steps, d.hplane, d.unit, plane);
  else if (small_k)
    forward_batch_kernel<T, NG, BT, 4, FU, 0><<<grid, dim3(64 * 4), 0, st>>>(p, steps, d.hplane, d.unit, plane);
  else if (d.cell)
    forward_batch_kernel<T, NG, BT, 8, FU, 1><<<grid, dim3(64 * 8), 0, st>>>(p, steps, d.hplane, d.unit, plane);
  else
    forward_batch_kernel<T, NG, BT, 8, FU, 0><<<grid, dim3(64 * 8), 0, st>>>(p, steps, d.hplane, d.unit, plane);
}

hipError_t launch_forward_batch(const Dims& d, const void* Wp, const float* bp, int n, const float* const* x,
                                const float* const* src, float* const* dst, hipStream_t st) {
  if (n < 1 || n > FWD_BATCH_MAX_STEPS) return hipErrorInvalidValue;
  FwdParams p = make_fwd_params(d, Wp, bp, x[0], src[0], dst[0], dst[0] + d.unit);
  FwdBatchSteps steps{};
  for (int j = 0; j < n; ++j) {
    steps.x[j] = x[j];
    steps.src[j] = src[j];
    steps.dst[j] = dst[j];
  }
  if (d.dtype)
    launch_forward_batch_t<__bf16>(d, p, steps, n, st);
  else
    launch_forward_batch_t<float>(d, p, steps, n, st);
  return hipGetLastError();
}

// ---- measurement: the bytes of a forward launch, streamed -----------------------------------
// The grid and block of the forward launch of this shape; every workgroup reads the weight panel
// (its gate rows x K, GEMM operand type) and the activation panel (its sequences x K: x in fp32, h
// in the operand type) its forward counterpart reads, from the same weight array, with the same
// 16-byte-per-lane loads, eight in flight per wave -- and does nothing else.  What this takes is
// what the memory system needs to deliver the launch's bytes to the compute units.
__global__ __launch_bounds__(512) void stream_panels_kernel(const uint4* __restrict__ w, size_t w_panel, const uint4* __restrict__ a,
                                                            size_t a_panel, float* __restrict__ sink) {
  constexpr int U = 8;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
  float acc = 0.0f;
  for (int part = 0; part < 2; ++part) {
    const uint4* base = part ? a + (size_t)blockIdx.y * a_panel : w + (size_t)blockIdx.x * w_panel;
    const size_t nblk = (part ? a_panel : w_panel) / 64;   // blocks of 64 x 16 bytes
    for (size_t b0 = wave; b0 < nblk; b0 += (size_t)nwaves * U) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        size_t b = b0 + (size_t)u * nwaves;
        if (b >= nblk) b = nblk - 1;
        v[u] = base[b * 64 + lane];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) acc += __uint_as_float(v[u].x ^ v[u].y ^ v[u].z ^ v[u].w);
    }
  }
  if (acc == 12345.678f) sink[0] = acc;   // keeps the loads alive; never true in practice
}

template <class T>
static void forward_launch_shape(const Dims& d, int& ng, int& bt, int& ks) {
  if (wide_shape(d).groups) {
    const WideFwdConfig c = wide_forward_config(d);
    ng = c == WIDE_FWD_82 ? 8 : (c == WIDE_FWD_21 || c == WIDE_FWD_22 ? 2 : 4), bt = c == WIDE_FWD_21 ? 1 : 2, ks = WIDE_FWD_KS;
    return;
  }
  switch (forward_config<T>(d)) {
    case FWD_TINY: ng = 1, bt = 1, ks = 4; break;
    case FWD_SMALLK: ng = 4, bt = 1, ks = 4; break;
    case FWD_82: ng = 8, bt = 2, ks = 8; break;
    case FWD_42: ng = 4, bt = 2, ks = 8; break;
    default: ng = PAIR_NG, bt = 1, ks = PAIR_FKS; break;
  }
}

hipError_t launch_forward_stream(const Dims& d, const void* Wp, const void* act, size_t act_bytes, float* sink,
                                 size_t* delivered_bytes, hipStream_t st) {
  int ng, bt, ks;
  if (d.dtype)
    forward_launch_shape<__bf16>(d, ng, bt, ks);
  else
    forward_launch_shape<float>(d, ng, bt, ks);
  const size_t op = d.op_bytes();
  const dim3 grid((d.HP / 4 + ng - 1) / ng, (d.BP / 16 + bt - 1) / bt);
  // 16-byte vectors per panel, rounded down to whole 1 KiB blocks
  const size_t w_panel = (size_t)ng * 16 * d.KP * op / 1024 * 64;
  const size_t a_panel = ((size_t)bt * 16 * ((size_t)d.KX * 4 + (size_t)d.KH * op)) / 1024 * 64;
  if (w_panel == 0 || a_panel == 0 || a_panel * 16 * grid.y > act_bytes) return hipErrorInvalidValue;
  if ((size_t)grid.x * w_panel * 16 > (size_t)d.G4 * d.KP * op) return hipErrorInvalidValue;
  if (delivered_bytes) *delivered_bytes = (size_t)grid.x * grid.y * (w_panel + a_panel) * 16;
  stream_panels_kernel<<<grid, dim3(64 * ks), 0, st>>>(reinterpret_cast<const uint4*>(Wp), w_panel,
                                                      reinterpret_cast<const uint4*>(act), a_panel, sink);
  return hipGetLastError();
}

template <class T, int NT, int BT, int KS, int U, int PARTS = 1, bool HALVES = false>
static hipError_t launch_backward_cfg(const Dims& d, const BwdParams& p, hipStream_t st) {
  dim3 grid((d.HP / 16 + NT - 1) / NT, (d.BP / 16 + BT - 1) / BT), block(64 * KS);
  backward_kernel<T, NT, BT, KS, U, PARTS, HALVES><<<grid, block, 0, st>>>(p);
  return hipGetLastError();
}

template <class T>
static hipError_t launch_backward_t(const Dims& d, const BwdParams& p, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    if (wide_shape(d).groups) switch (wide_backward_config(d)) {
      case BWD_11: return launch_backward_cfg<T, 1, 1, 8, PAIR_BU, 2>(d, p, st);
      case BWD_21: return launch_backward_cfg<T, 2, 1, 8, 4, 2>(d, p, st);
      default: return launch_backward_cfg<T, 2, 2, 8, 4, 2>(d, p, st);
    }
    if (backward_in_halves(d)) return launch_backward_cfg<T, 1, 1, PAIR_BKS, PAIR_BU, 2, true>(d, p, st);
  }
  switch (backward_config<T>(d)) {
    case BWD_SMALLK: return launch_backward_cfg<T, 1, 1, 4, 4>(d, p, st);
    case BWD_22: return launch_backward_cfg<T, 2, 2, 8, 4>(d, p, st);
    case BWD_12: return launch_backward_cfg<T, 1, 2, 8, 6>(d, p, st);
    default: return launch_backward_cfg<T, 1, 1, PAIR_BKS, PAIR_BU>(d, p, st);
  }
}

static BwdParams make_bwd_params(const Dims& d, const BackwardArgs& a) {
  const size_t plane = (size_t)d.B * d.H;
  BwdParams p{};
  p.WTh = a.WTh;
  p.dG_next = a.dG_next;
  p.h = a.state;
  p.c = a.state + d.hplane;
  p.g_i = a.state + d.unit;
  p.g_f = a.state + d.unit + plane;
  p.g_g = a.state + 2 * d.unit;
  p.g_o = a.state + 2 * d.unit + plane;
  p.h_prev = a.prev;
  p.cell = d.cell;
  p.c_prev = a.prev + d.hplane;
  p.dy_s = a.dy_s;
  p.dy_is_h = a.dy_is_h;
  p.dc = a.dc;
  p.dG_cur = a.dG_cur;
  p.dGT = a.dGT;
  p.aT = a.aT;
  p.col0 = a.col0;
  p.y_out_s = a.y_out_s;
  p.B = d.B;
  p.H = d.H;
  p.HP = d.HP;
  p.KH = d.KH;
  p.G4 = d.G4;
  p.NX = d.NX;
  p.KC = d.KC;
  p.BP = d.BP;
  return p;
}

hipError_t launch_backward(const Dims& d, const BackwardArgs& a, hipStream_t st) {
  BwdParams p = make_bwd_params(d, a);
  return d.dtype ? launch_backward_t<__bf16>(d, p, st) : launch_backward_t<float>(d, p, st);
}

// Shape classes for which a fused launch is instantiated: 1 = large K (forward 4 x 1, backward
// 1 x 1, 8 waves each); 2 = small-K forward (4 waves) with the 1 x 2 backward (8 waves); 3 = as 1 with the K splits of
// a wide shape (forward 2 x 1 by four waves: a gradient step without resident launches, B = 8, H = 1100 859 us apart, 741 fused,
// B = 32, H = 2048 1975 and 1905).  0 = none.
template <class T>
static int pair_class(const Dims& d) {
  const FwdConfig fc = forward_config<T>(d);
  const BwdConfig bc = backward_config<T>(d);
  if (fc == FWD_B1 && bc == BWD_11) return wide_shape(d).groups ? 3 : 1;
  if (fc == FWD_SMALLK && bc == BWD_12) return 2;
  return 0;
}

bool can_fuse_pair(const Dims& d) { return (d.dtype ? pair_class<__bf16>(d) : pair_class<float>(d)) != 0; }

template <class T, int CELL>
static void launch_pair_t(const Dims& d, const FwdParams& f, const BwdParams& b, hipStream_t st) {
  const int nfx = (d.HP / 4 + PAIR_NG - 1) / PAIR_NG, nfy = d.BP / 16;   // classes 1 and 2: forward 4 x 1
  const int cls = pair_class<T>(d);
  if constexpr (sizeof(T) == 2) {
    if (cls == 3) {
      const int nwx = (d.HP / 4 + 1) / 2, nbx = d.HP / 16, nby = d.BP / 16;
      pair_kernel<T, CELL, 2, WIDE_FWD_KS, 2, 1, 1, PAIR_BKS, PAIR_BU, 2>
          <<<dim3(nwx * nfy + nbx * nby), dim3(64 * PAIR_BKS), 0, st>>>(f, b, nwx, nwx * nfy, nbx);
      return;
    }
  }
  if constexpr (sizeof(T) == 2) {
    if (cls == 1 && backward_in_halves(d)) {
      const int nbx = d.HP / 16, nby = d.BP / 16;
      pair_kernel<T, CELL, PAIR_NG, PAIR_FKS, PAIR_FU, 1, 1, PAIR_BKS, PAIR_BU, 2, true>
          <<<dim3(nfx * nfy + nbx * nby), dim3(64 * PAIR_BKS), 0, st>>>(f, b, nfx, nfx * nfy, nbx);
      return;
    }
  }
  if (cls == 1) {
    const int nbx = d.HP / 16, nby = d.BP / 16;
    pair_kernel<T, CELL, PAIR_NG, PAIR_FKS, PAIR_FU, 1, 1, PAIR_BKS, PAIR_BU>
        <<<dim3(nfx * nfy + nbx * nby), dim3(64 * PAIR_BKS), 0, st>>>(f, b, nfx, nfx * nfy, nbx);
  } else {
    const int nbx = d.HP / 16, nby = (d.BP / 16 + 1) / 2;
    pair_kernel<T, CELL, 4, 4, 1, 1, 2, 8, 2><<<dim3(nfx * nfy + nbx * nby), dim3(512), 0, st>>>(f, b, nfx, nfx * nfy, nbx);
  }
}

hipError_t launch_backward_forward_pair(const Dims& d, const BackwardArgs& a, const void* Wp, const float* bp,
                                        const float* x_s, const float* src_unit, float* dst_unit, float* gates_units,
                                        hipStream_t st) {
  BwdParams b = make_bwd_params(d, a);
  FwdParams f = make_fwd_params(d, Wp, bp, x_s, src_unit, dst_unit, gates_units);
  if (d.dtype)
    d.cell ? launch_pair_t<__bf16, 1>(d, f, b, st) : launch_pair_t<__bf16, 0>(d, f, b, st);
  else
    d.cell ? launch_pair_t<float, 1>(d, f, b, st) : launch_pair_t<float, 0>(d, f, b, st);
  return hipGetLastError();
}

// ---- data-gradient GEMM: out[row][n] = sum_k dG[row][k] * WT[n][k] ---------------------------

// One workgroup = NT column tiles (16 outputs n each) x RT row tiles (16 (step, sequence) rows each);
// its KS waves split K = 4*HP, every wave covering all NT x RT tiles.  Partial sums meet in LDS;
// the NT*RT*4 output quarter-tiles are dealt round-robin to the waves for the store.
template <class T, int NT, int RT, int KS, int U>
__global__ __launch_bounds__(64 * KS) void dgrad_kernel(const T* __restrict__ WT, int N, const T* __restrict__ dG,
                                                        int nrow_tiles, int B, int BP, int G4,
                                                        float* __restrict__ out, int ld_out) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, NTILE = NT * RT, NPIECE = NTILE * 4, PPW = (NPIECE + KS - 1) / KS;
  extern __shared__ __attribute__((aligned(16))) unsigned char dgrad_smem[];
  float* red = reinterpret_cast<float*>(dgrad_smem);   // [KS][NTILE][4][64]
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: see wave_index note
  const int lrow = lane & 15, lq = lane >> 4;
  // Workgroups are handed to the 8 XCDs round-robin by their linear id.  As launched, an XCD would
  // own every 8th column group and see all of dG.  The id is re-mapped so that each XCD works
  // through a contiguous range of (row group, column group) pairs, column group fastest: the
  // workgroups that share a dG row group then share an L2, every XCD fetches only its own eighth
  // of dG, and the weight operand streams through each L2 once per round of resident workgroups
  // (measured: 136 -> 34 MB fetched per chunk on the 256 -> 1024 shape, 569 -> about 200 MB on
  // 512 -> 2048).
  const int gx = (int)gridDim.x, total = gx * (int)gridDim.y;
  const int id = (int)blockIdx.x + gx * (int)blockIdx.y;
  const int xcd = id & 7;
  const int work = xcd * (total >> 3) + min(xcd, total & 7) + (id >> 3);
  const int bx = work % gx, by = work / gx;
  const int ncol_tiles = (N + 15) / 16;
  const int nsteps = G4 / KSTEP;
  const T* abase[NT];
  const T* bbase[RT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
    abase[i] = WT + ((size_t)min(bx * NT + i, ncol_tiles - 1) * nsteps * 64 + lane) * VEC;
#pragma unroll
  for (int j = 0; j < RT; ++j)
    bbase[j] = dG + ((size_t)min(by * RT + j, nrow_tiles - 1) * nsteps * 64 + lane) * VEC;
  f32x4 acc[NT][RT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < RT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = wave; s0 < nsteps; s0 += KS * U) {
    typename M::Frag af[U][NT], bf[U][RT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t off = (size_t)min(s0 + u * KS, nsteps - 1) * 64 * VEC;
#pragma unroll
      for (int i = 0; i < NT; ++i) af[u][i] = M::load(abase[i] + off);
#pragma unroll
      for (int j = 0; j < RT; ++j) bf[u][j] = M::load(bbase[j] + off);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u * KS < nsteps) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int j = 0; j < RT; ++j) acc[i][j] = M::mma(af[u][i], bf[u][j], acc[i][j]);
      }
  }
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < RT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((wave * NTILE + i * RT + j) * 4 + r) * 64 + lane] = acc[i][j][r];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PPW; ++q) {
    const int piece = wave + q * KS;
    if (piece >= NPIECE) break;
    float v = 0.0f;
    for (int w = 0; w < KS; ++w) v += red[(w * NPIECE + piece) * 64 + lane];   // fixed order
    const int tile = piece >> 2, r = piece & 3;
    const int tn = tile / RT, tr = tile % RT;
    const int row = (by * RT + tr) * 16 + lrow;   // padded row: slot * BP + b
    const int n = (bx * NT + tn) * 16 + 4 * lq + r;
    const int slot = row / BP, b = row % BP;
    if (row >= nrow_tiles * 16 || b >= B || n >= N) continue;
    out[((size_t)slot * B + b) * ld_out + n] = v;
  }
}

template <class T, int NT, int RT, int KS, int U>
static hipError_t launch_dgrad_cfg(dim3 grid, const T* WT, int N, const T* dG, int nrow_tiles, const Dims& d, float* out,
                                   int ld_out, hipStream_t st) {
  const size_t lds = (size_t)KS * NT * RT * 4 * 64 * sizeof(float);
  hipError_t e = allow_dynamic_lds<dgrad_kernel<T, NT, RT, KS, U>>(lds);   // needed above 64 KiB only, harmless below
  if (e != hipSuccess) return e;
  dgrad_kernel<T, NT, RT, KS, U><<<grid, dim3(64 * KS), lds, st>>>(WT, N, dG, nrow_tiles, d.B, d.BP, d.G4, out, ld_out);
  return hipGetLastError();
}

template <class T>
static hipError_t launch_dgrad_t(const Dims& d, const void* WT, int N, const void* dG, int nslots, float* out, int ld_out,
                                 hipStream_t st) {
  const int ncol_tiles = round_up(N, 16) / 16, nrow_tiles = nslots * d.BP / 16;
  // The largest output block per workgroup that still gives every compute unit one: each operand
  // byte a workgroup fetches is used for 64, 32 or 16 outputs.
  if (((ncol_tiles + 3) / 4) * ((nrow_tiles + 3) / 4) >= TARGET_WGS)
    return launch_dgrad_cfg<T, 4, 4, 8, 4>(dim3((ncol_tiles + 3) / 4, (nrow_tiles + 3) / 4), (const T*)WT, N, (const T*)dG,
                                           nrow_tiles, d, out, ld_out, st);
  if (((ncol_tiles + 1) / 2) * ((nrow_tiles + 3) / 4) >= TARGET_WGS)
    return launch_dgrad_cfg<T, 2, 4, 8, 4>(dim3((ncol_tiles + 1) / 2, (nrow_tiles + 3) / 4), (const T*)WT, N, (const T*)dG,
                                           nrow_tiles, d, out, ld_out, st);
  if (((ncol_tiles + 1) / 2) * ((nrow_tiles + 1) / 2) >= TARGET_WGS)
    return launch_dgrad_cfg<T, 2, 2, 8, 4>(dim3((ncol_tiles + 1) / 2, (nrow_tiles + 1) / 2), (const T*)WT, N, (const T*)dG,
                                           nrow_tiles, d, out, ld_out, st);
  return launch_dgrad_cfg<T, 1, 1, 8, 4>(dim3(ncol_tiles, nrow_tiles), (const T*)WT, N, (const T*)dG, nrow_tiles, d, out, ld_out,
                                         st);
}

hipError_t launch_dgrad_gemm(const Dims& d, const void* WT, int N, const void* dG, int nslots, float* out, int ld_out,
                             hipStream_t st) {
  return d.dtype ? launch_dgrad_t<__bf16>(d, WT, N, dG, nslots, out, ld_out, st)
                 : launch_dgrad_t<float>(d, WT, N, dG, nslots, out, ld_out, st);
}

// ---- time-batched GEMM on 256 x 256 workgroup tiles --------------------------------------------
// D[i][j] (+)= sum_k A[i][k] B[j][k] for the weight gradient over a chunk of steps (K = CH*B), used
// when dW has enough 256 x 256 tiles to fill the chip (the dx GEMM's output never has).  Both operands are fragment-tiled, so a 16-row tile of
// one macro step is a contiguous 1 KiB block.  A workgroup of 8 waves (2 along i, 4 along j) owns
// 256 x 256 outputs, each wave 128 x 64 (8 x 4 MFMA tiles, 128 accumulator registers); two waves
// share a SIMD, so one wave's LDS reads hide behind the other's MFMAs.  Per round of two macro
// steps (K = 64) the workgroup copies 32 + 32 operand fragments (64 KiB) from L2 into one of two
// LDS stages -- fetched into registers one round ahead -- and every wave reads the 8 + 4
// fragments per macro step it needs: each operand byte enters the compute unit once per
// workgroup, and there is one barrier per 64 of K.
// Workgroup ids are re-mapped so that the workgroups sharing an XCD (ids equal modulo 8) work
// through a contiguous range of (i-block, j-block) pairs, j fastest: they stream the same A panel
// through the L2 they share.
struct TgemmParams {
  const void* A;      // rows i: mt_total 16-row tiles, a_steps macro steps per tile
  const void* B;      // rows j
  int mt_total, nt_total, a_steps, b_steps;
  int nk;             // macro steps to contract over (from step 0)
  int gx, gy;         // workgroup grid: i-blocks, j-blocks
  float* acc;         // tile-ordered accumulator
  int accumulate;     // 0: overwrite it, 1: add to it
  // The first `full` workgroups (a multiple of the compute units) take one output block each over
  // the whole of K; the blocks left over, too few for a round of their own, are shared out `split`
  // ways along K so that the last round is short instead of mostly empty: part 0 adds into the
  // block's place in `acc`, part q > 0 into `extra` block (q - 1) * (gx * gy - full) + (block - full).
  // Which part sums what is fixed by the shape, so results do not depend on scheduling.
  int full, split;
  float* extra;
};

template <class T>
__global__ __launch_bounds__(512) void tgemm_kernel(TgemmParams p) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, FRAG = 64 * VEC;
  constexpr int TI = 8, TJ = 4;           // MFMA tiles per wave along i and j
  constexpr int WGT = 16;                 // 16-row tiles per workgroup along each axis
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T* lds = reinterpret_cast<T*>(smem);    // [stage 2][macro step 2][16 tiles of A][FRAG]
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: see wave_index note
  const int wi = wave & 1, wj = wave >> 1;
  const int id = (int)blockIdx.x;
  int work, part = 0, nparts = 1;
  if (id < p.full) {
    const int xcd = id & 7;
    work = xcd * (p.full >> 3) + min(xcd, p.full & 7) + (id >> 3);
  } else {
    work = p.full + (id - p.full) / p.split;
    part = (id - p.full) % p.split;
    nparts = p.split;
  }
  const int bx = work / p.gy, by = work % p.gy;
  // this workgroup's share of K: rounds [r0, r1) of two macro steps each
  const int rounds_all = (p.nk + 1) >> 1;
  const int r0 = part * rounds_all / nparts, r1 = (part + 1) * rounds_all / nparts;
  const int nk = min(p.nk, 2 * r1) - 2 * r0;   // macro steps of the share (may be 0)
  const int nrounds = (nk + 1) >> 1;
  // a wave whose 128 x 64 outputs all lie outside the matrix (the last block of a ragged edge) only
  // helps to stage A
  const bool active = bx * WGT + wi * TI < p.mt_total && by * WGT + wj * TJ < p.nt_total;
  // A (the i operand, shared by the four waves of a row) goes L2 -> registers -> LDS: this wave
  // copies fragments f = wave*4 .. +4 of every round, f = ks * 16 + tile.  B (the j operand,
  // shared by two waves only) is fetched by each wave straight into its MFMA registers: LDS
  // carries 2/3 of the reads and half of the writes it would carry for both operands.
  const T* srcA[4];
  int ks_of[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int f = wave * 4 + q, ks = f >> 4, tile = f & 15;
    ks_of[q] = ks;
    srcA[q] = reinterpret_cast<const T*>(p.A) + ((size_t)min(bx * WGT + tile, p.mt_total - 1) * p.a_steps * 64 + lane) * VEC +
              (size_t)2 * r0 * FRAG;
  }
  const T* srcB[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
    srcB[j] = reinterpret_cast<const T*>(p.B) + ((size_t)min(by * WGT + wj * TJ + j, p.nt_total - 1) * p.b_steps * 64 + lane) * VEC +
              (size_t)2 * r0 * FRAG;
  u32x4 ringA[2][4];
  typename M::Frag ringB[2][2][TJ];   // [set][macro step of the round][tile]
  auto fetch = [&](int set, int round) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int s = min(round * 2 + ks_of[q], nk - 1);   // a macro step past the end is fetched (clamped) and never used
      ringA[set][q] = *reinterpret_cast<const u32x4*>(srcA[q] + (size_t)s * FRAG);
    }
    if (!active) return;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int s = min(round * 2 + ks, nk - 1);
#pragma unroll
      for (int j = 0; j < TJ; ++j) ringB[set][ks][j] = M::load(srcB[j] + (size_t)s * FRAG);
    }
  };
  auto stash = [&](int set, int stage) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<u32x4*>(&lds[((size_t)stage * 32 + wave * 4 + q) * FRAG + lane * VEC]) = ringA[set][q];
  };
  f32x4 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int r, int stage, int set) {
    if (!active) return;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if (r * 2 + ks < nk) {   // uniform
        const T* base = &lds[((size_t)stage * 32 + ks * 16) * FRAG + lane * VEC];
        // The wave's TI fragments of A come from LDS two ahead of the MFMAs that use them: two
        // reads, then TJ MFMAs and one more read in turn, so an LDS round trip always has eight
        // MFMAs to hide behind.  (Left to itself the scheduler puts every read right before its
        // MFMAs and waits for it.)  The group barriers fix that order for the instructions of
        // this block: 0x100 = LDS read, 0x008 = MFMA.
        typename M::Frag a[TI];
#pragma unroll
        for (int i = 0; i < TI; ++i) a[i] = M::load(base + (size_t)(wi * TI + i) * FRAG);
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[i][j] = M::mma(a[i], ringB[set][ks][j], acc[i][j]);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int i = 0; i < TI - 2; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, TJ, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * TJ, 0);
      }
    }
  };

  if (nrounds > 0) {
    // Register set r & 1 holds round r: its A part is moved to LDS stage r & 1 one round early, its
    // B part is consumed in place; the set is refilled with round r + 2 once round r is computed.
    fetch(0, 0);
    fetch(1, 1);           // clamped when there is a single round
    stash(0, 0);
    __syncthreads();
    for (int r = 0; r < nrounds; r += 2) {   // unrolled by two so that sets and stages are static
      if (r + 1 < nrounds) stash(1, 1);
      compute(r, 0, 0);
      fetch(0, r + 2);
      __syncthreads();
      if (r + 1 < nrounds) {
        if (r + 2 < nrounds) stash(0, 0);
        compute(r + 1, 1, 1);
        fetch(1, r + 3);
        __syncthreads();
      }
    }
  }

  // Running sum in a tile-ordered accumulator: a wave's 32 tiles are one contiguous run and a
  // lane's four rows one float4, so the read-modify-write of every chunk is fully coalesced;
  // wgrad_finish_kernel converts it to the caller's row-major dW once at the end of the run.
  if (!active) return;   // nobody reads blocks outside the matrix
  const size_t block = part == 0 ? (size_t)work : (size_t)(part - 1) * (p.gx * p.gy - p.full) + (work - p.full);
  float4* accp = reinterpret_cast<float4*>(part == 0 ? p.acc : p.extra) + ((block * 8 + wave) * (TI * TJ)) * 64 + lane;
#pragma unroll
  for (int half = 0; half < 2; ++half) {   // two batches of 16 tiles: the old values pass through few registers
    float4 old[TI * TJ / 2];
    if (p.accumulate) {
#pragma unroll
      for (int q = 0; q < TI * TJ / 2; ++q) old[q] = accp[(size_t)(half * (TI * TJ / 2) + q) * 64];
    }
#pragma unroll
    for (int q = 0; q < TI * TJ / 2; ++q) {
      const int t = half * (TI * TJ / 2) + q;
      f32x4 v = acc[t / TJ][t % TJ];
      if (p.accumulate) {
        v[0] += old[q].x;
        v[1] += old[q].y;
        v[2] += old[q].z;
        v[3] += old[q].w;
      }
      accp[(size_t)t * 64] = float4{v[0], v[1], v[2], v[3]};
    }
  }
}

constexpr int TGEMM_LDS_BYTES = 2 * 32 * 1024;
constexpr int TGEMM_MIN_TILES = 192;   // below this the output does not fill the chip with 256 x 256 tiles

template <class T>
static hipError_t launch_tgemm(const TgemmParams& p, hipStream_t st) {
  hipError_t e = allow_dynamic_lds<tgemm_kernel<T>>(TGEMM_LDS_BYTES);
  if (e != hipSuccess) return e;
  tgemm_kernel<T><<<dim3(p.full + (p.gx * p.gy - p.full) * p.split), dim3(512), TGEMM_LDS_BYTES, st>>>(p);
  return hipGetLastError();
}

// How the 256 x 256 output blocks are dealt out: whole rounds of one block per compute unit over all
// of K, and the blocks left over split along K as many ways as fit one more round (at most four).
constexpr int TGEMM_ROUND = 256;
static void tgemm_shares(int blocks, int& full, int& split) {
  full = blocks / TGEMM_ROUND * TGEMM_ROUND;
  const int rest = blocks - full;
  split = rest == 0 ? 1 : std::max(1, std::min(4, TGEMM_ROUND / rest));
  if (split == 1) full = blocks;
}

// ---- dx GEMM on the 256 x 256 blocks ---------------------------------------------------------
// dx[(step, b)][n] = sum_k dG[(step, b)][k] W_ih^T[n][k] over a chunk of steps has few output blocks
// (cfg3: 2 x 16) and a long K = 4H, so every block's K is shared out over `split` workgroups, each
// writing its partial block; dx_finish_kernel adds the parts in a fixed order and stores the rows
// of real sequences.  The partial blocks live in a scratch buffer the caller lends (the chunk's
// dG^T buffer, which nobody reads between this chunk's dW GEMM and the next chunk that fills it).
// Used when that gives the chip at least 192 workgroups with at least 16 macro steps each.
constexpr int DX_MAX_SPLIT = 8;
struct DxBlocks {
  int gx, gy, split;   // blocks along n, along the rows of a full chunk, K shares per block (0: not used)
};
static DxBlocks dx_blocks(const Dims& d, size_t scratch_bytes) {
  DxBlocks b{0, 0, 0};
  if (!d.dtype || d.NX < 256) return b;
  b.gx = (d.NX / 16 + 15) / 16;
  b.gy = (d.CH * d.BP / 16 + 15) / 16;
  const int blocks = b.gx * b.gy, nk = d.G4 / 32;
  const size_t fit = scratch_bytes / ((size_t)blocks * 256 * 256 * sizeof(float));
  const int split = (int)std::min<size_t>(std::min(DX_MAX_SPLIT, std::min(TGEMM_ROUND / blocks, nk / 16)), fit);
  if (split >= 1 && blocks * split >= 192) b.split = split;
  return b;
}

// partial[part][block][wave][tile][lane] (tgemm_kernel's accumulator order) -> dx rows.  One thread
// per float4 of a block: four consecutive n of one (step, b) row.
__global__ void dx_finish_kernel(const float4* __restrict__ partial, int blocks, int split, int gy, int nrows, int B, int BP,
                                 int I, float* __restrict__ out, int ld_out) {
  const size_t total = (size_t)blocks * (256 * 256 / 4), stride = (size_t)gridDim.x * blockDim.x;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
    const int lane = (int)(idx & 63), tile = (int)((idx >> 6) & 31), wave = (int)((idx >> 11) & 7);
    const int block = (int)(idx >> 14);
    const int bx = block / gy, by = block % gy;
    const int wi = wave & 1, wj = wave >> 1, ti = tile >> 2, tj = tile & 3;
    const int n = ((bx * 16 + wi * 8 + ti) * 16) + 4 * (lane >> 4);
    const int row = ((by * 16 + wj * 4 + tj) * 16) + (lane & 15);   // padded row: slot * BP + b
    const int slot = row / BP, b = row % BP;
    if (row >= nrows || b >= B || n >= I) continue;
    float4 u[DX_MAX_SPLIT];   // all parts fetched before the first addition: the loads overlap
#pragma unroll
    for (int q = 0; q < DX_MAX_SPLIT; ++q)
      if (q < split) u[q] = partial[(size_t)q * total + idx];
    float4 v = u[0];
#pragma unroll
    for (int q = 1; q < DX_MAX_SPLIT; ++q)   // fixed order
      if (q < split) {
        v.x += u[q].x;
        v.y += u[q].y;
        v.z += u[q].z;
        v.w += u[q].w;
      }
    float* dst = out + ((size_t)slot * B + b) * ld_out + n;
    if (n + 3 < I && (ld_out & 3) == 0) {
      *reinterpret_cast<float4*>(dst) = v;
    } else {
      const float e[4] = {v.x, v.y, v.z, v.w};
      for (int r = 0; r < 4 && n + r < I; ++r) dst[r] = e[r];
    }
  }
}

bool dx_gemm_uses_blocks(const Dims& d, size_t scratch_bytes) { return dx_blocks(d, scratch_bytes).split > 0; }

hipError_t launch_dx_gemm(const Dims& d, const void* WTx, const void* dG, int nslots, float* dx, void* scratch,
                          size_t scratch_bytes, hipStream_t st) {
  const DxBlocks b = dx_blocks(d, scratch_bytes);
  if (b.split == 0) return launch_dgrad_gemm(d, WTx, d.I, dG, nslots, dx, d.I, st);
  TgemmParams p{};
  p.A = WTx;
  p.B = dG;
  p.mt_total = d.NX / 16;
  p.nt_total = nslots * d.BP / 16;
  p.a_steps = p.b_steps = d.G4 / 32;
  p.nk = d.G4 / 32;
  p.gx = b.gx;
  p.gy = (p.nt_total + 15) / 16;   // a short chunk has fewer blocks; the shares stay those of the shape
  p.acc = reinterpret_cast<float*>(scratch);
  p.accumulate = 0;
  p.full = 0;
  p.split = b.split;
  p.extra = p.acc + (size_t)p.gx * p.gy * 256 * 256;
  hipError_t e = launch_tgemm<__bf16>(p, st);
  if (e != hipSuccess) return e;
  const int blocks = p.gx * p.gy;
  dx_finish_kernel<<<dim3(std::min(blocks * 64, 4096)), dim3(256), 0, st>>>(reinterpret_cast<const float4*>(scratch), blocks, b.split,
                                                                           p.gy, nslots * d.BP, d.B, d.BP, d.I, dx, d.I);
  return hipGetLastError();
}

// The weight gradient runs on the 256 x 256 tiles when the operands are bf16 and dW has enough tiles.
static bool wgrad_uses_big_tiles(const Dims& d) {
  if (!d.dtype) return false;
  const int gx = (d.G4 / 16 + 15) / 16, gy = (d.NA / 16 + 15) / 16;
  return gx * gy >= TGEMM_MIN_TILES;
}

// ---- x transposed into the weight-gradient operand ----------------------------------------------

template <class T>
__global__ void transpose_x_kernel(const float* __restrict__ x, int rows, int I, int KC, int ones_row,
                                   T* __restrict__ aT) {
  // x: [rows][I] (rows = nslots*B consecutive (step, b) pairs) -> aT[i][row]; the first column of
  // blocks also sets aT[ones_row][row] = 1, the operand row that turns db into a column of dW.
  __shared__ float tile[32][33];
  const int r0 = blockIdx.x * 32, i0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  for (int rr = ty; rr < 32; rr += 8) {
    int r = r0 + rr, i = i0 + tx;
    tile[rr][tx] = (r < rows && i < I) ? x[(size_t)r * I + i] : 0.0f;
  }
  __syncthreads();
  for (int ii = ty; ii < 32; ii += 8) {
    int i = i0 + ii, r = r0 + tx;
    if (i < I && r < rows) aT[ft_offset<T>(i, r, KC / (4 * Mma<T>::VEC))] = (T)tile[tx][ii];
  }
  if (blockIdx.y == 0 && ty == 0 && r0 + tx < rows) aT[ft_offset<T>(ones_row, r0 + tx, KC / (4 * Mma<T>::VEC))] = (T)1.0f;
}

hipError_t launch_transpose_x(const Dims& d, const float* x_first, int nslots, void* aT, hipStream_t st) {
  const int rows = nslots * d.B;
  dim3 grid((rows + 31) / 32, (d.I + 31) / 32), block(256);
  if (d.dtype)
    transpose_x_kernel<__bf16><<<grid, block, 0, st>>>(x_first, rows, d.I, d.KC, d.NX + d.HP, (__bf16*)aT);
  else
    transpose_x_kernel<float><<<grid, block, 0, st>>>(x_first, rows, d.I, d.KC, d.NX + d.HP, (float*)aT);
  return hipGetLastError();
}

// Zeroes columns [c0, c1) of the two weight-gradient operands (dGT: G4 rows, aT: NA rows).
template <class T>
__global__ void zero_operand_columns_kernel(T* __restrict__ dGT, int G4, T* __restrict__ aT, int NA, int KC, int c0, int c1) {
  const int ncols = c1 - c0, ncs = KC / (4 * Mma<T>::VEC);
  const size_t total = (size_t)(G4 + NA) * ncols;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int row = (int)(i / ncols), col = c0 + (int)(i % ncols);
    if (row < G4)
      dGT[ft_offset<T>(row, col, ncs)] = (T)0.0f;
    else
      aT[ft_offset<T>(row - G4, col, ncs)] = (T)0.0f;
  }
}

hipError_t launch_zero_operand_columns(const Dims& d, void* dGT, void* aT, int c0, int c1, hipStream_t st) {
  if (c1 <= c0) return hipSuccess;
  if (c0 < 0 || c1 > d.KC) return hipErrorInvalidValue;
  const size_t total = (size_t)(d.G4 + d.NA) * (c1 - c0);
  size_t blocks = (total + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  if (d.dtype)
    zero_operand_columns_kernel<__bf16><<<dim3((unsigned)blocks), dim3(256), 0, st>>>((__bf16*)dGT, d.G4, (__bf16*)aT, d.NA, d.KC, c0, c1);
  else
    zero_operand_columns_kernel<float><<<dim3((unsigned)blocks), dim3(256), 0, st>>>((float*)dGT, d.G4, (float*)aT, d.NA, d.KC, c0, c1);
  return hipGetLastError();
}

// ---- weight-gradient GEMM: dW[row(m)][n] (+)= sum_k dGT[m][k] * aT[n][k] ------------------------

// A workgroup of 2 x 2 waves owns a block of 2*WT x 2*WT MFMA tiles of dW (128 x 128 elements for
// WT = 4, 64 x 64 for WT = 2, used when the larger block would leave most compute units idle);
// each wave a WT x WT quarter.  Per macro step the workgroup copies the 2*WT fragments of dGT (1 KiB each, already
// in fragment order) into LDS with fully coalesced 16-byte loads, from which the two waves of a row read
// them; the fragments of aT every wave fetches straight into its MFMA registers.  Both are fetched PD macro steps
// ahead.  (Both operands through LDS: 39.6 us per chunk on H = 1024, B = 64, so: 37.0; two macro steps per barrier: 37.8.)  gridDim.z workgroups may share one
// output block, each with its own part of K and its own partial accumulator.
// EXTRA (wgrad_plan says where, blocks of 128): aT has one row tile (the row of ones, whose product is the bias gradient) more than whole blocks,
// which would cost a column of blocks that are nearly empty.  Its 2 * WT products per row block are dealt out over the waves of the first
// blocks instead: one more MFMA per macro step; the fragment comes through a buffer that gives waves without a product zeros and moves
// nothing for them.  A chunk of H = 256, I = 256, B = 64 12.4 -> 10.5 us.
template <class T, int WT, bool EXTRA>
__global__ __launch_bounds__(256) void wgrad_kernel(const T* __restrict__ dGT, const T* __restrict__ aT, int K, int KC,
                                                    int G4, int NTOT, int accumulate, float* __restrict__ dWacc) {
  using M = Mma<T>;
  constexpr int VEC = M::VEC, KSTEP = 4 * VEC, PD = 3;
  constexpr int FRAG = 64 * VEC;                  // elements of one fragment block (1 KiB)
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  __shared__ __attribute__((aligned(16))) T lds[2][2 * WT * FRAG];
  constexpr int SW = WT / 2;                      // fragments of dGT this wave copies per macro step
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;   // scalar: see wave_index note
  const int wm = wave & 1, wn = wave >> 1;
  const int MT = G4 / 16, NT = NTOT / 16;
  const int mt_wg = blockIdx.x * 2 * WT, nt_wg = blockIdx.y * 2 * WT;
  const int ncs = KC / KSTEP;    // macro steps per row tile in the fragment-tiled operands
  // gridDim.z workgroups share one output tile, each taking a contiguous part of the macro steps
  // that hold data and keeping its own partial accumulator (summed, in a fixed order, by
  // wgrad_finish_kernel).  A part may be empty (short last chunk): it then only initialises or
  // keeps its partial sum.
  const int nk_all = K / KSTEP;
  const int k_begin = (int)((long long)nk_all * blockIdx.z / gridDim.z);
  const int nk = (int)((long long)nk_all * (blockIdx.z + 1) / gridDim.z) - k_begin;
  const T* src[SW];   // row tiles q*4 + wave of dGT
  const T* srcB[WT];  // this wave's row tiles of aT
#pragma unroll
  for (int q = 0; q < SW; ++q) src[q] = dGT + (((size_t)min(mt_wg + q * 4 + wave, MT - 1) * ncs + k_begin) * 64 + lane) * VEC;
#pragma unroll
  for (int i = 0; i < WT; ++i) srcB[i] = aT + (((size_t)min(nt_wg + wn * WT + i, NT - 1) * ncs + k_begin) * 64 + lane) * VEC;
  const int extra_i = (int)blockIdx.y * 2 + wn;   // of this wave's row tiles, the one it multiplies with the extra tile (from WT on: none)
  const __amdgpu_buffer_rsrc_t extra_src =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(aT + (size_t)(NT - 1) * ncs * FRAG), 0, 0x7fffffff, 0x00020000);
  const int extra_off = extra_i < WT ? lane * 16 : (int)0x80000000u;
  const T* extra_a = &lds[0][(wm * WT + min(extra_i, WT - 1)) * FRAG + lane * VEC];
  u32x4 ring[PD][SW];
  typename M::Frag ringB[PD][WT], ringE[PD];
  auto fetch = [&](int stage, int ks) {
    const size_t off = (size_t)min(ks, nk - 1) * FRAG;
    if constexpr (EXTRA)
      ringE[stage] = as_frag<typename M::Frag>(__builtin_amdgcn_raw_buffer_load_b128(extra_src, extra_off, (k_begin + min(ks, nk - 1)) * 1024, 0));
#pragma unroll
    for (int q = 0; q < SW; ++q) ring[stage][q] = *reinterpret_cast<const u32x4*>(src[q] + off);
#pragma unroll
    for (int i = 0; i < WT; ++i) ringB[stage][i] = M::load(srcB[i] + off);
  };
  auto stash = [&](int stage, int buf) {
#pragma unroll
    for (int q = 0; q < SW; ++q)
      *reinterpret_cast<u32x4*>(&lds[buf][(q * 4 + wave) * FRAG + lane * VEC]) = ring[stage][q];
  };
  f32x4 acc[WT][WT], acc_extra{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  if (nk > 0) {   // uniform over the workgroup
#pragma unroll
  for (int st = 0; st < PD; ++st) fetch(st, st);
  stash(0, 0);
  __syncthreads();
  for (int k0 = 0; k0 < nk; k0 += PD) {
#pragma unroll
    for (int j = 0; j < PD; ++j) {
      const int ks = k0 + j;           // macro step computed now (held in lds[ks & 1])
      if (ks < nk) {
        typename M::Frag af[WT];
#pragma unroll
        for (int i = 0; i < WT; ++i) af[i] = M::load(&lds[ks & 1][(wm * WT + i) * FRAG + lane * VEC]);
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
          for (int jj = 0; jj < WT; ++jj) acc[i][jj] = M::mma(af[i], ringB[j][jj], acc[i][jj]);
        // order of this block's LDS reads (0x100) and MFMAs (0x008): two reads ahead, then a row of MFMAs
        // and one read in turn, so that only the first reads of a macro step are waited for
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int i = 0; i < WT - 2; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, WT, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * WT, 0);
        if constexpr (EXTRA)
          if (extra_i < WT) acc_extra = M::mma(M::load(extra_a + (ks & 1) * 2 * WT * FRAG), ringE[j], acc_extra);   // a scalar branch
        fetch(j, ks + PD);             // ring slot j has been used for step ks; refill it PD steps ahead
        if (ks + 1 < nk) stash((j + 1) % PD, (ks + 1) & 1);
      }
      __syncthreads();
    }
  }
  }

  // Epilogue: the running sum lives in a tile-ordered accumulator (each wave's quarter is one
  // contiguous run, a lane's four accumulator rows one float4), so the
  // read-modify-write of every chunk is fully coalesced; wgrad_finish_kernel converts it to the
  // caller's row-major dW once at the end of the run.
  // A part's accumulator: all blocks' tiles, then the extra tile's products, one after the other.
  float4* accp = reinterpret_cast<float4*>(dWacc) +
                 (((size_t)blockIdx.z * gridDim.x * gridDim.y + blockIdx.x * gridDim.y + blockIdx.y) * 4 + wave) * (WT * WT) * 64 + lane;
  if constexpr (EXTRA) {
    const size_t whole = (size_t)gridDim.x * gridDim.y * 4 * (WT * WT) * 64, extra = (size_t)gridDim.x * 2 * WT * 64;
    accp += blockIdx.z * extra;
    if (extra_i < WT) {
      float4* to = reinterpret_cast<float4*>(dWacc) + blockIdx.z * (whole + extra) + whole + (size_t)(mt_wg + wm * WT + extra_i) * 64 + lane;
      const float4 old = accumulate ? *to : float4{0.f, 0.f, 0.f, 0.f};
      *to = float4{acc_extra[0] + old.x, acc_extra[1] + old.y, acc_extra[2] + old.z, acc_extra[3] + old.w};
    }
  }
  if (accumulate) {
    float4 old[WT * WT];
#pragma unroll
    for (int q = 0; q < WT * WT; ++q) old[q] = accp[q * 64];
#pragma unroll
    for (int q = 0; q < WT * WT; ++q) {
      acc[q / WT][q % WT][0] += old[q].x;
      acc[q / WT][q % WT][1] += old[q].y;
      acc[q / WT][q % WT][2] += old[q].z;
      acc[q / WT][q % WT][3] += old[q].w;
    }
  }
#pragma unroll
  for (int q = 0; q < WT * WT; ++q)
    accp[q * 64] = float4{acc[q / WT][q % WT][0], acc[q / WT][q % WT][1], acc[q / WT][q % WT][2], acc[q / WT][q % WT][3]};
}

// dW_ih[row][n] / dW_hh[row][n] <- the tile-ordered accumulator (see wgrad_kernel's epilogue).
// The accumulator's column NX + HP (operand row of ones) holds the bias gradient.  ngates = 4
// (LSTM: db [4H]) or 3 (GRU: db = [db_ih | db_hh], 6H); the packed row of a gate block differs
// between the input and the recurrent side for the GRU (packed_gate_x / packed_gate_h).
// The first `nw` blocks do this, those behind them write the start state's gradients, whose arguments take scalar registers: seven
// waves per SIMD instead of eight.  2048 blocks, which filled eight, then leave an eighth part to wait for the others; 8192 do
// not (H = 3000, I = 128 121 us without the start state's part, 141 with it, 114 with 8192 blocks; H = 4096 325, 330, 209).
__global__ void wgrad_finish_kernel(const float* __restrict__ dWacc, int WT, int grid_y, int nsplit, size_t split_stride,
                                    int NX, int HP, int I, int H, int cell, float* __restrict__ dW_ih,
                                    float* __restrict__ dW_hh, float* __restrict__ db, int blocks, const float* __restrict__ dc,
                                    float* __restrict__ dh0, float* __restrict__ dc0, size_t plane, unsigned nw) {
  const int ngates = cell ? 3 : 4;
  const size_t nih = (size_t)ngates * H * I, nhh = (size_t)ngates * H * H, nb = (size_t)(cell ? 6 : 4) * H;
  const size_t total = nih + nhh + nb;
  const size_t stride = (size_t)nw * blockDim.x;
  if (blockIdx.x >= nw) {   // the start state's gradients from the running plane (dh0 holds dG_1 W_hh already)
    const size_t e = (size_t)(blockIdx.x - nw) * blockDim.x + threadIdx.x;
    if (e < plane) {
      if (cell) dh0[e] += dc[e];
      dc0[e] = cell ? 0.0f : dc[e];
    }
    return;
  }
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
    int row, np;
    bool recurrent;
    float* dst;
    if (idx < nih) {
      row = (int)(idx / I);
      np = (int)(idx % I);
      recurrent = false;
      dst = dW_ih + idx;
    } else if (idx < nih + nhh) {
      const size_t j = idx - nih;
      row = (int)(j / H);
      np = NX + (int)(j % H);
      recurrent = true;
      dst = dW_hh + j;
    } else {
      row = (int)(idx - nih - nhh);
      recurrent = row >= ngates * H;   // only the GRU has a second (recurrent) bias block
      if (recurrent) row -= ngates * H;
      np = NX + HP;
      dst = db + (idx - nih - nhh);
    }
    const int gate = row / H, u = row % H;
    int prow = gate;                                    // packed row of this gate block
    if (cell) prow = recurrent ? (gate == 2 ? 3 : gate) : gate;
    const int mp = 4 * u + prow;
    const int mt = mp >> 4, lq = (mp & 15) >> 2, r = mp & 3;
    const int nt = np >> 4, lrow = np & 15;
    size_t off;
    if (WT == 0) {   // tgemm_kernel's blocks: 2 x 4 waves of 8 x 4 tiles per 256 x 256 workgroup
      const int wgx = mt >> 4, wi = (mt & 15) >> 3, ti = mt & 7;
      const int wgy = nt >> 4, wj = (nt & 15) >> 2, tj = nt & 3;
      const size_t inner = (((size_t)(wi + 2 * wj) * 32 + (ti * 4 + tj)) * 64 + (lq * 16 + lrow)) * 4 + r;
      const int block = wgx * grid_y + wgy, first_shared = (int)split_stride;
      constexpr size_t BLOCK = 256 * 256;
      float v = dWacc[(size_t)block * BLOCK + inner];
      if (block >= first_shared)   // a block whose K was shared out: the other parts' sums, fixed order
        for (int sp = 1; sp < nsplit; ++sp)
          v += dWacc[((size_t)blocks + (size_t)(sp - 1) * (blocks - first_shared) + (block - first_shared)) * BLOCK + inner];
      *dst = v;
      continue;
    } else {
      const int wgx = mt / (2 * WT), wm = (mt % (2 * WT)) / WT, i = mt % WT;
      const int wgy = nt / (2 * WT), wn = (nt % (2 * WT)) / WT, jj = nt % WT;
      if (wgy == grid_y)   // the extra tile
        off = ((size_t)blocks * 4 * (WT * WT) * 64 + (size_t)mt * 64 + (lq * 16 + lrow)) * 4 + r;
      else
        off = ((((size_t)(wgx * grid_y + wgy) * 4 + (wm + 2 * wn)) * (WT * WT) + (i * WT + jj)) * 64 + (lq * 16 + lrow)) * 4 + r;
    }
    float v = dWacc[off];
    for (int sp = 1; sp < nsplit; ++sp) v += dWacc[(size_t)sp * split_stride + off];   // partial sums, fixed order
    *dst = v;
  }
}

// Blocks of the weight-gradient GEMM, and workgroups that share one along K.  Wave tiles of 4 x 4 MFMA tiles, 128 x 128 per workgroup,
// whenever the output has at least one such block in each direction, else 2 x 2.
// Where the blocks alone do not fill the chip, K is split for about 1.5 workgroups per compute unit.  bf16 GEMMs that run beside the
// sweeps stay at that: with two, H = 512, B = 128 takes 21.5 us a chunk for 22.1 but a gradient step that stores everything 1192 us for 1185, and
// without blocks for the row of ones B = 112, H = 499, t = 58 takes 578 us for 575.  Others have the chip to themselves, and fp32 products
// take longer than what they hold up: they take two workgroups per compute unit, as many as it holds at a time, and leave out the blocks
// of the row of ones (EXTRA), where that makes a chunk cheaper.  A chunk's cost is that of the compute unit with the most workgroups, in
// macro steps of 4 x 4 products (EXTRA: 17 for 16), and of its partial accumulators, which a run also reads once more at its end: a workgroup's
// 64 KiB take the time of 0.17 macro steps in bf16, 0.06 in fp32, all compute units at it; fewer workgroups than those write no faster.
// us a chunk, and a gradient step, with the start's blocks / two workgroups / EXTRA:
//   H = 512, I = 128, B = 256        37.6 / 33.5 / 31.8, t = 128 1432 / 1417 / 1414       fp32 H = 512, I = 256, B = 64  90 / 71 / 63, 2454 / 2462 / 2443
//   H = 256, I = 256, B = 64         12.4 / 12.4 / 10.5, t = 128  669 /  669 /  662       fp32 H = 448, I = 64, B = 250  206 / 152 / 144, 5173 / 5102 / 5010
//   H = 448, I = 29, B = 250         32.9 / 33.5 / -,    t = 128 1356 / 1360: not taken    fp32 H = 256, I = 128, B = 32  25.3 / 25.3 / 26.1, 1096 / 1096 / 1101: not
//   H = 128, I = 128, B = 32          6.7 /  6.7 /  7.3, t = 128  540 /  540 /  544: not   fp32 H = 128, I = 128, B = 64  21.5 / 21.5 / 23.4, 828 / 828 / 839: not
//   H = 512, I = 128, B = 16         12.5 / 13.9 / 12.5, t = 128  694 /   -  /  697: not
// (Above one block per compute unit, where K is not split, EXTRA costs as well: H = 1024, I = 256, 352 -> 320 blocks 36.3 -> 39.3 us.)
// More accumulators than the first choice's are taken only by shapes that mebptt_run_static, whose workspace is of a fixed size, refuses anyway.
struct WgradPlan {
  int wt, gx, gy, splits;
  bool extra;
  int blocks() const { return gx * gy; }
  size_t partial_floats() const { return ((size_t)blocks() * 4 * wt * wt + (extra ? (size_t)gx * 2 * wt : 0)) * 64 * 4; }   // one partial accumulator
  size_t accumulator_bytes() const { return partial_floats() * splits * sizeof(float); }
};
static WgradPlan wgrad_plan(const Dims& d) {
  const int MT = d.G4 / 16, NT = d.NA / 16, wt = MT >= 8 && NT >= 8 ? 4 : 2;
  auto split = [](int blocks, int workgroups) { return std::max(1, std::min(workgroups / blocks, 8)); };
  WgradPlan p{wt, (MT + 2 * wt - 1) / (2 * wt), (NT + 2 * wt - 1) / (2 * wt), 0, false};
  p.splits = split(p.blocks(), 384 + p.blocks() / 2);
  if (wt == 2 || p.blocks() > TARGET_WGS || (d.dtype && gemms_beside(d))) return p;
  const double steps = d.KC / (d.dtype ? 32 : 16), accumulator = d.dtype ? 0.17 : 0.06;
  auto cost = [&](const WgradPlan& q) {
    const int workgroups = q.blocks() * q.splits;
    return (workgroups + TARGET_WGS - 1) / TARGET_WGS * steps / q.splits * (q.extra ? 17.0 / 16 : 1) + accumulator * std::max(workgroups, TARGET_WGS);
  };
  const size_t chunk_buffers = 2 * ((size_t)d.CH * d.BP * d.G4 + (size_t)(d.G4 + d.NA) * d.KC) * d.op_bytes();
  const size_t most = p.accumulator_bytes() + chunk_buffers > MEBPTT_STATIC_WORKSPACE_BYTES ? ~(size_t)0 : p.accumulator_bytes();
  WgradPlan two = p;
  two.splits = split(p.blocks(), 2 * TARGET_WGS);
  if (two.accumulator_bytes() <= most && cost(two) < 0.99 * cost(p)) p = two;
  if (NT % (2 * wt) == 1 && 2 * (p.gy - 1) >= wt) {   // 2 * gy >= wt: the extra products are dealt out over that many waves a row
    WgradPlan best = p;
    for (const int workgroups : {384 + (p.gx * (p.gy - 1)) / 2, 2 * TARGET_WGS}) {
      WgradPlan q = p;
      q.gy = p.gy - 1;
      q.extra = true;
      q.splits = split(q.blocks(), workgroups);
      if (q.accumulator_bytes() <= most && cost(q) < std::min(0.95 * cost(p), cost(best))) best = q;
    }
    p = best;
  }
  return p;
}
size_t wgrad_accumulator_bytes(const Dims& d) {
  if (wgrad_uses_big_tiles(d)) {   // one padded 256 x 256 block per workgroup
    const size_t gx = (d.G4 / 16 + 15) / 16, gy = (d.NA / 16 + 15) / 16;
    int full, split;
    tgemm_shares((int)(gx * gy), full, split);
    return (gx * gy + (gx * gy - full) * (split - 1)) * 256 * 256 * sizeof(float);
  }
  return wgrad_plan(d).accumulator_bytes();
}

template <class T>
static void launch_wgrad_t(const Dims& d, const void* dGT, const void* aT, int K, int accumulate, float* dWacc,
                           hipStream_t st) {
  const WgradPlan plan = wgrad_plan(d);
  const dim3 grid(plan.gx, plan.gy, plan.splits), block(256);
  auto launch = [&](auto kernel) { kernel<<<grid, block, 0, st>>>((const T*)dGT, (const T*)aT, K, d.KC, d.G4, d.NA, accumulate, dWacc); };
  if (plan.wt == 2)
    launch(wgrad_kernel<T, 2, false>);
  else
    plan.extra ? launch(wgrad_kernel<T, 4, true>) : launch(wgrad_kernel<T, 4, false>);
}

hipError_t launch_wgrad(const Dims& d, const void* dGT, const void* aT, int nslots, int accumulate, float* dWacc,
                        hipStream_t st) {
  const int kstep = d.dtype ? 32 : 16;
  const int K = round_up(nslots * d.B, kstep);   // columns past nslots*B are zero
  if (wgrad_uses_big_tiles(d)) {
    TgemmParams p{};
    p.A = dGT;
    p.B = aT;
    p.mt_total = d.G4 / 16;
    p.nt_total = d.NA / 16;
    p.a_steps = p.b_steps = d.KC / 32;
    p.nk = K / 32;
    p.gx = (p.mt_total + 15) / 16;
    p.gy = (p.nt_total + 15) / 16;
    p.acc = dWacc;
    p.accumulate = accumulate;
    tgemm_shares(p.gx * p.gy, p.full, p.split);
    p.extra = dWacc + (size_t)p.gx * p.gy * 256 * 256;
    return launch_tgemm<__bf16>(p, st);
  }
  if (d.dtype)
    launch_wgrad_t<__bf16>(d, dGT, aT, K, accumulate, dWacc, st);
  else
    launch_wgrad_t<float>(d, dGT, aT, K, accumulate, dWacc, st);
  return hipGetLastError();
}

hipError_t launch_wgrad_finish(const Dims& d, const float* dWacc, float* dW_ih, float* dW_hh, float* db, const float* dc,
                               float* dh0, float* dc0, hipStream_t st) {
  const size_t plane = (size_t)d.B * d.H;
  const size_t values = (size_t)(d.cell ? 3 : 4) * d.H * ((size_t)d.I + d.H) + (size_t)(d.cell ? 6 : 4) * d.H;
  const unsigned nw = (unsigned)std::min<size_t>((values + 255) / 256, 8192);
  const dim3 grid(nw + (unsigned)((plane + 255) / 256));
  if (wgrad_uses_big_tiles(d)) {
    const int gx = (d.G4 / 16 + 15) / 16, gy = (d.NA / 16 + 15) / 16;
    int full, split;
    tgemm_shares(gx * gy, full, split);
    // nsplit and split_stride: here the shares of the left-over blocks and the first of those blocks
    wgrad_finish_kernel<<<grid, dim3(256), 0, st>>>(dWacc, 0, gy, split, (size_t)full, d.NX, d.HP, d.I, d.H, d.cell,
                                                          dW_ih, dW_hh, db, gx * gy, dc, dh0, dc0, plane, nw);
    return hipGetLastError();
  }
  const WgradPlan plan = wgrad_plan(d);
  wgrad_finish_kernel<<<grid, dim3(256), 0, st>>>(dWacc, plan.wt, plan.gy, plan.splits, plan.partial_floats(), d.NX, d.HP,
                                                        d.I, d.H, d.cell, dW_ih, dW_hh, db, plan.blocks(), dc, dh0, dc0, plane, nw);
  return hipGetLastError();
}

}  // namespace mebptt
