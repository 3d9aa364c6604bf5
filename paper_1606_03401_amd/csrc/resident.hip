// Resident launches: forward chains and sweeps, whose workgroups keep weights on the chip for many
// time steps (see the comments at each kernel).
#include <algorithm>

#include "resident_wide.h"

namespace mebptt {

// The bound every wait of a resident launch runs under, in ticks of the 100 MHz wall clock.  A
// host-side setting so that a test can make the waits give up at once -- every workgroup then leaves
// through the same path as after a real time-out -- without anything hanging.
constexpr long long RES_WAIT_TICKS = 50000000;   // 0.5 s
static long long g_wait_ticks = RES_WAIT_TICKS;
void set_resident_wait_ticks(long long ticks) { g_wait_ticks = ticks < 0 ? RES_WAIT_TICKS : ticks; }

// How long a workgroup waits for the first exchange before it gives the launch up and runs alone: about as long
// as that then takes (so giving up costs at most twice what knowing beforehand would have), and no less than
// another resident launch or a chunk's GEMMs hold the chip.  A workgroup that runs alone streams its weights from
// its L2, at 50 - 80 GB/s (H = 1024, B = 64: 47 ms a gradient step of 60 steps, 1.4 ms together).
// (g_patience: what a test asks for; negative: nothing, 0: nobody to wait for.)
static long long g_patience = -1;
void set_resident_patience(long long ticks) { g_patience = ticks; }
constexpr double ALONE_BYTES_PER_TICK = 600.0;   // 60 GB/s
constexpr long long MIN_PATIENCE = 50000;        // 0.5 ms
static long long patience(const Dims& d, int steps, size_t weights_per_step) {
  if (g_patience >= 0) return std::min(g_patience > 0 ? g_patience : 100LL, g_wait_ticks);
  const double ticks = (double)steps * (double)weights_per_step * d.op_bytes() / ALONE_BYTES_PER_TICK;
  return std::min(std::max(MIN_PATIENCE, (long long)ticks), g_wait_ticks / 4);
}

// ---- which shapes have forward chains -------------------------------------------------------------------
// Sequences per XCD: as few as keep all of them on the chip at once, in whole halves of an MFMA tile, so
// that no group straddles tiles (a step takes the same time for 1 and for 8 sequences, so with B < 64
// fewer XCDs work rather than all of them on less).  Returns 0 for a batch that does not fit.
static int group_share(const Dims& d) { return d.B <= 64 ? 8 : (d.B <= 128 ? 16 : (d.B <= 256 ? 32 : 0)); }

// What a shape asks of an instantiation.
struct ResidentShape {
  int nrt, nsx, nsh, ksf, nsb, ksb, nbt;   // units per workgroup / 4; macro steps and K splits; batch tiles per XCD
};
template <class T>
static bool resident_shape_t(const Dims& d, ResidentShape& s) {
  const int share = group_share(d), kstep = 4 * Mma<T>::VEC;
  if (share == 0 || d.H < 8) return false;
  const FwdConfig fc = forward_config<T>(d);
  s.nrt = (d.KH + 127) / 128;
  s.nsx = d.KX / kstep;
  s.nsh = d.KH / kstep;
  s.nsb = d.G4 / kstep;
  s.ksf = (fc == FWD_TINY || fc == FWD_SMALLK) ? 4 : 8;   // the K splits of the per-step kernels
  s.ksb = backward_config<T>(d) == BWD_SMALLK ? 4 : 8;
  s.nbt = share / 16;   // 0: half a tile
  return true;
}
static bool resident_shape(const Dims& d, ResidentShape& s) {
  return d.dtype ? resident_shape_t<__bf16>(d, s) : resident_shape_t<float>(d, s);
}
// A row of x is fetched in windows of 16 bytes of operands: it has to be at least that long.
static bool x_wide_enough(const Dims& d) { return d.I >= (d.dtype ? 8 : 4); }

// The smallest instantiation the shape fits (a table lists them in rising order of x width), or NULL.
static const ChainConfig* chain_config(const Dims& d) {
  ResidentShape s;
  if (!x_wide_enough(d) || !resident_shape(d, s)) return nullptr;
  const Table<ChainConfig> table = d.dtype ? (s.ksf == 4 ? chain_table_bf16_k4() : chain_table_bf16_k8())
                                           : (s.ksf == 4 ? chain_table_fp32_k4() : chain_table_fp32_k8());
  for (int i = 0; i < table.n; ++i) {
    const ChainConfig& c = table.at[i];
    if (c.nrt == s.nrt && c.ks == s.ksf && c.nbt == s.nbt && c.nhw * s.ksf >= s.nsh && c.nxw * s.ksf >= s.nsx) return &c;
  }
  return nullptr;
}

// The wide launches of a shape, or NULL; see wide_shape.
static const WideConfig* wide_config(const Dims& d) {
  const WideShape w = wide_shape(d);
  if (!w.groups) return nullptr;
  for (const Table<WideConfig>& table : {wide_table_1(), wide_table_2(), wide_table_3()})
    for (int i = 0; i < table.n; ++i) {
      const WideConfig& c = table.at[i];
      if (c.nr == w.nr && c.nhw * 4 * 32 >= d.KH && c.nb * 16 >= w.share) return &c;
    }
  return nullptr;
}
// Blocks of 16 * nr units of a wide sweep, and a slot of its partial sums: every four workgroups of a block send each other
// a quarter of the block's units of their sequences.
static int wide_blocks(const Dims& d, const WideConfig& c) { return (d.HP + 16 * c.nr - 1) / (16 * c.nr); }
static size_t wide_part_bytes(const Dims& d, const WideConfig& c) {
  return (size_t)wide_shape(d).groups * wide_blocks(d, c) * 16 * (4 * c.nr * 16 * c.nb) * sizeof(float);
}

bool runs_wide(const Dims& d) { return wide_config(d) != nullptr; }
bool can_run_forward_chain(const Dims& d) { return chain_config(d) != nullptr || runs_wide(d); }
// A wide chain launch reads x as operands, which a kernel ahead of it lays out for all its steps.
static size_t x_step_bytes(const Dims& d) { return (size_t)d.BP * d.KX * d.op_bytes(); }
int forward_chain_max_steps(const Dims& d) {
  return runs_wide(d) ? (int)std::min<size_t>(RES_MAX_STEPS, WIDE_X_BYTES / x_step_bytes(d)) : RES_MAX_STEPS;
}
size_t forward_chain_x_bytes(const Dims& d) { return runs_wide(d) ? forward_chain_max_steps(d) * x_step_bytes(d) : 0; }
size_t forward_chain_ring_bytes(const Dims& d) { return (size_t)(runs_wide(d) ? WIDE_RING : RES_RING) * d.BP * d.KH * d.op_bytes(); }
size_t resident_sync_bytes() { return (RES_SYNC_STATUS + 64) * sizeof(unsigned); }
size_t resident_status_offset() { return RES_SYNC_STATUS * sizeof(unsigned); }

hipError_t launch_forward_chain(const Dims& d, const void* Wp, const float* bp, const float* x_first, const float* src_unit,
                                const ChainStep* steps, int count, void* ring, float* spare, unsigned* sync, unsigned published,
                                unsigned launch, unsigned nth, void* xs, hipStream_t st) {
  const WideConfig* wide = wide_config(d);
  const ChainConfig* cfg = wide ? nullptr : chain_config(d);
  if ((!cfg && !wide) || count < 1 || count > forward_chain_max_steps(d)) return hipErrorInvalidValue;
  WideChainParams p{};
  p.Wp = Wp;
  p.bp = bp;
  p.x0 = x_first;
  p.src = src_unit;
  p.ring = ring;
  p.spare = spare;
  p.sync = sync;
  p.published = published;
  p.launch = launch;
  p.wait_ticks = g_wait_ticks;
  const int share = wide ? wide_shape(d).share : group_share(d);
  p.patience = patience(d, count, (size_t)d.G4 * d.KP * ((share + 15) / 16));
  p.alone = g_patience == 0;
  p.count = count;
  p.B = d.B;
  p.I = d.I;
  p.H = d.H;
  p.HP = d.HP;
  p.KX = d.KX;
  p.KH = d.KH;
  p.BP = d.BP;
  p.nb = share;
  p.unit = d.unit;
  p.hplane = d.hplane;
  for (int j = 0; j < count; ++j) p.step[j] = ResStep{steps[j].out, steps[j].gates};
  if (wide) {
    p.groups = wide_shape(d).groups;
    p.arrived = nth * (unsigned)((d.KH + 4 * wide->nr - 1) / (4 * wide->nr));
    p.xs = xs;
    const hipError_t e = launch_x_operands(d, x_first, count, xs, st);
    return e == hipSuccess ? wide->chain[d.cell](p, st) : e;
  }
  return cfg->launch[d.cell](p, st);
}

// ---- which shapes have sweeps ------------------------------------------------------------------------------
static const SweepConfig* sweep_config(const Dims& d) {   // with forward operations: LSTM only
  ResidentShape s;
  if (d.cell || !x_wide_enough(d) || !resident_shape(d, s)) return nullptr;
  // fp32 stores are twice as wide: spread over all 8 waves (a whole tile, half of it empty) they are faster than packed
  // into 4 (H = 256, B = 32: 43 against 48 us a launch of 9 steps)
  if (!d.dtype && s.nbt == 0) s.nbt = 1;
  const Table<SweepConfig> table = d.dtype ? sweep_table_bf16() : sweep_table_fp32();
  for (int i = 0; i < table.n; ++i) {
    const SweepConfig& c = table.at[i];
    if (c.nrt == s.nrt && c.ksf == s.ksf && c.ksb == s.ksb && c.nbt == s.nbt && c.nxw * s.ksf >= s.nsx &&
        c.nhw * s.ksf >= s.nsh && c.nbw * s.ksb >= s.nsb)
      return &c;
  }
  return nullptr;
}
// For launches of backward operations on stored internal states, which read neither x nor the gate weights:
// any input width.
static const BackSweepConfig* back_sweep_config(const Dims& d) {
  ResidentShape s;
  if (!resident_shape(d, s)) return nullptr;
  const Table<BackSweepConfig> table = d.dtype ? back_sweep_table_bf16() : back_sweep_table_fp32();
  for (int i = 0; i < table.n; ++i) {
    const BackSweepConfig& c = table.at[i];
    if (c.nrt == s.nrt && c.ksb == s.ksb && c.nbt == s.nbt && c.nbw * s.ksb >= s.nsb) return &c;
  }
  return nullptr;
}

bool can_run_sweep(const Dims& d) { return sweep_config(d) != nullptr; }
bool can_run_backward_sweep(const Dims& d) { return back_sweep_config(d) != nullptr || runs_wide(d); }

// Whether the time-batched GEMMs go to a stream of their own, beside the sequential work.  Launch-per-step
// kernels fill the device, and the two only get in each other's way (H = 2048: 2.8 % slower beside,
// H = 4096: 1.4 %).  A resident launch needs every compute unit at once: GEMMs beside it run in the gaps
// between launches and hold the next one up, each chunk costs two events and their waits, and a sweep launch may not
// run on into a chunk whose buffers are still being read.  That pays only where a chunk's GEMMs are long
// against the launches and the launches short.  Own stream against beside, a gradient step:
//   below 3 GFLOP a chunk: H = 32 (fp32) 163 / 206 us, H = 200, B = 37 1.04 / 1.13 ms, H = 256, B = 64 1.99 / 2.00;
//   B <= 32 (chunks of 64 steps): H = 512, 768, 1024 0.4 - 3.1 % faster, hidden and internal states stored;
//   B > 128: H = 384, 512 0.4 - 3.9 % faster;
//   between, -2.3 - +4.4 % (the sign turns with what the plan stores, which the rule does not look at): H = 384, 512
//   with internal states stored 1.6 - 2.3 % slower, with hidden states -0.4 - +1.8 %;
//   H = 1024, B = 64 1.4 % slower (GRU 1.8 %), H = 768, B = 128 1.5 % slower;
//   fp32, whose GEMMs take eight times as long, from 3 GFLOP on: H = 512, B = 32 0.9 % slower, H = 256, B = 256
//   0.6 % slower with hidden states stored, 7.8 % faster with internal ones (beside all the same: a rule by sizes alone).
//   wide launches: H = 2048, B = 128 0.4 % faster on the run's own stream, H = 4096, B = 32 even.
bool gemms_beside(const Dims& d) {
  if ((!can_run_forward_chain(d) && !can_run_backward_sweep(d)) || runs_wide(d)) return false;
  const double chunk_flops = 8.0 * d.CH * d.B * d.H * ((double)d.I + d.H);
  return chunk_flops >= 3e9 && (d.dtype == 0 || (d.B > 32 && d.B <= 128));
}

int sweep_max_steps() { return SWEEP_MAX_STEPS; }
size_t sweep_ring_bytes(const Dims& d) {
  const size_t slot = (size_t)d.BP * d.G4 * d.op_bytes();
  if (const WideConfig* c = wide_config(d)) return WIDE_RING * slot + WIDE_PART_RING * wide_part_bytes(d, *c);   // slots of dG, then of partial sums
  return RES_RING * slot;
}

hipError_t launch_sweep(const Dims& d, const SweepArgs& a, hipStream_t st) {
  const WideConfig* wide = a.state ? wide_config(d) : nullptr;
  const SweepConfig* with_forward = a.state ? nullptr : sweep_config(d);
  const BackSweepConfig* backward_only = a.state && !wide ? back_sweep_config(d) : nullptr;
  if ((!with_forward && !backward_only && !wide) || a.count < 1 || a.count > SWEEP_MAX_STEPS) return hipErrorInvalidValue;
  if ((a.s_hi - 1) / d.CH - (a.s_hi - a.count) / d.CH > 1) return hipErrorInvalidValue;   // two chunk buffers
  WideSweepParams p{};
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
  p.ring = a.ring;
  p.sync = a.sync;
  p.published = a.published;
  p.launch = a.launch;
  p.wait_ticks = g_wait_ticks;
  const int share = wide ? wide_shape(d).share : group_share(d);
  p.patience = patience(d, a.count, (size_t)d.G4 * (d.HP + (a.state ? 0 : d.KP)) * ((share + 15) / 16));
  p.alone = g_patience == 0;
  p.s_hi = a.s_hi;
  p.count = a.count;
  p.B = d.B;
  p.I = d.I;
  p.H = d.H;
  p.HP = d.HP;
  p.KX = d.KX;
  p.KH = d.KH;
  p.BP = d.BP;
  p.nb = share;
  p.G4 = d.G4;
  p.NX = d.NX;
  p.KC = d.KC;
  p.CH = d.CH;
  p.unit = d.unit;
  p.hplane = d.hplane;
  for (int j = 0; j < a.count; ++j) {
    p.src[j] = a.src[j];
    p.state[j] = a.state ? a.state[j] : nullptr;
  }
  if (wide) {
    p.groups = wide_shape(d).groups;
    p.arrived = a.nth * 4u * (unsigned)wide_blocks(d, *wide);
    p.parts = reinterpret_cast<char*>(a.ring) + (size_t)WIDE_RING * d.BP * d.G4 * d.op_bytes();
    return wide->sweep[d.cell](p, st);
  }
  return with_forward ? with_forward->launch(p, st) : backward_only->launch[d.cell](p, st);
}

}  // namespace mebptt
