// Resident launches: forward chains and sweeps, whose workgroups keep weights on the chip for many
// time steps (see the comments at each kernel).
#include "resident_sweep.h"

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
size_t resident_sync_bytes() { return (RES_SYNC_STATUS + 64) * sizeof(unsigned); }
size_t resident_status_offset() { return RES_SYNC_STATUS * sizeof(unsigned); }

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

// ---- which shapes have sweeps ------------------------------------------------------------------------------
struct SweepConfig {
  int nrt, nxw, nhw, ksf, nbw, ksb, nbt;
  hipError_t (*launch)(const SweepParams&, hipStream_t);
};
#define SWEEP(T, NRT, NXW, NHW, KSF, NBW, NBL, KSB, NBT) \
  {NRT, NXW, NHW, KSF, NBW, KSB, NBT, launch_sweep_cell<T, true, NRT, NXW, NHW, KSF, NBW, NBL, KSB, NBT, 0>}
static const SweepConfig SWEEP_BF16[] = {
    SWEEP(__bf16, 4, 1, 4, 4, 8, 0, 8, 1), SWEEP(__bf16, 4, 1, 4, 4, 8, 8, 8, 2),   // H = 512, I <= 128
    SWEEP(__bf16, 2, 2, 2, 4, 4, 0, 8, 1), SWEEP(__bf16, 2, 2, 2, 4, 4, 0, 8, 2),   // H = 256, I <= 256
    SWEEP(__bf16, 1, 1, 1, 4, 4, 0, 4, 1), SWEEP(__bf16, 1, 1, 1, 4, 4, 0, 4, 2),   // H = 128, I <= 128
};
struct BackSweepConfig {
  int nrt, nbw, ksb, nbt;
  hipError_t (*launch[2])(const SweepParams&, hipStream_t);   // by cell
};
#define BACK_SWEEP(T, NRT, NBW, NBL, KSB, NBT)                                           \
  {NRT, NBW, KSB, NBT, {launch_sweep_cell<T, false, NRT, 1, 1, 8, NBW, NBL, KSB, NBT, 0>, \
                        launch_sweep_cell<T, false, NRT, 1, 1, 8, NBW, NBL, KSB, NBT, 1>}}
static const BackSweepConfig BACK_SWEEP_BF16[] = {
    BACK_SWEEP(__bf16, 8, 16, 4, 8, 1),                                        // H = 1024
    BACK_SWEEP(__bf16, 4, 8, 0, 8, 1), BACK_SWEEP(__bf16, 4, 8, 0, 8, 2),         // H = 512
    BACK_SWEEP(__bf16, 2, 4, 0, 8, 1), BACK_SWEEP(__bf16, 2, 4, 0, 8, 2),         // H = 256
    BACK_SWEEP(__bf16, 1, 4, 0, 4, 1), BACK_SWEEP(__bf16, 1, 4, 0, 4, 2),         // H = 128
};

struct SweepShape {
  int nrt, nsx, nsh, ksf, nsb, ksb, nbt;
};
static bool sweep_shape(const Dims& d, SweepShape& s) {
  const int share = group_share(d);
  if (!d.dtype || share == 0) return false;
  const int kstep = 32;
  const FwdConfig fc = forward_config<__bf16>(d);
  s.nrt = (d.KH + 127) / 128;
  s.nsx = d.KX / kstep;
  s.nsh = d.KH / kstep;
  s.nsb = d.G4 / kstep;
  s.ksf = (fc == FWD_TINY || fc == FWD_SMALLK) ? 4 : 8;   // the K splits of the per-step kernels
  s.ksb = backward_config<__bf16>(d) == BWD_SMALLK ? 4 : 8;
  s.nbt = share > 16 ? 2 : 1;
  return true;
}
static const SweepConfig* sweep_config(const Dims& d) {   // with forward operations: LSTM only
  SweepShape s;
  if (d.cell || d.I < 8 || !sweep_shape(d, s)) return nullptr;
  for (const SweepConfig& c : SWEEP_BF16)
    if (c.nrt == s.nrt && c.ksf == s.ksf && c.ksb == s.ksb && c.nbt == s.nbt && c.nxw * s.ksf >= s.nsx &&
        c.nhw * s.ksf >= s.nsh && c.nbw * s.ksb >= s.nsb)
      return &c;
  return nullptr;
}
// For launches of backward operations on stored internal states, which read neither x nor the gate weights:
// any input width.
static const BackSweepConfig* back_sweep_config(const Dims& d) {
  SweepShape s;
  if (!sweep_shape(d, s)) return nullptr;
  for (const BackSweepConfig& c : BACK_SWEEP_BF16)
    if (c.nrt == s.nrt && c.ksb == s.ksb && c.nbt == s.nbt && c.nbw * s.ksb >= s.nsb) return &c;
  return nullptr;
}

bool can_run_sweep(const Dims& d) { return sweep_config(d) != nullptr; }
bool can_run_backward_sweep(const Dims& d) { return back_sweep_config(d) != nullptr; }
int sweep_max_steps() { return SWEEP_MAX_STEPS; }
size_t sweep_ring_bytes(const Dims& d) { return (size_t)RES_RING * d.BP * d.G4 * d.op_bytes(); }

hipError_t launch_sweep(const Dims& d, const SweepArgs& a, hipStream_t st) {
  const SweepConfig* with_forward = a.state ? nullptr : sweep_config(d);
  const BackSweepConfig* backward_only = a.state ? back_sweep_config(d) : nullptr;
  if ((!with_forward && !backward_only) || a.count < 1 || a.count > SWEEP_MAX_STEPS) return hipErrorInvalidValue;
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
  p.ring = a.ring;
  p.sync = a.sync;
  p.published = a.published;
  p.launch = a.launch;
  p.wait_ticks = g_wait_ticks;
  p.s_hi = a.s_hi;
  p.count = a.count;
  p.B = d.B;
  p.I = d.I;
  p.H = d.H;
  p.HP = d.HP;
  p.KX = d.KX;
  p.KH = d.KH;
  p.BP = d.BP;
  p.nb = group_share(d);
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
  return with_forward ? with_forward->launch(p, st) : backward_only->launch[d.cell](p, st);
}

}  // namespace mebptt
