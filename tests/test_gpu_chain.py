"""GPU tests of the forward-chain and sweep launches (a chain of forward operations, or a run of
forward+backward pairs, in one launch, weights resident on the chip, the batch split over the
XCDs): against the float64 oracle, bit for
bit against the launch-per-step path on the same inputs, for every strategy and many budgets, on
every shape class the kernel is instantiated for, with ragged batches, and from two host threads
at once."""
import threading

import numpy as np
import pytest

from oracle import lstm_bptt as ob
from paper_1606_03401_amd import binding as mb
from paper_1606_03401_amd import workloads as wl

pytestmark = pytest.mark.gpu

FIELDS = ("dW_ih", "dW_hh", "db", "dh0", "dc0", "dx", "y")


def _same(a, b, what=""):
    for f in FIELDS:
        assert np.array_equal(getattr(a, f), getattr(b, f)), (what, f)


def _run(w, inp, kind, m, chain):
    from paper_1606_03401_amd.session import Session
    mb.mebptt_forward_chain_enable(chain)
    try:
        s = Session(w, inp, kind=kind, m=m)
        out = s.run_and_fetch()          # raises if a chain launch gave up
    finally:
        mb.mebptt_forward_chain_enable(True)
    return out


SHAPES = [
    # B, I, H, t: (H/128, steps per wave, K split, batch tiles per XCD) in the comment
    (64, 128, 128, 40),     # (1, 2, 4, 1)
    (37, 100, 128, 33),     # (1, 2, 4, 2): ragged batch, groups straddle tiles, ragged I
    (5, 128, 128, 20),      # fewer sequences than XCDs
    (64, 256, 256, 60),     # (2, 4, 4, 1): the paper's experiment
    (150, 250, 256, 25),    # (2, 4, 4, 2)
    (256, 128, 512, 30),    # (4, 5, 4, 2): configuration 4's shape
    (100, 128, 512, 30),    # (4, 5, 4, 1)
    (64, 256, 1024, 60),    # (8, 5, 8, 1): configuration 2's shape
    (40, 250, 1024, 20),    # same class, ragged batch and input width
]


@pytest.mark.parametrize("B,I,H,t", SHAPES)
def test_chain_matches_per_step_path_and_oracle(B, I, H, t):
    from test_gpu_parity import TOL, check_against_oracle
    w = wl.Workload("chain", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=4, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, dy_first_step=2, seed=900 + B + H)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    ref = ob.lstm_bptt(inp.W_ih, inp.W_hh, inp.b, inp.x, inp.h0, inp.c0, inp.dy, w.dy_first_step)
    base = _run(w, inp, wl.KIND_HSM, 3, chain=False)
    check_against_oracle(w, inp, base, ref, TOL[w.gemm_dtype], label=f"chain {B}x{I}x{H} per-step: ")
    cases = [(wl.KIND_HSM, 1), (wl.KIND_HSM, 2), (wl.KIND_HSM, 3), (wl.KIND_HSM, 7), (wl.KIND_HSM, t),
             (wl.KIND_ISM, 1), (wl.KIND_ISM, 3), (wl.KIND_ISM, t), (wl.KIND_MSM, 2), (wl.KIND_MSM, 9), (wl.KIND_MSM, 4 * t)]
    for kind, m in cases:
        out = _run(w, inp, kind, m, chain=True)
        _same(out, base, (kind, m))
        assert out.stats.backward_ops == t


def test_chain_launch_count_and_status():
    """The launches really are chains: with the chain path on, a store-everything HSM plan of a
    long sequence needs far fewer forward launches than forward operations, and the status word
    stays clear."""
    from paper_1606_03401_amd.session import Session
    w = wl.Workload("chain-count", B=64, I=128, H=128, t=200, kind=wl.KIND_HSM, m=200, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, seed=31)
    inp = wl.make_inputs(w)
    s = Session(w, inp)
    mb.mebptt_profile_enable(1)
    out = s.run_and_fetch()
    prof = mb.mebptt_profile_collect()
    mb.mebptt_profile_enable(0)
    assert mb.mebptt_run_status(s.desc, s.workspace) == 0
    assert out.stats.forward_ops == 2 * w.t - 1
    assert prof.chain_steps >= w.t - 2                     # the initial forward pass went out as chains
    assert prof.launches[mb.K_CHAIN] <= (w.t + 47) // 48 + 1
    assert prof.sweep_steps >= w.t - 40                    # and the way back as sweep launches, one per chunk of steps
    assert prof.launches[mb.K_SWEEP] <= (w.t + 31) // 32 + 1
    assert prof.sweep_forward_steps == prof.sweep_steps    # these sweep launches recompute the internal states themselves
    assert (prof.launches[mb.K_FORWARD] + prof.launches[mb.K_PAIR] + prof.chain_steps + prof.sweep_forward_steps
            + prof.batch_steps == out.stats.forward_ops)
    assert prof.launches[mb.K_BACKWARD] + prof.launches[mb.K_PAIR] + prof.sweep_steps == w.t
    # store-everything BPTT (an internal-state slot per step): the forward pass as chains, the backward pass
    # through the stored states as backward-only sweep launches
    s2 = Session(w, inp, kind=wl.KIND_ISM, m=w.t)
    mb.mebptt_profile_enable(1)
    out2 = s2.run_and_fetch()
    prof2 = mb.mebptt_profile_collect()
    mb.mebptt_profile_enable(0)
    assert out2.stats.forward_ops == w.t and prof2.chain_steps >= w.t - 2 and prof2.sweep_forward_steps == 0
    assert prof2.sweep_steps >= w.t - 40 and prof2.launches[mb.K_BACKWARD] + prof2.sweep_steps == w.t
    for f in FIELDS:
        assert np.array_equal(getattr(out2, f), getattr(out, f)), f


@pytest.mark.parametrize("B,I,H,t", [(64, 256, 1024, 70), (64, 120, 1024, 45), (128, 64, 1024, 40), (16, 30, 1024, 37), (100, 120, 1024, 45)])
def test_batched_recomputation(B, I, H, t):
    """H = 1024: the weights of both directions do not fit on the chip together, so the way back
    through a stretch of stored hidden states is one launch of independent forward operations (the
    internal states of up to a chunk of steps, into the stage) followed by one backward-only sweep
    launch.  The launches really are those, every forward operation is accounted for, and the
    gradients are the per-step path's bit for bit and the oracle's within tolerance."""
    from paper_1606_03401_amd.session import Session
    from test_gpu_parity import TOL, check_against_oracle
    w = wl.Workload("batch", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=t, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, dy_first_step=3, seed=400 + B)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    ref = ob.lstm_bptt(inp.W_ih, inp.W_hh, inp.b, inp.x, inp.h0, inp.c0, inp.dy, w.dy_first_step)
    base = _run(w, inp, wl.KIND_HSM, t, chain=False)
    for kind, m in ((wl.KIND_HSM, t), (wl.KIND_HSM, 9), (wl.KIND_HSM, 4), (wl.KIND_MSM, 30), (wl.KIND_ISM, t)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        assert mb.mebptt_run_status(s.desc, s.workspace) == 0
        _same(out, base, ("batched recomputation", kind, m))
        assert prof.sweep_forward_steps == 0 and prof.sweep_steps > 0
        assert prof.launches[mb.K_FWD_BATCH] <= prof.launches[mb.K_SWEEP]
        assert (prof.launches[mb.K_FORWARD] + prof.launches[mb.K_PAIR] + prof.chain_steps + prof.batch_steps
                == out.stats.forward_ops)
        assert prof.launches[mb.K_BACKWARD] + prof.launches[mb.K_PAIR] + prof.sweep_steps == t
        if kind == wl.KIND_HSM:   # a sweep launch may start with a step whose state a forward run left in the core
            assert prof.batch_steps <= prof.sweep_steps <= prof.batch_steps + prof.launches[mb.K_SWEEP]
        if kind == wl.KIND_HSM and m == t:
            assert prof.batch_steps >= t - 8     # all but single steps left over at chunk boundaries
        if kind == wl.KIND_ISM:
            assert prof.batch_steps == 0         # the internal states were stored on the way forward
    check_against_oracle(w, inp, base, ref, TOL[w.gemm_dtype], label=f"batched recomputation {B}x{I}x{H}: ")


# Batches of operations on 128 x 32 and 128 x 64 tiles (last value: which, test_gpu_routes asks by name): rows of x that are no whole fragments;
# operations of one, two, three and more batch tiles whose tiles straddle workgroups, the last one partly empty; odd numbers of macro steps;
# K split 8 and 4 ways for both cores; padding units.
TILED = [(20, 650, 650, 33, 0, 32), (37, 201, 600, 33, 0, 64), (48, 333, 1024, 33, 0, 64), (16, 250, 990, 33, 1, 32), (32, 256, 1024, 33, 1, 64),
         (120, 194, 520, 33, 1, 64), (64, 203, 515, 20, 0, 32), (33, 40, 1100, 18, 0, 64), (33, 301, 1100, 20, 0, 32), (130, 203, 600, 21, 1, 64),
         (20, 72, 2100, 12, 1, 32), (20, 72, 2100, 12, 0, 32), (17, 1300, 900, 33, 0, 64)]


@pytest.mark.parametrize("B,I,H,t,cell,columns", TILED)
def test_batches_on_large_tiles(B, I, H, t, cell, columns):
    w = wl.Workload("tiles", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=t, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY, dy_first_step=2,
                    cell=cell, seed=B + I + H)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    mb.mebptt_profile_enable(1)
    out = _run(w, inp, wl.KIND_HSM, t, chain=True)
    prof = mb.mebptt_profile_collect()
    mb.mebptt_profile_enable(0)
    assert prof.batch_steps >= t - 4
    _same(out, _run(w, inp, wl.KIND_HSM, t, chain=False), (B, I, H))


def test_chains_from_two_host_threads():
    """Two host threads with their own streams run chain-eligible workloads at the same time: the
    library orders the two runs on the device (each chain launch wants the whole chip) and both
    give the single-threaded result."""
    import torch
    from paper_1606_03401_amd.session import Session
    ws = [wl.Workload("cthr-a", B=64, I=128, H=128, t=90, kind=wl.KIND_HSM, m=6, gemm_dtype=wl.GEMM_BF16,
                      loss=wl.LOSS_EXTERNAL_DY, seed=81),
          wl.Workload("cthr-b", B=64, I=256, H=256, t=70, kind=wl.KIND_MSM, m=12, gemm_dtype=wl.GEMM_BF16,
                      loss=wl.LOSS_EXTERNAL_DY, seed=82)]
    inps = [wl.make_inputs(w, nonzero_state=True) for w in ws]
    want = [Session(w, i).run_and_fetch() for w, i in zip(ws, inps)]
    sessions = [Session(w, i) for w, i in zip(ws, inps)]
    streams = [torch.cuda.Stream() for _ in ws]
    torch.cuda.synchronize()
    errors, results = [], [[], []]

    def worker(k):
        try:
            for _ in range(5):
                sessions[k].run(stream=streams[k].cuda_stream)
                streams[k].synchronize()
                results[k].append(sessions[k].fetch())
        except Exception as exc:   # noqa: BLE001 - reported by the main thread
            errors.append(exc)

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join(timeout=100)
    assert not errors, errors
    assert all(not th.is_alive() for th in threads)
    for k in range(2):
        assert len(results[k]) == 5
        for got in results[k]:
            _same(got, want[k])


def test_bounded_waits_give_up_and_report():
    """With the wait bound set to zero from the host, a workgroup that does not find the others'
    data at its first look gives up: every kernel still runs to its end, the run returns, the status
    word says a wait gave up and the session refuses the results.  With the default bound restored
    the same session computes the right gradients again."""
    from paper_1606_03401_amd.session import Session
    w = wl.Workload("give-up", B=64, I=128, H=128, t=60, kind=wl.KIND_HSM, m=60, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, seed=77)
    inp = wl.make_inputs(w)
    s = Session(w, inp)
    good = s.run_and_fetch()
    mb.mebptt_resident_wait_limit(0)
    try:
        with pytest.raises(RuntimeError):
            s.run_and_fetch()
        assert mb.mebptt_run_status(s.desc, s.workspace) == 1
    finally:
        mb.mebptt_resident_wait_limit(-1)
    _same(s.run_and_fetch(), good, "after restoring the bound")


@pytest.mark.parametrize("B,I,H,t", [(64, 128, 128, 40), (37, 100, 128, 33), (64, 256, 256, 50), (150, 128, 512, 30),
                                     (64, 256, 1024, 40)])
def test_gru_forward_chains(B, I, H, t):
    """The GRU core through forward-chain launches (h kept in full precision in registers from step
    to step), backward-only sweep launches and forward batches: bit for bit the launch-per-step
    path's gradients for every strategy and several budgets, and the oracle's within tolerance."""
    from paper_1606_03401_amd.session import Session
    from test_gpu_parity import TOL, check_against_oracle, oracle_gradients
    w = wl.Workload("gru-chain", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=4, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, dy_first_step=2, seed=1200 + B + H, cell=wl.CELL_GRU)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 3, chain=False)
    check_against_oracle(w, inp, base, oracle_gradients(w, inp), TOL[w.gemm_dtype], label=f"gru chain {B}x{I}x{H} per-step: ")
    for kind, m in ((wl.KIND_HSM, 1), (wl.KIND_HSM, 3), (wl.KIND_HSM, t), (wl.KIND_ISM, 2), (wl.KIND_ISM, t), (wl.KIND_MSM, 7)):
        _same(_run(w, inp, kind, m, chain=True), base, (kind, m))
    s = Session(w, inp, kind=wl.KIND_ISM, m=t)
    mb.mebptt_profile_enable(1)
    out = s.run_and_fetch()
    prof = mb.mebptt_profile_collect()
    mb.mebptt_profile_enable(0)
    _same(out, base, "profiled")
    assert prof.chain_steps >= t - 2 and prof.batch_steps == 0 and prof.sweep_forward_steps == 0
    assert mb.mebptt_run_status(s.desc, s.workspace) == 0
    assert prof.sweep_steps >= t - 40          # stored internal states: backward-only sweep launches
    s = Session(w, inp, kind=wl.KIND_HSM, m=t)
    mb.mebptt_profile_enable(1)
    out = s.run_and_fetch()
    prof = mb.mebptt_profile_collect()
    mb.mebptt_profile_enable(0)
    _same(out, base, "profiled, hidden states")
    assert prof.batch_steps >= t - 40 and prof.sweep_steps >= prof.batch_steps   # forward batches feed the sweeps


@pytest.mark.parametrize("B,I,H", [(64, 128, 128), (64, 256, 1024)])
def test_runs_join_the_chain_before_them(B, I, H):
    """Where memory runs out the schedule ends a re-forwarding chain with a run that leaves an internal
    state in the working core, then the backward operation on it, then the pairs for the steps below.
    That backward operation does not get a launch of its own: the sweep launch that follows carries
    it (recomputing the state itself and the chain stopping one step short, or taking the state from
    the core).  Counted from the launches, with every forward and backward operation still accounted
    for exactly once and the gradients those of the launch-per-step path bit for bit."""
    from paper_1606_03401_amd.session import Session
    t, m = 150, 7
    w = wl.Workload("join", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=m, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, seed=733 + H)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, m, chain=False)
    s = Session(w, inp)
    sched = s.plan.schedule()
    CH = mb.mebptt_chunk_steps(s.desc)

    def pair_below(i):      # entries i, i + 1: forward operation of one step keeping its state, backward operation of it
        return (i + 1 < len(sched) and sched[i]["op"] == 1 and sched[i]["count"] == 1 and sched[i]["keep"]
                and sched[i + 1]["op"] == 2 and sched[i + 1]["step"] == sched[i]["step"])
    lone = [i for i in range(1, len(sched)) if sched[i]["op"] == 2 and sched[i - 1]["op"] == 1 and sched[i - 1]["count"] >= 2]
    joinable = [i for i in lone if pair_below(i + 1) and sched[i + 1]["step"] == sched[i]["step"] - 1
                and (sched[i]["step"] - 1) // CH == (sched[i]["step"] - 2) // CH]
    assert len(joinable) >= 10              # the schedule has many such backward operations ...
    lone, joinable = len(lone), len(joinable)
    mb.mebptt_profile_enable(1)
    out = s.run_and_fetch()
    prof = mb.mebptt_profile_collect()
    mb.mebptt_profile_enable(0)
    _same(out, base, "joined runs")
    assert mb.mebptt_run_status(s.desc, s.workspace) == 0
    # ... and none of them is launched alone (what is, are the ones no pair follows, and single pairs)
    assert prof.launches[mb.K_BACKWARD] + prof.launches[mb.K_PAIR] <= lone - joinable + 3
    assert (prof.launches[mb.K_FORWARD] + prof.launches[mb.K_PAIR] + prof.chain_steps + prof.sweep_forward_steps
            + prof.batch_steps == out.stats.forward_ops == s.plan.forward_ops)
    assert prof.launches[mb.K_BACKWARD] + prof.launches[mb.K_PAIR] + prof.sweep_steps == t


def test_batched_recomputation_with_the_loss_on_h():
    """The same path when the loss is half the sum of the squared outputs (dy_t = h_t): the backward-only
    sweep launch then takes the injected gradient from the states the forward-batch launch left in the
    stage."""
    from test_gpu_parity import TOL, check_against_oracle, oracle_gradients
    w = wl.Workload("batch-h2", B=64, I=64, H=1024, t=40, kind=wl.KIND_HSM, m=7, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_HALF_SUM_H2, seed=515)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 7, chain=False)
    for kind, m in ((wl.KIND_HSM, 7), (wl.KIND_HSM, 40), (wl.KIND_MSM, 25)):
        _same(_run(w, inp, kind, m, chain=True), base, (kind, m))
    check_against_oracle(w, inp, base, oracle_gradients(w, inp), TOL[w.gemm_dtype], label="batched recomputation, loss on h: ")


@pytest.mark.parametrize("B,I,H,t,m", [(64, 128, 128, 70, 6), (64, 256, 1024, 45, 8)])
def test_resident_launches_in_a_captured_graph(B, I, H, t, m):
    """A run whose sequential work goes out as chain, sweep and forward-batch launches, captured into
    a HIP graph: every replay -- with eager runs, clobbered outputs and synchronisations between
    them -- reproduces the eager result bit for bit and leaves the status word clear (the rank
    counters and exchange slots the captured launches start from are reset by the run's own first kernel)."""
    import torch
    from paper_1606_03401_amd.session import Session
    w = wl.Workload("graph-resident", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=m, gemm_dtype=wl.GEMM_BF16,
                    loss=wl.LOSS_EXTERNAL_DY, seed=610 + H)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, m, chain=False)
    s = Session(w, inp)
    eager = s.run_and_fetch()
    _same(eager, base, "eager")
    s.capture()
    for rep in range(4):
        for tsr in (s.dW_ih, s.dW_hh, s.db, s.dh0, s.dc0, s.dx, s.y):
            tsr.fill_(float("nan"))
        torch.cuda.synchronize()
        s.replay()
        _same(s.fetch(), eager, ("replay", rep))
        assert mb.mebptt_run_status(s.desc, s.workspace) == 0
        if rep % 2 == 0:          # the program's own eager work between replays
            _same(s.run_and_fetch(), eager, ("eager after replay", rep))


def test_random_shapes_budgets_and_strategies_bit_identical():
    """Seeded random cases over the shape classes with resident launches, both cores, every strategy,
    budgets from 1 to beyond t, sequences from 2 steps to several chunks, losses starting anywhere:
    with the chain, sweep and forward-batch launches (and everything the executor does to join and
    lengthen them) the gradients are those of the launch-per-step path bit for bit and finite."""
    rng = np.random.default_rng(20260)
    for case in range(160):
        H = int(rng.choice([128, 256, 512, 1024]))
        I = {128: int(rng.choice([8, 40, 64, 100, 128])), 256: int(rng.choice([136, 200, 256])),
             512: int(rng.choice([16, 64, 100, 128])), 1024: int(rng.choice([32, 128, 250, 256]))}[H]
        B = int(rng.choice([1, 3, 8, 17, 32, 50, 64, 100, 128, 200, 256]))
        if H == 1024 and B > 128:
            B = 64
        t = int(rng.integers(2, 90)) if rng.random() < 0.85 else int(rng.integers(90, 300))
        kind = int(rng.choice([wl.KIND_HSM, wl.KIND_ISM, wl.KIND_MSM]))
        m = int(rng.integers(1, t + 2)) if kind != wl.KIND_MSM else int(rng.integers(2, 4 * t + 2))
        w = wl.Workload("random", B=B, I=I, H=H, t=t, kind=kind, m=m, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY,
                        dy_first_step=int(rng.integers(1, t + 1)), seed=int(rng.integers(1, 10**6)),
                        cell=int(rng.random() < 0.2))
        inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
        what = (case, B, I, H, t, kind, m, w.dy_first_step, w.cell)
        base = _run(w, inp, kind, m, chain=False)
        got = _run(w, inp, kind, m, chain=True)
        _same(got, base, what)
        for f in FIELDS:
            assert np.all(np.isfinite(getattr(got, f))), (what, f)


# (B, I, H, core) around the edges of the resident instantiations: units that do not divide by 32 or by the
# compute units of an XCD, x rows that end inside a 16-byte window, inputs wider than the state, batches
# that leave XCDs idle or take two MFMA tiles per XCD.
EDGE_BF16 = [
    (4, 16, 32, 0), (5, 8, 9, 0), (64, 600, 100, 0), (70, 1000, 64, 0), (3, 2000, 128, 0), (37, 100, 200, 0), (130, 300, 200, 0),
    (20, 960, 160, 0), (20, 200, 384, 0), (200, 300, 300, 0), (40, 700, 384, 0), (20, 200, 500, 0), (150, 180, 512, 0),
    (16, 512, 512, 0), (200, 1000, 500, 0), (24, 90, 600, 0), (24, 512, 576, 0), (20, 650, 650, 0), (128, 300, 700, 0),
    (33, 1000, 768, 0), (17, 128, 896, 0), (17, 500, 800, 0), (100, 200, 1000, 0), (37, 100, 200, 1), (65, 77, 333, 1), (20, 650, 650, 1),
]
EDGE_FP32 = [
    (4, 16, 32, 0), (9, 100, 50, 0), (64, 256, 60, 0), (130, 4, 64, 0), (30, 64, 100, 0), (20, 500, 128, 0), (20, 900, 70, 0),
    (32, 64, 256, 0), (32, 128, 256, 0), (150, 300, 200, 0), (20, 700, 256, 0), (8, 32, 288, 0), (16, 200, 384, 0),
    (32, 200, 500, 0), (16, 1000, 512, 0), (200, 300, 512, 0), (9, 101, 50, 1), (16, 203, 301, 1),
]


@pytest.mark.parametrize("dtype,B,I,H,cell", [(wl.GEMM_BF16, *s) for s in EDGE_BF16] + [(wl.GEMM_FP32, *s) for s in EDGE_FP32])
def test_resident_launches_at_the_edges_of_their_shapes(dtype, B, I, H, cell):
    from paper_1606_03401_amd.session import Session
    t = 37
    w = wl.Workload("edge", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=5, gemm_dtype=dtype, loss=wl.LOSS_EXTERNAL_DY,
                    dy_first_step=3, seed=4000 + B + I + H, cell=cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 5, chain=False)
    for kind, m in ((wl.KIND_HSM, 5), (wl.KIND_HSM, t), (wl.KIND_ISM, t), (wl.KIND_MSM, 13)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        _same(out, base, (kind, m))
        assert mb.mebptt_run_status(s.desc, s.workspace) == 0
        assert prof.chain_steps > 0          # the shape really runs as resident launches


@pytest.mark.parametrize("dtype,B,I,H", [(wl.GEMM_BF16, 20, 40, 200), (wl.GEMM_FP32, 20, 40, 72), (wl.GEMM_BF16, 64, 64, 1024)])
def test_resident_launches_pass_on_every_nan(dtype, B, I, H):
    """The exchange marks what has not arrived by a bit pattern that is a NaN: an input that produces
    exactly that NaN must neither stall a launch nor reach a sequence it does not belong to."""
    w = wl.Workload("nan", B=B, I=I, H=H, t=24, kind=wl.KIND_HSM, m=6, gemm_dtype=dtype, loss=wl.LOSS_EXTERNAL_DY, seed=5)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    clean = _run(w, inp, wl.KIND_HSM, 6, chain=True)
    bad = 11
    inp.x[2, bad] = np.uint32(0xFFFFFFFF).view(np.float32)
    inp.h0[bad + 1] = np.uint32(0xFFFFFFFF).view(np.float32)
    inp.x[3, bad + 2, 0] = np.inf
    base = _run(w, inp, wl.KIND_HSM, 6, chain=False)
    out = _run(w, inp, wl.KIND_HSM, 6, chain=True)        # raises if a launch gave up
    others = [b for b in range(B) if b not in (bad, bad + 1, bad + 2)]
    assert np.array_equal(out.y[:, others], clean.y[:, others]) and np.array_equal(out.dx[:, others], clean.dx[:, others])
    assert np.isnan(out.y[2:, bad]).all()
    assert np.array_equal(np.isnan(out.y), np.isnan(base.y)) and np.array_equal(out.y[:, bad + 2], base.y[:, bad + 2], equal_nan=True)


# Weights that are infinite: a macro step that shares an instruction with an infinite weight's has to keep out of it (zero times
# infinity would be a NaN), and so has a zero that stands for a part's missing macro step.  Outputs are compared for infinite weights of h and
# x, gradients for those of x.  With infinite weights of h they are not: a sweep multiplies the zeros that stand for the step after the last
# one as well, which a launch per step leaves out, and is NaN a step sooner.
@pytest.mark.parametrize("B,I,H,cell", [(64, 64, 1024, 0), (20, 650, 650, 0), (16, 40, 705, 1)])
def test_infinite_weights(B, I, H, cell):
    w = wl.Workload("inf", B=B, I=I, H=H, t=20, kind=wl.KIND_HSM, m=6, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY, seed=6, cell=cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    inp.W_hh[5, 7], inp.W_hh[H + 9, H - 1], inp.W_ih[11, I - 1] = np.inf, -np.inf, np.inf
    base = _run(w, inp, wl.KIND_HSM, 6, chain=False)
    assert np.isfinite(base.y).all()     # an infinite gate sum is a gate of 0 or 1
    for kind, m in ((wl.KIND_HSM, 6), (wl.KIND_HSM, 20), (wl.KIND_ISM, 20)):
        assert np.array_equal(_run(w, inp, kind, m, chain=True).y, base.y)
    inp.W_hh[5, 7], inp.W_hh[H + 9, H - 1] = 0.25, -0.25
    base = _run(w, inp, wl.KIND_HSM, 6, chain=False)
    for name in ("dW_ih", "dW_hh", "db", "dh0", "dc0", "y"):
        assert np.isfinite(getattr(base, name)).all(), name
    for kind, m in ((wl.KIND_HSM, 6), (wl.KIND_HSM, 20), (wl.KIND_ISM, 20)):
        out = _run(w, inp, kind, m, chain=True)
        for name in FIELDS:
            assert np.array_equal(getattr(out, name), getattr(base, name), equal_nan=True), (kind, m, name)   # dx: infinite in one column


@pytest.mark.parametrize("B,I,H", [(32, 128, 512), (33, 300, 512), (128, 130, 384), (129, 130, 384), (40, 64, 256)])
def test_gemms_beside_or_between_resident_launches(B, I, H):
    """On both sides of every line of the rule that puts the time-batched GEMMs on a stream of their own:
    several chunks, with sweep launches that may run on from one chunk into the next."""
    t = 140
    w = wl.Workload("chunks", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=9, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY,
                    dy_first_step=20, seed=77 + B)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 9, chain=False)
    for kind, m in ((wl.KIND_HSM, 9), (wl.KIND_HSM, t), (wl.KIND_ISM, t), (wl.KIND_MSM, 30)):
        _same(_run(w, inp, kind, m, chain=True), base, (kind, m))


# as EDGE_*: both K splits of either direction, one and two batch tiles per XCD, padded units and x rows
ALONE = [(wl.GEMM_BF16, 5, 8, 9, 0), (wl.GEMM_BF16, 37, 100, 200, 0), (wl.GEMM_BF16, 70, 1000, 64, 0), (wl.GEMM_BF16, 150, 180, 500, 0),
         (wl.GEMM_BF16, 33, 300, 500, 1), (wl.GEMM_BF16, 100, 200, 1000, 0), (wl.GEMM_BF16, 65, 77, 333, 1), (wl.GEMM_BF16, 20, 650, 650, 1),
         (wl.GEMM_FP32, 4, 16, 32, 0), (wl.GEMM_FP32, 70, 100, 50, 0), (wl.GEMM_FP32, 130, 300, 200, 0), (wl.GEMM_FP32, 9, 101, 50, 1),
         (wl.GEMM_FP32, 32, 200, 500, 0), (wl.GEMM_FP32, 100, 203, 301, 1)]


@pytest.fixture(params=[0, 1], ids=["alone", "impatient"])
def patience(request):
    import torch   # noqa: F401 - its HIP runtime is the one the library uses
    mb.mebptt_resident_patience(request.param)
    yield
    mb.mebptt_resident_patience(-1)


@pytest.mark.parametrize("dtype,B,I,H,cell", ALONE)
def test_launches_that_are_given_up(patience, dtype, B, I, H, cell):
    """One workgroup per XCD instead of all of them gives the launch-per-step path's bits, and so does any
    mixture of those who wait and those who have lost their patience, whoever is there by then."""
    from paper_1606_03401_amd.session import Session
    t = 37
    w = wl.Workload("given-up", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=5, gemm_dtype=dtype, loss=wl.LOSS_EXTERNAL_DY,
                    dy_first_step=3, seed=5000 + B + I + H, cell=cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 5, chain=False)
    for kind, m in ((wl.KIND_HSM, 5), (wl.KIND_HSM, t), (wl.KIND_ISM, t), (wl.KIND_MSM, 13)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        _same(out, base, (kind, m))
        assert prof.chain_steps > 0 and prof.sweep_steps > 0
    w = w.scaled(loss=wl.LOSS_HALF_SUM_H2)
    base = _run(w, inp, wl.KIND_HSM, 5, chain=False)
    for kind, m in ((wl.KIND_HSM, 5), (wl.KIND_ISM, t)):
        _same(_run(w, inp, kind, m, chain=True), base, ("loss on h", kind, m))


def test_launches_given_up_and_not_in_turn():
    """What a launch leaves behind is the same either way: the exchange of the next one starts from it."""
    from paper_1606_03401_amd.session import Session
    for dtype, B, I, H in ((wl.GEMM_BF16, 64, 100, 200), (wl.GEMM_FP32, 20, 40, 72)):
        w = wl.Workload("turns", B=B, I=I, H=H, t=60, kind=wl.KIND_HSM, m=6, gemm_dtype=dtype, loss=wl.LOSS_EXTERNAL_DY, seed=B)
        s = Session(w, wl.make_inputs(w, nonzero_state=True, nonzero_bias=True))
        want = s.run_and_fetch()
        for ticks in (0, -1, 0, 1, 0, 1, -1):
            mb.mebptt_resident_patience(ticks)
            try:
                _same(s.run_and_fetch(), want, ticks)
            finally:
                mb.mebptt_resident_patience(-1)


@pytest.mark.parametrize("shapes", [((64, 128, 512), (64, 100, 500)), ((37, 100, 200), (20, 64, 300)), ((64, 256, 1024), (37, 100, 200))])
def test_replays_of_two_graphs_at_the_same_time(shapes):
    """Two captured runs replayed on two streams without any order between them: their resident launches
    meet on the chip and get into each other's way; both give the eager result every time, status 0."""
    import torch
    from paper_1606_03401_amd.session import Session
    sessions, want = [], []
    for k, (B, I, H) in enumerate(shapes):
        w = wl.Workload("meet", B=B, I=I, H=H, t=60, kind=wl.KIND_HSM, m=6, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY, seed=40 + k)
        s = Session(w, wl.make_inputs(w, nonzero_state=True, nonzero_bias=True))
        want.append(s.run_and_fetch())
        s.capture()
        sessions.append(s)
    streams = [torch.cuda.Stream() for _ in sessions]
    torch.cuda.synchronize()
    for rep in range(8):
        for s in sessions:
            s.dW_hh.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(3):
            for s, st in zip(sessions, streams):
                with torch.cuda.stream(st):
                    s.replay()
        torch.cuda.synchronize()
        for k, s in enumerate(sessions):
            _same(s.fetch(), want[k], (rep, k))      # fetch raises if a launch gave up


CHILD = """
import sys
import numpy as np
from paper_1606_03401_amd import binding as mb, workloads as wl
from paper_1606_03401_amd.session import Session
B, I, H = (int(v) for v in sys.argv[1:])
w = wl.Workload("process", B=B, I=I, H=H, t=60, kind=wl.KIND_HSM, m=6, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY, seed=B)
s = Session(w, wl.make_inputs(w, nonzero_state=True, nonzero_bias=True))
mb.mebptt_forward_chain_enable(False)
want = s.run_and_fetch()
mb.mebptt_forward_chain_enable(True)
for rep in range(30):
    for _ in range(10):
        s.run()
    out = s.run_and_fetch()          # raises if a launch failed
    assert all(np.array_equal(getattr(out, f), getattr(want, f)) for f in ("dW_ih", "dW_hh", "db", "dh0", "dc0", "dx", "y")), rep
"""


def test_two_processes_on_one_device():
    """Nothing orders the resident launches of two processes: they meet on the chip, and both compute the
    launch-per-step path's gradients every time."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    procs = [subprocess.Popen([sys.executable, "-c", CHILD, *map(str, shape)], cwd=root) for shape in ((64, 128, 512), (64, 100, 500))]
    try:
        assert [p.wait(timeout=90) for p in procs] == [0, 0]
    finally:
        for p in procs:
            if p.poll() is None:
                p.kill()


# (B, I, H, core): one shape for every instantiation of the resident kernels -- units per compute unit, macro steps of
# x, h and dG per wave, K splits, batch tiles per XCD, both cores -- that the shapes above do not select.
INSTANCES_BF16 = [
    (1, 21, 404, 0), (1, 52, 401, 1), (1, 54, 553, 1), (1, 62, 559, 0), (1, 83, 701, 1), (1, 93, 290, 1), (1, 93, 652, 0),
    (1, 111, 535, 1), (1, 171, 931, 1), (1, 176, 895, 1), (1, 267, 426, 1), (1, 291, 783, 1), (1, 308, 107, 0),
    (1, 313, 330, 1), (1, 317, 149, 0), (1, 414, 200, 1), (1, 727, 520, 0), (1, 782, 141, 1), (1, 818, 432, 0),
    (1, 836, 486, 1), (1, 945, 519, 1), (1, 956, 651, 1), (1, 1826, 24, 1), (2, 128, 28, 1), (2, 136, 59, 1),
    (2, 157, 461, 1), (2, 159, 20, 0), (2, 180, 424, 0), (2, 657, 11, 1), (16, 278, 9, 1), (65, 18, 281, 0),
    (65, 58, 783, 1), (65, 133, 401, 0), (65, 280, 14, 0), (65, 283, 790, 0), (65, 826, 653, 0), (66, 8, 403, 1),
    (66, 17, 129, 1), (66, 18, 523, 1), (66, 53, 773, 0), (66, 139, 400, 1), (66, 297, 769, 1), (66, 358, 282, 0),
    (66, 426, 9, 1), (66, 477, 170, 1), (66, 568, 400, 1), (66, 923, 671, 1), (67, 19, 680, 1), (67, 51, 141, 0),
    (67, 165, 453, 0), (67, 398, 286, 1), (68, 15, 900, 1), (68, 121, 515, 1), (68, 148, 514, 0), (68, 191, 9, 0),
    (68, 273, 133, 1), (68, 287, 147, 0), (69, 29, 531, 0), (69, 204, 426, 1), (70, 531, 674, 1), (70, 637, 535, 1),
    (71, 517, 534, 0), (71, 718, 394, 0), (72, 531, 137, 0), (72, 722, 16, 1), (73, 18, 17, 1), (77, 561, 647, 0),
    (84, 145, 11, 1), (85, 1069, 11, 1), (93, 18, 9, 0), (121, 1048, 9, 0), (129, 1214, 10, 0), (130, 57, 532, 0),
    (130, 257, 135, 1), (130, 483, 153, 1), (130, 1197, 9, 1), (132, 855, 10, 1), (133, 33, 517, 1), (135, 537, 402, 1),
    (136, 9, 392, 1), (136, 251, 408, 1), (136, 552, 9, 0), (137, 34, 140, 1), (138, 717, 129, 0), (139, 140, 413, 0),
    (139, 439, 257, 0), (140, 136, 11, 1), (140, 149, 385, 1), (142, 811, 11, 0), (143, 44, 10, 0), (144, 16, 260, 1),
    (149, 9, 9, 1), (154, 145, 9, 0), (154, 365, 265, 1), (180, 290, 9, 1),
]
INSTANCES_FP32 = [
    (1, 50, 148, 1), (1, 61, 449, 1), (1, 139, 99, 1), (1, 258, 167, 0), (1, 266, 467, 1), (1, 366, 497, 0),
    (1, 407, 129, 1), (1, 621, 155, 1), (1, 808, 397, 1), (2, 226, 145, 1), (3, 585, 15, 1), (4, 290, 16, 1),
    (6, 16, 264, 1), (65, 9, 420, 0), (65, 20, 403, 1), (65, 166, 129, 1), (65, 284, 406, 1), (65, 603, 130, 0),
    (65, 699, 9, 0), (66, 143, 71, 0), (66, 545, 391, 0), (67, 154, 73, 1), (67, 280, 385, 0), (68, 41, 137, 0),
    (68, 260, 147, 1), (68, 277, 134, 0), (68, 530, 389, 1), (69, 12, 268, 0), (69, 668, 11, 1), (70, 183, 142, 0),
    (70, 358, 14, 1), (71, 18, 263, 1), (71, 33, 257, 0), (73, 10, 11, 1), (73, 52, 264, 1), (76, 29, 132, 1),
    (82, 570, 137, 1), (88, 26, 10, 0), (95, 292, 15, 0), (129, 26, 392, 1), (130, 9, 286, 0), (132, 144, 78, 0),
    (133, 13, 275, 1), (133, 19, 407, 0), (133, 224, 130, 1), (134, 41, 270, 1), (134, 181, 138, 0), (135, 268, 385, 1),
    (135, 729, 9, 0), (136, 537, 140, 1), (138, 14, 85, 0), (138, 266, 136, 1), (139, 38, 266, 0), (140, 31, 131, 0),
    (140, 536, 12, 1), (142, 297, 10, 0), (144, 560, 129, 0), (149, 148, 12, 0), (151, 159, 65, 1), (153, 14, 131, 1),
    (173, 235, 65, 0), (239, 9, 17, 1), (256, 294, 9, 1),
]


@pytest.mark.parametrize("dtype,B,I,H,cell", [(wl.GEMM_BF16, *s) for s in INSTANCES_BF16] + [(wl.GEMM_FP32, *s) for s in INSTANCES_FP32])
def test_every_instantiation(dtype, B, I, H, cell):
    """Bit for bit the launch-per-step path, and really by chain and sweep launches: with hidden states stored
    the sweeps recompute the internal ones or a forward batch does, with internal states stored neither."""
    from paper_1606_03401_amd.session import Session
    t = 20
    w = wl.Workload("instance", B=B, I=I, H=H, t=t, kind=wl.KIND_HSM, m=5, gemm_dtype=dtype, loss=wl.LOSS_EXTERNAL_DY,
                    dy_first_step=2, seed=B + I + H, cell=cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 5, chain=False)
    for kind, m in ((wl.KIND_HSM, 5), (wl.KIND_HSM, t), (wl.KIND_ISM, t)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        _same(out, base, (kind, m))
        assert prof.chain_steps > 0
        if B > 128 and H > (512 if dtype == wl.GEMM_BF16 else 256):   # two batch tiles per XCD: the way back does not fit
            assert prof.sweep_steps == 0
        elif kind == wl.KIND_ISM:
            assert prof.batch_steps == 0 and prof.sweep_forward_steps == 0 and prof.sweep_steps >= t - 2
        elif mb.mebptt_stage_steps(s.desc):
            assert prof.batch_steps > 0 and prof.sweep_forward_steps == 0 and prof.sweep_steps > 0
        else:
            assert prof.batch_steps == 0 and prof.sweep_forward_steps > 0


# Half tiles, where one matrix instruction takes two macro steps, in sweeps (all of these) and in chains (seven and eight row tiles, see
# test_gpu_routes): a group of sequences that is full, has one or lacks one; an odd and an even number of row tiles, the last one
# short; parts of K of unequal length, and x that ends inside a macro step.
HALVES = [(1, 200, 500, 0), (9, 520, 512, 1), (8, 40, 705, 0), (63, 264, 769, 0), (57, 33, 1000, 1), (64, 1, 1024, 0), (16, 130, 897, 0), (64, 256, 1024, 1),
          (63, 250, 769, 0), (5, 8, 896, 1), (64, 256, 1024, 0)]
HALVES_T = 40


@pytest.mark.parametrize("B,I,H,cell", HALVES)
def test_two_macro_steps_per_instruction(B, I, H, cell):
    from oracle import gru_bptt as og
    from test_gpu_parity import TOL
    t = HALVES_T
    w = wl.Workload("halves", B=B, I=I, H=H, t=t, kind=wl.KIND_ISM, m=t, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY,
                    dy_first_step=1, seed=70 + B + I + H, cell=cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_HSM, 3, chain=False)
    if cell:
        ref = og.gru_bptt(inp.W_ih, inp.W_hh, inp.b, inp.x, inp.h0, inp.dy, w.dy_first_step)
    else:
        ref = ob.lstm_bptt(inp.W_ih, inp.W_hh, inp.b, inp.x, inp.h0, inp.c0, inp.dy, w.dy_first_step)
    for name in ("dW_ih", "dW_hh", "db", "dh0", "dx", "y") + (() if cell else ("dc0",)):
        got, want = getattr(base, name).astype(np.float64), getattr(ref, name)
        assert np.linalg.norm(got - want) <= TOL[w.gemm_dtype] * np.linalg.norm(want), name
    from paper_1606_03401_amd.session import Session
    for kind, m in ((wl.KIND_HSM, 3), (wl.KIND_ISM, t)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        _same(out, base, (kind, m))
        assert prof.sweep_steps > 0 and (prof.chain_steps > 0) == (I >= 8)


def test_random_widths_types_and_budgets_bit_identical():
    """As the seeded random cases above, over any width, both operand types, batches up to 256 and inputs
    wider and narrower than the state."""
    rng = np.random.default_rng(20261)
    for case in range(80):
        dtype = wl.GEMM_FP32 if rng.random() < 0.4 else wl.GEMM_BF16
        H = int(rng.integers(8, 513 if dtype == wl.GEMM_FP32 else 1025))
        I = int(np.exp(rng.uniform(np.log(4), np.log(1200))))
        B = int(np.exp(rng.uniform(0, np.log(257))))
        t = int(rng.integers(2, 60))
        kind = int(rng.choice([wl.KIND_HSM, wl.KIND_ISM, wl.KIND_MSM]))
        m = int(rng.integers(1, t + 2)) if kind != wl.KIND_MSM else int(rng.integers(2, 4 * t + 2))
        w = wl.Workload("random-any", B=B, I=I, H=H, t=t, kind=kind, m=m, gemm_dtype=dtype,
                        loss=wl.LOSS_HALF_SUM_H2 if rng.random() < 0.2 else wl.LOSS_EXTERNAL_DY,
                        dy_first_step=int(rng.integers(1, t + 1)), seed=int(rng.integers(1, 10**6)), cell=int(rng.random() < 0.3))
        inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
        what = (case, dtype, B, I, H, t, kind, m, w.dy_first_step, w.cell)
        _same(_run(w, inp, kind, m, chain=True), _run(w, inp, kind, m, chain=False), what)


def test_step_handed_over_at_the_start_of_a_chunk():
    """A policy that leads to a chain handing the first step of a chunk over to a sweep launch while the
    time-batched GEMMs that read the buffers of the chunk below have only just been issued beside it: the launch waits for
    them.  (Hidden states stored at 31, 33 .. 63 and 65 .., the rest recomputed in runs of two.)"""
    from paper_1606_03401_amd.session import Session
    hidden, internal, t = lambda y: (mb.STORE_HIDDEN, y), lambda y: (mb.STORE_INTERNAL, y), 100
    plan = mb.mebptt_plan_from_policy(t, 90, [hidden(31), hidden(34)] + [hidden(1)] * (t - 66) + [hidden(2)] + [hidden(1)] * 30
                                      + [internal(2)] * 2 + [hidden(1)] * 30)
    w = wl.Workload("policy", B=64, I=128, H=512, t=t, kind=wl.KIND_MSM, m=90, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY, seed=9)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    s = Session(w, inp, plan=plan)
    assert mb.mebptt_chunk_steps(s.desc) == 32
    out = s.run_and_fetch()
    _same(out, _run(w, inp, wl.KIND_HSM, 90, chain=False))
    assert out.stats.forward_ops == plan.forward_ops and out.stats.backward_ops == t
