"""GPU tests of the wide resident launches (weights spread once over the device or a part of it, exchange across
XCDs): against the float64 oracle, bit for bit the launch-per-step path on every instantiation, at the edges of its range, for
every strategy, however the launches come about (together, one workgroup alone, given up by some), on infinities and NaNs, and in
replays of graphs."""
import numpy as np
import pytest

from paper_1606_03401_amd import binding as mb
from paper_1606_03401_amd import workloads as wl
import test_gpu_chain
from test_gpu_chain import _run, _same

pytestmark = pytest.mark.gpu

# (B, I, H): row tiles and batch tiles of a compute unit in the comment.  Widths that are a multiple of nothing, rows of x
# shorter than a macro step and wider than the weights of x that stay on the chip, batches that leave a part of a batch tile, whole
# batch tiles or a whole group empty.
SHAPES = [
    (129, 130, 530), (256, 64, 768), (200, 700, 601),             # 3 x 4, four groups
    (130, 77, 700), (193, 40, 800), (256, 256, 1024), (140, 1100, 1001),   # (3 and) 4 x 4, four groups
    (1, 8, 1025), (20, 100, 1301), (32, 256, 1536),               # 3 x 1, two groups
    (33, 9, 1100), (50, 513, 1499),                               # 3 x 2
    (65, 60, 1057), (128, 128, 1280), (100, 333, 1500),           # 3 x 4
    (5, 64, 1700), (32, 900, 1601),                               # 4 x 1
    (40, 128, 1990), (64, 512, 2048),                             # 4 x 2
    (70, 31, 1537), (100, 640, 2001), (128, 512, 2048),           # 4 x 4
    (9, 65, 2050), (16, 200, 3000), (17, 64, 3071), (32, 300, 2560),   # 3 x 1 and 3 x 2, one group
    (7, 40, 3073), (16, 128, 4000), (20, 33, 3301), (32, 96, 4096),    # 4 x 1 and 4 x 2, one group
]

def _workload(B, I, H, t, cell, **kw):
    return wl.Workload("wide", B=B, I=I, H=H, t=t, kind=wl.KIND_ISM, m=4, gemm_dtype=wl.GEMM_BF16, loss=wl.LOSS_EXTERNAL_DY,
                       dy_first_step=2, seed=B + I + H, cell=cell, **kw)


@pytest.mark.parametrize("cell", [0, 1], ids=["lstm", "gru"])
@pytest.mark.parametrize("B,I,H", SHAPES)
def test_every_instantiation(B, I, H, cell):
    """All steps go out in wide launches, and the gradients are those of the launch-per-step path bit for bit."""
    from paper_1606_03401_amd.session import Session
    t = 11
    w = _workload(B, I, H, t, cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_ISM, 4, chain=False)
    for kind, m in ((wl.KIND_ISM, 4), (wl.KIND_ISM, t), (wl.KIND_HSM, 4)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        _same(out, base, (kind, m))
        assert prof.sweep_steps == t and prof.chain_steps + prof.batch_steps == out.stats.forward_ops


@pytest.mark.parametrize("cell", [0, 1], ids=["lstm", "gru"])
@pytest.mark.parametrize("B,I,H", [(130, 77, 700), (33, 1100, 1101), (66, 40, 1600), (9, 65, 2050), (20, 33, 3301)])
def test_against_the_oracle(B, I, H, cell):
    """One, two and four groups of XCDs, one, two and four batch tiles, weights that are fetched again in every step."""
    from test_gpu_parity import TOL, check_against_oracle, oracle_gradients
    w = _workload(B, I, H, 6, cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    ref = oracle_gradients(w, inp)
    for kind, m in ((wl.KIND_ISM, 2), (wl.KIND_HSM, 6)):
        check_against_oracle(w, inp, _run(w, inp, kind, m, chain=True), ref, TOL[w.gemm_dtype], label=f"wide {B}x{I}x{H} {cell}: ")


@pytest.mark.parametrize("B,I,H", [(40, 64, 1100), (130, 77, 700), (20, 40, 2051)])
def test_every_nan_is_passed_on(B, I, H):
    test_gpu_chain.test_resident_launches_pass_on_every_nan(wl.GEMM_BF16, B, I, H)


def test_input_wider_than_a_launch_stages():
    """x of seven steps fills the staging: a chain of eleven goes out in two launches, nearly all weights of x streamed."""
    w = _workload(128, 16500, 1040, 11, 0)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    _same(_run(w, inp, wl.KIND_ISM, 4, chain=True), _run(w, inp, wl.KIND_ISM, 4, chain=False))


# (B, I, H), forward tile (unit groups x batch tiles, macro steps in flight), backward tile, whether steps are fused
PER_STEP = [(8, 64, 1100, True),       # 2 x 1; 1 x 1
            (1, 700, 1537, True),      # the same, rows of x that are no whole fragments
            (20, 33, 1056, True),      # 2 x 2; 1 x 1
            (32, 512, 2048, True),     # the same, as many workgroups as that tile is used for
            (40, 520, 2040, False),    # 4 x 2, four; 2 x 1
            (61, 130, 1270, True),     # 4 x 2, two; 2 x 1
            (129, 64, 600, True),      # the same, four groups of XCDs
            (100, 100, 1500, False),   # 4 x 2, two; 2 x 2
            (120, 513, 2041, False),   # 8 x 2; 2 x 2
            (250, 520, 1000, False)]   # the same, four groups of XCDs


@pytest.mark.parametrize("cell", [0, 1], ids=["lstm", "gru"])
@pytest.mark.parametrize("B,I,H,fused", PER_STEP)
def test_launch_per_step_kernels(B, I, H, fused, cell):
    """What runs these shapes where resident launches do not: every tile, alone and fused, the same bits as the wide launches."""
    from paper_1606_03401_amd.session import Session
    w = _workload(B, I, H, 9, cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    want = _run(w, inp, wl.KIND_HSM, 3, chain=True)
    mb.mebptt_forward_chain_enable(False)
    try:
        for kind, m in ((wl.KIND_HSM, 3), (wl.KIND_ISM, 9)):
            s = Session(w, inp, kind=kind, m=m)
            mb.mebptt_profile_enable(1)
            out = s.run_and_fetch()
            prof = mb.mebptt_profile_collect()
            mb.mebptt_profile_enable(0)
            _same(out, want, (kind, m))
            pairs = prof.launches[5]
            assert (pairs > 0) == (fused and kind == wl.KIND_HSM) and prof.chain_steps + prof.sweep_steps + prof.batch_steps == 0
    finally:
        mb.mebptt_forward_chain_enable(True)


@pytest.mark.parametrize("cell", [0, 1], ids=["lstm", "gru"])
def test_every_backward_step_goes_out_in_a_sweep(cell):
    """Also the last but one of a stretch whose first state is the run's start, which is in no slot."""
    from paper_1606_03401_amd.session import Session
    w = _workload(18, 40, 1100, 12, cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_ISM, 1, chain=False)
    for kind, m in ((wl.KIND_ISM, 1), (wl.KIND_ISM, 2), (wl.KIND_ISM, 3), (wl.KIND_HSM, 1), (wl.KIND_MSM, 2), (wl.KIND_MSM, 5)):
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        _same(out, base, (kind, m))
        assert prof.sweep_steps == w.t and prof.launches[1] == 0, (kind, m)
        assert prof.chain_steps + prof.batch_steps == out.stats.forward_ops and prof.launches[0] == 0, (kind, m)


@pytest.mark.parametrize("B,I,H", [(20, 60, 1100), (140, 80, 600)])
def test_short_sequences_go_out_a_launch_per_step(B, I, H):
    """One or two steps, and up to five that are recomputed again and again; the same bits either way."""
    from paper_1606_03401_amd.session import Session
    for t, kind, m, wide in ((1, wl.KIND_HSM, 1, False), (1, wl.KIND_ISM, 1, False), (2, wl.KIND_HSM, 2, False), (2, wl.KIND_ISM, 2, False),
                             (3, wl.KIND_HSM, 1, False), (3, wl.KIND_ISM, 3, True), (5, wl.KIND_ISM, 1, False), (5, wl.KIND_HSM, 5, True),
                             (6, wl.KIND_HSM, 1, True)):
        w = _workload(B, I, H, t, 0).scaled(dy_first_step=1)
        inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
        s = Session(w, inp, kind=kind, m=m)
        mb.mebptt_profile_enable(1)
        out = s.run_and_fetch()
        prof = mb.mebptt_profile_collect()
        mb.mebptt_profile_enable(0)
        assert (prof.chain_steps + prof.batch_steps + prof.sweep_steps > 0) == wide, (t, kind, m)
        _same(out, _run(w, inp, kind, m, chain=False), (t, kind, m))


@pytest.mark.parametrize("B,I,H", [(3, 20, 1056), (40, 40, 1100)])
def test_chains_longer_than_a_launch(B, I, H):
    """More steps than one launch carries and several chunks of time-batched work, every strategy."""
    t = 230
    w = _workload(B, I, H, t, 0)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    base = _run(w, inp, wl.KIND_ISM, 12, chain=False)
    for kind, m in ((wl.KIND_ISM, 12), (wl.KIND_ISM, t), (wl.KIND_HSM, 9), (wl.KIND_HSM, t), (wl.KIND_MSM, 30)):
        _same(_run(w, inp, kind, m, chain=True), base, (kind, m))


@pytest.mark.parametrize("ticks", [0, 1], ids=["alone", "impatient"])
@pytest.mark.parametrize("B,I,H,cell", [(3, 20, 1056, 0), (37, 40, 1101, 1), (130, 77, 700, 0), (70, 33, 1300, 0), (5, 9, 2051, 1)])
def test_launches_that_are_given_up(ticks, B, I, H, cell):
    """One workgroup per group of XCDs gives the same bits, and so does any mixture of groups that are complete and
    groups that are given up; what a launch leaves behind for the next one is the same either way."""
    t = 7
    w = _workload(B, I, H, t, cell)
    inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
    from paper_1606_03401_amd.session import Session
    for kind, m in ((wl.KIND_ISM, 3), (wl.KIND_HSM, 3)):
        s = Session(w, inp, kind=kind, m=m)
        want = s.run_and_fetch()
        for patience in (ticks, -1, ticks):
            mb.mebptt_resident_patience(patience)
            try:
                _same(s.run_and_fetch(), want, (kind, m, patience))
            finally:
                mb.mebptt_resident_patience(-1)


def test_bounded_waits_give_up_and_report():
    """With every wait stopping after one look the kernels run to their end and the run reports it; then all is well again."""
    from paper_1606_03401_amd.session import Session
    w = _workload(40, 64, 1100, 9, 0)
    s = Session(w, wl.make_inputs(w, nonzero_state=True, nonzero_bias=True))
    want = s.run_and_fetch()
    mb.mebptt_resident_wait_limit(0)
    try:
        s.run()
        assert mb.mebptt_run_status(s.desc, s.workspace) == 1
    finally:
        mb.mebptt_resident_wait_limit(-1)
    _same(s.run_and_fetch(), want)


def test_replays_of_two_graphs_at_the_same_time():
    """Two captured runs without any order between them, a wide one and one with a copy of the weights per XCD or two wide
    ones: both give the eager result every time."""
    import torch
    from paper_1606_03401_amd.session import Session
    for shapes in (((64, 64, 1100), (40, 40, 1056)), ((64, 64, 1100), (64, 100, 500))):
        sessions, want = [], []
        for B, I, H in shapes:
            w = _workload(B, I, H, 12, 0)
            s = Session(w, wl.make_inputs(w, nonzero_state=True, nonzero_bias=True))
            want.append(s.run_and_fetch())
            s.capture()
            sessions.append(s)
        streams = [torch.cuda.Stream() for _ in sessions]
        for rep in range(4):
            for s in sessions:
                s.dW_hh.fill_(float("nan"))
            torch.cuda.synchronize()
            for _ in range(2):
                for s, st in zip(sessions, streams):
                    with torch.cuda.stream(st):
                        s.replay()
            torch.cuda.synchronize()
            for k, s in enumerate(sessions):
                _same(s.fetch(), want[k], (shapes, rep, k))      # fetch raises if a launch failed


def test_random_shapes_budgets_and_strategies_bit_identical():
    rng = np.random.default_rng(20262)
    for case in range(24):
        if rng.random() < 0.25:
            H, B = int(rng.integers(513, 1025)), int(rng.integers(129, 257))
        else:
            H, B = int(np.exp(rng.uniform(np.log(1025), np.log(2300)))), int(np.exp(rng.uniform(0, np.log(129))))
        I = int(np.exp(rng.uniform(np.log(8), np.log(1100))))
        t = int(rng.integers(2, 40))
        kind = int(rng.choice([wl.KIND_HSM, wl.KIND_ISM, wl.KIND_MSM]))
        m = int(rng.integers(1, t + 2)) if kind != wl.KIND_MSM else int(rng.integers(2, 4 * t + 2))
        w = wl.Workload("random-wide", B=B, I=I, H=H, t=t, kind=kind, m=m, gemm_dtype=wl.GEMM_BF16,
                        loss=wl.LOSS_HALF_SUM_H2 if rng.random() < 0.2 else wl.LOSS_EXTERNAL_DY,
                        dy_first_step=int(rng.integers(1, t + 1)), seed=int(rng.integers(1, 10**6)), cell=int(rng.random() < 0.3))
        inp = wl.make_inputs(w, nonzero_state=True, nonzero_bias=True)
        what = (case, B, I, H, t, kind, m, w.dy_first_step, w.cell)
        _same(_run(w, inp, kind, m, chain=True), _run(w, inp, kind, m, chain=False), what)
