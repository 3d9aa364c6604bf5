"""GPU parity of mebptt_chain_run (appendix "Generalizing to deep feed-forward networks": a chain
of dense tanh layers of differing widths under the three-dimensional policy) against the float64
oracle, through the C ABI: gradients within the fp32 tolerance at every budget, bit-identical
across budgets, forward cost equal to the oracle's C(n, m, 0), pool use within the budget (guard
bytes around the pool and the workspace)."""
import threading

import numpy as np
import pytest

from oracle import chain_bptt as cb
from oracle import chain_dp as cd
from paper_1606_03401_amd import binding as mb

pytestmark = pytest.mark.gpu

TOL = 1e-4
GUARD = 4096
PATTERN = 0xA5


def _inputs(widths, B, seed):
    rng = np.random.default_rng(seed)
    n = len(widths) - 1
    W = [(rng.uniform(-1, 1, size=(widths[i + 1], widths[i])) / np.sqrt(widths[i])).astype(np.float32) for i in range(n)]
    b = [rng.uniform(-0.3, 0.3, size=(widths[i + 1],)).astype(np.float32) for i in range(n)]
    x0 = rng.standard_normal((B, widths[0])).astype(np.float32)
    dy = (0.1 * rng.standard_normal((B, widths[-1]))).astype(np.float32)
    return W, b, x0, dy


def _errs(got, ref):
    ref = np.asarray(ref, np.float64)
    d = np.asarray(got, np.float64) - ref
    return (np.linalg.norm(d) / max(np.linalg.norm(ref), 1e-300), np.abs(d).max() / max(np.abs(ref).max(), 1e-300))


def _run(widths, B, unit_bytes, m, W, b, x0, dy, dx0_over_x0=False):
    import torch
    dev = torch.device("cuda:0")
    desc = mb.make_chain_desc(widths, B, unit_bytes)
    layers = mb.mebptt_chain_layers(desc)
    plan = mb.mebptt_chain_plan(layers, m)
    up = lambda a: torch.from_numpy(a).to(dev)
    tW, tb, tx, tdy = [up(w) for w in W], [up(v) for v in b], up(x0), up(dy)
    dW = [torch.full_like(w, float("nan")) for w in tW]
    db = [torch.full_like(v, float("nan")) for v in tb]
    dx0, y = tx if dx0_over_x0 else torch.full_like(tx, float("nan")), torch.full_like(tdy, float("nan"))
    pool_bytes = m * unit_bytes
    pool_outer = torch.full((pool_bytes + 2 * GUARD,), PATTERN, dtype=torch.uint8, device=dev)
    ws_bytes = mb.mebptt_chain_workspace_bytes(desc)
    ws_outer = torch.full((ws_bytes + 2 * GUARD,), PATTERN, dtype=torch.uint8, device=dev)
    pool, ws = pool_outer[GUARD:GUARD + pool_bytes], ws_outer[GUARD:GUARD + ws_bytes]
    stats = mb.mebptt_chain_run(desc, plan, tW, tb, tx, tdy, pool if m else None, ws, dW, db, dx0, y)
    torch.cuda.synchronize()
    for outer, nbytes in ((pool_outer, pool_bytes), (ws_outer, ws_bytes)):
        assert bool((outer[:GUARD] == PATTERN).all()) and bool((outer[GUARD + nbytes:] == PATTERN).all())
    assert stats.peak_units == plan.peak <= m
    assert bool((pool[stats.peak_units * unit_bytes:] == PATTERN).all())      # nothing written above the reported peak
    assert stats.backward_ops == len(widths) - 1
    assert stats.forward_cost == plan.forward_cost
    out = dict(dW=[t.cpu().numpy() for t in dW], db=[t.cpu().numpy() for t in db], dx0=dx0.cpu().numpy(), y=y.cpu().numpy())
    return out, stats, layers


@pytest.mark.parametrize("widths,B,unit_bytes", [
    ([48, 96, 33, 128, 64, 17, 80, 40], 37, 1024),     # nothing a multiple of anything, states of 3 .. 19 units
    ([16, 16, 16, 16, 16, 16], 16, 1024),              # homogeneous: the HSM special case
    ([300, 520, 70, 1000, 250, 130], 130, 65536),      # several tiles per GEMM, large and small states
    ([5, 7], 3, 64),                                    # a single layer
])
def test_chain_run_matches_oracle_at_every_budget(widths, B, unit_bytes):
    W, b, x0, dy = _inputs(widths, B, 1234 + len(widths) + B)
    ref = cb.chain_backprop(W, b, x0, dy)
    n = len(widths) - 1
    s = [-(-B * widths[i + 1] * 4 // unit_bytes) for i in range(n)]
    u = [widths[i] * widths[i + 1] for i in range(n)]
    chain = cd.Chain(u, s, [0] * n)
    budgets = sorted(set([0, 1, min(s), max(s), max(s) + min(s), sum(s) // 2, sum(s), sum(s) + 3]))
    C, _ = cd.chain_tables(chain, max(budgets))
    first = None
    for m in budgets:
        out, stats, layers = _run(widths, B, unit_bytes, m, W, b, x0, dy)
        assert [(c, st, 0) for c, st in zip(u, s)] == layers
        assert stats.forward_cost == C(n, m, 0)                      # the optimum of the oracle's recursion, bit-exact
        for i in range(n):
            assert max(_errs(out["dW"][i], ref.dW[i])) <= TOL, (m, i)
            assert max(_errs(out["db"][i], ref.db[i])) <= TOL, (m, i)
        assert max(_errs(out["dx0"], ref.dx0)) <= TOL and max(_errs(out["y"], ref.y)) <= TOL
        if first is None:
            first = out
        else:      # recomputation repeats the same arithmetic: every budget gives the same bits
            for i in range(n):
                assert np.array_equal(out["dW"][i], first["dW"][i]) and np.array_equal(out["db"][i], first["db"][i])
            assert np.array_equal(out["dx0"], first["dx0"]) and np.array_equal(out["y"], first["y"])
    assert C(n, 0, 0) > C(n, sum(s), 0) or n == 1      # memory buys time


# Forward products whose operands pass through LDS, on 1 x 1, 1 x 2 and 2 x 2 tiles (test_gpu_routes: which): steps of 32 that leave remainders of 0,
# 4, 8 and 28; as many steps as waves, one more and several times as many; rows and columns that end inside a tile; rows that are no whole
# slots beside them; memorised states that lie on slots (4096) and that do not (1004).
STAGED = [([256, 260, 1000, 300, 257, 528, 288, 2044], 70), ([284, 256, 512, 16], 16), ([1024, 300, 640, 272], 300),
          ([288, 1000, 512, 1024, 500, 256], 250), ([1052, 130, 1000, 200, 1028, 60], 60)]


@pytest.mark.parametrize("unit_bytes", [4096, 1004])
@pytest.mark.parametrize("widths,B", STAGED)
def test_forward_products_through_lds(widths, B, unit_bytes):
    test_chain_run_matches_oracle_at_every_budget(widths, B, unit_bytes)


def test_chain_run_rejects_a_plan_for_another_chain():
    import torch
    widths, B = [32, 48, 16, 64], 8
    W, b, x0, dy = _inputs(widths, B, 7)
    desc = mb.make_chain_desc(widths, B, 256)
    other = mb.make_chain_desc([32, 48, 24, 64], B, 256)
    plan = mb.mebptt_chain_plan(mb.mebptt_chain_layers(other), 10)
    dev = torch.device("cuda:0")
    up = lambda a: torch.from_numpy(a).to(dev)
    tW, tb = [up(w) for w in W], [up(v) for v in b]
    dW, db = [torch.zeros_like(w) for w in tW], [torch.zeros_like(v) for v in tb]
    pool = torch.zeros(10 * 256, dtype=torch.uint8, device=dev)
    ws = torch.zeros(mb.mebptt_chain_workspace_bytes(desc), dtype=torch.uint8, device=dev)
    with pytest.raises(mb.MebpttError) as e:
        mb.mebptt_chain_run(desc, plan, tW, tb, up(x0), up(dy), pool, ws, dW, db)
    assert e.value.code == mb.ESHAPE


@pytest.mark.parametrize("widths,B", [
    ([3, 5, 2, 4, 1, 9], 7),                     # narrower than a 16-byte vector
    ([4, 4, 17, 33], 1), ([16, 64, 65, 63], 15), ([64, 128, 64], 16), ([67, 1, 67], 17),
    ([600, 1030, 514], 129),                     # every output block size of the data and weight products
    ([1100, 2100, 1025], 70), ([2048, 1024], 512),
])
def test_chain_products_at_the_edges_of_their_tiles(widths, B):
    W, b, x0, dy = _inputs(widths, B, 99 + len(widths) + B)
    ref = cb.chain_backprop(W, b, x0, dy)
    out, _, _ = _run(widths, B, 4096, sum(-(-B * d * 4 // 4096) for d in widths[1:]), W, b, x0, dy)
    for i in range(len(widths) - 1):
        assert max(_errs(out["dW"][i], ref.dW[i])) <= TOL and max(_errs(out["db"][i], ref.db[i])) <= TOL, i
    assert max(_errs(out["dx0"], ref.dx0)) <= TOL and max(_errs(out["y"], ref.y)) <= TOL


def test_chain_runs_from_two_host_threads():
    """The call takes no lock: two threads that make their first calls at the same time each set up the
    launches they need."""
    shapes = [([600, 1030, 514], 129), ([1100, 2100, 1025], 70)]
    args = [(w, B, 4096, sum(-(-B * d * 4 // 4096) for d in w[1:]), *_inputs(w, B, 7 + B)) for w, B in shapes]
    got, errors = [[], []], []

    def worker(k):
        try:
            for _ in range(3):
                got[k].append(_run(*args[k])[0])
        except Exception as exc:   # noqa: BLE001 - reported by the main thread
            errors.append(exc)

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join(timeout=100)
    assert not errors, errors
    for k in range(2):
        want = _run(*args[k])[0]
        assert len(got[k]) == 3
        for out in got[k]:
            assert np.array_equal(out["dx0"], want["dx0"]) and np.array_equal(out["y"], want["y"])
            assert all(np.array_equal(a, b) for f in ("dW", "db") for a, b in zip(out[f], want[f]))


@pytest.mark.parametrize("widths,B", [([1030, 600, 514], 129), ([3, 5], 7), ([2048, 1024], 512)])
def test_input_gradient_over_the_input(widths, B):
    """dx0 may be x0's own buffer: it is written after the last reader of x0."""
    args = (widths, B, 4096, sum(-(-B * d * 4 // 4096) for d in widths[1:]), *_inputs(widths, B, 31 + B))
    want, out = _run(*args)[0], _run(*args, dx0_over_x0=True)[0]
    assert np.array_equal(out["dx0"], want["dx0"]) and np.array_equal(out["y"], want["y"])
    assert all(np.array_equal(a, b) for f in ("dW", "db") for a, b in zip(out[f], want[f]))


@pytest.mark.parametrize("widths,B", [
    ([70, 2047, 65], 510),       # forward product on 4 x 4 tiles
    ([130, 1030, 40], 250),      # and on 2 x 2
])
def test_forward_products_on_their_largest_blocks(widths, B):
    W, b, x0, dy = _inputs(widths, B, 199 + B)
    ref = cb.chain_backprop(W, b, x0, dy)
    out, _, _ = _run(widths, B, 4096, sum(-(-B * d * 4 // 4096) for d in widths[1:]), W, b, x0, dy)
    for i in range(len(widths) - 1):
        assert max(_errs(out["dW"][i], ref.dW[i])) <= TOL and max(_errs(out["db"][i], ref.db[i])) <= TOL, i
    assert max(_errs(out["dx0"], ref.dx0)) <= TOL and max(_errs(out["y"], ref.y)) <= TOL
