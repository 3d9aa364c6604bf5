"""Which kernels a call launches, by name: the cases that other tests compare with the oracle or bit for bit really reach the kernels they
are there for, and calls on either side of a dispatch rule go where the rule says.  The names come from a traced run of every call in one
process of its own."""
import json
import os
import re
import subprocess
import sys

import pytest

import test_gpu_chain as chain
import test_gpu_chain_run as chain_run
import test_gpu_parity as parity

pytestmark = pytest.mark.gpu

CHILD = """
import json, sys, time
import torch
from torch.profiler import profile, ProfilerActivity
from paper_1606_03401_amd import binding as mb
from paper_1606_03401_amd import workloads as wl
from paper_1606_03401_amd.session import Session

def rnn(B, I, H, t, kind, m, bf16=1, cell=0):
    w = wl.Workload("route", B=B, I=I, H=H, t=t, kind=kind, m=m, gemm_dtype=bf16, loss=wl.LOSS_EXTERNAL_DY, dy_first_step=1, seed=1, cell=cell)
    return Session(w, wl.make_inputs(w)).run

def dense(widths, B):
    desc = mb.make_chain_desc(widths, B, 4096)
    layers = mb.mebptt_chain_layers(desc)
    m = sum(s for _, s, _ in layers)
    plan = mb.mebptt_chain_plan(layers, m)
    f = lambda *shape: torch.zeros(shape, device="cuda")
    W, b = [f(o, i) for i, o in zip(widths, widths[1:])], [f(o) for o in widths[1:]]
    pool, ws = [torch.zeros(n, dtype=torch.uint8, device="cuda") for n in (m * 4096, mb.mebptt_chain_workspace_bytes(desc))]
    x0, dy, dx0, y, dW, db = f(B, widths[0]), f(B, widths[-1]), f(B, widths[0]), f(B, widths[-1]), [f(*w.shape) for w in W], [f(*v.shape) for v in b]
    return lambda: mb.mebptt_chain_run(desc, plan, W, b, x0, dy, pool, ws, dW, db, dx0, y)

for call in json.load(sys.stdin):
    step = globals()[call[0]](*call[1:])
    step()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        time.sleep(0.05)     # the two clocks differ a little, and what seems to lie outside the traced time is dropped
        step()
        torch.cuda.synchronize()
        time.sleep(0.05)
    names = {}
    for e in p.events():
        if "mebptt" in e.name or "chain_" in e.name:
            names[e.name] = names.get(e.name, 0) + 1
    print("NAMES " + json.dumps(names), flush=True)
    del step
"""
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def launched(calls):
    """Of each call, {kernel name: launches}."""
    r = subprocess.run([sys.executable, "-c", CHILD], input=json.dumps(calls), capture_output=True, text=True, cwd=ROOT, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [json.loads(l[6:]) for l in r.stdout.splitlines() if l.startswith("NAMES ")]
    assert len(got) == len(calls)
    return got


def count(names, kernel, flag=None):
    """Launches of a kernel; `flag`: of its instantiations whose last template argument is this truth value."""
    end = {None: "", True: r"(Lb1EEEv|, true>)", False: r"(Lb0EEEv|, false>)"}[flag]
    return sum(n for name, n in names.items() if re.search(rf"\d*{kernel}(I|<).*{end}" if flag is not None else rf"{kernel}(I|<)", name))


def test_chains_that_take_two_macro_steps_per_instruction():
    """Up to 64 sequences, 769 to 1024 units, at most 256 columns of x, launches of 16 steps and more; shorter launches and
    other widths take one macro step.  (H = 500, I = 768: 20 % more time a launch with two; H = 896, I = 512: 10 %.)"""
    from paper_1606_03401_amd import workloads as wl
    two = [(B, I, H, c) for B, I, H, c in chain.HALVES if H > 768 and 8 <= I <= 256]
    one = [s for s in chain.HALVES if s not in two and s[1] >= 8] + [(20, 768, 500, 0), (64, 512, 896, 0), (65, 256, 1024, 0), (20, 300, 880, 0)]
    assert len(two) >= 4 and len(one) >= 7
    calls = [["rnn", B, I, H, t, wl.KIND_ISM, t, 1, c] for t in (chain.HALVES_T, 15) for B, I, H, c in two + one]
    for call, names in zip(calls, launched(calls)):
        expected = tuple(call[1:4] + call[8:]) in two and call[4] >= 16
        assert count(names, "forward_chain_kernel", expected) > 0, (call, names)
        if not expected:
            assert count(names, "forward_chain_kernel", True) == 0, (call, names)


def forward_tiles(names):
    """Of every dense layer's forward launch: (row tiles, column tiles, through LDS)."""
    found = [(n, re.search(r"chain_forward_kernel<(\d+), (\d+), \w+, (\w+)>", name)) for name, n in names.items() if "chain_forward_kernel" in name]
    return {(int(m[1]), int(m[2]), m[3] == "true"): n for n, m in found}


@pytest.mark.parametrize("what", ["single", "compared"])
def test_dense_layers_whose_operands_pass_through_lds(what):
    """On the sides of the rule: whole and broken steps of 32, and 2 x 2 tiles that give every compute unit one workgroup or more.  (Broken steps cost
    up to 35 % of a launch, second workgroups 10 %.)  And of the chains that are compared with the oracle, every staged instantiation."""
    single = [(256, 288, 1024, 2, 2, True), (250, 512, 1000, 2, 2, True), (250, 284, 1024, 2, 2, False), (461, 832, 832, 2, 2, False),
              (192, 2044, 2048, 2, 2, False), (128, 512, 1000, 1, 2, True), (128, 284, 1000, 1, 2, False), (128, 1028, 1000, 1, 2, False),
              (16, 256, 512, 1, 1, True), (16, 284, 1024, 1, 1, False), (16, 872, 64, 1, 1, False), (60, 900, 256, 1, 1, True), (60, 1000, 200, 1, 1, True),
              (60, 920, 200, 1, 1, False), (60, 1052, 130, 1, 1, True), (16, 255, 512, 1, 1, False), (16, 252, 512, 1, 1, False)]
    if what == "single":
        for (B, K, N, *tiles), names in zip(single, launched([["dense", [K, N], B] for B, K, N, *_ in single])):
            assert forward_tiles(names) == {tuple(tiles): 1}, (B, K, N, names)
    else:
        seen = {}
        for names in launched([["dense", widths, B] for widths, B in chain_run.STAGED]):
            for k, n in forward_tiles(names).items():
                seen[k] = seen.get(k, 0) + n
        assert {(1, 1, True), (1, 2, True), (2, 2, True), (1, 1, False), (1, 2, False)} <= set(seen), seen


def test_weight_gradients_without_blocks_for_the_row_of_ones():
    """Of the shapes compared with the oracle, those that say so; and not where every workgroup has a compute unit of its own already (H = 128,
    fp32: 1.3 % of a gradient step) or the GEMMs run beside the sweeps."""
    shapes = [(B, I, H, dtype, cell, ones) for B, I, H, _, dtype, cell, ones in parity.WGRAD_BLOCKS]
    shapes += [(64, 256, 256, 1, 0, True), (64, 256, 256, 0, 0, True), (64, 128, 128, 0, 0, False), (32, 128, 256, 0, 0, False), (32, 128, 128, 1, 0, False),
               (128, 128, 512, 1, 0, False), (96, 1023, 512, 1, 0, False), (16, 128, 512, 1, 0, False), (64, 256, 1024, 1, 0, False)]
    for (B, I, H, dtype, cell, ones), names in zip(shapes, launched([["rnn", B, I, H, 4, 0, 2, dtype, cell] for B, I, H, dtype, cell, _ in shapes])):
        assert count(names, "wgrad_kernel", ones) == 1 and count(names, "wgrad_kernel", not ones) == 0, (B, I, H, dtype, names)


def test_forward_batches_on_large_tiles():
    """Of the shapes compared bit for bit, those tiles that they say; and the small ones where large tiles would be slower (H = 2048, I = 33, B = 33: 8.1 and
    17.6 us for one operation; H = 600, I = 193, B = 20 6.5 and 10.1 for five), or where GEMMs run beside and rows of x are whole 16 bytes."""
    from paper_1606_03401_amd import workloads as wl
    small = [(20, 193, 600, 6, 0), (64, 36, 1024, 20, 0), (128, 69, 1024, 3, 0), (4, 650, 896, 6, 0), (64, 256, 1024, 33, 0), (33, 33, 2048, 4, 0)]
    calls = [["rnn", B, I, H, t, wl.KIND_HSM, t, 1, cell] for B, I, H, t, cell in [s[:5] for s in chain.TILED] + small]
    got = launched(calls)
    for (B, I, H, t, cell, columns), names in zip(chain.TILED, got):
        tiles = {int(m[1]) * 16: n for m, n in ((re.search(r"forward_batch_tiles_kernel<2, (\d), \d>", k), n) for k, n in names.items()) if m}
        assert columns in tiles, (B, I, H, names)
    for s, names in zip(small, got[len(chain.TILED):]):
        assert count(names, "forward_batch_tiles_kernel") == 0 and (count(names, "forward_batch_kernel") > 0 or s[3] == 4), (s, names)
