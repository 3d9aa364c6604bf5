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

pytestmark = pytest.mark.gpu

CHILD = """
import json, sys
import torch
from torch.profiler import profile, ProfilerActivity
from paper_1606_03401_amd import binding as mb
from paper_1606_03401_amd import workloads as wl
from paper_1606_03401_amd.session import Session

def rnn(B, I, H, t, kind, m, bf16=1, cell=0):
    w = wl.Workload("route", B=B, I=I, H=H, t=t, kind=kind, m=m, gemm_dtype=bf16, loss=wl.LOSS_EXTERNAL_DY, dy_first_step=1, seed=1, cell=cell)
    return Session(w, wl.make_inputs(w)).run

for call in json.load(sys.stdin):
    step = globals()[call[0]](*call[1:])
    step()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        step()
        torch.cuda.synchronize()
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
