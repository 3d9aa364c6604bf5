"""Work that a program has this library do, as cases that a timing harness can run.

Each case is one gradient step through a public entry point of the C ABI: ``mebptt_run`` or
``mebptt_run_prepared`` for a recurrent core under a checkpointing plan, ``mebptt_chain_run`` for a
chain of dense layers of differing widths.  The listed cases are the named workloads of
``paper_1606_03401_amd.workloads``, the shape of the paper's own experiment, and shapes beside them
(other cores, other strategies, fp32 operands, sizes that are no multiple of anything); ``draw``
spreads over the ranges these stand for.

A case of a recurrent core ("rnn") holds the sizes B, I, H, t, the strategy and its budget m, the
operand type, the core, where the loss sits (at every step from `dy_first` on, or on h itself), whether bias and
start state are there, whether dx is wanted, and the entry point.  A case of a chain ("dense") holds
the batch, the widths (spaces between them), and the budget as a share of all states.
"""
import math

import torch

from paper_1606_03401_amd import binding as mb

KINDS = {"hsm": mb.HSM, "ism": mb.ISM, "msm": mb.MSM}
UNIT_BYTES = 4096          # memory unit of the dense chains


def _rnn(name, B, I, H, t, kind, m, dtype="bf16", cell="lstm", loss="dy", dy_first=1, state=True, dx=True, entry="run"):
    return {"name": name, "what": "rnn", "B": B, "I": I, "H": H, "t": t, "kind": kind, "m": m, "dtype": dtype, "cell": cell,
            "loss": loss, "dy_first": dy_first, "state": state, "dx": dx, "entry": entry}


def _dense(name, B, widths, share):
    return {"name": name, "what": "dense", "B": B, "widths": " ".join(str(w) for w in widths), "share": share}


def listed():
    return [
        # the smallest call: a toy model in fp32, where launches are everything
        _rnn("tiny fp32", 4, 16, 32, 20, "hsm", 4, dtype="fp32", loss="h", state=False),
        # the headline workload, weights prepared once for several sequences
        _rnn("1024 hsm 50", 64, 256, 1024, 1000, "hsm", 50, state=False, entry="prepared"),
        # internal states in the slots, a model whose weights are re-read by every step
        _rnn("2048 ism 100", 128, 512, 2048, 1000, "ism", 100, state=False),
        # a very long sequence with the loss at its end
        _rnn("512 long", 256, 128, 512, 10000, "hsm", 100, dy_first=9901, state=False),
        # the largest weights, a small batch, the mixed strategy
        _rnn("4096 msm 50", 32, 1024, 4096, 1000, "msm", 50, state=False),
        # the paper's experiment: 256 -> 256, batch 64, a budget of 50 hidden states
        _rnn("paper 256", 64, 256, 256, 400, "hsm", 50),
        # the other core, with the built-in loss
        _rnn("gru 1024", 64, 256, 1024, 300, "hsm", 30, cell="gru", loss="h"),
        # store-everything BPTT, what every budget is compared with
        _rnn("512 store all", 128, 128, 512, 200, "ism", 200),
        # sizes that are a multiple of nothing, a small model and a truncated sequence
        _rnn("ragged 200", 37, 100, 200, 150, "msm", 24, dy_first=101),
        # a stack's inner layer: as wide as its input, a small batch, no multiple of 64
        _rnn("650 stack layer", 20, 650, 650, 200, "hsm", 20),
        # fp32 operands, as a check of a bf16 run is made
        _rnn("fp32 256", 32, 128, 256, 200, "hsm", 20, dtype="fp32"),
        # the appendix's chain of layers of differing widths, half the memory it would like
        _dense("dense chain", 256, [512, 1024, 1024, 768, 1536, 1000, 640, 2048, 512, 900, 1024, 256], 0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """Half of all widths are round, half are whatever they are."""
    v = _log(rng, lo, hi)
    if rng.random() < 0.5:
        step = 64 if v >= 128 else 16
        v = max(step, (v + step // 2) // step * step)
    return max(lo, min(hi, v))


def draw(rng):
    if rng.random() < 0.15:
        n = rng.randint(3, 14)
        c = _dense("", _size(rng, 16, 512), [_size(rng, 64, 2048) for _ in range(n + 1)], round(rng.uniform(0.1, 1.0), 2))
        del c["name"]
        return c
    while True:
        fp32 = rng.random() < 0.2
        B, t = _size(rng, 4, 256), _log(rng, 20, 1000)
        H, I = _size(rng, 32, 512 if fp32 else 2048), _size(rng, 16, 1024)
        kind = rng.choice(["hsm", "ism", "msm"])
        m = _log(rng, 8 if kind == "msm" else 4, t)
        c = _rnn("", B, I, H, t, kind, m, dtype="fp32" if fp32 else "bf16", cell="gru" if rng.random() < 0.2 else "lstm",
                 loss="h" if rng.random() < 0.2 else "dy", state=rng.random() < 0.7, dx=rng.random() < 0.8,
                 entry=rng.choice(["run", "prepared"]))
        if c["loss"] == "dy" and rng.random() < 0.4:
            c["dy_first"] = rng.randint(1, min(t, 60))
        del c["name"]
        if work(c)["flops"] <= (1.0e12 if fp32 else 1.2e13):
            return c


# ---- inputs -------------------------------------------------------------------------------------


def _widths(case):
    return [int(v) for v in case["widths"].split()]


def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _uniform(g, shape, k):
    return (torch.rand(shape, generator=g, device="cuda") * 2 - 1) * k


def _normal(g, shape, s):
    return torch.randn(shape, generator=g, device="cuda") * s


def _rnn_inputs(case, seed):
    g = _rng(seed)
    B, I, H, t = case["B"], case["I"], case["H"], case["t"]
    gru = case["cell"] == "gru"
    k = H ** -0.5
    v = {"W_ih": _uniform(g, ((3 if gru else 4) * H, I), k), "W_hh": _uniform(g, ((3 if gru else 4) * H, H), k),
         "x": _normal(g, (t, B, I), 1.0), "dy": None, "b": None, "h0": None, "c0": None}
    if case["loss"] == "dy":
        v["dy"] = _normal(g, (t - case["dy_first"] + 1, B, H), 0.1)
    if case["state"]:
        v["b"] = _uniform(g, ((6 if gru else 4) * H,), k)
        v["h0"] = _normal(g, (B, H), 0.5)
        v["c0"] = None if gru else _normal(g, (B, H), 0.5)
    return v


def _dense_inputs(case, seed):
    g = _rng(seed)
    w, B = _widths(case), case["B"]
    return {"W": [_uniform(g, (w[i + 1], w[i]), (3.0 / w[i]) ** 0.5) for i in range(len(w) - 1)],
            "b": [_uniform(g, (w[i + 1],), 0.3) for i in range(len(w) - 1)],
            "x0": _normal(g, (B, w[0]), 1.0), "dy": _normal(g, (B, w[-1]), 0.1)}


def _desc(case):
    return mb.make_desc(case["B"], case["I"], case["H"], case["t"], 1 if case["dtype"] == "bf16" else 0,
                        1 if case["loss"] == "h" else 0, case["dy_first"], mb.CELL_GRU if case["cell"] == "gru" else mb.CELL_LSTM)


def _plan(case):
    return mb.mebptt_plan(case["t"], case["m"], KINDS[case["kind"]])


def _chain_plan(case):
    desc = mb.make_chain_desc(_widths(case), case["B"], UNIT_BYTES)
    layers = mb.mebptt_chain_layers(desc)
    m = int(case["share"] * sum(s for _, s, _ in layers))
    return desc, m, mb.mebptt_chain_plan(layers, m)


def _bytes(n):
    return torch.zeros(max(int(n), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    if case["what"] == "dense":
        v = _dense_inputs(case, seed)
        desc, m, plan = _chain_plan(case)
        return {"case": dict(case), **v, "desc": desc, "plan": plan, "pool": _bytes(m * UNIT_BYTES),
                "ws": _bytes(mb.mebptt_chain_workspace_bytes(desc)), "dW": [torch.zeros_like(w) for w in v["W"]],
                "db": [torch.zeros_like(b) for b in v["b"]], "dx0": torch.zeros_like(v["x0"]), "y": torch.zeros_like(v["dy"])}
    v = _rnn_inputs(case, seed)
    desc, plan = _desc(case), _plan(case)
    B, H, t = case["B"], case["H"], case["t"]
    s = {"case": dict(case), **v, "desc": desc, "plan": plan, "slots": _bytes(mb.mebptt_slot_pool_bytes(desc, plan)),
         "ws": _bytes(mb.mebptt_workspace_bytes(desc)), "dW_ih": torch.zeros_like(v["W_ih"]), "dW_hh": torch.zeros_like(v["W_hh"]),
         "db": torch.zeros((6 if case["cell"] == "gru" else 4) * H, device="cuda"), "dh0": torch.zeros((B, H), device="cuda"),
         "dc0": torch.zeros((B, H), device="cuda"), "dx": torch.zeros_like(v["x"]) if case["dx"] else None,
         "y": torch.zeros((t, B, H), device="cuda")}
    if case["entry"] == "prepared":
        mb.mebptt_prepare(desc, s["W_ih"], s["W_hh"], s["b"], s["ws"])
    return s


def run(s):
    if s["case"]["what"] == "dense":
        mb.mebptt_chain_run(s["desc"], s["plan"], s["W"], s["b"], s["x0"], s["dy"], s["pool"], s["ws"], s["dW"], s["db"],
                            s["dx0"], s["y"])
        return {"dW": s["dW"], "db": s["db"], "dx0": s["dx0"], "y": s["y"]}
    out = (s["slots"], s["ws"], s["dW_ih"], s["dW_hh"], s["db"], s["dh0"], s["dc0"], s["dx"], s["y"])
    if s["case"]["entry"] == "prepared":
        mb.mebptt_run_prepared(s["desc"], s["plan"], s["x"], s["dy"], s["h0"], s["c0"], *out)
    else:
        mb.mebptt_run(s["desc"], s["plan"], s["W_ih"], s["W_hh"], s["b"], s["x"], s["dy"], s["h0"], s["c0"], *out)
    got = {k: s[k] for k in ("dW_ih", "dW_hh", "db", "dh0", "y")}
    if s["case"]["cell"] == "lstm":
        got["dc0"] = s["dc0"]
    if s["case"]["dx"]:
        got["dx"] = s["dx"]
    return got


# ---- what a pass cannot do without -----------------------------------------------------------------


def work(case):
    if case["what"] == "dense":
        w, B = _widths(case), case["B"]
        params = sum(w[i] * w[i + 1] + w[i + 1] for i in range(len(w) - 1))
        _, _, plan = _chain_plan(case)
        macs = plan.forward_cost * B + 2 * B * sum(w[i] * w[i + 1] for i in range(len(w) - 1))
        return {"bytes": 4.0 * (2 * params + 2 * B * (w[0] + w[-1])), "flops": 2.0 * macs}
    B, I, H, t = case["B"], case["I"], case["H"], case["t"]
    gates = 3 if case["cell"] == "gru" else 4
    params = gates * H * (I + H) + (6 if gates == 3 else 4) * H
    values = 2 * params + t * B * (I + H) + 2 * B * H + (t * B * I if case["dx"] else 0)
    if case["loss"] == "dy":
        values += (t - case["dy_first"] + 1) * B * H
    # the forward operations that the plan's budget makes necessary, and one backward step each: dh (and dx), dW
    forward = _plan(case).forward_ops
    one = 2.0 * B * gates * H * (I + H)
    back = 2.0 * B * gates * H * ((I if case["dx"] else 0) + H) + one
    return {"bytes": 4.0 * values, "flops": forward * one + t * back}


def tolerance(case):
    # bf16 operands: one rounding of h and of dG per step; fp32: sums in another order
    if case["what"] == "rnn" and case["dtype"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": 1e-5}


# ---- the same step in 64 bits ----------------------------------------------------------------------


def _exact_dense(case, seed):
    v = _dense_inputs(case, seed)
    W, b = [w.double() for w in v["W"]], [u.double() for u in v["b"]]
    a = [v["x0"].double()]
    for Wi, bi in zip(W, b):
        a.append(torch.tanh(a[-1] @ Wi.t() + bi))
    g, dW, db = v["dy"].double(), [None] * len(W), [None] * len(W)
    for i in reversed(range(len(W))):
        dz = g * (1 - a[i + 1] ** 2)
        dW[i], db[i], g = dz.t() @ a[i], dz.sum(0), dz @ W[i]
    return {"dW": dW, "db": db, "dx0": g, "y": a[-1]}


def _exact_lstm(case, v):
    B, H, t, first = case["B"], case["H"], case["t"], case["dy_first"]
    Wi, Wh = v["W_ih"].double(), v["W_hh"].double()
    b = v["b"].double() if v["b"] is not None else torch.zeros(4 * H, dtype=torch.float64, device="cuda")
    z = torch.zeros((B, H), dtype=torch.float64, device="cuda")
    h0 = v["h0"].double() if v["h0"] is not None else z
    h, c = h0, v["c0"].double() if v["c0"] is not None else z
    acts, cs, hs, WiT, WhT = [], [c], torch.empty((t, B, H), dtype=torch.float64, device="cuda"), Wi.t().contiguous(), Wh.t().contiguous()
    for s in range(t):
        G = torch.addmm(b, v["x"][s].double(), WiT) + h @ WhT
        act = torch.sigmoid(G)
        act[:, 2 * H:3 * H] = torch.tanh(G[:, 2 * H:3 * H])
        i, f, g, o = act.split(H, 1)
        c = f * c + i * g
        h = o * torch.tanh(c)
        acts.append(act)
        cs.append(c)
        hs[s] = h
    dWi, dWh, db = torch.zeros_like(Wi), torch.zeros_like(Wh), torch.zeros_like(b)
    dx = torch.zeros((t, B, case["I"]), dtype=torch.float32, device="cuda")   # kept in 32 bits for room: 6e-8
    dh, dc = torch.zeros_like(z), torch.zeros_like(z)
    for s in reversed(range(t)):
        i, f, g, o = acts[s].split(H, 1)
        if case["loss"] == "h":
            dh = dh + hs[s]
        elif s + 1 >= first:
            dh = dh + v["dy"][s + 1 - first].double()
        tc = torch.tanh(cs[s + 1])
        dc = dc + dh * o * (1 - tc * tc)
        dG = torch.cat([dc * g * i * (1 - i), dc * cs[s] * f * (1 - f), dc * i * (1 - g * g), dh * tc * o * (1 - o)], 1)
        dc = dc * f
        dWi.addmm_(dG.t(), v["x"][s].double())
        dWh.addmm_(dG.t(), hs[s - 1] if s else h0)
        db += dG.sum(0)
        if case["dx"]:
            dx[s] = dG @ Wi
        dh = dG @ Wh
        acts[s] = None
    return {"dW_ih": dWi, "dW_hh": dWh, "db": db, "dh0": dh, "dc0": dc, "dx": dx, "y": hs}


def _exact_gru(case, v):
    B, H, t, first = case["B"], case["H"], case["t"], case["dy_first"]
    Wi, Wh = v["W_ih"].double(), v["W_hh"].double()
    b = v["b"].double() if v["b"] is not None else torch.zeros(6 * H, dtype=torch.float64, device="cuda")
    h0 = v["h0"].double() if v["h0"] is not None else torch.zeros((B, H), dtype=torch.float64, device="cuda")
    h, kept, hs = h0, [], torch.empty((t, B, H), dtype=torch.float64, device="cuda")
    for s in range(t):
        gi = torch.addmm(b[:3 * H], v["x"][s].double(), Wi.t())
        gh = torch.addmm(b[3 * H:], h, Wh.t())
        r = torch.sigmoid(gi[:, :H] + gh[:, :H])
        z = torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
        nh = gh[:, 2 * H:]
        n = torch.tanh(gi[:, 2 * H:] + r * nh)
        h = (1 - z) * n + z * h
        kept.append((r, z, n, nh))
        hs[s] = h
    dWi, dWh, db = torch.zeros_like(Wi), torch.zeros_like(Wh), torch.zeros_like(b)
    dx = torch.zeros((t, B, case["I"]), dtype=torch.float64, device="cuda")
    dh = torch.zeros_like(h0)
    for s in reversed(range(t)):
        r, z, n, nh = kept[s]
        prev = hs[s - 1] if s else h0
        if case["loss"] == "h":
            dh = dh + hs[s]
        elif s + 1 >= first:
            dh = dh + v["dy"][s + 1 - first].double()
        dn = dh * (1 - z) * (1 - n * n)
        dr, dz = dn * nh * r * (1 - r), dh * (prev - n) * z * (1 - z)
        dGi, dGh = torch.cat([dr, dz, dn], 1), torch.cat([dr, dz, dn * r], 1)
        dWi.addmm_(dGi.t(), v["x"][s].double())
        dWh.addmm_(dGh.t(), prev)
        db += torch.cat([dGi, dGh], 1).sum(0)
        if case["dx"]:
            dx[s] = dGi @ Wi
        dh = dGh @ Wh + dh * z
    return {"dW_ih": dWi, "dW_hh": dWh, "db": db, "dh0": dh, "dx": dx, "y": hs}


def exact(case, seed):
    if case["what"] == "dense":
        return _exact_dense(case, seed)
    v = _rnn_inputs(case, seed)
    got = _exact_gru(case, v) if case["cell"] == "gru" else _exact_lstm(case, v)
    if not case["dx"]:
        del got["dx"]
    if case["dy_first"] > 100 and case["loss"] == "dy":
        # the gradient of the start state has vanished below what 32 bits hold
        for k in ("dh0", "dc0"):
            if k in got:
                got[k] = None
    return got
