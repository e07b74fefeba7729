"""Performance cases: the contractions that users of this library run.

Coupled-cluster-shaped work (ladder and ring terms, their gradients, a
sequence with an intermediate), batches of uneven block contractions as
block-sparse codes issue them, and the plain building blocks around them
(small contractions, batch labels, products with a small matrix), through
the public entry points: ``contract`` with its cached plans, a kept plan and
``famlies_execute``, ``famlies_batch_*``, ``Network`` and ``contract_ad``.

A case is a dict of plain values; ``kind`` selects the family.  Inputs are
made on the GPU from the seed.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_2604_07311_amd as fm
import synth

DTYPES = {"f64": torch.float64, "f32": torch.float32}
CODES = {"f64": fm.FAMLIES_F64, "f32": fm.FAMLIES_F32}
COMPUTES = {"native": fm.FAMLIES_NATIVE, "bf16x3": fm.FAMLIES_BF16X3, "bf16x6": fm.FAMLIES_BF16X6,
            "int8x6": fm.FAMLIES_INT8X6, "int8x7": fm.FAMLIES_INT8X7}


def listed():
    return [
        # One small FP64 contraction, every extent 16, plan kept by the
        # caller: the innermost call of an iterative solver, where latency
        # and the number of launches decide.
        {"name": "plain16_f64", "kind": "plain", "dtype": "f64", "a": 16, "b": 16, "i": 16, "j": 16, "e": 16,
         "f": 16, "pad": 0, "entry": "plan"},
        # One ragged FP32 block with padded strides through contract(): a
        # block of a block-sparse tensor, odd extents everywhere.
        {"name": "plain_ragged_f32", "kind": "plain", "dtype": "f32", "a": 37, "b": 21, "i": 11, "j": 29, "e": 23,
         "f": 19, "pad": 1, "entry": "contract"},
        # The FP64 particle-particle ladder that bench.py quotes, v=128 o=32.
        {"name": "ladder_f64", "kind": "ladder", "dtype": "f64", "compute": "native", "v": 128, "o": 32},
        # The FP32 ladder at odd sizes: runs that are not 16-byte aligned, a
        # contracted range that no K slice divides.
        {"name": "ladder_odd_f32", "kind": "ladder", "dtype": "f32", "compute": "native", "v": 93, "o": 27},
        # The ring term at o=48 v=192 in split-BF16 precision (three
        # products): the mixed-precision option on the largest tensors.
        {"name": "ring_bf16x3", "kind": "ring", "dtype": "f32", "compute": "bf16x3", "v": 192, "o": 48},
        # The FP32-accurate split (six products) at odd sizes.
        {"name": "ring_odd_bf16x6", "kind": "ring", "dtype": "f32", "compute": "bf16x6", "v": 115, "o": 31},
        # FP64 emulated on INT8 MFMA, six slices, an ordinary ladder.
        {"name": "ladder_int8x6", "kind": "ladder", "dtype": "f64", "compute": "int8x6", "v": 96, "o": 24},
        # A tenth of bench.py's batched workload: 2,000 uneven FP32 problems
        # in random layouts in one call (block-sparse contractions).
        {"name": "batched_f32", "kind": "batched", "dtype": "f32", "n": 2000, "hi": 48},
        # One training step through the contraction: forward, dA and dB.
        {"name": "autograd_f32", "kind": "autograd", "dtype": "f32", "v": 96, "o": 24},
        # A coupled-cluster-like sequence with an intermediate, the constant
        # operand kept packed, and an elementwise-batched reduction.
        {"name": "network_f32", "kind": "network", "dtype": "f32", "v": 72, "o": 20},
        # Labels in all three tensors: one product per k-point.
        {"name": "batch_labels_f64", "kind": "labels", "dtype": "f64", "l": 96, "a": 120, "b": 104, "e": 136},
        # A large tensor times a small matrix along its slowest mode (a
        # Tucker / basis change step): bound by memory, not by MFMA.
        {"name": "mode_product_f64", "kind": "mode", "dtype": "f64", "a": 96, "b": 80, "c": 88, "d": 64, "r": 16},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "ladder", "ladder", "ring", "batched", "autograd", "network", "labels",
                       "mode"])
    dtype = rng.choice(["f64", "f32"])
    if kind == "plain":
        c = {"kind": kind, "dtype": dtype}
        for lab in "abijef":
            c[lab] = _log(rng, 4, 40)
        c.update(pad=rng.randint(0, 2), entry=rng.choice(["plan", "contract"]))
        return c
    if kind in ("ladder", "ring"):
        compute = rng.choice(["native", "int8x6", "int8x7"] if dtype == "f64" else ["native", "bf16x3", "bf16x6"])
        v = _log(rng, 24, 112)
        return {"kind": kind, "dtype": dtype, "compute": compute, "v": v, "o": max(4, v // rng.choice([3, 4, 5]))}
    if kind == "batched":
        return {"kind": kind, "dtype": dtype, "n": _log(rng, 32, 1500 if dtype == "f32" else 700),
                "hi": rng.randint(12, 48)}
    if kind == "autograd":
        v = _log(rng, 24, 96)
        return {"kind": kind, "dtype": dtype, "v": v, "o": max(4, v // rng.choice([3, 4, 5]))}
    if kind == "network":
        v = _log(rng, 24, 80)
        return {"kind": kind, "dtype": dtype, "v": v, "o": max(4, v // rng.choice([3, 4, 5]))}
    if kind == "labels":
        return {"kind": kind, "dtype": dtype, "l": _log(rng, 4, 256), "a": _log(rng, 16, 200),
                "b": _log(rng, 16, 200), "e": _log(rng, 16, 200)}
    return {"kind": "mode", "dtype": dtype, "a": _log(rng, 16, 96), "b": _log(rng, 16, 96), "c": _log(rng, 16, 96),
            "d": _log(rng, 16, 96), "r": _log(rng, 1, 32)}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _values(g, n, dtype, dist):
    if dist == "uniform":
        return torch.rand(n, generator=g, device="cuda", dtype=dtype).mul_(2).sub_(1)
    x = torch.randn(n, generator=g, device="cuda", dtype=dtype)
    if dist == "outliers":  # one value in a thousand ten thousand times larger
        x.mul_(1 + 9999.0 * (torch.rand(n, generator=g, device="cuda") < 1e-3).to(dtype))
    return x


def _tensor(g, labels, ext, dtype, dist="uniform", order=None, pad=0):
    """A strided tensor in column-major storage (or `order`, fastest first)
    with `pad` unused elements after each run of the two fastest modes."""
    order = list(range(len(labels))) if order is None else [labels.index(ch) for ch in order]
    pads = [0] * len(labels)
    for d in order[:2]:
        pads[d] = pad
    lay = synth.layout([ext[ch] for ch in labels], order=order, pad=pads)
    return _values(g, lay.size, dtype, dist).as_strided(lay.extents, lay.strides, lay.base)


def _desc(t, labels):
    return fm.make_desc(tuple(t.shape), t.stride(), labels)


class _Plan:
    """A plan that lives as long as the state that keeps it."""

    def __init__(self, plan):
        self.plan = plan

    def __del__(self):
        torch.cuda.synchronize()
        fm.famlies_plan_destroy(self.plan)


class _Net:
    def __init__(self, net):
        self.net = net

    def __del__(self):
        torch.cuda.synchronize()
        self.net.close()


# The labels and storage of each single-contraction family: A, B, C labels,
# A's storage order, alpha, beta, value distribution.
FAMILIES = {
    "plain": ("aeif", "ebfj", "abij", None, 1.0, 0.5, "uniform"),
    "ladder": ("abef", "efij", "abij", "eafb", 1.0, 1.0, "uniform"),
    "ring": ("akic", "cbkj", "aibj", None, 1.0, 0.0, "outliers"),
    "labels": ("aeL", "ebL", "abL", None, 1.0, 0.0, "uniform"),
    "mode": ("abcd", "dr", "abcr", None, 1.0, 0.0, "uniform"),
    "autograd": ("aeif", "ebfj", "abij", None, 1.0, 0.0, "uniform"),
}


def _extents(case):
    kind = case["kind"]
    if kind == "plain":
        return {ch: case[ch] for ch in "abijef"}
    if kind == "labels":
        return {"L": case["l"], "a": case["a"], "b": case["b"], "e": case["e"]}
    if kind == "mode":
        return {ch: case[ch] for ch in "abcdr"}
    v, o = case["v"], case["o"]
    if kind == "ring":
        return {"a": v, "b": v, "c": v, "i": o, "j": o, "k": o}
    return {"a": v, "b": v, "e": v, "f": v, "i": o, "j": o, "k": o, "l": o}


def _inputs(case, seed):
    la, lb, lc, order, alpha, beta, dist = FAMILIES[case["kind"]]
    ext, dtype, g = _extents(case), DTYPES[case["dtype"]], _gen(seed)
    pad = case.get("pad", 0)
    A = _tensor(g, la, ext, dtype, dist, order, pad)
    B = _tensor(g, lb, ext, dtype, dist, None, pad)
    C = _tensor(g, lc, ext, dtype, "normal" if case["kind"] == "autograd" else "uniform", None, pad)
    return la, lb, lc, alpha, beta, A, B, C


def _network_inputs(case, seed):
    ext, dtype, g = _extents(case), DTYPES[case["dtype"]], _gen(seed)
    t = {}
    for name, labels, order in (("W", "abef", "eafb"), ("T", "efkl", None), ("V", "klij", None),
                                ("R", "abij", None), ("Q", "abij", None), ("Z", "ij", None)):
        t[name] = _tensor(g, labels, ext, dtype, "uniform", order)
    return t


def _batched_problems(case):
    """The problems' shapes and layouts, drawn from the case; the seed gives
    their values."""
    rng = np.random.default_rng([5, case["n"], case["hi"]])
    return [synth.random_problem(rng, 4, case["hi"]) for _ in range(case["n"])]


def _batched_inputs(case, seed):
    """Problems and one flat buffer per operand with a 256-byte aligned block
    for each problem."""
    probs, dtype, g = _batched_problems(case), DTYPES[case["dtype"]], _gen(seed)
    bufs, starts = [], []
    for side in ("a", "b", "c"):
        pos, at = 0, []
        for p in probs:
            at.append(pos)
            pos += (getattr(p, side).size + 63) // 64 * 64
        bufs.append(_values(g, pos, dtype, "uniform"))
        starts.append(at)
    return probs, bufs, starts


def prepare(case, seed):
    kind = case["kind"]
    dev = torch.cuda.current_device()
    if kind == "batched":
        table = os.path.join(os.path.dirname(fm.__file__), "tables", "batch_mi355x.txt")
        fm.famlies_load_tune_table(fm.handle(dev), table)
        probs, bufs, starts = _batched_inputs(case, seed)
        descs = [[fm.make_desc(lay.extents, lay.strides, lab) for lay, lab in side] for side in
                 ([(p.a, p.la) for p in probs], [(p.b, p.lb) for p in probs], [(p.c, p.lc) for p in probs])]
        plan = _Plan(fm.famlies_batch_plan(fm.handle(dev), CODES[case["dtype"]], *descs))
        es = bufs[0].element_size()
        ptrs = [torch.tensor([b.data_ptr() + es * (s + getattr(p, side).base) for p, s in zip(probs, at)],
                             dtype=torch.int64).cuda() for b, at, side in zip(bufs, starts, "abc")]
        return {"kind": kind, "plan": plan, "bufs": bufs, "ptrs": ptrs}
    if kind == "network":
        t = _network_inputs(case, seed)
        net = fm.Network(CODES[case["dtype"]], device=dev)
        keep = _Net(net)
        ext = _extents(case)
        ids = {n: net.tensor(tuple(t[n].shape), t[n].stride(), lab) for n, lab in
               (("W", "abef"), ("T", "efkl"), ("V", "klij"), ("R", "abij"), ("Q", "abij"), ("Z", "ij"))}
        lay = synth.layout([ext[ch] for ch in "abkl"])
        ids["I"] = net.tensor(lay.extents, lay.strides, "abkl", intermediate=True)
        net.contract(1.0, ids["W"], ids["T"], 0.0, ids["I"], pack_a=True)
        net.contract(1.0, ids["I"], ids["V"], 0.5, ids["R"])
        net.contract(2.0, ids["R"], ids["Q"], 0.0, ids["Z"])
        net.compile()
        for n, x in t.items():
            net.bind(ids[n], x.data_ptr())
        return {"kind": kind, "net": keep, "t": t}
    la, lb, lc, alpha, beta, A, B, C = _inputs(case, seed)
    state = {"kind": kind, "A": A, "B": B, "C": C, "labels": (la, lb, lc), "alpha": alpha, "beta": beta,
             "compute": case.get("compute", "native"), "entry": case.get("entry", "contract")}
    if kind == "autograd":
        A.requires_grad_(True)
        B.requires_grad_(True)
    elif state["entry"] == "plan":
        state["plan"] = _Plan(fm.famlies_plan_contract(fm.handle(dev), CODES[case["dtype"]],
                                                       COMPUTES[state["compute"]], _desc(A, la), _desc(B, lb),
                                                       _desc(C, lc)))
    return state


# --------------------------------------------------------------------- pass
def run(state):
    kind = state["kind"]
    if kind == "batched":
        a, b, c = (p.data_ptr() for p in state["ptrs"])
        fm.famlies_batch_execute(state["plan"].plan, 1.0, 0.5, a, b, c, torch.cuda.current_stream().cuda_stream)
        return state["bufs"][2]
    if kind == "network":
        state["net"].net.execute(torch.cuda.current_stream().cuda_stream)
        return {"R": state["t"]["R"], "Z": state["t"]["Z"]}
    A, B, C, (la, lb, lc) = state["A"], state["B"], state["C"], state["labels"]
    if kind == "autograd":
        out = fm.contract_ad(state["alpha"], A, la, B, lb, 0.0, None, lc)
        dA, dB = torch.autograd.grad(out, (A, B), C)
        return {"C": out.detach(), "dA": dA, "dB": dB}
    if state["entry"] == "plan":
        fm.famlies_execute(state["plan"].plan, state["alpha"], A.data_ptr(), B.data_ptr(), state["beta"],
                           C.data_ptr(), torch.cuda.current_stream().cuda_stream)
        return C
    return fm.contract(state["alpha"], A, la, B, lb, state["beta"], C, lc, compute=state["compute"])


# ------------------------------------------------------------------- 64 bits
def _matmul64(A, la, B, lb, lc):
    """sum A B over the labels not in lc, in float64, modes in lc's order."""
    ext = dict(zip(la, A.shape))
    ext.update(zip(lb, B.shape))
    L = [ch for ch in lc if ch in la and ch in lb]
    I = [ch for ch in lc if ch in la and ch not in L]
    J = [ch for ch in lc if ch in lb and ch not in L]
    P = [ch for ch in la if ch in lb and ch not in L]

    def size(g):
        return math.prod(ext[ch] for ch in g)

    X = A.double().permute([la.index(ch) for ch in L + I + P]).reshape(size(L), size(I), size(P))
    Y = B.double().permute([lb.index(ch) for ch in L + P + J]).reshape(size(L), size(P), size(J))
    if size(L) > 1 and size(I) == 1 and size(J) == 1:
        out = (X[:, 0, :] * Y[:, :, 0]).sum(-1)
    else:
        out = torch.stack([torch.mm(x, y) for x, y in zip(X, Y)])
    got = L + I + J
    return out.reshape([ext[ch] for ch in got]).permute([got.index(ch) for ch in lc])


def exact(case, seed):
    kind = case["kind"]
    if kind == "batched":
        probs, (ab, bb, cb), (sa, sb, sc) = _batched_inputs(case, seed)
        want = cb.double()
        for p, i, j, k in zip(probs, sa, sb, sc):
            A, B, C = (buf.as_strided(lay.extents, lay.strides, s + lay.base) for buf, lay, s in
                       ((ab, p.a, i), (bb, p.b, j), (want, p.c, k)))
            C.mul_(0.5).add_(_matmul64(A, p.la, B, p.lb, p.lc))
        return want
    if kind == "network":
        t = _network_inputs(case, seed)
        inter = _matmul64(t["W"], "abef", t["T"], "efkl", "abkl")
        R = _matmul64(inter, "abkl", t["V"], "klij", "abij") + 0.5 * t["R"].double()
        return {"R": R, "Z": 2.0 * _matmul64(R, "abij", t["Q"], "abij", "ij")}
    la, lb, lc, alpha, beta, A, B, C = _inputs(case, seed)
    out = alpha * _matmul64(A, la, B, lb, lc)
    if kind == "autograd":
        return {"C": out, "dA": alpha * _matmul64(C, lc, B, lb, la), "dB": alpha * _matmul64(A, la, C, lc, lb)}
    return out + beta * C.double() if beta else out


def work(case):
    es = 8 if case["dtype"] == "f64" else 4
    kind = case["kind"]
    if kind == "batched":
        mnk = [synth.sizes(p) for p in _batched_problems(case)]
        return {"bytes": sum(m * k + k * n + 2 * m * n for m, n, k in mnk) * es,
                "flops": 2.0 * sum(m * n * k for m, n, k in mnk)}
    ext = _extents(case)

    def size(labels):
        return math.prod(ext[ch] for ch in labels)

    if kind == "network":
        read = sum(size(x) for x in ("abef", "efkl", "klij", "abij", "abij"))
        return {"bytes": (read + size("abij") + size("ij")) * es,
                "flops": 2.0 * (size("abefkl") + size("abklij") + size("abij"))}
    la, lb, lc = FAMILIES[kind][:3]
    a, b, c = size(la), size(lb), size(lc)
    flops = 2.0 * size("".join(dict.fromkeys(la + lb)))
    if kind == "autograd":  # A, B, G read; C, dA, dB written
        return {"bytes": (2 * a + 2 * b + 2 * c) * es, "flops": 3 * flops}
    return {"bytes": (a + b + (2 if FAMILIES[kind][5] else 1) * c) * es, "flops": flops}
