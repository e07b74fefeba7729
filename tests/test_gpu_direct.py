"""The direct kernel (small and narrow FP64 / FP32 contractions): tile edges,
K steps and padded K runs at their remainders, both gather directions, batch
labels, unaligned bases and non-finite values, against the oracle at the
componentwise bounds of the FP64 and FP32 paths (gamma_{K+2}(2^-53) D,
gamma_{K+4}(2^-24) D)."""
import numpy as np
import pytest

import synth
from tests.famlies_testutil import DeviceRunner, check_fp32, check_fp64, oracle_full, round_inputs, used_offsets

pytestmark = pytest.mark.gpu

CHECK = {"f64": check_fp64, "f32": check_fp32}


@pytest.fixture(scope="module")
def gpu():
    return DeviceRunner()


def _problem(ext, la, lb, lc, orders=(None, None, None), seed=1, beta=0.5, shift=0, dist="uniform"):
    lays = []
    for lab, order in zip((la, lb, lc), orders):
        t = synth.layout([ext[ch] for ch in lab], order=None if order is None else [lab.index(ch) for ch in order])
        lays.append(synth.Strided(t.extents, t.strides, t.base + shift, t.size + shift))
    p = synth.Problem("direct", la, lb, lc, *lays, 1.25, beta)
    rng = np.random.default_rng(seed)
    p.abuf, p.bbuf, p.cbuf = (synth.fill(rng, t, dist) for t in (p.a, p.b, p.c))
    return p


def _run(gpu, p, dtype, K):
    p = round_inputs(p, dtype)
    want, d = oracle_full(p)
    got = gpu.run(p, dtype)
    used = np.zeros(p.cbuf.size, dtype=bool)
    used[used_offsets(p.c)] = True
    np.testing.assert_array_equal(got[~used], p.cbuf[~used])
    CHECK[dtype](got, want, d, K, where=used)


# (M, N, first contracted extent, second): remainders of the 16 / 32 / 64
# tiles, K from one to several steps, runs of every remainder of 16 bytes.
SIZES = [(1, 1, 1, 1), (1, 1, 5184, 1), (16, 16, 16, 1), (15, 17, 13, 5), (33, 31, 15, 4), (32, 64, 18, 7),
         (64, 16, 23, 19), (1, 700, 77, 1), (130, 3, 7, 9), (5, 2100, 40, 1), (2100, 20, 31, 2), (100, 90, 50, 3),
         (40, 40, 3, 11), (16, 48, 64, 2)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("orders", ["kk", "kr", "rk", "rr"])
def test_direct_sizes(gpu, dtype, size, orders):
    """k: an operand stored along the contracted modes, r: along its rows."""
    m, n, k, q = size
    ext = {"m": m, "n": n, "k": k, "q": q}
    oa, ob = ("kmq" if orders[0] == "k" else "mkq"), ("knq" if orders[1] == "k" else "nkq")
    p = _problem(ext, "mkq", "knq", "mn", (oa, ob, "nm"), seed=m + 3 * n + k, shift=1)
    _run(gpu, p, dtype, k * q)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_direct_batch_labels_and_long_dot(gpu, dtype):
    ext = {"a": 21, "b": 37, "e": 29, "L": 19}
    _run(gpu, _problem(ext, "aeL", "ebL", "abL", seed=5), dtype, 29)
    ext = {"L": 24, "p": 611, "q": 3}
    _run(gpu, _problem(ext, "pqL", "pqL", "L", seed=6, beta=0.0), dtype, 611 * 3)
    # one output, K cut over many workgroups; positive data keep the normwise bound meaningful
    p = _problem({"p": 100003}, "p", "p", "", seed=7)
    p.abuf, p.bbuf = np.abs(p.abuf), np.abs(p.bbuf)
    _run(gpu, p, dtype, 100003)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_direct_repeated_entries_and_tails_do_not_spread_nonfinite(gpu, dtype):
    """Runs of 13 (padded with repeated entries) and K tails: an Inf or NaN
    gives exactly what the sum over the real entries gives."""
    ext = {"m": 18, "n": 35, "k": 13, "q": 3}
    p = _problem(ext, "mkq", "knq", "mn", ("kmq", "nkq", "mn"), seed=8, beta=0.0)
    p = round_inputs(p, dtype)
    A = np.lib.stride_tricks.as_strided(p.abuf[p.a.base:], p.a.extents, [8 * s for s in p.a.strides])
    B = np.lib.stride_tricks.as_strided(p.bbuf[p.b.base:], p.b.extents, [8 * s for s in p.b.strides])
    A[3, 12, 1], A[4, 8, 0], A[5, 0, 2] = np.inf, -np.inf, np.nan
    B[10, 7, 2] = np.inf
    B[9, 8, 0] = np.inf
    # plain sums (the oracle's compensated ones turn an Inf into NaN)
    want = p.cbuf.copy()
    C = np.lib.stride_tricks.as_strided(want[p.c.base:], p.c.extents, [8 * s for s in p.c.strides])
    C[...] = p.alpha * np.einsum("mkq,knq->mn", A, B, optimize=False)
    got = gpu.run(p, dtype)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf]) and np.array_equal(np.isinf(got), inf)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("mask", [1, 2, 3])
def test_direct_packed_equals_gathered(gpu, dtype, mask):
    """Pre-packed operands of a plan that runs direct: same sums, same bits."""
    import torch
    fm = gpu.fm
    p = round_inputs(_problem({"m": 45, "n": 70, "k": 27, "q": 5}, "mkq", "knq", "mn", ("kmq", "nkq", "nm"), seed=9),
                     dtype)
    es = 8 if dtype == "f64" else 4
    plan = gpu.plan(p, dtype)
    a, b, c0 = (gpu.to_dev(x, dtype) for x in (p.abuf, p.bbuf, p.cbuf))
    s = torch.cuda.current_stream().cuda_stream
    src = [a.data_ptr() + es * p.a.base, b.data_ptr() + es * p.b.base]
    outs = []
    keep = []
    for m in (0, mask):
        ptrs = list(src)
        for op in (0, 1):
            if m & (1 << op):
                buf = torch.empty(fm.famlies_pack_size(plan, op) // 4 + 4, dtype=torch.int32, device="cuda")
                fm.famlies_pack(plan, op, src[op], buf.data_ptr(), s)
                keep.append(buf)
                ptrs[op] = buf.data_ptr()
        c = c0.clone()
        fm.famlies_execute_packed(plan, p.alpha, ptrs[0], ptrs[1], p.beta, c.data_ptr() + es * p.c.base, m, s)
        torch.cuda.synchronize()
        outs.append(c.cpu().numpy())
    fm.famlies_plan_destroy(plan)
    np.testing.assert_array_equal(outs[0], outs[1])
    want, d = oracle_full(p)
    CHECK[dtype](outs[1].astype(np.float64), want, d, 27 * 5)
