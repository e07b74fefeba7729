"""Operands read in 16-byte runs along K whose length no run or slice divides
(the padded contracted order and its void mask) in the tiled FP64, FP32,
bf16x3 and bf16x6 kernels: forced tiles, split-K, unaligned bases, non-finite
values, against the oracle at each precision's componentwise bound."""
import numpy as np
import pytest

import synth
from tests.famlies_testutil import (DeviceRunner, U32, bf16x3_bound, check_fp32, check_fp64, gamma, oracle_full,
                                    round_inputs, used_offsets)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    return DeviceRunner()


def _problem(ext, orders, seed, shift=1, beta=0.5):
    lays = []
    for lab, order in zip(("mkq", "knq", "mn"), orders):
        t = synth.layout([ext[ch] for ch in lab], order=[lab.index(ch) for ch in order])
        lays.append(synth.Strided(t.extents, t.strides, t.base + shift, t.size + shift))
    p = synth.Problem("runs", "mkq", "knq", "mn", *lays, 1.25, beta)
    rng = np.random.default_rng(seed)
    p.abuf, p.bbuf, p.cbuf = (synth.fill(rng, t, "uniform") for t in (p.a, p.b, p.c))
    return p


def _plan(gpu, tmp_path, p, dtype, compute, bm, split, tail=0):
    """A plan whose tile table forces bm x bm tiles and the K split (so the
    tiled kernel runs at sizes the oracle checks in full)."""
    fm = gpu.fm
    code = fm.FAMLIES_F64 if dtype == "f64" else fm.FAMLIES_F32
    comp = fm._compute_code(compute)
    descs = [fm.make_desc(t.extents, t.strides, lab) for t, lab in ((p.a, p.la), (p.b, p.lb), (p.c, p.lc))]
    info, _ = fm.famlies_analyze(code, comp, *descs)
    lg = lambda x: int(np.ceil(np.log2(max(x, 1))))
    path = tmp_path / "t.txt"
    path.write_text("plain %d %d %d %d %d %d %d %d %d 0 %d\n" % (
        code, comp, lg(info["m"]), lg(info["n"]), lg(info["k"]), bm, bm, 8 if dtype == "f64" else 32, split, tail))
    h = fm.famlies_create(0)
    fm.famlies_load_tune_table(h, str(path))
    plan = fm.famlies_plan_contract(h, code, comp, *descs)
    assert fm.famlies_plan_get_info(plan)["tile_m"] == bm
    return h, plan


MODES = [("f64", "native"), ("f32", "native"), ("f32", "bf16x3"), ("f32", "bf16x6")]


@pytest.mark.parametrize("dtype,compute", MODES)
@pytest.mark.parametrize("bm,split,tail", [(64, 1, 0), (128, 1, 0), (64, 3, 0), (64, 3, 2)])
@pytest.mark.parametrize("orders", [("kmq", "knq", "nm"), ("kmq", "nkq", "nm"), ("mkq", "knq", "mn"),
                                    ("kqm", "kqn", "nm")])
@pytest.mark.parametrize("run", [(13, 9), (93, 3), (50, 5), (6, 31)])
def test_runs_match_oracle(gpu, tmp_path, dtype, compute, bm, split, tail, orders, run):
    p = round_inputs(_problem({"m": 150, "n": 170, "k": run[0], "q": run[1]}, orders, seed=run[0]), dtype)
    K = run[0] * run[1]
    h, plan = _plan(gpu, tmp_path, p, dtype, compute, bm, split, tail)
    try:
        got = gpu.run(p, dtype, compute=compute, plan=plan)
    finally:
        gpu.fm.famlies_plan_destroy(plan)
        gpu.fm.famlies_destroy(h)
    want, d = oracle_full(p)
    used = np.zeros(p.cbuf.size, dtype=bool)
    used[used_offsets(p.c)] = True
    np.testing.assert_array_equal(got[~used], p.cbuf[~used])
    if compute == "native":
        (check_fp64 if dtype == "f64" else check_fp32)(got, want, d, K, where=used)
        return
    _, dp = oracle_full(p, None, 0.0)
    if compute == "bf16x3":
        bound = bf16x3_bound(K, dp, d)
    else:  # dropped products 2^-22, FP32 accumulation, FP64 epilogue and FP32 store
        bound = (2.0 ** -22 + gamma(3 * K, 2.0 ** -23) * (1 + 2.0 ** -7)) * dp + 2.0 ** -23 * d
    assert np.all(np.abs(got - want)[used] <= bound[used])


@pytest.mark.parametrize("dtype,compute", MODES[:3])
@pytest.mark.parametrize("orders", [("kmq", "knq", "mn"), ("kmq", "nkq", "mn")])
def test_void_entries_do_not_spread_nonfinite(gpu, tmp_path, dtype, compute, orders):
    p = round_inputs(_problem({"m": 70, "n": 66, "k": 13, "q": 3}, orders, seed=5, beta=0.0), dtype)
    A, B = (np.lib.stride_tricks.as_strided(buf[t.base:], t.extents, [8 * s for s in t.strides])
            for buf, t in ((p.abuf, p.a), (p.bbuf, p.b)))
    A[3, 12, 1] = A[4, 9, 0] = A[5, 0, 2] = np.nan
    B[10, 7, 2] = B[9, 8, 0] = np.nan
    h, plan = _plan(gpu, tmp_path, p, dtype, compute, 64, 1)
    try:
        got = gpu.run(p, dtype, compute=compute, plan=plan, beta=0.0)
    finally:
        gpu.fm.famlies_plan_destroy(plan)
        gpu.fm.famlies_destroy(h)
    C = np.lib.stride_tricks.as_strided(got[p.c.base:], p.c.extents, [8 * s for s in p.c.strides])
    want = np.zeros((70, 66), dtype=bool)
    want[3:6, :] = True
    want[:, 7:9] = True
    np.testing.assert_array_equal(np.isnan(C), want)
