"""FP64 on INT8 at the edges of its tiles, plane tiles, K blocks, pairs and K
ranges (128 x 128 and 128 x 64 tiles, odd runs, both gather directions,
unaligned bases), against the emulation oracle: same digits, so the error is
that of the FP64 recombination alone, gamma_{s+4+r} (2^-53) D' with r the
number of partial sums per entry (at most 16 K ranges and their reduction)."""
import numpy as np
import pytest

import oracle
import synth
from tests.famlies_testutil import DeviceRunner, U64, gamma, used_offsets

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    return DeviceRunner()


def _scale_exp(mx):
    f, e = np.frexp(mx)
    return np.where(mx == 0, 0, np.where(f <= 127 / 128, e, e + 1))


# (M, N, run of K, runs)
SIZES = [(1, 1, 1, 1), (64, 64, 64, 1), (130, 65, 13, 9), (127, 129, 93, 3), (40, 200, 50, 5), (200, 63, 3, 50),
         (129, 257, 128, 2), (70, 70, 2, 700)]


@pytest.mark.parametrize("s", [3, 6, 7])
@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("orders", [("kmq", "knq"), ("kmq", "nkq"), ("mkq", "nkq")])
def test_int8_edges(gpu, s, size, orders):
    m, n, k, q = size
    ext = {"m": m, "n": n, "k": k, "q": q}
    lays = []
    for lab, order in (("mkq", orders[0]), ("knq", orders[1]), ("mn", "nm")):
        t = synth.layout([ext[ch] for ch in lab], order=[lab.index(ch) for ch in order])
        lays.append(synth.Strided(t.extents, t.strides, t.base + 1, t.size + 1))
    p = synth.Problem("i8", "mkq", "knq", "mn", *lays, 1.25, -0.5)
    rng = np.random.default_rng(m + 7 * n + k)
    p.abuf, p.bbuf, p.cbuf = (synth.fill(rng, t, "normal") for t in (p.a, p.b, p.c))
    got = gpu.run(p, "f64", "int8x%d" % s)
    emul = oracle.contract(p.alpha, *p.oracle_args()[:4], p.beta, *p.oracle_args()[4:], split=oracle.int8_slices(s))
    _, d = oracle.contract(p.alpha, *p.oracle_args()[:4], p.beta, *p.oracle_args()[4:], want_cond=True)
    K = k * q
    view = lambda buf, t: np.lib.stride_tricks.as_strided(buf[t.base:], t.extents, [8 * x for x in t.strides])
    ea = _scale_exp(np.abs(view(p.abuf, p.a)).max(axis=(1, 2)))
    eb = _scale_exp(np.abs(view(p.bbuf, p.b)).max(axis=(0, 2)))
    scale = abs(p.alpha) * np.exp2((ea[:, None] + eb[None, :]).astype(np.float64))
    dprime = view(d, p.c) + K * scale * (2.0 ** (1 - 7 * s) + 2.0 ** (-14 * s))
    err = np.abs(view(got, p.c) - view(emul, p.c))
    assert np.all(err <= gamma(s + 4 + 17, U64) * dprime), np.max(err / dprime)
    used = np.zeros(p.cbuf.size, dtype=bool)
    used[used_offsets(p.c)] = True
    np.testing.assert_array_equal(got[~used], p.cbuf[~used])
