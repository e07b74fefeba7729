"""Every wave tile of the direct kernel (16 x 16, 32 x 32, 16 x 64, 64 x 16), one
wave per tile or four sharing it, one accumulator or three, with and without K
ranges over workgroups: the dry run's log says that each size takes its
route, and results are compared with an FP64 product at the componentwise
bounds (gamma_{K+2}(2^-53) D, gamma_{K+4}(2^-24) D).  M and N are multiples of no
tile edge; with one wave per tile the tiles are no multiple of a workgroup's
four."""
import os
import re
import subprocess
import sys

import pytest

from tests.famlies_testutil import U32, U64, gamma

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# dtype, (tile M, tile N, waves), accumulators, K ranges > 1, gather of A and B
# (k: along k, r: by rows), M, N, K
CASES = [
    ("f64", (16, 16, 1), 1, 0, "kk", 21480, 2, 29), ("f64", (16, 16, 1), 1, 0, "kr", 9110, 7, 38),
    ("f64", (16, 16, 1), 1, 0, "rk", 1, 11346, 37), ("f64", (16, 16, 1), 1, 0, "rr", 1, 20571, 32),
    ("f64", (16, 16, 4), 1, 0, "kk", 4, 71, 98), ("f64", (16, 16, 4), 1, 0, "rk", 6, 51, 87),
    ("f64", (16, 16, 4), 1, 1, "kk", 38, 5, 2857), ("f64", (16, 16, 4), 1, 1, "rk", 92, 3, 2447),
    ("f64", (16, 16, 4), 3, 0, "kk", 3, 297, 202), ("f64", (16, 16, 4), 3, 0, "rk", 3, 227, 226),
    ("f64", (16, 64, 1), 1, 0, "kk", 7, 194237, 19), ("f64", (16, 64, 1), 1, 0, "kr", 3, 138905, 48),
    ("f64", (16, 64, 1), 1, 0, "rk", 5, 111179, 42), ("f64", (16, 64, 1), 1, 0, "rr", 2, 44364, 260),
    ("f64", (16, 64, 1), 3, 0, "kk", 1, 70439, 270), ("f64", (16, 64, 1), 3, 0, "kr", 10, 38305, 278),
    ("f64", (16, 64, 1), 3, 0, "rk", 69635, 36, 279), ("f64", (16, 64, 1), 3, 0, "rr", 2, 37449, 275),
    ("f64", (16, 64, 4), 1, 0, "kk", 2, 16469, 183), ("f64", (16, 64, 4), 1, 0, "rk", 3, 21598, 91),
    ("f64", (16, 64, 4), 1, 1, "kk", 15, 489, 2609), ("f64", (16, 64, 4), 1, 1, "rk", 3, 578, 2065),
    ("f64", (16, 64, 4), 3, 0, "kk", 1, 98810, 288), ("f64", (16, 64, 4), 3, 0, "rk", 23, 33400, 203),
    ("f64", (32, 32, 1), 1, 0, "kk", 19, 63382, 137), ("f64", (32, 32, 1), 1, 0, "kr", 18, 231953, 293),
    ("f64", (32, 32, 1), 1, 0, "rk", 52649, 17, 216), ("f64", (32, 32, 1), 1, 0, "rr", 20, 22711, 114),
    ("f64", (32, 32, 4), 1, 0, "kk", 359, 774, 185), ("f64", (32, 32, 4), 1, 0, "rk", 18, 9831, 269),
    ("f64", (32, 32, 4), 1, 1, "kk", 84, 525, 2005), ("f64", (32, 32, 4), 1, 1, "rk", 245, 69, 2311),
    ("f64", (32, 32, 4), 3, 0, "kk", 283, 813, 671), ("f64", (32, 32, 4), 3, 0, "rk", 273, 555, 528),
    ("f64", (64, 16, 1), 1, 0, "kk", 187049, 2, 86), ("f64", (64, 16, 1), 1, 0, "kr", 125862, 4, 59),
    ("f64", (64, 16, 1), 1, 0, "rk", 46526, 4, 183), ("f64", (64, 16, 1), 1, 0, "rr", 91737, 9, 44),
    ("f64", (64, 16, 1), 3, 0, "kk", 38448, 29, 280), ("f64", (64, 16, 1), 3, 0, "kr", 68693, 4, 275),
    ("f64", (64, 16, 1), 3, 0, "rk", 40750, 4, 288), ("f64", (64, 16, 1), 3, 0, "rr", 34324, 11, 165),
    ("f64", (64, 16, 4), 1, 0, "kk", 9784, 19, 50), ("f64", (64, 16, 4), 1, 0, "rk", 7494, 4, 223),
    ("f64", (64, 16, 4), 1, 1, "kk", 857, 3, 2720), ("f64", (64, 16, 4), 1, 1, "rk", 166, 34, 2117),
    ("f64", (64, 16, 4), 3, 0, "kr", 11242, 10, 260), ("f64", (64, 16, 4), 3, 0, "rr", 20250, 2, 244),
    ("f32", (16, 16, 1), 1, 0, "kk", 4, 21791, 8), ("f32", (16, 16, 1), 1, 0, "kr", 2, 22764, 70),
    ("f32", (16, 16, 1), 1, 0, "rk", 3, 117906, 5), ("f32", (16, 16, 1), 1, 0, "rr", 20495, 6, 4),
    ("f32", (16, 16, 4), 1, 0, "kk", 1, 241, 237), ("f32", (16, 16, 4), 1, 0, "rk", 19, 12, 348),
    ("f32", (16, 16, 4), 1, 1, "kk", 3, 122, 2369), ("f32", (16, 16, 4), 1, 1, "rk", 88, 12, 2753),
    ("f32", (16, 16, 4), 3, 0, "kk", 8, 120, 447), ("f32", (16, 16, 4), 3, 0, "rk", 12, 81, 462),
    ("f32", (16, 64, 1), 1, 0, "kk", 2, 128162, 59), ("f32", (16, 64, 1), 1, 0, "kr", 1, 102408, 141),
    ("f32", (16, 64, 1), 1, 0, "rk", 3, 36647, 175), ("f32", (16, 64, 1), 1, 0, "rr", 2, 198276, 41),
    ("f32", (16, 64, 4), 1, 0, "kk", 3, 11478, 114), ("f32", (16, 64, 4), 1, 0, "rk", 3, 5560, 233),
    ("f32", (16, 64, 4), 3, 0, "kk", 33, 5003, 779), ("f32", (32, 32, 1), 1, 0, "kk", 21982, 25, 232),
    ("f32", (32, 32, 1), 1, 0, "kr", 52, 17944, 33), ("f32", (32, 32, 1), 1, 0, "rk", 39098, 17, 299),
    ("f32", (32, 32, 1), 1, 0, "rr", 23047, 26, 210), ("f32", (32, 32, 4), 1, 0, "kk", 6244, 58, 99),
    ("f32", (32, 32, 4), 1, 0, "rk", 53, 7154, 129), ("f32", (32, 32, 4), 1, 1, "kk", 412, 151, 2846),
    ("f32", (32, 32, 4), 1, 1, "rr", 874, 74, 2927), ("f32", (32, 32, 4), 3, 0, "kk", 446, 463, 1122),
    ("f32", (32, 32, 4), 3, 0, "rk", 727, 364, 1133), ("f32", (64, 16, 1), 1, 0, "kk", 30790, 3, 258),
    ("f32", (64, 16, 1), 1, 0, "kr", 210979, 8, 13), ("f32", (64, 16, 1), 1, 0, "rk", 50324, 4, 109),
    ("f32", (64, 16, 1), 1, 0, "rr", 175511, 13, 13), ("f32", (64, 16, 4), 1, 0, "kk", 5491, 29, 51),
    ("f32", (64, 16, 4), 1, 0, "rk", 10077, 6, 141), ("f32", (64, 16, 4), 3, 0, "kk", 5003, 33, 779),
]


def _descs(fm, o, m, n, k):
    return (fm.make_desc((m, k), (k, 1) if o[0] == "k" else (1, m), "mk"),
            fm.make_desc((k, n), (1, k) if o[1] == "k" else (n, 1), "kn"), fm.make_desc((m, n), (n, 1), "mn"))


def test_sizes_take_their_routes():
    code = ("import paper_2604_07311_amd as fm\n"
            "from tests.test_gpu_direct_shapes import CASES, _descs\n"
            "for c in CASES:\n"
            "    fm.famlies_analyze(fm.FAMLIES_F64 if c[0] == 'f64' else fm.FAMLIES_F32, 0, *_descs(fm, *c[4:]))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, FAMLIES_LOG="1"))
    lines = [ln for ln in r.stderr.splitlines() if "analyze" in ln]
    assert len(lines) == len(CASES), r.stderr
    for c, ln in zip(CASES, lines):
        g = re.search(r"direct=(\d+)x(\d+)/(\d+) waves/split (\d+)/chains (\d+)", ln)
        assert g, (c, ln)
        bm, bn, wk, split, chains = map(int, g.groups())
        assert ((bm, bn, wk), chains, int(split > 1)) == c[1:4], (c, ln)
    assert {c[1] for c in CASES} == {(a, b, w) for a, b in ((16, 16), (32, 32), (16, 64), (64, 16)) for w in (1, 4)}


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%dx%d-%dw-c%d-s%d-%s-%d-%d-%d" % (c[0], *c[1], *c[2:]))
def test_route_matches_fp64(case):
    import torch
    import paper_2604_07311_amd as fm
    dtype, _, _, _, o, m, n, k = case
    dt = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(m + 3 * n + 5 * k)
    rnd = lambda size: torch.rand(size, generator=g, device="cuda", dtype=dt) * 2 - 1
    # one element before and behind each operand, unaligned bases
    a, b, c0 = rnd(m * k + 2), rnd(k * n + 2), rnd(m * n + 2)
    A = a[1:-1].view(m, k) if o[0] == "k" else a[1:-1].view(k, m).t()
    B = b[1:-1].view(n, k).t() if o[1] == "k" else b[1:-1].view(k, n)
    prod, absp = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    plan = fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F64 if dtype == "f64" else fm.FAMLIES_F32, 0,
                                    *_descs(fm, o, m, n, k))
    s = torch.cuda.current_stream().cuda_stream
    for beta in (0.0, -0.5):
        got = []
        for packed in (0, 0, 3):
            ptr, keep = [A.data_ptr(), B.data_ptr()], []
            for op in (0, 1):
                if packed:
                    keep.append(torch.empty(fm.famlies_pack_size(plan, op) // 4 + 4, dtype=torch.int32, device="cuda"))
                    fm.famlies_pack(plan, op, ptr[op], keep[op].data_ptr(), s)
                    ptr[op] = keep[op].data_ptr()
            c = c0.clone()
            fm.famlies_execute_packed(plan, 1.25, ptr[0], ptr[1], beta, c[1:].data_ptr(), packed, s)
            torch.cuda.synchronize()
            got.append(c)
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
        C0 = c0[1:-1].view(m, n).double()
        d = 1.25 * absp + abs(beta) * C0.abs()
        bound = (gamma(k + 2, U64) if dtype == "f64" else gamma(k + 4, U32)) * d + gamma(k + 4, U64) * d
        assert bool(((got[0][1:-1].view(m, n).double() - (1.25 * prod + beta * C0)).abs() <= bound).all())
        assert got[0][0] == c0[0] and got[0][-1] == c0[-1]
    fm.famlies_plan_destroy(plan)
