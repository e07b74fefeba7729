"""bf16x3 and bf16x6 through part planes (256 x 128 tiles): every entry against
an FP64 product on the GPU at the precision's componentwise bound, with ragged
tiles, odd runs, each gather direction, batch planes, levelled rounds,
pre-packed operands equal to gathered ones, and run-to-run equality; the dry run's log says which of them take the path (not
bf16x3 with both operands in runs along K, where the tiled kernel is as fast:
its pairs are checked all the same)."""
import os
import subprocess
import sys

import pytest

from tests.famlies_testutil import U64, bf16x3_bound, gamma

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# M, N, run of K, runs, batch: a round and part of one, odd runs; exact tiles;
# batch planes; a 128-column remainder with few tiles along N
SIZES = {"odd": (4200, 4170, 93, 45, 1), "even": (4096, 4096, 128, 32, 1), "planes": (4050, 4030, 1499, 1, 2),
         "wide": (7010, 2500, 50, 90, 1)}
ORDERS = ["kk", "kr", "rk", "rr"]


def _descs(fm, size, orders):
    m, n, k, q, L = size
    A = fm.make_desc([k, q, m, L], [1, k * m, k, k * q * m] if orders[0] == "k" else [m, k * m, 1, k * q * m], "kqmL")
    B = fm.make_desc([k, q, n, L], [1, k, k * q, k * q * n] if orders[1] == "k" else [n, k * n, 1, k * q * n], "kqnL")
    C = fm.make_desc([n, m, L], [1, n, n * m], "nmL")
    return A, B, C


def test_planes_are_chosen():
    code = ("import paper_2604_07311_amd as fm\n"
            "from tests.test_gpu_planes import SIZES, ORDERS, _descs\n"
            "for c in ('bf16x3', 'bf16x6'):\n"
            "    for s in SIZES.values():\n"
            "        for o in ORDERS:\n"
            "            fm.famlies_analyze(fm.FAMLIES_F32, fm._compute_code(c), *_descs(fm, s, o))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, FAMLIES_LOG="1"))
    lines = [ln for ln in r.stderr.splitlines() if "analyze" in ln]
    assert len(lines) == 2 * len(SIZES) * len(ORDERS), r.stderr
    expected = [c == "bf16x6" or o != "kk" for c in ("bf16x3", "bf16x6") for _ in SIZES for o in ORDERS]
    assert ["planes 256x128" in ln for ln, e in zip(lines, expected) if e] == [True] * sum(expected), lines


@pytest.mark.gpu
@pytest.mark.parametrize("compute", ["bf16x3", "bf16x6"])
@pytest.mark.parametrize("which", sorted(SIZES))
@pytest.mark.parametrize("orders", ORDERS)
def test_planes_match_fp64(compute, which, orders):
    import torch
    import paper_2604_07311_amd as fm
    m, n, k, q, L = SIZES[which]
    K, beta = k * q, -0.5 if orders[0] == "k" else 0.0
    g = torch.Generator(device="cuda").manual_seed(23)
    a = torch.rand(L * m * K, generator=g, device="cuda") * 2 - 1
    b = torch.rand(L * n * K, generator=g, device="cuda") * 2 - 1
    c0 = torch.rand(L * m * n, generator=g, device="cuda") * 2 - 1
    plan = fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F32, fm._compute_code(compute),
                                    *_descs(fm, SIZES[which], orders))
    s = torch.cuda.current_stream().cuda_stream
    outs = []
    packs = []
    for op, t in ((0, a), (1, b)):
        packs.append(torch.empty(fm.famlies_pack_size(plan, op), dtype=torch.uint8, device="cuda"))
        fm.famlies_pack(plan, op, t.data_ptr(), packs[op].data_ptr(), s)
    for mask in (0, 0, 1, 2, 3):
        c = c0.clone()
        fm.famlies_execute_packed(plan, 1.25, (packs[0] if mask & 1 else a).data_ptr(),
                                  (packs[1] if mask & 2 else b).data_ptr(), beta, c.data_ptr(), mask, s)
        torch.cuda.synchronize()
        outs.append(c)
    fm.famlies_plan_destroy(plan)
    assert all(torch.equal(outs[0], c) for c in outs[1:])
    if orders[0] == "k":
        A = a.double().view(L, q, m, k).permute(0, 2, 1, 3).reshape(L, m, K)
    else:
        A = a.double().view(L, q, k, m).permute(0, 3, 1, 2).reshape(L, m, K)
    if orders[1] == "k":
        B = b.double().view(L, n, K)
    else:
        B = b.double().view(L, q, k, n).permute(0, 3, 1, 2).reshape(L, n, K)
    for i in range(L):
        got, C0 = outs[0].double().view(L, m, n)[i], c0.double().view(L, m, n)[i]
        absp = 1.25 * torch.mm(A[i].abs(), B[i].t().abs())
        d = absp + abs(beta) * C0.abs()
        bound = (bf16x3_bound(K, absp, d) if compute == "bf16x3" else
                 (2.0 ** -22 + gamma(3 * K, 2.0 ** -23) * (1 + 2.0 ** -7)) * absp + 2.0 ** -23 * d)
        err = (got - (1.25 * torch.mm(A[i], B[i].t()) + beta * C0)).abs()
        assert bool((err <= bound + gamma(K + 2, U64) * d).all()), float((err / bound).max())
