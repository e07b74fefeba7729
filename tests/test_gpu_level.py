"""Levelled last round of the 128 x 128 kernels (first parts and runs of the
tiles that do not fill a round, blocks of partial sums reduced afterwards):
every entry against an FP64 product on the GPU, at the componentwise bounds of
each precision, and run-to-run equality."""
import os
import subprocess
import sys

import numpy as np
import pytest

from tests.famlies_testutil import U32, U64, bf16x3_bound, gamma

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# M, N, run of K, runs, batch: fewer tiles than a round; a round and part of
# one; batch planes sharing the rounds; ragged edges in all.
SIZES = {"part": (950, 1000, 250, 24, 1), "rounds": (3500, 3480, 93, 60, 1), "planes": (1150, 1150, 5997, 1, 4)}
MODES = [("f64", "native"), ("f32", "native"), ("f32", "bf16x3"), ("f32", "bf16x6")]


def _descs(fm, size):
    m, n, k, q, L = size
    A = fm.make_desc([k, q, m, L], [1, k * m, k, k * q * m], "kqmL")
    B = fm.make_desc([k, q, n, L], [1, k, k * q, k * q * n], "kqnL")
    C = fm.make_desc([n, m, L], [1, n, n * m], "nmL")
    return A, B, C


def test_levels_are_chosen():
    """The sizes below take a levelled round in the dry run's log (and a small
    problem does not)."""
    code = ("import paper_2604_07311_amd as fm\n"
            "from tests.test_gpu_level import SIZES, MODES, _descs\n"
            "for d, c in MODES:\n"
            "    for s in list(SIZES.values()) + [(64, 64, 64, 1, 1)]:\n"
            "        fm.famlies_analyze(fm.FAMLIES_F64 if d == 'f64' else fm.FAMLIES_F32, fm._compute_code(c),\n"
            "                           *_descs(fm, s))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, FAMLIES_LOG="1"))
    lines = [ln for ln in r.stderr.splitlines() if "analyze" in ln]
    assert len(lines) == 4 * len(MODES), r.stderr
    for i, ln in enumerate(lines):
        assert ("level=" in ln) == (i % 4 != 3), ln


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,compute", MODES)
@pytest.mark.parametrize("which", sorted(SIZES))
@pytest.mark.parametrize("beta", [0.0, -0.5])
def test_level_matches_fp64(dtype, compute, which, beta):
    import torch
    import paper_2604_07311_amd as fm
    size = SIZES[which]
    m, n, k, q, L = size
    K = k * q
    dt = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(17)
    a = torch.rand(L * m * K, generator=g, device="cuda", dtype=dt) * 2 - 1
    b = torch.rand(L * n * K, generator=g, device="cuda", dtype=dt) * 2 - 1
    c0 = torch.rand(L * m * n, generator=g, device="cuda", dtype=dt) * 2 - 1
    plan = fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F64 if dtype == "f64" else fm.FAMLIES_F32,
                                    fm._compute_code(compute), *_descs(fm, size))
    s = torch.cuda.current_stream().cuda_stream
    outs = []
    for _ in range(2):
        c = c0.clone()
        fm.famlies_execute(plan, 1.25, a.data_ptr(), b.data_ptr(), beta, c.data_ptr(), s)
        torch.cuda.synchronize()
        outs.append(c)
    fm.famlies_plan_destroy(plan)
    assert torch.equal(outs[0], outs[1])
    A = a.double().view(L, q, m, k).permute(0, 2, 1, 3).reshape(L, m, K)
    B = b.double().view(L, n, K)
    for i in range(L):
        got = outs[0].double().view(L, m, n)[i]
        C0 = c0.double().view(L, m, n)[i]
        prod = torch.mm(A[i], B[i].t())
        absp = 1.25 * torch.mm(A[i].abs(), B[i].t().abs())
        d = absp + abs(beta) * C0.abs()
        # the reference is itself an FP64 sum of K terms
        ref = gamma(K + 2, U64) * d
        if dtype == "f64":
            bound = gamma(K + 2, U64) * d
        elif compute == "native":
            bound = gamma(K + 4, U32) * d
        elif compute == "bf16x3":
            bound = bf16x3_bound(K, absp, d)
        else:
            bound = (2.0 ** -22 + gamma(3 * K, 2.0 ** -23) * (1 + 2.0 ** -7)) * absp + 2.0 ** -23 * d
        err = (got - (1.25 * prod + beta * C0)).abs()
        assert bool((err <= bound + ref).all()), "%s" % float((err / (bound + ref)).max())
