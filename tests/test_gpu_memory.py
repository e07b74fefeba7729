"""Plans where memory is short: calls that just fit the static scratch array,
plans past the handle's budget of extra workspace and plans on a nearly full
device run as the tile choice alone would (results against an FP64 product)."""
import os
import subprocess
import sys

import numpy as np
import pytest

from tests.famlies_testutil import U64, gamma

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_noalloc_at_the_limit():
    """The longest dot product whose plain indexing vectors and K ranges fit
    64 MiB, and one slice more."""
    import torch
    import paper_2604_07311_amd as fm
    desc = lambda k: (fm.make_desc([k, 3], [1, k], "km"), fm.make_desc([k], [1], "k"), fm.make_desc([3], [1], "m"))
    info, _ = fm.famlies_analyze(fm.FAMLIES_F64, 0, *desc(8000000))
    tm, tn, bk, split = (info[x] for x in ("tile_m", "tile_n", "tile_k", "split_k"))
    work = split * tm * tn * 8
    # image: rows and columns of X / Y and C, both contracted vectors (one slice
    # of padding), three batch offsets; in whole 256 bytes beside the K ranges
    words = ((64 << 20) - work - 24) // 4 - 2 * (tm + tn)
    kp = words // 2 // bk * bk
    k = kp - bk
    a = torch.rand(3, k, device="cuda", dtype=torch.float64) - 0.5
    b = torch.rand(k, device="cuda", dtype=torch.float64) - 0.5
    c = torch.zeros(3, device="cuda", dtype=torch.float64)
    s = torch.cuda.current_stream().cuda_stream
    args = lambda kk: (fm.handle(0), fm.FAMLIES_F64, 0, 1.0, desc(kk)[0], a.data_ptr(), desc(kk)[1], b.data_ptr(), 0.0,
                       desc(kk)[2], c.data_ptr(), s)
    fm.famlies_contract_noalloc(*args(k))
    torch.cuda.synchronize()
    want, d = a @ b, a.abs() @ b.abs()
    assert bool(((c - want).abs() <= 2 * gamma(k + 2, U64) * d).all())
    with pytest.raises(fm.FamliesError) as e:
        fm.famlies_contract_noalloc(*args(k + 1024))
    assert e.value.code == fm.FAMLIES_ERR_UNSUPPORTED


BUDGET = """
import torch, paper_2604_07311_amd as fm
m, n, k, q = 4200, 4170, 93, 45
d = (fm.make_desc([k, q, m], [1, k * m, k], "kqm"), fm.make_desc([k, q, n], [1, k, k * q], "kqn"),
     fm.make_desc([n, m], [1, n], "nm"))
a = torch.rand(m * k * q, device="cuda") - 0.5
b = torch.rand(n * k * q, device="cuda") - 0.5
A = a.double().view(q, m, k).permute(1, 0, 2).reshape(m, q * k)
want = A @ b.double().view(n, q * k).t()
plans = []
for i in range(60):
    plans.append(fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F32, fm.FAMLIES_BF16X6, *d))
for p in (plans[0], plans[-1]):
    c = torch.empty(m, n, device="cuda")
    fm.famlies_execute(p, 1.0, a.data_ptr(), b.data_ptr(), 0.0, c.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    print("err %.3e" % float((c.double() - want).norm() / want.norm()))
for p in plans[:30]:
    fm.famlies_plan_destroy(p)
plans.append(fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F32, fm.FAMLIES_BF16X6, *d))
"""


def test_plans_past_the_budget_keep_runs_and_rounds():
    """The planes of 60 such plans pass the budget: the later plans split while
    staging, with K in runs and a levelled round as long as that fits, then as
    the tile choice alone; after half are destroyed planes come again."""
    r = subprocess.run([sys.executable, "-c", BUDGET], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, FAMLIES_LOG="1"))
    assert r.returncode == 0, r.stderr
    lines = [ln for ln in r.stderr.splitlines() if "[famlies] plan" in ln]
    planes = ["planes" in ln for ln in lines]
    assert len(lines) == 61 and planes[0] and not planes[59] and planes[60], planes
    first = planes.index(False)
    assert not any(planes[first:60]) and "level=" in lines[first], lines[first]
    errs = [float(ln.split()[1]) for ln in r.stdout.splitlines()]
    # FP32 sums of K = 4185 terms: within a third of each other (the runs differ
    # by the two kernels' order of the small products only)
    assert errs[1] <= 1.33 * errs[0], errs


@pytest.mark.parametrize("compute", ["native", "int8x6"])
def test_plan_on_a_nearly_full_device(compute):
    """Levelled blocks (INT8: K ranges) that no longer fit are done without."""
    import torch
    import paper_2604_07311_amd as fm
    m, n, k = (3500, 3480, 5584) if compute == "native" else (512, 512, 20000)
    A = torch.rand(m, k, device="cuda", dtype=torch.float64) - 0.5
    B = torch.rand(n, k, device="cuda", dtype=torch.float64) - 0.5
    want, d = A @ B.t(), A.abs() @ B.abs().t()
    c = torch.empty(m, n, device="cuda", dtype=torch.float64)
    descs = (fm.make_desc((m, k), (k, 1), "mk"), fm.make_desc((n, k), (k, 1), "nk"), fm.make_desc((m, n), (n, 1), "mn"))
    h = fm.handle(0)
    code = (fm.FAMLIES_F64, fm._compute_code(compute))
    free = lambda: torch.cuda.mem_get_info()[0]
    free0 = free()
    plan = fm.famlies_plan_contract(h, *code, *descs)
    full = free0 - free()
    fm.famlies_plan_destroy(plan)
    hogs = []
    try:
        # leave less than that plan took, but more than the tile choice needs
        short = (150 << 20) if compute == "native" else (25 << 20)
        while free() > full - short + (4 << 20):
            hogs.append(torch.empty(free() - (full - short), device="cuda", dtype=torch.uint8))
        free0 = free()
        plan = fm.famlies_plan_contract(h, *code, *descs)
        assert free0 - free() < full - short + (4 << 20)
        fm.famlies_execute(plan, 1.0, A.data_ptr(), B.data_ptr(), 0.0, c.data_ptr(),
                           torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        fm.famlies_plan_destroy(plan)
    finally:
        del hogs
        torch.cuda.empty_cache()
    bound = 2 * gamma(k + 2, U64) * d if compute == "native" else 1e-10 * d.max()
    assert bool(((c - want).abs() <= bound).all())
