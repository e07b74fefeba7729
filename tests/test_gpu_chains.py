"""Error of the direct, levelled and part-plane routes against that of the
tiled kernel with the tile choice's own K ranges, on the same inputs: equal
chains of additions give equal errors.  The bound of 1.1 is five standard
deviations of the ratio at the fewest entries compared (4000: 5 / sqrt(4000)
= 0.08) and leaves out a chain twice as long (at least 1.4)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# m, n, k, which of A and B are gathered along k (bits): routes as the planner
# takes them
CASES = {"direct": (81, 1296, 1296, 3), "direct-deep": (256, 256, 1024, 1), "level": (2376, 2376, 2376, 3),
         "level-rounds": (3680, 3680, 3680, 3), "wide": (484, 12544, 12544, 3)}
MODES = [("f64", "native"), ("f32", "native"), ("f32", "bf16x6")]


@pytest.mark.parametrize("dtype,compute", MODES)
@pytest.mark.parametrize("which", sorted(CASES))
def test_error_is_that_of_the_k_ranges(tmp_path, dtype, compute, which):
    import torch
    import paper_2604_07311_amd as fm
    m, n, k, o = CASES[which]
    dt = torch.float64 if dtype == "f64" else torch.float32
    code = fm.FAMLIES_F64 if dtype == "f64" else fm.FAMLIES_F32
    comp = fm._compute_code(compute)
    g = torch.Generator(device="cuda").manual_seed(23)
    a = torch.rand(m * k, generator=g, device="cuda", dtype=dt) * 2 - 1
    b = torch.rand(k * n, generator=g, device="cuda", dtype=dt) * 2 - 1
    A = a.view(m, k) if o & 1 else a.view(k, m).t()
    B = b.view(n, k).t() if o & 2 else b.view(k, n)
    descs = [fm.make_desc(tuple(t.shape), t.stride(), lab) for t, lab in ((A, "mk"), (B, "kn"))]
    descs.append(fm.make_desc((m, n), (n, 1), "mn"))
    info, _ = fm.famlies_analyze(code, comp, *descs)
    lg = lambda x: int(np.ceil(np.log2(max(x, 1))))
    path = tmp_path / "t.txt"
    path.write_text("plain %d %d %d %d %d %d %d %d %d 0 %d\n" % (
        code, comp, lg(info["m"]), lg(info["n"]), lg(info["k"]), info["tile_m"], info["tile_n"],
        8 if dtype == "f64" else 32, info["split_k"],
        info["split_tiles"] if info["split_k"] > 1 and compute == "native" else 0))
    h = fm.famlies_create(0)
    fm.famlies_load_tune_table(h, str(path))
    outs = []
    for hd in (fm.handle(0), h):
        plan = fm.famlies_plan_contract(hd, code, comp, *descs)
        c = torch.empty(m, n, device="cuda", dtype=dt)
        fm.famlies_execute(plan, 1.0, A.data_ptr(), B.data_ptr(), 0.0, c.data_ptr(),
                           torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        if hd is h:
            got = fm.famlies_plan_get_info(plan)
            assert (got["tile_m"], got["split_k"]) == (info["tile_m"], info["split_k"])
        fm.famlies_plan_destroy(plan)
        outs.append(c)
    fm.famlies_destroy(h)
    if dtype == "f32":
        want = A.double() @ B.double()
        err = [float((c.double() - want).norm()) for c in outs]
    else:  # 4000 entries in extended precision
        i = torch.randint(m, (4000,), generator=g, device="cuda")
        j = torch.randint(n, (4000,), generator=g, device="cuda")
        want = np.concatenate([(A[p].cpu().numpy().astype(np.longdouble)
                                * B[:, q].t().cpu().numpy().astype(np.longdouble)).sum(1)
                               for p, q in zip(i.split(500), j.split(500))])
        err = [float(np.sqrt(((c[i, j].cpu().numpy() - want) ** 2).sum())) for c in outs]
    print("%s %s %s: %.3e against %.3e" % (which, dtype, compute, err[0], err[1]))
    assert err[0] <= 1.1 * err[1]
