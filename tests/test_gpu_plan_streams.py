"""One plan on two streams at once, each with its own operands and outputs,
where the tile choice splits nothing along K but the plan's route has a
workspace (levelled rounds, part planes): every result is that of the same
plan run alone on that data, on either route's rounding bound."""
import pytest

from tests.famlies_testutil import U32, U64, bf16x3_bound, gamma

pytestmark = pytest.mark.gpu

# (m, n, k, batch), dtype, compute: unsplit, with a part of a round
CASES = [((1150, 1150, 3000, 4), "f64", "native"), ((1150, 1150, 3000, 4), "f32", "native"),
         ((4096, 4160, 1024, 1), "f32", "bf16x3"), ((4096, 4160, 1024, 1), "f32", "bf16x6")]


def _setup(size, dtype, compute):
    import torch
    import paper_2604_07311_amd as fm
    m, n, k, L = size
    dt = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=dt) * 2 - 1
    descs = (fm.make_desc((k, m, L), (1, k, k * m), "kmL"), fm.make_desc((k, n, L), (1, k, k * n), "knL"),
             fm.make_desc((n, m, L), (1, n, n * m), "nmL"))
    plan = fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F64 if dtype == "f64" else fm.FAMLIES_F32,
                                    fm._compute_code(compute), *descs)
    assert fm.famlies_plan_get_info(plan)["split_k"] == 1
    data = [(rnd(L, m, k), rnd(L, n, k), torch.zeros(L, m, n, device="cuda", dtype=dt)) for _ in range(2)]
    return fm, torch, plan, data


def _check(size, dtype, compute, data):
    import torch
    k = size[2]
    for a, b, c in data:
        for i in range(size[3]):
            want, d = (torch.mm(x, y.t()) for x, y in ((a[i].double(), b[i].double()),
                                                       (a[i].double().abs(), b[i].double().abs())))
            bound = gamma(k + 4, U64 if dtype == "f64" else U32) * d
            if compute == "bf16x3":
                bound = bf16x3_bound(k, d, d)
            elif compute == "bf16x6":
                bound = (2.0 ** -22 + gamma(3 * k, 2.0 ** -23) * (1 + 2.0 ** -7)) * d + 2.0 ** -23 * d
            assert bool(((c[i].double() - want).abs() <= bound + gamma(k + 2, U64) * d).all())


@pytest.mark.parametrize("size,dtype,compute", CASES)
def test_two_streams(size, dtype, compute):
    fm, torch, plan, data = _setup(size, dtype, compute)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(6):
        for (a, b, c), s in zip(data, streams):
            fm.famlies_execute(plan, 1.0, a.data_ptr(), b.data_ptr(), 0.0, c.data_ptr(), s.cuda_stream)
    torch.cuda.synchronize()
    _check(size, dtype, compute, data)
    fm.famlies_plan_destroy(plan)


def test_captured_and_eager():
    """A graph launched beside eager calls of the same plan on another stream."""
    size, dtype, compute = CASES[3]
    fm, torch, plan, data = _setup(size, dtype, compute)
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    run = lambda i, st: fm.famlies_execute(plan, 1.0, data[i][0].data_ptr(), data[i][1].data_ptr(), 0.0,
                                           data[i][2].data_ptr(), st.cuda_stream)
    run(0, s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        run(0, s)
    torch.cuda.synchronize()
    for _ in range(3):
        data[0][2].zero_()
        data[1][2].zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(t):
            g.replay()
        run(1, s)
        torch.cuda.synchronize()
        _check(size, dtype, compute, data)
    fm.famlies_plan_destroy(plan)


@pytest.mark.parametrize("packed", [1, 2, 3])
def test_packed_planes_on_two_streams(packed):
    size, dtype, compute = CASES[3]
    fm, torch, plan, data = _setup(size, dtype, compute)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    calls = []
    for a, b, c in data:
        ptr = [a.data_ptr(), b.data_ptr()]
        keep = []
        for op in (0, 1):
            if packed >> op & 1:
                keep.append(torch.empty(fm.famlies_pack_size(plan, op) // 4 + 4, dtype=torch.int32, device="cuda"))
                fm.famlies_pack(plan, op, ptr[op], keep[-1].data_ptr(), torch.cuda.current_stream().cuda_stream)
                ptr[op] = keep[-1].data_ptr()
        calls.append((ptr, c, keep))
    torch.cuda.synchronize()
    for _ in range(4):
        for (ptr, c, _), s in zip(calls, streams):
            fm.famlies_execute_packed(plan, 1.0, ptr[0], ptr[1], 0.0, c.data_ptr(), packed, s.cuda_stream)
    torch.cuda.synchronize()
    _check(size, dtype, compute, data)
    fm.famlies_plan_destroy(plan)
