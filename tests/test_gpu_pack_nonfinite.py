"""Infinities beside a pre-packed operand: in the contracted order padded to
16-byte runs some entries repeat an element and do not count, and the operand
that is gathered next to a packed one must hold 0 there too (0 * Inf is NaN).
Packed results against the gathered ones and against NumPy."""
import numpy as np
import pytest

from tests.famlies_testutil import DeviceRunner, round_inputs
from tests.test_gpu_k_runs import _plan, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    return DeviceRunner()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bm", [64, 128])
@pytest.mark.parametrize("packed", [0, 1])
@pytest.mark.parametrize("partner", ["rows", "k"])
def test_inf_beside_packed_runs(gpu, tmp_path, dtype, bm, packed, partner):
    """The packed operand has unit stride along k; its partner is gathered by
    rows, or along its contracted modes with q the fastest (by elements)."""
    import torch
    fm = gpu.fm
    orders = [["mkq", "qkm"], ["nkq", "qkn"]]
    own = ["kmq", "knq"][packed]
    other = orders[1 - packed][partner == "k"]
    a, b = (own, other) if packed == 0 else (other, own)
    p = round_inputs(_problem({"m": 150, "n": 170, "k": 13, "q": 3}, (a, b, "nm"), seed=3, beta=0.0), dtype)
    A, B = (np.lib.stride_tricks.as_strided(buf[t.base:], t.extents, [8 * s for s in t.strides])
            for buf, t in ((p.abuf, p.a), (p.bbuf, p.b)))
    T = B if packed == 0 else A  # (k, n, q) or (m, k, q): infinities in the partner only
    for i, k in enumerate((9, 10, 11, 12, 8)):
        T[(k, 5 + i, i % 3) if packed == 0 else (5 + i, k, i % 3)] = np.inf
    with np.errstate(invalid="ignore"):
        want = sum(A[:, k, q][:, None] * B[k, :, q][None, :] for k in range(13) for q in range(3))
    assert np.isinf(want).any() and not np.isnan(want).any()
    h, plan = _plan(gpu, tmp_path, p, dtype, "native", bm, 1)
    try:
        gathered = gpu.run(p, dtype, plan=plan, alpha=1.0, beta=0.0)
        es, s = (8 if dtype == "f64" else 4), torch.cuda.current_stream().cuda_stream
        ta, tb, tc = (gpu.to_dev(x, dtype) for x in (p.abuf, p.bbuf, p.cbuf))
        ptr = [ta.data_ptr() + es * p.a.base, tb.data_ptr() + es * p.b.base]
        buf = torch.empty(fm.famlies_pack_size(plan, packed) // 4 + 4, dtype=torch.int32, device="cuda")
        fm.famlies_pack(plan, packed, ptr[packed], buf.data_ptr(), s)
        ptr[packed] = buf.data_ptr()
        fm.famlies_execute_packed(plan, 1.0, ptr[0], ptr[1], 0.0, tc.data_ptr() + es * p.c.base, 1 << packed, s)
        torch.cuda.synchronize()
        got = tc.cpu().numpy().astype(np.float64)
    finally:
        fm.famlies_plan_destroy(plan)
        fm.famlies_destroy(h)
    np.testing.assert_array_equal(got, gathered)
    C = np.lib.stride_tricks.as_strided(got[p.c.base:], p.c.extents, [8 * s for s in p.c.strides])
    np.testing.assert_array_equal(np.isnan(C), np.zeros_like(want, dtype=bool))
    np.testing.assert_array_equal(np.where(np.isinf(want), C, 0.0), np.where(np.isinf(want), want, 0.0))
