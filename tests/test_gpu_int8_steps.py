"""FP64 on INT8 over the step counts of its GEMM's K loop (three buffers, six
steps a turn): small integers, whose digits and sums are exact, so every entry
must equal the integer product."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [3, 4, 5, 6, 7])
@pytest.mark.parametrize("n", [50, 200])
def test_every_step_count(s, n):
    import torch
    import paper_2604_07311_amd as fm
    rng = np.random.default_rng(s)
    for k in (1, 33, 64, 100, 128, 192, 200, 256, 320, 384, 448, 512, 700, 1500):
        a, b = rng.integers(-60, 61, (70, k)), rng.integers(-60, 61, (k, n))
        A, B = (torch.from_numpy(x.astype(np.float64)).cuda() for x in (a, b))
        C = fm.contract(1.0, A, "mk", B, "kn", 0.0, None, "mn", compute="int8x%d" % s)
        np.testing.assert_array_equal(C.cpu().numpy(), (a @ b).astype(np.float64), err_msg="k=%d" % k)
