"""bf16x3 with both operands gathered by elements along K (no unit stride):
part planes are weighed against the 256 x 128 tile that such plans split
while staging in, and taken where each element meets enough tiles."""
import os
import re
import subprocess
import sys

import pytest

from tests.famlies_testutil import U64, bf16x3_bound, gamma

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SIZES = [(4096, 4096, 4096), (3001, 2999, 3003), (1024, 1024, 64)]  # the last is too small


def _descs(fm, m, n, k):
    return (fm.make_desc((m, k), (2 * k, 2), "mk"), fm.make_desc((k, n), (2, 2 * k), "kn"),
            fm.make_desc((m, n), (n, 1), "mn"))


def test_planes_replace_the_tall_tile():
    code = ("import paper_2604_07311_amd as fm\n"
            "from tests.test_tall_planes import SIZES, _descs\n"
            "for s in SIZES:\n"
            "    fm.famlies_analyze(fm.FAMLIES_F32, fm.FAMLIES_BF16X3, *_descs(fm, *s))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, FAMLIES_LOG="1"))
    lines = [ln for ln in r.stderr.splitlines() if "analyze" in ln]
    assert [bool(re.search("planes", ln)) for ln in lines] == [True, True, False], r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("size", SIZES)
def test_tall_planes_match_fp64(size):
    import torch
    import paper_2604_07311_amd as fm
    m, n, k = size
    g = torch.Generator(device="cuda").manual_seed(29)
    a = torch.rand(m, 2 * k, generator=g, device="cuda") * 2 - 1
    b = torch.rand(n, 2 * k, generator=g, device="cuda") * 2 - 1
    c = torch.empty(m, n, device="cuda")
    A, B = a[:, ::2], b[:, ::2].t()
    fm.contract(1.0, A, "mk", B, "kn", 0.0, c, "mn", compute="bf16x3")
    want, d = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    assert bool(((c.double() - want).abs() <= bf16x3_bound(k, d, d) + gamma(k + 2, U64) * d).all())
