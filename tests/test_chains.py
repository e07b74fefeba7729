"""No kernel or round that a plan takes instead of its tile choice's K ranges
adds more contracted entries into one accumulator than they do (the error of a
sum over K grows with that chain).  Read from the dry run's log."""
import os
import re
import subprocess
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MODES = [("f64", "native"), ("f32", "native"), ("f32", "bf16x3"), ("f32", "bf16x6")]


def problems():
    """Plain products (k in whole 16-byte runs, gathered along k or by rows)
    from a few tiles to several rounds of them."""
    rng = np.random.default_rng(41)
    out = []
    for _ in range(60):
        m, n = (int(2 ** rng.uniform(3, 12.3)) for _ in range(2))
        k = 32 * int(2 ** rng.uniform(0, 9))
        out.append((m, n, k, int(rng.integers(4))))
    return out + [(2376, 2376, 2368, 0), (3680, 3680, 3680, 1), (484, 12544, 12544, 2), (1024, 1024, 50016, 0)]


def _log():
    code = ("import paper_2604_07311_amd as fm\n"
            "from tests.test_chains import MODES, problems\n"
            "for d, c in MODES:\n"
            "    for m, n, k, o in problems():\n"
            "        info, _ = fm.famlies_analyze(\n"
            "            fm.FAMLIES_F64 if d == 'f64' else fm.FAMLIES_F32, fm._compute_code(c),\n"
            "            fm.make_desc([m, k], [k, 1] if o & 1 else [1, m], 'mk'),\n"
            "            fm.make_desc([k, n], [1, k] if o & 2 else [n, 1], 'kn'), fm.make_desc([m, n], [n, 1], 'mn'))\n"
            "        print(d, c, info['m'], info['n'], info['k'], info['tile_m'], info['tile_n'], info['tile_k'],\n"
            "              info['split_k'], info['split_tiles'])\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, FAMLIES_LOG="1"))
    assert r.returncode == 0, r.stderr
    lines = [ln for ln in r.stderr.splitlines() if "analyze" in ln]
    return list(zip((ln.split() for ln in r.stdout.splitlines()), lines))


def up(a, b):
    return -(-a // b)


def test_chains_are_no_longer_than_the_tile_choices():
    seen = {"direct": 0, "level": 0, "planes": 0}
    for (dtype, compute, *nums), line in _log():
        m, n, k, tm, tn, bk, split, cut = map(int, nums)
        if split == 1:
            continue  # one chain over all of K
        chunk = up(up(k, split), bk) * bk
        cut = cut or up(m, tm) * up(n, tn)
        direct = re.search(r"direct=\d+x\d+/(\d+) waves/split (\d+)(?:/chains (\d+))?", line)
        level = re.search(r"level=(\d+) whole, (\d+) x (\d+) \+ (\d+) x (\d+) slices", line)
        planes = re.search(r"planes 256x128(?: fold=(\d+) steps)?", line)
        if direct:
            wk, ds, chains = (int(x or 1) for x in direct.groups())
            ks = 8 if dtype == "f64" else 16
            of_wave = up(up(up(k, ds), ks), wk)
            assert min(up(of_wave, chains) * ks, k) <= chunk, line
            seen["direct"] += 1
        elif compute == "bf16x3" and k <= 12544:
            continue  # the dropped low products' error is ten times that of one chain
        elif planes:
            assert planes.group(1) and 0 < 32 * int(planes.group(1)) <= chunk, line
            seen["planes"] += 1
        elif level:
            _, rem, q, _, part = map(int, level.groups())
            assert rem >= cut and max(q, part) * bk <= chunk, line
            seen["level"] += 1
    assert min(seen.values()) >= 1, seen
