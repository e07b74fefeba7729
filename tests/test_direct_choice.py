"""Which kernel the planner takes for small and narrow problems, from the dry
run's log: strided operands, and tall against wide problems."""
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def routes(problems):
    """(tile, waves, split) of the direct kernel, or None, per problem (dtype
    code, A and B each as (extents, strides), C's strides)."""
    code = ("import sys, json, paper_2604_07311_amd as fm\n"
            "for dt, a, b, c in json.loads(sys.argv[1]):\n"
            "    fm.famlies_analyze(dt, 0, fm.make_desc(*a, 'mk'), fm.make_desc(*b, 'kn'),\n"
            "                       fm.make_desc((a[0][0], b[0][1]), c, 'mn'))\n")
    import json
    r = subprocess.run([sys.executable, "-c", code, json.dumps(problems)], cwd=ROOT, capture_output=True, text=True,
                       timeout=300, env=dict(os.environ, FAMLIES_LOG="1"))
    lines = [ln for ln in r.stderr.splitlines() if "analyze" in ln]
    assert len(lines) == len(problems), r.stderr
    got = [re.search(r"direct=(\d+)x(\d+)/(\d+) waves/split (\d+)", ln) for ln in lines]
    return [tuple(map(int, g.groups())) if g else None for g in got]


def _strided(dt, m, n, k):
    """No unit stride in A or B along k, rows of B's columns two elements apart."""
    return [dt, [[m, k], [2 * k, 2]], [[k, n], [2, 2 * k]], [n, 1]]


def test_strided_operands_do_not_take_large_direct_tiles():
    """Loads that touch a line per lane: 32 x 32 wave tiles took 17.7 us where
    the tiled kernel takes 11.1 (FP32) and 12.4 against 11.7 (FP64)."""
    for r in routes([_strided(2, 300, 300, 300), _strided(1, 300, 300, 300)]):
        assert r is None or r[:2] == (16, 16), r
    # a small one keeps the direct kernel
    assert all(routes([_strided(1, 24, 24, 200)]))


def test_long_sides_are_walked_in_long_segments():
    """64 x 16 wave tiles where the kernel's M is the long side, 16 x 64 where N
    is (or 32 x 32), so that memory is touched in segments of 64 elements."""
    for dt in (1, 2):
        for big, k in ((500000, 64), (799223, 64)):
            tall = [dt, [[big, k], [1, big]], [[k, 14], [1, k]], [14, 1]]
            wide = [dt, [[14, k], [k, 1]], [[k, big], [big, 1]], [big, 1]]
            t, w = routes([tall, wide])
            assert t and t[:2] in ((64, 16), (32, 32)), (dt, big, k, t)
            assert w and w[:2] in ((16, 64), (32, 32)), (dt, big, k, w)


def test_rows_whole_lines_apart_on_unevenly_filled_units():
    """FP64 rows whole cache lines apart: one and a half direct workgroups per
    CU took 30 us at 6000 x 64 x 800 where the tiles take 23, 17 against 14 at 458
    x 150 x 832.  Rows off the lines, or full rounds, keep the direct kernel."""
    def kk(m, n, k):
        return [1, [[m, k], [k, 1]], [[k, n], [1, k]], [n, 1]]
    assert routes([kk(6000, 64, 800), kk(64, 6000, 800), kk(458, 150, 832)]) == [None] * 3
    assert all(routes([kk(100, 4000, 700), kk(4000, 64, 1024), kk(2000, 100, 800)]))
