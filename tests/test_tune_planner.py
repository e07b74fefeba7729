"""Tile-table entries that leave their size class to the planner (bk 0), and
the autotuner's use of them: a tuned handle is not slower than an untuned one
where the planner's route beats every tile."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PLAN = """
import sys, torch, paper_2604_07311_amd as fm
h = fm.famlies_create(0)
fm.famlies_load_tune_table(h, sys.argv[1])
p = fm.famlies_plan_contract(h, fm.FAMLIES_F64, 0, fm.make_desc([64, 64], [64, 1], "mk"),
                             fm.make_desc([64, 64], [1, 64], "kn"), fm.make_desc([64, 64], [64, 1], "mn"))
print(fm.famlies_plan_get_info(p)["tile_m"])
"""


@pytest.mark.gpu
def test_planner_entry_keeps_the_direct_kernel(tmp_path):
    for bk, direct in ((0, True), (8, False)):
        path = tmp_path / "t.txt"
        path.write_text("plain 1 0 6 6 6 64 64 %d 1\n" % bk)
        r = subprocess.run([sys.executable, "-c", PLAN, str(path)], cwd=ROOT, capture_output=True, text=True,
                           timeout=100, env=dict(os.environ, FAMLIES_LOG="1"))
        assert r.returncode == 0, r.stderr
        line = [ln for ln in r.stderr.splitlines() if "[famlies] plan" in ln][0]
        assert ("direct=" in line) == direct and ("tile table" in line) != direct, line


@pytest.mark.gpu
def test_tuner_leaves_small_products_to_the_planner(tmp_path):
    import paper_2604_07311_amd as fm
    h = fm.famlies_create(0)
    path = str(tmp_path / "t.txt")
    fm.famlies_tune(h, path, fm.FAMLIES_TUNE_QUICK | fm.FAMLIES_TUNE_PLAIN_ONLY)
    fm.famlies_destroy(h)
    rows = [ln.split() for ln in open(path) if ln.strip() and not ln.startswith("#")]
    # 64 x 64 x 1024: one direct launch takes no longer than tiles and their
    # reduction (FP64 8.1 against 9.2 us, FP32 7.5 against 7.4: a tie)
    small = [r for r in rows if r[3:6] == ["6", "6", "10"] and r[2] == "0"]
    assert len(small) == 2 and all(r[8] == "0" for r in small), small


def test_planner_entries_are_for_plain_classes(tmp_path):
    # loading into a handle needs a device: the reader by itself
    from tests.test_host_sanitize import CSRC, HOST_SOURCES
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                    os.path.join(ROOT, "tests", "sanitize", "driver.cpp")] +
                   [os.path.join(CSRC, s) for s in HOST_SOURCES] + ["-o", exe], check=True)
    for text, want in (("plain 1 0 6 6 6 64 64 0 1\n", "ok 1"), ("batch 1 0 6 6 6 64 64 0 1\n", "err"),
                       ("plain 1 0 6 6 6 0 64 0 1\n", "err"), ("plain 1 0 6 6 6 64 64 -8 1\n", "err")):
        path = tmp_path / "t.txt"
        path.write_text(text)
        r = subprocess.run([exe, "table", str(path)], capture_output=True, text=True, timeout=60)
        assert r.stdout.strip() == want, text
