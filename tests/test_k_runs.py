"""The contracted order padded to 16-byte runs (csrc/planner.cpp
``padded_k_runs``), checked on the host: every index counts exactly once."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_07311_amd", "csrc")


def test_padded_runs_count_every_index_once(tmp_path):
    exe = str(tmp_path / "krun")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-I" + CSRC,
                    "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "krun_driver.cpp"),
                    os.path.join(CSRC, "planner.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert int(r.stdout.split()[-1]) > 500
