"""Split launch lists (plan.cpp, split_units) on random problems, built with g++
(tests/split_units.cpp).  No GPU code is built or run."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_34318_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_units_cover_each_items_tiles_once(tmp_path):
    exe = tmp_path / "split_units"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}",
                        os.path.join(ROOT, "tests", "split_units.cpp"), os.path.join(CSRC, "plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    counts = r.stdout.split()
    assert int(counts[1]) > 100 and int(counts[3]) > 100, r.stdout
