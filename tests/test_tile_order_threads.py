"""The tile order of the interpolation's lists (csrc/lists.h) over worker
threads: no allocation off the calling thread, the same order for any number
of threads."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tile_order_threads(tmp_path):
    exe = str(tmp_path / "list_alloc_harness")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I", os.path.join(ROOT, "paper_1311_4120_amd", "csrc"),
                        os.path.join(ROOT, "tests", "sanitize", "list_alloc_harness.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stderr[-4000:])
