"""Rows that a compressed root level does not store: where they go in the list made at creation and how long the gaps between
stored rows are, for lists that the default creation does not check (repeated, descending or outside the mode).  Runs on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_places_and_gaps_stay_inside_for_every_list(tmp_path):
    exe = str(tmp_path / "root_rows")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", os.path.join(ROOT, "tests", "sanitize", "root_rows_driver.cpp"), "-o", exe]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and " ok" in res.stdout, res.stdout + res.stderr
