"""The search of segment offsets that launches of few blocks run, compiled
and run on the CPU (its index arithmetic has no HIP dependency): no offset
outside the caller's array is read, also by a search that ends before the
other one it shares its rounds with."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_probe_is_inside_the_offsets(tmp_path):
    exe = str(tmp_path / "segment_search_test")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_1604_04815_amd", "csrc"),
                    os.path.join(ROOT, "tests", "segment_search_test.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all checks passed" in r.stdout
