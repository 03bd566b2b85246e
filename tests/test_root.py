"""The outlier rejection's square root and quotient (root.hpp) on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_root_host_build(tmp_path):
    exe = tmp_path / "root_test"
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I",
                        os.path.join(ROOT, "paper_1808_06194_amd", "csrc"),
                        os.path.join(ROOT, "tests", "cpp", "root_test.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
