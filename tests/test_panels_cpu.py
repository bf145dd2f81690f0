"""How the rows of a matrix are cut into panels, without a GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_xcd_gets_the_same_share_of_the_rows(tmp_path):
    exe = str(tmp_path / "panels_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2004_13940_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host_stub", "panels_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "", f"exit {r.returncode}\n{r.stdout}"
