"""The built library on a stub of the runtime, without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "host_stub")
PACKAGE = os.path.join(ROOT, "paper_2004_13940_amd")


@pytest.mark.parametrize("check", [
    # with every call that can fail failing in turn: nothing that is half built is taken for whole, nothing stays allocated, and
    # the same call succeeds afterwards with all of its launches
    "build_check",
    # stratified epochs are captured once per set of arguments where that is asked for, and replayed
    "graph_check",
])
def test_library_on_a_stub_of_the_runtime(tmp_path, check):
    if not os.path.exists(os.path.join(PACKAGE, "libfm_mi355x.so")):
        from paper_2004_13940_amd import build
        build.build()
    exe = str(tmp_path / check)
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"),
           os.path.join(STUB, check + ".cpp"), "-o", exe, os.path.join(PACKAGE, "libfm_mi355x.so"), f"-Wl,-rpath,{PACKAGE}",
           "-Wl,--allow-shlib-undefined"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "", f"exit {r.returncode}\n{r.stdout}\n{r.stderr}"
