"""The upload ring's host code, compiled against a stub of the runtime calls it makes."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "host_stub")
CSRC = os.path.join(ROOT, "paper_2004_13940_amd", "csrc")


def test_uploads_stay_on_the_stream_of_the_caller(tmp_path):
    """The stub does a stream's work as late as it may, and its hipStreamPerThread is another stream in every thread: copies
    that a helper thread enqueues are not ordered before what the caller does next, blocks refilled too early show."""
    exe = str(tmp_path / "upload_check")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", STUB, "-I", CSRC, os.path.join(STUB, "upload_check.cpp"),
           "-x", "c++", os.path.join(CSRC, "fm_upload.hip"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "", f"exit {r.returncode}\n{r.stdout}"
