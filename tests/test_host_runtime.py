"""The runtime's host side where several streams, processes, contexts or threads meet.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_08490_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")


def _compile(tmp_path, name, sources=("api.cpp", "host_build.cpp", "sampler.cpp")):
    """tests/sanitize/<name>.cpp with the host runtime and the launcher stand-ins, without device code."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / name)
    srcs = [os.path.join(CSRC, f) for f in sources] + [os.path.join(SAN, f) for f in ("launch_stubs.cpp", name + ".cpp")]
    cmd = [gxx, "-std=c++20", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, "-w", "-o", exe] + srcs + \
          ["-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib", "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return exe


def test_every_call_waits_for_an_upload_that_is_not_known_to_have_finished(tmp_path):
    """Two calls with one stream handle while the upload is under way: both wait (the handle of the per-thread stream, or of
    a stream made where another one was destroyed, is another stream the second time).  Once the upload has finished
    none waits, whatever the handle."""
    run = subprocess.run([_compile(tmp_path, "upload_wait")], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "upload wait ok" in run.stdout, run.stdout + run.stderr
