"""The ring of plan buffers (plan_ring.h, no HIP): a slot is handed out again only after its call
has reported, waiting for one leaves the library's lock free, and calls that a device error
ended are not waited for for ever.  Built with the address and undefined-behaviour sanitizers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_17357_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("ring") / "plan_ring")
    subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, os.path.join(ROOT, "tests", "native", "plan_ring_main.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("case", ["order", "lock_is_free", "ended_calls", "failed_stream"])
def test_ring(program, case):
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)  # the sanitizer runtime must come first in the library list
    r = subprocess.run([program, case], capture_output=True, text=True, env=env, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_no_call_synchronises_the_device():
    """What include/cronus.h promises; a device-wide wait also breaks the capture of any other stream."""
    for name in os.listdir(CSRC):
        assert "hipDeviceSynchronize(" not in open(os.path.join(CSRC, name)).read(), name
