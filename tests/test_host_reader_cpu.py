"""The reader of device arrays into host memory, on the CPU.

csrc/host_read.cpp is compiled against a few HIP calls written for the CPU (tests/fake_hip), with the
thread sanitizer, so that its threads, its bookkeeping and its use of the runtime can be checked
without a device.
"""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_09118_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    out = tmp_path_factory.mktemp("host_reader") / "check"
    fake = os.path.join(HERE, "fake_hip")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=thread", "-I", fake, "-I", CSRC,
           os.path.join(fake, "host_reader_check.cpp"), os.path.join(CSRC, "host_read.cpp"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def run(name):
        res = subprocess.run([str(out), name], capture_output=True, text=True, timeout=120,
                             env=dict(os.environ, TSAN_OPTIONS="halt_on_error=1"))
        assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr

    return run


@pytest.mark.parametrize("name", [
    "error_of_a_worker", "capture_mode", "slots_are_shared", "known_memory_makes_no_slots", "small_reads",
    "filled_by_the_kernel", "readers_at_once", "no_pinned_memory", "slots_of_a_failed_stream"])
def test_reader(check, name):
    check(name)
