"""Copies of results to the host by several threads (copies_to_host), on the CPU:
the code of csrc/host.hpp linked against a model of the HIP calls it makes
(tests/copies_host_check.cpp).  2^21 doubles take the threaded path."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    tmp = tmp_path_factory.mktemp("copies")
    obj, out = str(tmp / "check.o"), str(tmp / "check")
    subprocess.check_call([HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-O1", "-fPIC",
                           "-I", os.path.join(ROOT, "include"), "-c", "-o", obj,
                           os.path.join(ROOT, "tests", "copies_host_check.cpp")])
    subprocess.check_call(["g++", "-o", out, obj, "-lpthread"])
    return out


@pytest.mark.parametrize("case", ["small", "large", "per_thread_stream", "other_device", "pinned", "partly_pinned",
                                  "several_threads"])
def test_copies_arrive_whole_and_in_order(exe, case):
    for _ in range(5):
        r = subprocess.run([exe, case], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (case, r.returncode, r.stderr)
