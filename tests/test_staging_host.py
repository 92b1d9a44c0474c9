"""Staged downloads (staging.h) on the host alone, against stand-ins for the HIP
calls they make (staging_host.cpp): the rows arrive, and the threads that ask
for copies are only those that may.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    out = tmp_path_factory.mktemp("staging") / "staging_host"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-pthread",
                    os.path.join(HERE, "staging_host.cpp"), "-o", str(out)], check=True)
    return str(out)


@pytest.mark.parametrize("case", [
    "pageable",             # chunks by several threads
    "per_thread_stream",    # the handle means the caller's stream in the caller's thread only
    "no_host_memory",       # threads that cannot be made: the caller does the work
    "pinned",               # a destination the copy engine writes in place: one copy a row
])
def test_staged_download(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, f"{r.returncode}: {r.stdout}{r.stderr}"
