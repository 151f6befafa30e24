"""What the library's host code asks of the HIP runtime, seen through a stand-in for it that runs on the CPU (hip_stub): what is
cleared, waited for, allocated and launched."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-shared", "-fPIC", "-Wall", "-Werror",
                    os.path.join(ROOT, "tests", "hip_stub", "hip_stub.c"), "-o", lib], check=True)
    return lib


def run(stub, code, timeout=120):
    """`code` in a process of its own, with J (the binding), `stub` and log(): the calls made since the last one."""
    head = f"""
import ctypes, sys, time
sys.path.insert(0, {ROOT!r})
stub = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
stub.stub_log.restype = ctypes.c_char_p
stub.stub_malloc_limit.argtypes = [ctypes.c_size_t]
import paper_2210_01238_amd as J
assert "torch" not in sys.modules                    # whose own HIP calls would come to the stand-in, too
def log():
    text = stub.stub_log().decode().splitlines()
    stub.stub_clear_log()
    return [line.split() for line in text]
GRIDS = lambda p: (1 << 20, (1 << 20) + J.jacobi_grid_bytes(p))        # addresses that nothing touches
"""
    r = subprocess.run([sys.executable, "-c", head + code], capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_set_up_waits_for_the_clearing_of_its_scratch(stub):
    """hipMemset goes to the default stream, which streams created as non-blocking do not wait for: the first launch on one
    must not meet words and messages that are cleared under it."""
    run(stub, """
for dims in ((256, 256), (1024, 1024), (64, 64, 64), (4096, 4096)):
    p = J.jacobi_create(dims, (1,) * len(dims), J.JACOBI_F64)
    log()
    J.jacobi_prepare(p)
    calls = [c[0] for c in log()]
    assert "hipMemset" in calls, calls
    after = calls[calls.index("hipMemset"):]
    assert "hipStreamSynchronize" in after or "hipDeviceSynchronize" in after, calls
    J.jacobi_destroy(p)
""")
