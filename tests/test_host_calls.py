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
stub.stub_live.restype = stub.stub_misuses.restype = ctypes.c_long
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


def test_first_launch_comes_after_the_clearing_of_the_scratch(stub):
    """hipMemset goes to the default stream, which streams created as non-blocking do not wait for: the first launch on one
    must not meet words and messages that are cleared under it.  Set-up waits for it where resident2d_kernel may run; block
    launches wait for an event recorded behind it; who uses neither has nothing cleared and waits for nothing."""
    run(stub, """
for dims, narrow, blocks in (((256, 256), 1, 1), ((256, 60), 1, 0), ((1024, 1024), 0, 1), ((64, 64, 64), 0, 1), ((4096, 4096), 0, 0), ((256, 256, 256), 0, 0)):
    p = J.jacobi_create(dims, (1,) * len(dims), J.JACOBI_F64)
    log()
    J.jacobi_prepare(p)
    calls = log()
    names = [c[0] for c in calls]
    assert (J.jacobi_get_option(p, "block_workgroups") > 0) == bool(blocks)
    assert ("hipMemset" in names) == bool(narrow or blocks), calls
    assert ("hipStreamSynchronize" in names) == bool(narrow), calls
    if narrow:
        assert names.index("hipStreamSynchronize") > names.index("hipMemset"), calls
    if blocks and not narrow:
        assert ["hipEventRecord", "(nil)"] in calls[names.index("hipMemset"):], calls
        J.jacobi_sweep(p, *GRIDS(p), 100, 1 << 12)
        names = [c[0] for c in log()]
        assert names.count("hipLaunchKernel") == 1 and "hipStreamWaitEvent" in names[:names.index("hipLaunchKernel")], names
    J.jacobi_destroy(p)
""")


def test_without_room_for_the_messages_a_plan_runs_by_launches(stub):
    """The block kernels' messages are an extra: where the device has room for the partial sums only, the plan is set up and runs
    launch by launch as without them; without room for those it is out of memory."""
    run(stub, """
for dims, tiles in (((1024, 1024), (4, 4)), ((64, 64, 64), (2, 2, 2))):
    p = J.jacobi_create(dims, tiles, J.JACOBI_F64)
    whole = J.jacobi_scratch_bytes(p)
    stub.stub_malloc_limit(whole - 1)
    J.jacobi_prepare(p)
    sizes = [int(c[1]) for c in log() if c[0] == "hipMalloc"]
    assert sizes[0] == whole and sizes[-1] < 1 << 20, sizes
    assert J.jacobi_scratch_bytes(p) == sizes[-1]
    a, b = GRIDS(p)
    J.jacobi_sweep(p, a, b, 50)
    assert sum(c[0] == "hipLaunchKernel" for c in log()) >= 50
    J.jacobi_destroy(p)
    p = J.jacobi_create(dims, tiles, J.JACOBI_F64)
    J.jacobi_run(p, a, b, 50, 25, 1 << 16)           # which sets the plan up itself
    assert sum(c[0] == "hipLaunchKernel" for c in log()) >= 50
    J.jacobi_destroy(p)
    p = J.jacobi_create(dims, tiles, J.JACOBI_F64)
    stub.stub_malloc_limit(1000)
    try:
        J.jacobi_prepare(p)
        raise SystemExit("prepared without memory")
    except J.JacobiError as e:
        assert e.code == J.binding.JACOBI_ENOMEM
    stub.stub_malloc_limit(1 << 40)
    J.jacobi_prepare(p)                              # and again, with room: in blocks after all
    log()
    J.jacobi_sweep(p, a, b, 50)
    assert sum(c[0] == "hipLaunchKernel" for c in log()) == 1
    J.jacobi_destroy(p)
""")


def test_scatter_of_very_many_tiles_stays_within_what_one_launch_takes(stub):
    """A launch of 2^32 threads and more is refused by the runtime; a workgroup per one-row tile gets there with 2^24 tiles."""
    run(stub, """
n = (1 << 24) + 300
for tiles, dtype in ((n, J.JACOBI_F64), (1000, J.JACOBI_F32)):
    p = J.jacobi_create((tiles, 3), (tiles, 1), dtype)
    J.jacobi_prepare(p)
    log()
    J.jacobi_scatter(p, 1 << 20, 1 << 20)
    launches = [(int(c[1]), int(c[2])) for c in log() if c[0] == "hipLaunchKernel"]
    assert sum(g for g, b in launches) == tiles, launches
    assert all(g * b < 1 << 32 for g, b in launches), launches
    J.jacobi_destroy(p)
""")


def test_gather_of_very_large_grids_stays_within_what_one_launch_takes(stub):
    """A wavefront takes 1 to 4 KiB of a row, so that 2^32 threads are reached by fp64 fields of 64 GiB with long rows, and by 2^26 short rows.  Every
    wavefront is launched once: the launches cover what the rows need, and no workgroup more than the last one's rest."""
    run(stub, """
def waves(dims, dtype):
    size, line = (8, 16) if dtype == J.JACOBI_F64 else (4, 32)
    vecs = -(-(dims[-1] + 2 + line - 1) * size // 16)
    rows = 1
    for n in dims[:-1]: rows *= n + 2
    grid = J.jacobi_grid_bytes(p)
    q = 1 if size == 8 and grid > 124 << 20 and vecs >= 16 * 64 else min(4, -(-vecs // 64))
    return rows * -(-vecs // (64 * q))
for dims, tiles, dtype, pieces in (((93000, 93000), (8, 8), J.JACOBI_F64, 2), ((2100, 2080, 2080), (10, 10, 10), J.JACOBI_F64, 2), ((67108900, 3), (100, 1), J.JACOBI_F64, 2),
                                   ((140000000, 2), (1000, 1), J.JACOBI_F32, 3), ((92000, 92000), (8, 8), J.JACOBI_F64, 1), ((1000, 300), (2, 2), J.JACOBI_F32, 1)):
    p = J.jacobi_create(dims, tiles, dtype)
    J.jacobi_prepare(p)
    log()
    J.jacobi_gather(p, 1 << 20, 1 << 20)
    launches = [(int(c[1]), int(c[2])) for c in log() if c[0] == "hipLaunchKernel"]
    assert all(g * b < 1 << 32 for g, b in launches), (dims, launches)
    assert len(launches) == pieces and sum(g for g, b in launches) == -(-waves(dims, dtype) // 4), (dims, launches, waves(dims, dtype))
    J.jacobi_destroy(p)
""")


PLANS = [((96, 200), (3, 2)), ((48, 48), (48, 48)), ((512, 512), (4, 4)), ((24, 20, 36), (2, 2, 3)), ((8, 8, 8), (8, 8, 8)), ((256, 256), (1, 1)),
         ((2304, 2304), (8, 8)), ((64, 64, 64), (2, 2, 2))]


def test_streams_events_and_memory_live_as_long_as_their_plan(stub):
    """Every stream, event and block of memory that a plan's calls make is destroyed exactly once, by jacobi_destroy, after it has waited for the
    device; nothing is used before it is made or after it is gone.  Plans that run tasks over their own streams, with task sizes and numbers
    of streams that change from call to call, in blocks with and without ghost cells, with profiling, and plans that never run."""
    run(stub, f"""
for dims, tiles in {PLANS!r}:
    for dtype in (J.JACOBI_F64, J.JACOBI_F32):
        for profile in (0, 1):
            p = J.jacobi_create(dims, tiles, dtype)
            J.jacobi_set_option(p, "profile", profile)
            J.jacobi_scatter(p, 1 << 40, 1 << 20)
            for iters, group, streams in ((7, 1, 4), (3, 1, 4), (8, 2, 3), (5, 100, 1), (6, 37, 16), (4, 1, 2)):
                J.jacobi_sweep_tasks(p, *GRIDS(p), iters, group, streams, 1 << 40)
            J.jacobi_run(p, *GRIDS(p), 60, 20, 1 << 16, 1 << 40)
            J.jacobi_sweep(p, *GRIDS(p), 60)
            if profile:
                J.jacobi_profile_read(p)
            log()
            J.jacobi_destroy(p)
            names = [c[0] for c in log()]
            assert names[0] == "hipDeviceSynchronize" and names.count("hipFree") == 1, names[:5]
            assert [stub.stub_live(k) for k in (0, 1, 2)] == [0, 0, 0] and stub.stub_misuses() == 0, (dims, dtype)
    p = J.jacobi_create(dims, tiles, J.JACOBI_F64)
    J.jacobi_prepare(p)
    J.jacobi_destroy(p)
    p = J.jacobi_create(dims, tiles, J.JACOBI_F64)
    J.jacobi_destroy(p)
    assert [stub.stub_live(k) for k in (0, 1, 2)] == [0, 0, 0] and stub.stub_misuses() == 0, dims
""")


def test_destroying_a_plan_reports_what_failed(stub):
    """The rest is destroyed all the same."""
    run(stub, """
for call in ("hipFree", "hipEventDestroy", "hipStreamDestroy"):
    p = J.jacobi_create((512, 512), (4, 4), J.JACOBI_F64)
    J.jacobi_sweep_tasks(p, *GRIDS(p), 3, 3, 5)
    stub.stub_fail(call.encode())
    try:
        J.jacobi_destroy(p)
        raise SystemExit(call + " failed unnoticed")
    except J.JacobiError as e:
        assert e.code == J.binding.JACOBI_EHIP and call in str(e), e
    assert [stub.stub_live(k) for k in (0, 1, 2)] == [0, 0, 0]
""")
