"""Which large 2-D grids run whole on the chip (chip2d_kernel), and as what: planned on the CPU, with a stand-in for the HIP runtime
(hip_stub) that counts launches; and the waits in the generated code, as for the other block kernels."""
import os
import re
import subprocess

import pytest

import test_device_waits as waits
from test_block_plans import text
from test_chip2d_gpu import EVERY, ITERS, PLAIN, VARIANTS
from test_host_calls import ROOT, run, stub  # noqa: F401  (stub: a fixture)

HEAD = """
from numpy import float64, float32
def plan(dims, tiles, dtype):
    return J.jacobi_create(dims, tiles, J.JACOBI_F64 if dtype is float64 else J.JACOBI_F32)
def figures(p, *names):
    return tuple(J.jacobi_get_option(p, "chip_" + n) for n in names)
def launches(p, iters, every):
    J.jacobi_prepare(p)
    J.jacobi_sweep(p, *GRIDS(p), 50)                     # the first one also clears the plan's words
    log()
    J.jacobi_run(p, *GRIDS(p), iters, every, 1 << 16) if every else J.jacobi_sweep(p, *GRIDS(p), iters)
    return sum(c[0] == "hipLaunchKernel" for c in log())
"""


def test_every_compiled_variant_is_reached(stub):  # noqa: F811
    run(stub, HEAD + f"""
for want, cases in {text(VARIANTS)}.items():
    for dims, tiles, dtype in cases:
        p = plan(dims, tiles, dtype)
        assert figures(p, "rows_in_registers", "even") == want and launches(p, {ITERS}, {EVERY}) == 1, (dims, dtype, want)
        assert J.jacobi_get_option(p, "block_workgroups") == 0
        J.jacobi_destroy(p)
for dims, tiles, dtype in {text(PLAIN)}:
    p = plan(dims, tiles, dtype)
    assert launches(p, 9, 3) == launches(p, 8, 0) == 1, (dims, dtype)
    J.jacobi_destroy(p)
""")
    with open(os.path.join(ROOT, "paper_2210_01238_amd", "csrc", "launchers.h")) as f:
        rows = {int(n) for n in re.findall(r"X\((\d+),", re.search(r"#define JK_CHIP2D_VARIANTS\(X\)(.*)", f.read()).group(1))}
    compiled = {((n, even), t) for n in rows for even in (0, 1) for t in ("float64", "float32")} - {((8, 1), "float64")}
    assert compiled == {(v, c[2].__name__) for v, cases in VARIANTS.items() for c in cases}


def test_cuts_cover_the_grid(stub):  # noqa: F811
    """Blocks of lanes x cells by wavefronts x rows, as few as cover the grid, at most one per CU; larger grids, narrow ones and those
    the other block kernel takes have none."""
    run(stub, HEAD + """
import random
rng = random.Random(7)
seen = 0
for _ in range(3000):
    dtype = rng.choice((float64, float32))
    ny, nx = (int(2 ** rng.uniform(6, 13.3)) for _ in range(2))
    p = plan((ny, nx), (1, 1), dtype)
    wg, cells, rows, regs, even = figures(p, "workgroups", "cells_per_lane", "rows_per_wave", "rows_in_registers", "even")
    if wg:
        seen += 1
        w, h = 64 * cells, 8 * rows
        assert cells * (8 if dtype is float64 else 4) == 32 and w < nx and h <= ny
        assert wg == -(-nx // w) * -(-ny // h) <= 256 and regs <= rows
        assert bool(even) == (nx % cells == 0 and ny % h == 0)
        assert J.jacobi_get_option(p, "block_workgroups") == 0
    J.jacobi_destroy(p)
assert seen > 300, seen
for dims in ((4096, 4100), (8192, 8192), (20000, 200), (1024, 1024), (2048, 2048)):
    p = plan(dims, (1, 1), float64)
    assert figures(p, "workgroups") == (0,), dims
    J.jacobi_destroy(p)
""")


def test_no_lane_sends_both_ways(stub):  # noqa: F811
    """A lane has one column to send.  Every width up to 64 blocks side by side, at heights that blocks divide: the starts of the columns are
    spread evenly, in whole lanes (in cells where a lane's cells do not divide the width), the first steps one longer; where the fewest
    columns would leave a lane with two, there is one column more."""
    seen = run(stub, HEAD + """
seen = set()
def both(nx, HW, C, nb):
    unit = C if nx % C == 0 else 1
    step, longer = divmod((nx - HW) // unit, nb - 1)
    start = [(b * step + min(b, longer)) * unit for b in range(nb)]
    assert start[-1] + HW == nx
    return any((start[b - 1] + HW - start[b]) // C == (start[b + 1] - 1 - start[b]) // C for b in range(1, nb - 1))
for dtype, C in ((float64, 4), (float32, 8)):
    HW = 64 * C
    for nx in range(HW + 1, 64 * HW + 1):
        nb = -(-nx // HW)
        shared = both(nx, HW, C, nb)
        if not shared and nx % 97:
            continue                                      # (a sample of the others)
        for rows in (8, 12, 16, 20, 24, 32):
            ny = 256 // nb // 2 * 8 * rows
            p = plan((ny, nx), (1, 1), dtype)
            wg, held = figures(p, "workgroups", "rows_per_wave")
            J.jacobi_destroy(p)
            if wg:
                seen.add((nx, C))
                columns = wg // -(-ny // (8 * held))
                assert columns == nb + shared and not both(nx, HW, C, columns), (nx, rows, wg)
print(sorted(s for s in seen if both(s[0], 64 * s[1], s[1], -(-s[0] // (64 * s[1])))), len(seen))
""")
    assert seen.strip().startswith("[(513, 4), (516, 4), (1025, 8), (1032, 8)]"), seen


# Calls timed both ways (us, MI355X), chip = 0 and chip = 1 forced: short ones near the line, with norms, with blocked passes
TIMED = [
    # dims, type, tblock, iterations, norm every, by launches, on the chip
    ((4672, 4836), "float32", 4, 4, 3, 80.5, 127.6), ((3968, 4172), "float32", 8, 4, 3, 64.4, 83.5), ((4224, 5780), "float32", 12, 5, 3, 95.1, 110.8),
    ((3568, 6300), "float32", 1, 4, 3, 122.4, 135.2), ((4999, 4318), "float32", 12, 9, 1, 304.5, 443.2), ((4999, 4318), "float32", 8, 3, 0, 64.0, 89.9),
    ((4208, 5082), "float32", 8, 23, 1, 743.0, 1027.0), ((4672, 5036), "float32", 4, 7, 0, 92.7, 112.9),
    ((5832, 3452), "float32", 4, 100, 3, 1490.3, 1812.6), ((2187, 3092), "float32", 4, 8, 0, 40.5, 49.7), ((2595, 2096), "float32", 1, 3, 2, 34.2, 37.0),
    ((1565, 1577), "float64", 8, 6, 6, 49.1, 40.3), ((2496, 3568), "float64", 4, 5, 0, 68.8, 56.0), ((3480, 3960), "float32", 4, 11, 11, 98.4, 80.0),
    ((4224, 5248), "float32", 8, 5, 3, 87.9, 76.6), ((4032, 4115), "float32", 12, 12, 1, 332.0, 293.5), ((5015, 3392), "float32", 1, 3, 0, 68.5, 55.5),
    ((3072, 2392), "float64", 8, 10, 10, 82.1, 69.0), ((3004, 2112), "float64", 8, 11, 5, 96.9, 78.0), ((2816, 4008), "float64", 8, 29, 0, 234.9, 188.5),
]


def test_calls_take_the_faster_path(stub):  # noqa: F811
    """(A call on the chip is one launch.)"""
    run(stub, HEAD + f"""
wrong = []
for dims, dtype, tblock, iters, every, other, chip in {TIMED!r}:
    p = plan(dims, (1, 1), float64 if dtype == "float64" else float32)
    J.jacobi_set_option(p, "tblock", tblock)
    if (launches(p, iters, every) == 1) != (chip < other):
        wrong.append((dims, dtype, tblock, iters, every, other, chip))
    J.jacobi_destroy(p)
assert not wrong, wrong
""")


def test_set_up_words_and_scratch(stub):  # noqa: F811
    """The plan's words are cleared by a kernel on the stream of the first launch, once; without room for the messages the plan runs by
    launches; calls of one or two iterations take the path that is faster for them."""
    run(stub, HEAD + """
p = plan((4096, 4096), (4, 4), float64)
J.jacobi_prepare(p)
assert "hipMemset" not in [c[0] for c in log()]
counts = []
for _ in range(3):
    J.jacobi_sweep(p, *GRIDS(p), 100, 1 << 12)
    counts.append(sum(c[0] == "hipLaunchKernel" for c in log()))
assert counts == [2, 1, 1], counts
J.jacobi_sweep(p, *GRIDS(p), 1)
assert ["512"] != [c[2] for c in log() if c[0] == "hipLaunchKernel"]
whole = J.jacobi_scratch_bytes(p)
J.jacobi_destroy(p)
p = plan((4096, 4096), (4, 4), float64)
stub.stub_malloc_limit(whole - 1)
J.jacobi_prepare(p)
assert J.jacobi_scratch_bytes(p) < whole
log()
J.jacobi_sweep(p, *GRIDS(p), 50)
assert sum(c[0] == "hipLaunchKernel" for c in log()) >= 50
J.jacobi_destroy(p)
""")


def test_a_launch_that_fails_leaves_its_clearing_waited_for(stub):  # noqa: F811
    """The first launch fails, the kernel that clears the words is on its way: the next launch, on whatever stream, waits for it."""
    run(stub, HEAD + """
p = plan((4096, 4096), (4, 4), float64)
J.jacobi_prepare(p)
log()
stub.stub_fail_launch(1)
try:
    J.jacobi_sweep(p, *GRIDS(p), 100, 1 << 40)
    raise SystemExit("the launch did not fail")
except J.JacobiError as e:
    assert e.code == J.binding.JACOBI_EHIP
calls = [c[0] for c in log()]
assert calls.index("hipEventRecord") > calls.index("hipLaunchKernel") and calls.count("hipLaunchKernel") == 1, calls
J.jacobi_sweep(p, *GRIDS(p), 100, 1 << 41)
calls = [c[0] for c in log()]
assert calls == ["hipStreamWaitEvent", "hipLaunchKernel", "hipEventRecord"], calls
J.jacobi_destroy(p)
""")


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """The instructions of one variant, in the order of the text."""
    from paper_2210_01238_amd import build
    d = tmp_path_factory.mktemp("asm")
    src, out = str(d / "one.hip"), str(d / "one.s")
    with open(src, "w") as f:
        f.write('#include "chip2d_kernel.h"\n'
                "template __global__ void jk::chip2d_kernel<float, 8, 0, 0, true>(jk::Geo, jk::Chip2d, float *, float *);\n")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "-I", build.CSRC, "-I", os.path.join(ROOT, "include"),
                    "--cuda-device-only", "-S", src, "-o", out], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.STDOUT)
    found, inside = [], False
    for line in open(out):
        if re.match(r"_ZN2jk\d+chip2d_kernelI.*:", line):
            inside = True
        elif line.startswith(".Lfunc_end"):
            inside = False
        elif inside and line.startswith(".LBB"):
            found.append("label")
        elif inside and line.startswith("\t") and not line.lstrip().startswith((";", ".")):
            found.append(line.split(";")[0].strip())
    assert found
    return found


def test_end_of_a_workgroup_and_its_barriers_wait_for_every_wavefront(code):
    for pattern in (r"buffer_wbl2", r"global_atomic_add v.* offset:8 sc0"):
        bad, n = waits.unwaited(code, [i for i, x in enumerate(code) if re.match(pattern, x)])
        assert n >= 1 and not bad, (pattern, bad)

