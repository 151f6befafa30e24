"""Which runs take their last norm from their last pass (test_norm_after_gpu.py compares the values, which says nothing about a run that takes
a pass of its own for it): the kernels launched, seen through a stand-in for the HIP runtime (hip_stub)."""
from test_block_plans import text
from test_host_calls import run, stub  # noqa: F401  (stub: a fixture)
from test_norm_after_gpu import LARGE, SHAPES, SHAPES_3D

HEAD = """
import re
from numpy import float64, float32
UPDATE, RESIDUAL, BOTH, AFTER, BOTH_AFTER = range(5)        # what a kernel delivers: its second template argument
def kernels(dims, tiles, dtype, iters, every, **options):
    "[(kernel, mode, third argument: levels of the blocked passes)] of a run, without the ring's copy and the final sums"
    p = J.jacobi_create(dims, tiles, J.JACOBI_F64 if dtype is float64 else J.JACOBI_F32)
    for k, v in options.items():
        J.jacobi_set_option(p, k, v)
    J.jacobi_prepare(p)
    log()
    J.jacobi_run(p, *GRIDS(p), iters, every, 1 << 16)
    names = [c[4] for c in log() if c[0] == "hipLaunchKernel"]
    size = J.jacobi_grid_bytes(p)
    last = J.jacobi_pass_schedule(p, every)[-1]
    J.jacobi_destroy(p)
    out = []
    for n in names:
        m = re.match(r"_ZN2jk\\d+(sweep[23]d_\\w*?kernel|residual2d_stack_kernel)I[df]Li(\\d+)E(?:Li(\\d+)E)?", n)
        if m:
            out.append((m.group(1), RESIDUAL if "stack" in n else int(m.group(2)), int(m.group(3) or 0)))
    finals = sum("residual_final_kernel" in n for n in names)
    assert finals == iters // every, (dims, names)
    return out, size, last
"""


def test_the_last_2d_pass_delivers_the_norm(stub):  # noqa: F811
    """Depths from 3 up to 7, from 240 MiB on up to 11, of tiles at least one row higher; with the norm of its source due as well where the run has
    a second stretch of one pass."""
    run(stub, HEAD + f"""
taken = set()
for shapes, depths, strips in (({text(SHAPES)}, range(2, 9), (0, 1, 5)), ({text(LARGE)}, range(8, 13), (0, 5))):
    for dims, tiles, dtype in shapes:
        for depth in depths:
            for iters in (depth, 2 * depth):
                for strip in strips:
                    seen, size, last = kernels(dims, tiles, dtype, iters, depth, tblock=depth, resident=0, rows_per_strip=strip)
                    th, tw, lane = dims[0] // tiles[0], dims[1] // tiles[1], 2 if dtype is float64 else 4
                    assert last == depth and th >= depth and tw % lane == 0          # the tests' shapes run in one pass a stretch
                    want = 3 <= depth < (12 if size >= 240 << 20 else 8) and th > depth
                    mode = BOTH_AFTER if iters > depth else AFTER
                    assert (seen[-1] == ("sweep2d_tp_kernel", mode, depth + 1)) == want, (dims, depth, iters, seen)
                    assert (seen[-1][1] == RESIDUAL) == (not want), (dims, depth, iters, seen)
                    assert len(seen) == iters // depth + (not want), (dims, depth, iters, seen)
                    taken.add((depth, mode, dtype.__name__, want))
for depth in range(3, 12):
    for mode in (AFTER, BOTH_AFTER):
        for t in ("float64", "float32"):
            assert (depth, mode, t, True) in taken
assert {{(8, AFTER, t, False) for t in ("float64", "float32")}} | {{(12, AFTER, t, False) for t in ("float64", "float32")}} <= taken
# tiles exactly as high as the pass is deep
seen, _, _ = kernels((35, 400), (7, 1), float64, 5, 5, tblock=5, resident=0)
assert [s[1] for s in seen] == [UPDATE, RESIDUAL], seen
# strips of one row: the scratch does not hold a sum of either norm for each of so many workgroups
seen, _, _ = kernels((5720, 5634), (8, 3), float64, 16, 8, tblock=8, resident=0, rows_per_strip=1)
assert [s[1] for s in seen] == [UPDATE, BOTH, RESIDUAL], seen
# 240 MiB: the line of the deeper passes
for rows, want in ((5605, False), (5620, True)):
    seen, size, _ = kernels((rows, 5600), (1, 1), float64, 9, 9, tblock=9, resident=0)
    assert (size >= 240 << 20) == want and (seen[-1][1] == AFTER) == want, (rows, size, seen)
""")


def test_the_last_3d_pass_delivers_the_norm(stub):  # noqa: F811
    """fp64 passes of three, of tiles at least four planes deep, grids from 24 MiB on, no norm of the source due."""
    run(stub, HEAD + f"""
count = 0
for dims, tiles in {text(SHAPES_3D)}:
    for iters, every, tblock, strip in ((3, 3, 3, 0), (3, 3, 3, 1), (10, 10, 4, 0), (10, 10, 4, 3), (6, 3, 3, 0)):
        seen, size, last = kernels(dims, tiles, float64, iters, every, tblock=tblock, resident=0, rows_per_strip=strip)
        assert size >= 24 << 20
        want = last == 3 and dims[0] // tiles[0] >= 4 and iters == every
        assert (seen[-1] == ("sweep3d_tc_kernel", AFTER, 4)) == want, (dims, iters, seen)
        assert (seen[-1][1] == RESIDUAL) == (not want), (dims, iters, seen)
        count += want
assert count == 3 * 4, count
seen, size, last = kernels((128, 128, 128), (1, 1, 1), float64, 3, 3, tblock=3, resident=0)      # 16 MB
assert size < 24 << 20 and last == 3 and seen[-1][1] == RESIDUAL
seen, size, last = kernels((200, 200, 200), (1, 1, 1), float32, 3, 3, tblock=3, resident=0)
assert size >= 24 << 20 and last == 3 and seen[-1][1] == RESIDUAL
seen, size, last = kernels((200, 200, 200), (1, 1, 1), float64, 4, 4, tblock=4, resident=0)
assert last == 4 and seen[-1][1] == RESIDUAL
""")
