"""Which calls run in blocks, and as what: planned on the CPU, with a stand-in for the HIP runtime (hip_stub) that counts launches.
The suite that runs them on a GPU compares them with the launch-per-iteration path - which says nothing about a call that
takes that path itself."""
import os
import re

from test_blocks_gpu import BLOCK_CASES, PLAIN, VARIANT_EVERY, VARIANT_ITERS, VARIANTS
from test_host_calls import ROOT, run, stub  # noqa: F401  (stub: a fixture)

HEAD = """
from numpy import float64, float32
def plan(dims, tiles, dtype):
    return J.jacobi_create(dims, tiles, J.JACOBI_F64 if dtype is float64 else J.JACOBI_F32)
def launches(p, iters, every):
    J.jacobi_prepare(p)
    log()
    J.jacobi_run(p, *GRIDS(p), iters, every, 1 << 16) if every else J.jacobi_sweep(p, *GRIDS(p), iters)
    return sum(c[0] == "hipLaunchKernel" for c in log())
def variant(p):
    return tuple(J.jacobi_get_option(p, "block_" + k) for k in ("cells_per_lane", "planes_per_wave", "rows_per_wave"))
"""


def text(cases):
    return repr(cases).replace("<class 'numpy.float64'>", "float64").replace("<class 'numpy.float32'>", "float32")


def test_calls_of_the_block_tests_run_in_blocks(stub):  # noqa: F811
    run(stub, HEAD + f"""
for dims, tiles, iters, every, dtype in {text(BLOCK_CASES + [(*c[:2], 24, 2, c[2]) for c in PLAIN])}:
    p = plan(dims, tiles, dtype)
    assert variant(p)[0] and launches(p, iters, every) == 1, (dims, tiles, iters, every, dtype)
    J.jacobi_set_option(p, "chip", 0)
    assert launches(p, iters, every) == 1, (dims, tiles, iters, every, dtype)
    J.jacobi_destroy(p)
""")


def test_every_compiled_variant_is_reached(stub):  # noqa: F811
    run(stub, HEAD + f"""
for want, cases in {text(VARIANTS)}.items():
    for dims, tiles, dtype in cases:
        p = plan(dims, tiles, dtype)
        J.jacobi_set_option(p, "chip", 0)
        assert variant(p) == want and launches(p, {VARIANT_ITERS}, {VARIANT_EVERY}) == 1, (dims, tiles, dtype, variant(p), want)
        J.jacobi_destroy(p)
""")
    with open(os.path.join(ROOT, "paper_2210_01238_amd", "csrc", "launchers.h")) as f:
        tables = {m.group(1): re.findall(r"X\((\d[\d., ]*)", m.group(2))
                  for m in re.finditer(r"#define JK_(BLOCKS\dD_VARIANTS\w*)\(X\)((?:.*\\\n)*.*)", f.read())}
    numbers = {name: [[int(n) for n in v.split(",")[:3] if n.strip().isdigit()] for v in vs] for name, vs in tables.items()}
    both = {(c, 0, rw) for c, rw, *_ in numbers["BLOCKS2D_VARIANTS"]} | {tuple(v) for v in numbers["BLOCKS3D_VARIANTS"]}
    f32_only = {(c, 0, rw) for c, rw, *_ in numbers["BLOCKS2D_VARIANTS_F32"]} | {tuple(v) for v in numbers["BLOCKS3D_VARIANTS_F32"]}
    compiled = {(v, t) for v in both for t in ("float64", "float32")} | {(v, "float32") for v in f32_only}
    assert compiled == {(v, c[2].__name__) for v, cases in VARIANTS.items() for c in cases}


# Calls timed both ways (us, MI355X): the launch-per-iteration path or, for the narrow grids, resident2d_kernel, and in blocks.
TIMED = [
    # dims, tiles, type, tblock, iterations, norm every, other, blocks
    ((27, 29, 119), (1, 1, 1), "float64", 1, 22, 0, 87.9, 107.3), ((27, 29, 119), (1, 1, 1), "float64", 1, 132, 0, 506.8, 559.3),
    ((19, 20, 128), (1, 4, 1), "float64", 1, 20, 20, 85.4, 98.0), ((14, 7, 64), (2, 1, 2), "float64", 4, 98, 98, 547.3, 312.1),
    ((51, 33, 256), (1, 3, 1), "float32", 12, 14, 0, 129.0, 73.4), ((77, 50, 256), (1, 5, 1), "float32", 1, 132, 22, 891.1, 596.3),
    ((64, 64, 64), (2, 2, 2), "float64", 1, 100, 50, 604.6, 345.4), ((29, 28, 128), (1, 4, 1), "float32", 1, 12, 10, 65.8, 52.3),
    ((23, 26, 64), (1, 2, 4), "float32", 1, 9, 4, 57.0, 40.2), ((26, 35, 64), (2, 1, 1), "float32", 1, 9, 0, 47.9, 35.6),
    ((96, 84), (3, 1), "float64", 1, 13, 0, 14.9, 17.4), ((76, 228), (1, 3), "float32", 8, 13, 0, 15.1, 17.3),
    ((96, 84), (3, 1), "float64", 1, 78, 0, 65.6, 45.3), ((76, 248), (2, 4), "float64", 8, 18, 9, 32.1, 25.0),
    ((352, 208), (1, 1), "float64", 1, 32, 0, 35.2, 25.5), ((256, 256), (1, 1), "float64", 1, 100, 100, 98.8, 63.7),
    ((295, 460), (1, 1), "float32", 1, 127, 25, 169.0, 91.7), ((68, 148), (1, 2), "float32", 4, 64, 2, 320.1, 140.0),
]


def test_calls_take_the_faster_path(stub):  # noqa: F811
    """(Block kernels are the launches of 512 threads.)"""
    run(stub, HEAD + f"""
for dims, tiles, dtype, tblock, iters, every, other, blocks in {TIMED!r}:
    p = plan(dims, tiles, float64 if dtype == "float64" else float32)
    J.jacobi_set_option(p, "tblock", tblock)
    J.jacobi_prepare(p)
    log()
    J.jacobi_run(p, *GRIDS(p), iters, every, 1 << 16)
    assert ("512" in [c[2] for c in log() if c[0] == "hipLaunchKernel"]) == (blocks < other), (dims, dtype, iters, other, blocks)
    J.jacobi_destroy(p)
""")
