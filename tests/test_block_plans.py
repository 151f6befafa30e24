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
    J.jacobi_destroy(p)
""")


def test_every_compiled_variant_is_reached(stub):  # noqa: F811
    run(stub, HEAD + f"""
for want, cases in {text(VARIANTS)}.items():
    for dims, tiles, dtype in cases:
        p = plan(dims, tiles, dtype)
        assert variant(p) == want and launches(p, {VARIANT_ITERS}, {VARIANT_EVERY}) == 1, (dims, tiles, dtype, variant(p), want)
        J.jacobi_destroy(p)
""")
    with open(os.path.join(ROOT, "paper_2210_01238_amd", "csrc", "launchers.h")) as f:
        tables = {m.group(1): re.findall(r"X\(([\d., ]+)\)", m.group(2))
                  for m in re.finditer(r"#define JK_(BLOCKS\dD_VARIANTS\w*)\(X\)((?:.*\\\n)*.*)", f.read())}
    numbers = {name: [tuple(int(float(n)) for n in v.split(",")) for v in vs] for name, vs in tables.items()}
    both = {(c, 0, rw) for c, rw, *_ in numbers["BLOCKS2D_VARIANTS"]} | set(numbers["BLOCKS3D_VARIANTS"])
    f32_only = {(c, 0, rw) for c, rw, *_ in numbers["BLOCKS2D_VARIANTS_F32"]} | set(numbers["BLOCKS3D_VARIANTS_F32"])
    compiled = {(v, t) for v in both for t in ("float64", "float32")} | {(v, "float32") for v in f32_only}
    assert compiled == {(v, c[2].__name__) for v, cases in VARIANTS.items() for c in cases}
