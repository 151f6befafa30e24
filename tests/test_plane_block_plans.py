"""How the cooperative 3-D blocked passes split their planes into blocks: the workgroups of a launch, seen through a stand-in for the HIP runtime
(hip_stub), against a search of all splits.  (test_plane_blocks_gpu.py compares the results of such passes with the oracle's.)"""
from test_host_calls import run, stub  # noqa: F401  (stub: a fixture)

HEAD = """
import random
CUS = 256
def up(a, b): return -(-a // b)
def units(dims, dtype, depth):
    "units of a pass per block of planes: row groups x column segments"
    own = 8 * {2: 8, 3: 6, 4: 5}[depth] - 2 * depth
    return up(dims[1], own) * up(dims[2], 120 if dtype == J.JACOBI_F64 else 240)
def plan(dims, tiles, dtype, depth, **options):
    p = J.jacobi_create(dims, tiles, dtype)
    for k, v in {"tblock": depth, "resident": 0, **options}.items(): J.jacobi_set_option(p, k, v)
    J.jacobi_prepare(p)
    return p
def blocks(dims, tiles, dtype, depth, **options):
    "blocks of planes in a cooperative pass of this depth"
    p = plan(dims, tiles, dtype, depth, **options)
    log()
    J.jacobi_sweep(p, *GRIDS(p), depth)
    n = [int(c[1]) for c in log() if c[0] == "hipLaunchKernel" and "sweep3d_tc_kernel" in c[4]]
    J.jacobi_destroy(p)
    assert len(n) == 1 and n[0] % units(dims, dtype, depth) == 0, (dims, n)
    return n[0] // units(dims, dtype, depth)
def searched(nz, across, depth):
    "the rule, every split looked at: planes per block"
    def rounds(r): return up(across * up(nz, r), CUS)
    def cost(r):
        return rounds(r) * (r + 2 * depth) + (rounds(r) == 1 and 8 <= r <= 21 - 2 * depth and r < nz and nz % r == 0)
    least = up(nz, max(16, up(24 * CUS, across)))
    R = min(range(least, nz + 1), key=lambda r: (cost(r), rounds(r), -r if rounds(r) == 1 else r))
    if depth <= 3:
        R = next(r for r in range(least, R + 1) if r == R or up(nz, r) > CUS // across and cost(r) * 16 <= cost(R) * 17)
    return R
"""


def test_the_split_is_the_best_of_all(stub):  # noqa: F811
    run(stub, HEAD + """
rng = random.Random(12)
for _ in range(1500):
    dtype, depth = rng.choice(((J.JACOBI_F64, 3), (J.JACOBI_F64, 4), (J.JACOBI_F32, 3)))
    td, tz = rng.choice((4, 5, 7, 16, 33, 64, 100)), rng.choice((1, 1, 2, 3, 7, 20))
    dims = (td * tz, int(2 ** rng.uniform(2, 10)), 4 * int(2 ** rng.uniform(1, 9)))
    nz, across = dims[0], units(dims, dtype, depth)
    assert blocks(dims, (tz, 1, 1), dtype, depth) == up(nz, searched(nz, across, depth)), (dims, tz, dtype, depth)
# one round, ten units to a block: 25 blocks of 8 planes are all full, 23 of 9 end with one of 2; thin and thick blocks stay full
assert blocks((200, 200, 200), (2, 2, 2), J.JACOBI_F64, 3) == 23 and blocks((198, 200, 200), (2, 2, 2), J.JACOBI_F64, 3) == 25
assert blocks((128, 128, 128), (1, 1, 1), J.JACOBI_F64, 3) == 32 and blocks((384, 384, 384), (4, 4, 4), J.JACOBI_F32, 3) == 12
assert blocks((96, 292, 384), (1, 1, 1), J.JACOBI_F64, 4) == 6
""")


def test_planes_that_are_given_are_taken_up_to_the_whole_column(stub):  # noqa: F811
    """Blocks may cross from tile to tile, and those that the library chooses do: the option can ask for the same ones, and for deeper."""
    run(stub, HEAD + """
for dims, tiles, dtype, depth in (((36, 200, 720), (9, 1, 1), J.JACOBI_F64, 4), ((33, 352, 366), (11, 11, 61), J.JACOBI_F64, 3), ((512, 512, 512), (4, 4, 4), J.JACOBI_F64, 4)):
    nz, td = dims[0], dims[0] // tiles[0]
    chosen = blocks(dims, tiles, dtype, depth)
    planes = searched(nz, units(dims, dtype, depth), depth)
    assert planes > td and chosen == up(nz, planes), (dims, planes)
    for given in (1, td - 1, td, td + 1, planes, nz - 1, nz, 4096):
        assert blocks(dims, tiles, dtype, depth, rows_per_strip=given) == up(nz, min(nz, given)), (dims, given)
""")


def test_planning_takes_no_longer_than_a_launch(stub):  # noqa: F811
    """The split is asked for with every pass: host time of a pass with the library's choice and with one that is given.  (A search of all
    splits takes 15 to 60 us here, as long as the pass itself.)"""
    run(stub, HEAD + """
for dims in ((2048, 64, 64), (4096, 30, 60), (16384, 30, 60), (768, 1024, 1024)):
    def per_pass(strip):
        p = plan(dims, (1, 1, 1), J.JACOBI_F64, 3, rows_per_strip=strip)
        a, b = GRIDS(p)
        best = 1e9
        for _ in range(9):
            stub.stub_clear_log()
            t = time.perf_counter()
            J.jacobi_sweep(p, a, b, 600)
            best = min(best, (time.perf_counter() - t) / 200)
        J.jacobi_destroy(p)
        return best
    given, chosen = per_pass(64), per_pass(0)
    print(dims, "us per pass, planes given %.2f, chosen %.2f" % (given * 1e6, chosen * 1e6))
    assert chosen < given + 6e-6, (dims, given, chosen)
""")
