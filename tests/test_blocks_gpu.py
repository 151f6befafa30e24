"""The path that runs a whole jacobi_run of a mid-sized grid in one launch, the grid cut into blocks that workgroups keep in
registers and whose borders they exchange as tagged messages.  fp64 grids bit for bit against the CPU oracle, fp32 within
1e-5*max|u|, norms within 1e-12 / 1e-5 (the bars of the other suites).  Shapes at the edges of the cut: one cell more than
a block, odd sizes, widths that only one or two cells per lane divide, tiles one cell wide, seams inside a lane's cells."""
import numpy as np
import pytest

from parity_util import random_padded
from test_parity_gpu import check

pytestmark = pytest.mark.gpu

CASES = [
    # (interior dims, tiles, iterations, norm every[, the only type that runs this way])
    ((513, 301), (1, 1), 37, 12), ((300, 1001), (3, 7), 40, 7), ((257, 770), (1, 5), 33, 33), ((1024, 1024), (4, 4), 60, 30),
    ((701, 613), (1, 1), 41, 8), ((640, 300), (64, 300), 32, 16), ((512, 264), (512, 2), 24, 6, np.float64), ((130, 514), (2, 1), 64, 2),
    ((1500, 1110), (5, 3), 48, 25), ((66, 2600), (1, 13), 30, 10), ((2000, 258), (8, 3), 50, 0), ((1536, 1536), (2, 3), 20, 10),
]


def run_whole(H, a, tiles, iters, every, **opts):
    r = H.JacobiRun([n - 2 for n in a.shape], tiles, a.dtype, **opts)
    try:
        r.load(a)
        r.other().fill_(255)                    # NaN: the other grid's ring has to come from the run
        res = r.run(iters, every, fuse_residual=True) if every else (r.sweep(iters) or [])
        where = r.cur is r.a
        return r.fetch(), res, where
    finally:
        r.close()


CASES_3D = [
    # rows of exactly one and two lanes' cells, one cell fewer, odd rows, one and many blocks per direction
    ((64, 64, 64), (2, 2, 2), 40, 20), ((64, 64, 64), (1, 1, 1), 33, 1, np.float64), ((64, 64, 64), (1, 1, 1), 33, 5), ((61, 53, 47), (1, 1, 1), 30, 7), ((48, 40, 60), (2, 2, 3), 41, 0),
    ((40, 70, 63), (4, 7, 21), 36, 12), ((6, 40, 64), (2, 4, 8), 60, 15), ((128, 128, 128), (2, 2, 2), 30, 10, np.float32), ((96, 96, 128), (3, 2, 1), 30, 10),
    ((90, 100, 126), (1, 5, 9), 28, 14, np.float32), ((30, 46, 33), (1, 1, 1), 40, 40),
]

# Every compiled variant of the kernels, each at about the smallest grid for which it is chosen; in 3-D once with rows that fill the
# wavefront and once with shorter ones.  Widths of tiles that 4 does not divide have seams inside a lane's cells.
F64, F32 = np.float64, np.float32
VARIANTS = {
    # (cells per lane, planes (0: 2-D), rows per wavefront): [(interior dims, tiles, type)]
    (1, 0, 2): [((20, 322), (4, 7), F64), ((20, 636), (4, 12), F32)], (1, 0, 4): [((37, 340), (1, 17), F64), ((37, 660), (1, 3), F32)],
    (1, 0, 6): [((56, 300), (8, 1), F64), ((56, 580), (8, 29), F32)], (1, 0, 8): [((101, 333), (1, 9), F64), ((101, 613), (1, 1), F32)],
    (1, 0, 12): [((3482, 113), (2, 1), F64), ((2065, 185), (7, 37), F32)], (1, 0, 16): [((265, 3093), (53, 3), F64), ((177, 3463), (59, 1), F32)],
    (1, 0, 24): [((365, 3095), (5, 5), F32)],
    (2, 0, 6): [((64, 3468), (8, 4), F64), ((1728, 228), (54, 12), F32)], (2, 0, 8): [((160, 2312), (32, 8), F64), ((2144, 188), (32, 4), F32)],
    (2, 0, 10): [((268, 2940), (4, 28), F64), ((3459, 244), (3, 4), F32)], (2, 0, 12): [((3306, 468), (38, 12), F64), ((3618, 356), (54, 4), F32)],
    (2, 0, 16): [((3189, 736), (3, 32), F64), ((3697, 468), (1, 12), F32)], (2, 0, 24): [((977, 3386), (1, 2), F32)],
    (4, 0, 8): [((2667, 976), (21, 16), F64), ((802, 3608), (2, 8), F32)], (4, 0, 10): [((2221, 1096), (1, 8), F64), ((3160, 916), (40, 4), F32)],
    (4, 0, 12): [((3410, 756), (2, 36), F64), ((3369, 1004), (3, 4), F32), ((2048, 2048), (2, 4), F64), ((2048, 2048), (2, 4), F32)],
    (1, 4, 2): [((7, 7, 36), (1, 1, 12), F64), ((7, 7, 64), (1, 1, 4), F64), ((7, 7, 34), (1, 1, 2), F32), ((7, 7, 64), (1, 1, 8), F32)],
    (1, 6, 3): [((219, 38, 35), (3, 2, 7), F64), ((64, 10, 64), (16, 2, 16), F64), ((200, 44, 33), (8, 4, 11), F32), ((37, 217, 64), (1, 7, 4), F32)],
    (2, 4, 2): [((8, 8, 65), (1, 2, 13), F64), ((8, 8, 128), (2, 2, 2), F64), ((7, 7, 65), (1, 1, 13), F32), ((7, 7, 128), (1, 1, 32), F32)],
    (2, 5, 2): [((225, 37, 65), (25, 1, 13), F64), ((217, 37, 128), (31, 1, 2), F64), ((11, 8, 128), (1, 1, 16), F32)],
    (2, 6, 3): [((38, 220, 67), (2, 4, 1), F32), ((49, 217, 128), (7, 7, 32), F32)],
    (4, 4, 2): [((8, 8, 130), (2, 1, 10), F32), ((7, 7, 256), (1, 1, 8), F32), ((190, 10, 255), (2, 1, 3), F32)],
    (4, 5, 2): [((45, 6, 159), (5, 2, 53), F32), ((37, 217, 256), (1, 7, 16), F32)],
}
VARIANT_ITERS, VARIANT_EVERY = 31, 9
# (Option chip = 0 in the tests below: blocks with ghost cells also where a call would run in those without.)


BLOCK_CASES = [(*c[:4], t) for c in CASES + CASES_3D for t in (c[4:] or (np.float64, np.float32))]


@pytest.mark.parametrize("dims,tiles,iters,every,dtype", BLOCK_CASES)
def test_blocks_match_the_oracle(H, oracle_mod, dims, tiles, iters, every, dtype):
    """(That these calls are one launch each is checked without a GPU: test_block_plans.py.)"""
    a = random_padded(dims, dtype=dtype, seed=sum(dims) + iters)
    ref, ref_res = oracle_mod.run(a, iters, every)
    out, res, in_a = run_whole(H, a, tiles, iters, every, resident=1)
    check(out, res, ref, ref_res)
    # the launch-per-iteration path: the same grid to the bit (fp32 too), the result in the same buffer
    out0, res0, in_a0 = run_whole(H, a, tiles, iters, every, resident=0)
    assert np.array_equal(out, out0) and in_a == in_a0
    out2, res2, _ = run_whole(H, a, tiles, iters, every, resident=1)
    assert np.array_equal(out2, out) and res2 == res                # and the same bits on every run
    if len(dims) == 3:                                              # which may have been without ghost cells: with them
        out3, res3, in_a3 = run_whole(H, a, tiles, iters, every, resident=1, chip=0)
        check(out3, res3, ref, ref_res)
        assert np.array_equal(out3, out) and in_a3 == in_a


@pytest.mark.parametrize("variant,dims,tiles,dtype", [(v, *c) for v, cases in VARIANTS.items() for c in cases])
def test_every_variant_matches_the_oracle(H, oracle_mod, variant, dims, tiles, dtype):
    a = random_padded(dims, dtype=dtype, seed=sum(dims))
    ref, ref_res = oracle_mod.run(a, VARIANT_ITERS, VARIANT_EVERY)
    r = H.JacobiRun(dims, tiles, dtype, resident=1, chip=0, profile=1)
    try:
        got = tuple(H.B.jacobi_get_option(r.plan, "block_" + k) for k in ("cells_per_lane", "planes_per_wave", "rows_per_wave"))
        assert got == variant
        r.load(a)
        r.other().fill_(255)
        res = r.run(VARIANT_ITERS, VARIANT_EVERY, fuse_residual=True)
        check(r.fetch(), res, ref, ref_res)
        assert H.B.jacobi_profile_read(r.plan)[1] == 1             # one launch
    finally:
        r.close()


PLAIN = [((1024, 1024), (4, 4), np.float64), ((300, 701), (3, 1), np.float32), ((64, 64, 64), (2, 2, 2), np.float64),
         ((61, 53, 47), (1, 1, 1), np.float32)]


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_blocks_without_all_workgroups_take_the_plain_path(H, oracle_mod, dims, tiles, dtype):
    """Some workgroups come too late (resident_admitted: as many as are let in): the others do the work along the plain path, one
    iteration after the other through memory, with the same result; the next launch finds the plan's words as it needs
    them.  The norms' last bits show that it was that path: other workgroups' sums, in another order."""
    a = random_padded(dims, dtype=dtype, seed=77)
    r = H.JacobiRun(dims, tiles, dtype, resident=1, chip=0)
    try:
        n = H.B.jacobi_get_option(r.plan, "block_workgroups")
        for iters, every in ((120, 2), (24, 2), (23, 0), (26, 26), (25, 6)):
            ref, ref_res = oracle_mod.run(a, iters, every)
            norms = {}
            for admitted in (0, 1, n // 2, n - 1, 0, n - 1, n - 1, 0):
                r.set_option("resident_admitted", admitted)
                r.load(a)
                r.other().fill_(255)
                res = r.run(iters, every, fuse_residual=True) if every else (r.sweep(iters) or [])
                check(r.fetch(), res, ref, ref_res)
                assert norms.setdefault(admitted, res) == res, (iters, every, admitted)
            if len(ref_res) == 60:
                # one norm in three or so differs in its last bit; fp32: fewer (squares have 48 bits and are added up in 53)
                assert len({tuple(v) for v in norms.values()}) >= (4 if dtype == np.float64 else 3), norms
    finally:
        r.close()


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_blocks_that_do_not_wait_for_each_other_to_start(H, oracle_mod, dims, tiles, dtype):
    """resident_spin_limit = 1: the roll is called once, without waiting; whoever is there does the work, whichever path it is."""
    a = random_padded(dims, dtype=dtype, seed=77)
    for iters, every in ((24, 8), (23, 0), (26, 26)):
        ref, ref_res = oracle_mod.run(a, iters, every)
        r = H.JacobiRun(dims, tiles, dtype, resident=1, chip=0, resident_spin_limit=1)
        try:
            for limit in (1, 1, 0, 1, 0):
                r.set_option("resident_spin_limit", limit)
                r.load(a)
                res = r.run(iters, every, fuse_residual=True) if every else (r.sweep(iters) or [])
                check(r.fetch(), res, ref, ref_res)
        finally:
            r.close()


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_blocks_count_exchanges_from_zero_again(H, oracle_mod, dims, tiles, dtype):
    """Every launch (resident_epoch_limit = 1) and every third one clears the messages and starts with the same tags: other fields
    each time, so that a message left over would show."""
    r = H.JacobiRun(dims, tiles, dtype, resident=1, chip=0)
    try:
        for limit in (1, 130):
            r.set_option("resident_epoch_limit", limit)
            for k in range(5):
                a = random_padded(dims, dtype=dtype, seed=100 + k)
                ref, ref_res = oracle_mod.run(a, 50, 25)
                r.load(a)
                res = r.run(50, 25, fuse_residual=True)
                check(r.fetch(), res, ref, ref_res)
    finally:
        r.close()


def test_blocks_sweeps_keep_parity_and_residual_of_the_input(H, oracle_mod):
    """jacobi_sweep ends in the buffer the schedule says, also with blocked passes asked for; jacobi_sweep_residual gives
    the norm of the field that went in."""
    import torch
    a = random_padded((700, 900), seed=5)
    for iters, opts in ((40, {}), (41, {}), (40, dict(tblock=8)), (39, dict(tblock=12)), (30, dict(fused=0)), (30, dict(profile=1))):
        ref, _ = oracle_mod.run(a, iters)
        r = H.JacobiRun((700, 900), (7, 3), resident=1, **opts)
        try:
            r.load(a)
            passes = len(H.B.jacobi_pass_schedule(r.plan, iters))
            r.sweep(iters)
            assert (r.cur is r.a) == (passes % 2 == 0), (iters, opts)
            assert np.array_equal(r.fetch(), ref), (iters, opts)
            r.load(a)
            norm = torch.zeros(1, dtype=torch.float64, device="cuda")
            r.sweep_residual(iters, norm)
            assert np.array_equal(r.fetch(), ref), (iters, opts)
            want = oracle_mod.residual(a)
            assert abs(norm.item() - want) <= 1e-12 * want
            if opts.get("profile"):
                ms, n = H.B.jacobi_profile_read(r.plan)
                assert n == 2 and ms > 0.0
        finally:
            r.close()


def test_blocks_special_values_and_many_norms(H, oracle_mod):
    """Infinities and NaN in the field spread as on the other path; more norms than one launch delivers."""
    a = random_padded((520, 640), seed=9)
    a[100, 200] = np.inf
    a[300, 0] = -np.inf
    a[400, 641] = np.nan
    got = [run_whole(H, a, (2, 4), 30, 10, resident=k) for k in (1, 0)]
    assert np.array_equal(got[0][0], got[1][0], equal_nan=True)
    assert np.array_equal(np.isnan(got[0][1]), np.isnan(got[1][1]))
    b = random_padded((260, 300), seed=10)
    ref, ref_res = oracle_mod.run(b, 300, 2)                       # 150 norms
    out, res, _ = run_whole(H, b, (1, 1), 300, 2, resident=1)
    check(out, res, ref, ref_res)


def test_blocks_in_a_hip_graph_and_two_plans_on_two_streams(H, oracle_mod):
    import torch
    a = random_padded((512, 700), seed=12)
    iters = 32
    r = H.JacobiRun((512, 700), (4, 7), resident=1)
    q = H.JacobiRun((1024, 1024), (1, 1), resident=1)
    b = random_padded((1024, 1024), seed=13)
    ref_b, _ = oracle_mod.run(b, 40)
    try:
        H.B.jacobi_prepare(r.plan)
        g_dev = torch.from_numpy(a).cuda()
        res = torch.zeros(2, dtype=torch.float64, device="cuda")
        exp, exp_res = oracle_mod.run(a, iters, 16)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            st = int(torch.cuda.current_stream().cuda_stream)
            H.B.jacobi_scatter(r.plan, g_dev.data_ptr(), r.a.data_ptr(), st)
            fin = H.B.jacobi_run(r.plan, r.a.data_ptr(), r.b.data_ptr(), iters, 16, res.data_ptr(), st)
        for k in range(3):
            res.zero_()
            graph.replay()
            torch.cuda.synchronize()
            r.cur = r.a if fin == r.a.data_ptr() else r.b
            check(r.fetch(), res.cpu().tolist(), exp, exp_res)
            r.load(a)
            r.sweep(20 + k)                      # eager launches between the replays use up other tags
            r.residual()
        # one plan, two pairs of grids, two streams at once: launches of one plan share its messages and follow each other
        other = H.JacobiRun((512, 700), (4, 7), resident=1)
        c = random_padded((512, 700), seed=14)
        ref_c, _ = oracle_mod.run(c, 41)
        try:
            s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
            for k in range(4):
                r.load(a)
                other.load(c)
                torch.cuda.synchronize()
                f1 = H.B.jacobi_sweep(r.plan, r.a.data_ptr(), r.b.data_ptr(), iters, int(s1.cuda_stream))
                f2 = H.B.jacobi_sweep(r.plan, other.a.data_ptr(), other.b.data_ptr(), 41, int(s2.cuda_stream))
                torch.cuda.synchronize()
                r.cur = r.a if f1 == r.a.data_ptr() else r.b
                other.cur = other.a if f2 == other.a.data_ptr() else other.b
                assert np.array_equal(r.fetch(), exp), k
                assert np.array_equal(other.fetch(), ref_c), k
        finally:
            other.close()
        # two plans whose workgroups together are more than the chip has CUs, on two streams at once
        for k in range(4):
            r.load(a)
            q.load(b)
            torch.cuda.synchronize()
            with torch.cuda.stream(s1):
                r.sweep(iters)
            with torch.cuda.stream(s2):
                q.sweep(40)
            torch.cuda.synchronize()
            assert np.array_equal(r.fetch(), exp), k
            assert np.array_equal(q.fetch(), ref_b), k
    finally:
        r.close()
        q.close()
