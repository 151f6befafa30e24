"""The path that runs a whole jacobi_run of a 3-D grid in one launch, the grid in the chip's registers, without ghost cells.  fp64 grids
bit for bit against the CPU oracle, fp32 within 1e-5*max|u|, norms within 1e-12 / 1e-5 (the bars of the other suites), all of them
the same bits as by launches.  Shapes: every compiled variant; blocks of full height and one row or plane short; rows that fill the
lanes, that are one cell longer or shorter, odd ones; a number of blocks that two do not divide; tiles one cell wide, high and deep."""
import numpy as np
import pytest

from parity_util import random_padded
from test_blocks_gpu import VARIANT_EVERY, VARIANT_ITERS
from test_blocks_gpu import VARIANTS as GHOST_VARIANTS
from test_blocks_gpu import run_whole
from test_parity_gpu import check

pytestmark = pytest.mark.gpu

F64, F32 = np.float64, np.float32
# (cells per lane, planes, rows per wavefront, wavefronts per row): [(interior dims, tiles, type)]
VARIANTS = {
    (1, 2, 2, 1): [((64, 4, 64), (16, 1, 4), F64), ((18, 17, 9), (6, 17, 3), F64), ((64, 4, 64), (1, 2, 32), F32),
                   ((17, 19, 9), (17, 19, 9), F32)],
    (1, 3, 3, 1): [((162, 30, 64), (1, 10, 8), F64), ((49, 123, 9), (1, 1, 9), F64), ((186, 42, 64), (6, 6, 2), F32)],
    (1, 4, 4, 1): [((56, 224, 64), (1, 28, 64), F64), ((97, 163, 9), (1, 1, 3), F64), ((256, 32, 64), (16, 1, 8), F32),
                   ((116, 70, 9), (58, 35, 3), F32)],
    (1, 6, 6, 1): [((372, 84, 64), (1, 12, 8), F64), ((193, 173, 9), (193, 173, 3), F64), ((84, 372, 64), (28, 2, 1), F32),
                   ((178, 177, 9), (89, 1, 3), F32)],
    (1, 3, 3, 2): [((24, 42, 128), (6, 7, 2), F64), ((22, 47, 65), (1, 47, 1), F64), ((42, 24, 128), (21, 12, 16), F32),
                   ((35, 29, 66), (5, 1, 11), F32)],
    (1, 4, 3, 2): [((8, 126, 128), (2, 1, 16), F64), ((31, 139, 66), (31, 139, 66), F64), ((8, 126, 128), (1, 3, 8), F32),
                   ((15, 121, 66), (5, 11, 1), F32)],
    (1, 4, 4, 2): [((128, 8, 128), (2, 8, 32), F64), ((199, 31, 66), (199, 1, 1), F64), ((128, 8, 128), (1, 1, 8), F32),
                   ((196, 15, 75), (98, 15, 75), F32)],
    (1, 5, 5, 2): [((20, 390, 128), (10, 39, 8), F64), ((57, 19, 65), (19, 1, 1), F64), ((20, 320, 128), (5, 20, 8), F32),
                   ((19, 64, 66), (1, 16, 66), F32)],
    (1, 6, 6, 2): [((264, 72, 128), (4, 24, 32), F64), ((191, 122, 65), (1, 1, 65), F64), ((36, 420, 128), (9, 6, 128), F32),
                   ((82, 186, 66), (1, 6, 22), F32)],
    (2, 4, 4, 2): [((64, 16, 256), (1, 8, 128), F64), ((68, 15, 129), (4, 15, 43), F64), ((64, 16, 256), (32, 16, 1), F32),
                   ((22, 46, 130), (1, 2, 10), F32)],
    (2, 5, 4, 2): [((10, 104, 256), (1, 13, 2), F64), ((19, 65, 130), (19, 1, 65), F64), ((10, 104, 256), (2, 2, 128), F32),
                   ((19, 54, 130), (19, 2, 13), F32)],
    (2, 5, 5, 2): [((100, 10, 256), (100, 5, 64), F64), ((57, 19, 139), (19, 19, 1), F64), ((100, 10, 256), (5, 1, 256), F32),
                   ((65, 19, 130), (13, 19, 1), F32)],
    (2, 6, 6, 2): [((84, 12, 256), (6, 4, 1), F32), ((34, 45, 131), (2, 9, 131), F32)],
    (2, 7, 6, 2): [((98, 12, 256), (14, 12, 2), F32), ((41, 58, 129), (41, 58, 129), F32)],
    (2, 8, 7, 2): [((32, 518, 256), (1, 37, 64), F32), ((46, 41, 131), (1, 41, 131), F32)],
    (4, 4, 4, 2): [((64, 16, 512), (32, 8, 256), F32), ((47, 22, 259), (1, 1, 7), F32)],
    (4, 5, 5, 2): [((20, 50, 512), (1, 5, 1), F32), ((19, 55, 259), (1, 1, 7), F32)],
}
ITERS, EVERY = 23, 7                # odd and even stretches between norms, and iterations behind the last one


@pytest.mark.parametrize("variant,dims,tiles,dtype", [(v, *c) for v, cases in VARIANTS.items() for c in cases])
def test_every_variant_matches_the_oracle(H, oracle_mod, variant, dims, tiles, dtype):
    a = random_padded(dims, dtype=dtype, seed=sum(dims))
    ref, ref_res = oracle_mod.run(a, ITERS, EVERY)
    r = H.JacobiRun(dims, tiles, dtype, resident=1, profile=1)
    try:
        got = tuple(H.B.jacobi_get_option(r.plan, "chip_" + k) for k in ("cells_per_lane", "planes_per_wave", "rows_per_wave", "waves_per_row"))
        assert got == variant
        for _ in range(2):
            r.load(a)
            r.other().fill_(255)            # NaN: the other grid's ring has to come from the run
            res = r.run(ITERS, EVERY, fuse_residual=True)
            check(r.fetch(), res, ref, ref_res)
            assert H.B.jacobi_profile_read(r.plan)[1] == 1             # one launch
        if dtype == F32:
            out = r.fetch()
            r.set_option("resident", 0)
            r.load(a)
            r.run(ITERS, EVERY, fuse_residual=True)
            assert np.array_equal(r.fetch(), out)
    finally:
        r.close()


@pytest.mark.parametrize("variant,dims,tiles,dtype", [(v, *c) for v, cases in GHOST_VARIANTS.items() if v[1] for c in cases])
def test_variants_with_ghost_cells_match_the_oracle(H, oracle_mod, variant, dims, tiles, dtype):
    """Option chip = 0: blocks3d_kernel, also where a call would run without ghost cells."""
    a = random_padded(dims, dtype=dtype, seed=sum(dims))
    ref, ref_res = oracle_mod.run(a, VARIANT_ITERS, VARIANT_EVERY)
    out, res, _ = run_whole(H, a, tiles, VARIANT_ITERS, VARIANT_EVERY, resident=1, chip=0)
    check(out, res, ref, ref_res)


PLAIN = [((64, 64, 64), (2, 2, 2), F64), ((96, 90, 100), (1, 3, 2), F32), ((61, 53, 47), (1, 1, 1), F64)]


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_without_all_workgroups_the_plain_path_is_taken(H, oracle_mod, dims, tiles, dtype):
    """As for the other block kernels: fewer workgroups do the work through memory, with the same result, and the next launch
    finds the plan's words as it needs them."""
    a = random_padded(dims, dtype=dtype, seed=77)
    r = H.JacobiRun(dims, tiles, dtype, resident=1)
    try:
        n = H.B.jacobi_get_option(r.plan, "chip_workgroups")
        for iters, every in ((30, 3), (23, 0)):
            ref, ref_res = oracle_mod.run(a, iters, every)
            norms = {}
            for admitted in (0, 1, n // 2, n - 1, 0, n - 1):
                r.set_option("resident_admitted", admitted)
                r.load(a)
                r.other().fill_(255)
                res = r.run(iters, every, fuse_residual=True) if every else (r.sweep(iters) or [])
                check(r.fetch(), res, ref, ref_res)
                assert norms.setdefault(admitted, res) == res, (iters, every, admitted)
        r.set_option("resident_admitted", 0)
        for limit in (1, 1, 0):                            # the roll is called once, without waiting
            r.set_option("resident_spin_limit", limit)
            r.load(a)
            r.sweep(23)
            check(r.fetch(), [], ref, ref_res)
    finally:
        r.close()


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_tags_that_come_round(H, oracle_mod, dims, tiles, dtype):
    """More exchanges than there are tags, launches of all lengths one after the other, with and without ghost cells by turns (they share
    the plan's words): other fields each time, so that a message left over would show."""
    r = H.JacobiRun(dims, tiles, dtype, resident=1)
    try:
        for k, (iters, chip) in enumerate(((600, 1), (15, 1), (16, 0), (255, 1), (17, 1), (254, 0), (256, 1), (40, 1), (40, 1))):
            a = random_padded(dims, dtype=dtype, seed=100 + k)
            ref, ref_res = oracle_mod.run(a, iters, iters // 2)
            r.set_option("chip", chip)
            r.load(a)
            res = r.run(iters, iters // 2, fuse_residual=True)
            check(r.fetch(), res, ref, ref_res)
    finally:
        r.close()


@pytest.mark.parametrize("dims", [(26, 78, 58), (66, 30, 33), (38, 62, 54)])
def test_a_launch_without_ghost_cells_leaves_the_epoch_alone(H, oracle_mod, dims):
    """Both kinds of launch share the epoch, not the messages: one without ghost cells, however low the limit is set for it, must not have
    those with ghost cells count through tags again that their messages still carry.  Calls of one exchange, whose words nothing has
    overwritten when the tag would come again; other fields each time, so that one of those words would show."""
    r = H.JacobiRun(dims, (1, 1, 1), F32, resident=1, profile=1)
    try:
        assert H.B.jacobi_get_option(r.plan, "block_depth") == 2
        for k, (chip, limit, iters) in enumerate([(0, 0, 4), (1, 1, 40), (0, 0, 4), (1, 1, 40), (0, 0, 4), (0, 0, 30), (1, 1, 40), (0, 0, 30)]):
            a = random_padded(dims, dtype=F32, seed=200 + k)
            r.set_option("chip", chip)
            r.set_option("resident_epoch_limit", limit)
            r.load(a)
            r.sweep(iters)
            check(r.fetch(), [], oracle_mod.run(a, iters)[0], [])
            assert H.B.jacobi_profile_read(r.plan)[1] == 1
    finally:
        r.close()


@pytest.mark.parametrize("iters,every,opts", [(9, 0, {}), (10, 1, {}), (20, 3, dict(tblock=4)), (21, 21, dict(fused=0)), (300, 2, {})])
def test_short_calls_parity_of_the_buffers_and_many_norms(H, oracle_mod, iters, every, opts):
    dims, tiles = (61, 53, 47), (1, 1, 1)
    a = random_padded(dims, seed=iters)
    ref, ref_res = oracle_mod.run(a, iters, every)
    out, res, in_a = run_whole(H, a, tiles, iters, every, resident=1, **opts)
    check(out, res, ref, ref_res)
    out0, _, in_a0 = run_whole(H, a, tiles, iters, every, resident=0, **opts)
    assert np.array_equal(out, out0) and in_a == in_a0


def test_special_values_spread_as_by_launches(H):
    for dims in ((64, 60, 63), (60, 58, 101)):
        a = random_padded(dims, seed=9)
        for at, v in (((10, 20, 30), np.inf), ((33, 0, 17), -np.inf), ((4, 5, dims[2] + 1), np.nan), ((0, 7, 9), np.inf),
                      ((dims[0] + 1, 25, 2), np.nan), ((31, 31, 1), -0.0), ((1, 1, 50), 5e-324)):
            a[at] = v
        got = [run_whole(H, a, (1, 1, 1), 17, 5, resident=k) for k in (1, 0)]
        assert np.array_equal(got[0][0], got[1][0], equal_nan=True)
        assert np.array_equal(np.isnan(got[0][1]), np.isnan(got[1][1]))


def test_plans_and_streams_beside_each_other_and_graphs(H, oracle_mod):
    """Two plans on two streams, whose workgroups together are more than the chip has CUs; calls recorded into a graph run by launches."""
    import torch
    dims, tiles = (108, 108, 108), ((1, 1, 1), (2, 3, 4))
    fields = [random_padded(dims, seed=12 + k) for k in range(2)]
    refs = [oracle_mod.run(f, 40)[0] for f in fields]
    q = [H.JacobiRun(dims, t, resident=1) for t in tiles]
    streams = [torch.cuda.Stream() for _ in range(2)]
    try:
        for _ in range(3):
            for r, f in zip(q, fields):
                r.load(f)
            torch.cuda.synchronize()
            for r, s in zip(q, streams):
                with torch.cuda.stream(s):
                    r.sweep(40)
            torch.cuda.synchronize()
            for r, ref in zip(q, refs):
                assert np.array_equal(r.fetch(), ref)
        r = q[0]
        dev = torch.from_numpy(fields[0]).cuda()
        exp, exp_res = oracle_mod.run(fields[0], 10, 5)
        res = torch.zeros(2, dtype=torch.float64, device="cuda")
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            st = int(torch.cuda.current_stream().cuda_stream)
            H.B.jacobi_scatter(r.plan, dev.data_ptr(), r.a.data_ptr(), st)
            fin = H.B.jacobi_run(r.plan, r.a.data_ptr(), r.b.data_ptr(), 10, 5, res.data_ptr(), st)
        for _ in range(3):
            res.zero_()
            graph.replay()
            torch.cuda.synchronize()
            r.cur = r.a if fin == r.a.data_ptr() else r.b
            check(r.fetch(), res.cpu().tolist(), exp, exp_res)
            r.load(fields[0])
            r.sweep(20)                          # eager calls, in one launch each, between the replays
    finally:
        for r in q:
            r.close()
