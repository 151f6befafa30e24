"""The path that runs a whole jacobi_run of a large 2-D grid in one launch, the grid in the chip's registers and LDS, without
ghost cells.  fp64 grids bit for bit against the CPU oracle, fp32 within 1e-5*max|u|, norms within 1e-12 / 1e-5 (the bars of
the other suites).  Shapes: every compiled variant; blocks that end where the next one begins, that overlap by whole lanes, by single
cells, by rows; widths that no lane's cells divide; tiles one cell wide or high, seams inside a lane's cells."""
import numpy as np
import pytest

from parity_util import random_padded
from test_blocks_gpu import run_whole
from test_parity_gpu import check

pytestmark = pytest.mark.gpu

F64, F32 = np.float64, np.float32
# (rows per wavefront in registers, even cut): [(interior dims, tiles, type)]
VARIANTS = {
    (8, 0): [((735, 2045), (5, 5), F64), ((1501, 1501), (1, 1501), F64), ((127, 8155), (1, 7), F32), ((1601, 1607), (1601, 1), F32)],
    (8, 1): [((2048, 2544), (64, 3), F32), ((2560, 3072), (1, 1), F32)],
    (12, 0): [((1604, 2523), (4, 3), F64), ((2052, 3928), (3, 491), F32)],
    (12, 1): [((2304, 2304), (8, 8), F64), ((5952, 1368), (31, 9), F32)],
    (16, 0): [((4959, 1200), (1, 8), F64), ((2601, 2601), (1, 1), F64), ((4036, 2904), (4, 33), F32)],
    (16, 1): [((3584, 1280), (7, 20), F64), ((2560, 2560), (1, 5), F64), ((3328, 2392), (2, 13), F32)],
    (20, 0): [((5508, 1456), (27, 13), F64), ((3259, 4952), (1, 4), F32)],
    (20, 1): [((1600, 4088), (1, 7), F64), ((1600, 5624), (8, 19), F32)],
    (24, 0): [((4063, 2480), (1, 20), F64), ((3101, 3101), (7, 7), F64), ((4027, 4952), (1, 8), F32)],
    (24, 1): [((5568, 1200), (3, 3), F64), ((2496, 5120), (13, 5), F32)],
    (23, 0): [((4959, 2480), (9, 31), F64), ((3501, 3501), (3, 9), F64), ((4987, 4952), (1, 1), F32)],
    (23, 1): [((4096, 2560), (16, 1), F64), ((4096, 4096), (4, 4), F64), ((4096, 5120), (2, 64), F32)],
}
ITERS, EVERY = 17, 5                # odd and even stretches between norms, and some iterations behind the last one


@pytest.mark.parametrize("variant,dims,tiles,dtype", [(v, *c) for v, cases in VARIANTS.items() for c in cases])
def test_every_variant_matches_the_oracle(H, oracle_mod, variant, dims, tiles, dtype):
    a = random_padded(dims, dtype=dtype, seed=sum(dims))
    ref, ref_res = oracle_mod.run(a, ITERS, EVERY)
    r = H.JacobiRun(dims, tiles, dtype, resident=1, profile=1)
    try:
        assert tuple(H.B.jacobi_get_option(r.plan, "chip_" + k) for k in ("rows_in_registers", "even")) == variant
        for _ in range(2):
            r.load(a)
            r.other().fill_(255)            # NaN: the other grid's ring has to come from the run
            res = r.run(ITERS, EVERY, fuse_residual=True)
            check(r.fetch(), res, ref, ref_res)
            assert H.B.jacobi_profile_read(r.plan)[1] == 1             # one launch
        if dtype == F32:                                               # the same bits as by launches
            out = r.fetch()
            r.set_option("resident", 0)
            r.load(a)
            r.run(ITERS, EVERY, fuse_residual=True)
            assert np.array_equal(r.fetch(), out)
    finally:
        r.close()


# Widths at which the middle one of three columns of blocks would have, in one lane, the cell that the block W of it needs and the one the
# block E of it needs: by launches (False) where four columns are more blocks than CUs
BOTH_WAYS = [((8160, 516), (5, 3), F64, True), ((8192, 516), (1, 1), F64, True), ((9000, 513), (9, 19), F64, True),
             ((14000, 513), (1, 1), F64, True), ((16384, 516), (1, 129), F64, True), ((17000, 513), (17, 1), F64, False),
             ((5250, 1032), (1, 1), F32, True), ((8160, 1032), (8, 4), F32, True), ((9000, 1032), (1, 43), F32, True),
             ((4096, 1025), (1, 5), F32, True), ((6000, 1025), (3, 1), F32, True), ((17000, 1032), (1, 1), F32, False)]


@pytest.mark.parametrize("dims,tiles,dtype,whole", BOTH_WAYS)
def test_widths_just_over_two_blocks(H, oracle_mod, dims, tiles, dtype, whole):
    a = random_padded(dims, dtype=dtype, seed=sum(dims))
    ref, ref_res = oracle_mod.run(a, ITERS, EVERY)
    outs = []
    for resident in (1, 0):
        r = H.JacobiRun(dims, tiles, dtype, resident=resident, profile=1)
        try:
            r.load(a)
            r.other().fill_(255)
            res = r.run(ITERS, EVERY, fuse_residual=True)
            assert (H.B.jacobi_profile_read(r.plan)[1] == 1) == (bool(resident) and whole)
            outs.append(r.fetch())
            check(outs[-1], res, ref, ref_res)
        finally:
            r.close()
    assert np.array_equal(*outs)


PLAIN = [((2304, 2304), (8, 8), F64), ((1601, 1607), (1, 1), F32)]


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_without_all_workgroups_the_plain_path_is_taken(H, oracle_mod, dims, tiles, dtype):
    """As for the other block kernels: fewer workgroups do the work through memory, with the same result, and the next launch
    finds the plan's words as it needs them.  (Norms add up other workgroups' sums, in another order.)"""
    a = random_padded(dims, dtype=dtype, seed=77)
    r = H.JacobiRun(dims, tiles, dtype, resident=1)
    try:
        n = H.B.jacobi_get_option(r.plan, "chip_workgroups")
        for iters, every in ((9, 3), (8, 0)):
            ref, ref_res = oracle_mod.run(a, iters, every)
            norms = {}
            for admitted in (0, n // 2, n - 1, 0, n - 1):
                r.set_option("resident_admitted", admitted)
                r.load(a)
                r.other().fill_(255)
                res = r.run(iters, every, fuse_residual=True) if every else (r.sweep(iters) or [])
                check(r.fetch(), res, ref, ref_res)
                assert norms.setdefault(admitted, res) == res, (iters, every, admitted)
        r.set_option("resident_admitted", 0)
        r.set_option("resident_spin_limit", 1)             # the roll is called once, without waiting
        for limit in (1, 1, 0):
            r.set_option("resident_spin_limit", limit)
            r.load(a)
            r.sweep(8)
            check(r.fetch(), [], ref, ref_res)
    finally:
        r.close()


@pytest.mark.parametrize("dims,tiles,dtype", PLAIN)
def test_exchanges_are_counted_from_zero_again(H, oracle_mod, dims, tiles, dtype):
    """Launches clear the messages and start with the same tags: other fields each time, so that a message left over would show."""
    r = H.JacobiRun(dims, tiles, dtype, resident=1)
    try:
        for limit in (1, 50):
            r.set_option("resident_epoch_limit", limit)
            for k in range(4):
                a = random_padded(dims, dtype=dtype, seed=100 + k)
                ref, ref_res = oracle_mod.run(a, 20, 10)
                r.load(a)
                res = r.run(20, 10, fuse_residual=True)
                check(r.fetch(), res, ref, ref_res)
    finally:
        r.close()


@pytest.mark.parametrize("iters,every,opts", [(1, 0, {}), (1, 1, {}), (2, 1, {}), (3, 0, {}), (20, 3, dict(tblock=8)), (21, 21, dict(fused=0)),
                                              (260, 2, {})])
def test_short_calls_parity_of_the_buffers_and_many_norms(H, oracle_mod, iters, every, opts):
    """The result lies in the buffer in which the passes would leave it; more norms than one launch delivers."""
    dims, tiles = (1501, 1501), (1, 19)
    a = random_padded(dims, seed=iters)
    ref, ref_res = oracle_mod.run(a, iters, every)
    out, res, in_a = run_whole(H, a, tiles, iters, every, resident=1, **opts)
    check(out, res, ref, ref_res)
    out0, _, in_a0 = run_whole(H, a, tiles, iters, every, resident=0, **opts)
    assert np.array_equal(out, out0) and in_a == in_a0


def test_special_values_spread_as_by_launches(H):
    a = random_padded((2304, 2305), seed=9)
    for at, v in (((100, 200), np.inf), ((1153, 0), -np.inf), ((400, 2306), np.nan), ((0, 1024), np.inf), ((2305, 257), np.nan),
                  ((768, 256), -0.0), ((769, 1), 5e-324)):
        a[at] = v
    got = [run_whole(H, a, (1, 5), 23, 10, resident=k) for k in (1, 0)]
    assert np.array_equal(got[0][0], got[1][0], equal_nan=True)
    assert np.array_equal(np.isnan(got[0][1]), np.isnan(got[1][1]))


def test_plans_grids_and_threads_beside_each_other(H, oracle_mod):
    """Two plans on two streams, whose workgroups together are more than the chip has CUs; one plan, two pairs of grids, calls from
    two threads on two streams: its launches follow each other."""
    import threading

    import torch
    dims = (2304, 2304)
    fields = [random_padded(dims, seed=12 + k) for k in range(2)]
    refs = [oracle_mod.run(f, 30)[0] for f in fields]
    q = [H.JacobiRun(dims, t, resident=1) for t in ((1, 1), (8, 8))]
    other = H.JacobiRun(dims, (1, 1), resident=1)                    # its grids only
    streams = [torch.cuda.Stream() for _ in range(2)]
    try:
        for _ in range(3):
            for r, f in zip(q, fields):
                r.load(f)
            torch.cuda.synchronize()
            for r, s in zip(q, streams):
                with torch.cuda.stream(s):
                    r.sweep(30)
            torch.cuda.synchronize()
            for r, ref in zip(q, refs):
                assert np.array_equal(r.fetch(), ref)
        pair = [q[0], other]
        for _ in range(3):
            for r, f in zip(pair, fields):
                r.load(f)
            torch.cuda.synchronize()
            fins = [None, None]

            def call(k):
                for n in (10, 10, 10):
                    g = pair[k]
                    fin = H.B.jacobi_sweep(q[0].plan, g.cur.data_ptr(), g.other().data_ptr(), n, int(streams[k].cuda_stream))
                    g.cur = g.a if fin == g.a.data_ptr() else g.b
                fins[k] = True
            threads = [threading.Thread(target=call, args=(k,)) for k in range(2)]
            [t.start() for t in threads]
            [t.join() for t in threads]
            torch.cuda.synchronize()
            assert all(fins)
            for r, ref in zip(pair, refs):
                assert np.array_equal(r.fetch(), ref)
    finally:
        for r in (*q, other):
            r.close()


def test_in_a_hip_graph_calls_run_by_launches(H, oracle_mod):
    import torch
    a = random_padded((2304, 2304), seed=3)
    ref, ref_res = oracle_mod.run(a, 10, 5)
    r = H.JacobiRun((2304, 2304), (8, 8), resident=1)
    try:
        H.B.jacobi_prepare(r.plan)
        dev = torch.from_numpy(a).cuda()
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
            check(r.fetch(), res.cpu().tolist(), ref, ref_res)
            r.load(a)
            r.sweep(20)                          # eager calls, in one launch each, between the replays
    finally:
        r.close()
