"""jacobi_run in blocked 2-D passes whose last pass also delivers the norm of its result (one more level of the pipeline).
fp64 grids bit for bit against the CPU oracle, fp32 within 1e-5*max|u|, norms within 1e-12 / 1e-5 (the bars of the other suites).
Every depth of the last pass, with and without a norm of its source due from the same pass (beyond 7 only grids of at least 240 MiB
take it: those against passes of one iteration); heights around the strips' and the pipeline's ends, tiles exactly one row too low
for the additional level, columns that end inside and at a wavefront's own."""
import numpy as np
import pytest

from parity_util import random_padded
from test_parity_gpu import check

pytestmark = pytest.mark.gpu

F64, F32 = np.float64, np.float32
# (interior dims, tiles, type): 8 rows a tile take the additional level up to depth 7
SHAPES = [((13, 2), (1, 1), F64), ((52, 208), (4, 1), F64), ((39, 210), (3, 105), F64), ((129, 330), (1, 3), F64),
          ((16, 224), (2, 2), F64), ((52, 472), (4, 2), F32), ((131, 228), (1, 3), F32), ((8, 236), (1, 59), F32)]


@pytest.mark.parametrize("depth", range(2, 9))
@pytest.mark.parametrize("dims,tiles,dtype", SHAPES)
def test_last_norm_from_the_last_pass(H, oracle_mod, dims, tiles, dtype, depth):
    a = random_padded(dims, dtype=dtype, seed=sum(dims) + depth)
    for iters, every in ((depth, depth), (2 * depth, depth)):         # the last pass: its result's norm; its source's as well
        ref, ref_res = oracle_mod.run(a, iters, every)
        for strip in (0, 1, 5):
            r = H.JacobiRun(dims, tiles, dtype, tblock=depth, resident=0)
            try:
                r.set_option("rows_per_strip", strip)
                r.load(a)
                r.other().fill_(255)        # NaN
                res = r.run(iters, every, fuse_residual=True)
                check(r.fetch(), res, ref, ref_res)
            finally:
                r.close()


LARGE = [((5720, 5634), (8, 3), F64), ((5605, 5798), (5, 1), F64), ((8113, 8008), (7, 11), F32)]


@pytest.mark.parametrize("depth", range(8, 13))
@pytest.mark.parametrize("dims,tiles,dtype", LARGE)
def test_deep_last_passes(H, dims, tiles, dtype, depth):
    a = random_padded(dims, dtype=dtype, seed=depth)
    results = []
    for tblock in (1, depth):
        r = H.JacobiRun(dims, tiles, dtype, tblock=tblock, resident=0)
        try:
            assert r.nbytes >= 240 << 20
            r.load(a)
            r.other().fill_(255)        # NaN
            norms = [r.run(depth, depth, fuse_residual=True)]
            norms.append(r.run(2 * depth, depth, fuse_residual=True))
            results.append((r.fetch(), np.concatenate(norms)))
        finally:
            r.close()
    assert np.array_equal(results[0][0], results[1][0])
    np.testing.assert_allclose(results[1][1], results[0][1], rtol=1e-12 if dtype == F64 else 1e-5)


# the three-dimensional passes of 3 iterations, taken from grids of 24 MiB on: planes, rows and columns at the ends of what a workgroup and
# a wavefront own; the last ones with a norm of the source due from the same pass, which keeps the pass of its own
SHAPES_3D = [((64, 65, 800), (1, 1, 1)), ((3, 1030, 1130), (1, 1, 5)), ((126, 161, 226), (9, 7, 1)), ((33, 352, 366), (11, 11, 61)), ((120, 97, 360), (24, 1, 3))]


@pytest.mark.parametrize("dims,tiles", SHAPES_3D)
def test_last_norm_from_the_last_3d_pass(H, oracle_mod, dims, tiles):
    a = random_padded(dims, dtype=F64, seed=sum(dims))
    for iters, every, tblock, strip in ((3, 3, 3, 0), (3, 3, 3, 1), (10, 10, 4, 0), (10, 10, 4, 3), (6, 3, 3, 0)):
        ref, ref_res = oracle_mod.run(a, iters, every)
        r = H.JacobiRun(dims, tiles, F64, tblock=tblock, resident=0)
        try:
            assert r.nbytes >= 24 << 20
            r.set_option("rows_per_strip", strip)
            r.load(a)
            r.other().fill_(255)        # NaN
            res = r.run(iters, every, fuse_residual=True)
            check(r.fetch(), res, ref, ref_res)
        finally:
            r.close()
