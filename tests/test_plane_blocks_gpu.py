"""Cooperative 3-D blocked passes: a workgroup's block of planes begins and ends anywhere in the column of tiles, and row groups
take turns with column segments in bands of four.  fp64 grids bit for bit against the CPU oracle, fp32 within 1e-5*max|u|, norms within
1e-12 / 1e-5 (the bars of the other suites).  Blocks that begin and end on, before and behind the seam of two tiles, tiles as deep as the
pass, blocks longer than a tile, over one, two and all seams (given, and as the library chooses them), a last block of one plane; one row group, exactly
a band, a band and a part of one, each with several segments."""
import numpy as np
import pytest

from parity_util import random_padded
from test_parity_gpu import check

pytestmark = pytest.mark.gpu

F64, F32 = np.float64, np.float32


@pytest.mark.parametrize("dims,tiles,dtype,depth", [((16, 33, 122), (4, 1, 1), F64, 4), ((21, 130, 250), (3, 2, 5), F64, 3), ((21, 168, 140), (7, 4, 7), F64, 3),
                                                    ((29, 129, 242), (1, 3, 1), F64, 4), ((25, 200, 362), (5, 5, 1), F64, 4), ((21, 171, 484), (7, 3, 1), F32, 3),
                                                    ((16, 30, 250), (4, 1, 1), F64, 4), ((21, 40, 500), (7, 2, 1), F32, 3), ((36, 200, 720), (9, 1, 1), F64, 4), ((33, 352, 366), (11, 11, 61), F64, 3)])
def test_blocks_of_planes_across_tiles(H, oracle_mod, dims, tiles, dtype, depth):
    a = random_padded(dims, dtype=dtype, seed=sum(dims))
    for iters, every in ((2 * depth, 0), (2 * depth, depth)):
        ref, ref_res = oracle_mod.run(a, iters, every)
        td = dims[0] // tiles[0]
        for strip in sorted({0, 1, 2, td - 1, td + 1, 2 * td + 1, dims[0] - 1, 4096}):
            r = H.JacobiRun(dims, tiles, dtype, tblock=depth, resident=0)
            try:
                r.set_option("rows_per_strip", strip)
                r.load(a)
                r.other().fill_(255)        # NaN
                res = r.run(iters, every, fuse_residual=True)
                check(r.fetch(), res, ref, ref_res)
            finally:
                r.close()
