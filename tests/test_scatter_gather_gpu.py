"""jacobi_scatter and jacobi_gather cell by cell: every padded cell of every tile against the padded global array,
and back into a destination at any element alignment, with guard cells on both sides.  Sizes at the edges of what
the kernels move at once: rows shorter than a vector, one cell more or less than a vector, a wavefront or a
workgroup's share of a row, tiles one cell wide, seams inside a vector.  Copies: exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [
    ((1, 1), (1, 1)), ((1, 2), (1, 2)), ((3, 5), (1, 1)), ((4, 7), (2, 7)), ((6, 9), (3, 3)), ((5, 30), (5, 10)),
    ((8, 126), (2, 1)), ((8, 127), (1, 1)), ((8, 254), (1, 2)), ((3, 257), (1, 1)), ((2, 1022), (1, 2)), ((2, 1023), (2, 1)),
    ((3, 2050), (1, 2)), ((2, 4094), (1, 1)), ((2, 8190), (1, 2)), ((1030, 3), (2, 1)), ((700, 2), (7, 1)),
    ((1, 1, 1), (1, 1, 1)), ((3, 4, 5), (3, 2, 5)), ((6, 10, 14), (2, 2, 2)), ((5, 7, 9), (1, 1, 1)), ((4, 6, 130), (2, 3, 1)),
    ((8, 8, 66), (2, 2, 11)), ((2, 130, 258), (1, 2, 3)),
]


def expected_tiles(a, lay):
    """Yields (tile, padded block of the global array) for a padded 2-D or 3-D array."""
    full = a if a.ndim == 3 else a[None]
    td, th, tw = lay.tile
    pk = 2 if lay.ndim == 3 else 0
    for t in range(lay.ntiles):
        tz, ty, tx = t // (lay.tiles[1] * lay.tiles[2]), t // lay.tiles[2] % lay.tiles[1], t % lay.tiles[2]
        yield t, full[tz * td:(tz * td + td + pk) if pk else 1, ty * th:ty * th + th + 2, tx * tw:tx * tw + tw + 2]


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("dims,tiles", SHAPES)
def test_scatter_gather_cells(H, dims, tiles, dtype):
    import torch
    a = (np.arange(np.prod([n + 2 for n in dims]), dtype=np.float64) + 1.0).reshape([n + 2 for n in dims]).astype(dtype)
    for streaming in (0, 2):
        r = H.JacobiRun(dims, tiles, dtype, nontemporal=streaming)
        try:
            lay = H.B.jacobi_get_layout(r.plan)
            stream = int(torch.cuda.current_stream().cuda_stream)
            for off in range(0, 5):
                src = torch.full((a.size + 16,), -1.0, dtype=torch.from_numpy(a).dtype, device="cuda")
                src[off:off + a.size] = torch.from_numpy(a).reshape(-1).cuda()
                r.a.zero_()
                H.B.jacobi_scatter(r.plan, src[off:].data_ptr(), r.a.data_ptr(), stream)
                raw = r.a.cpu().numpy().view(dtype)
                for t, block in expected_tiles(a, lay):
                    base = t * lay.tile_stride
                    n = lay.nplanes * (lay.tile[1] + 2)
                    rows = raw[base:base + n * lay.pitch].reshape(n, lay.pitch)[:, :lay.tile[2]]
                    flat = block.reshape(n, lay.tile[2] + 2)
                    assert np.array_equal(rows, flat[:, 1:-1]), (t, off)
                    assert np.array_equal(raw[base + lay.xhalo_offset:][:n], flat[:, 0]), (t, off)
                    assert np.array_equal(raw[base + lay.xhalo_offset + lay.xhalo_pitch:][:n], flat[:, -1]), (t, off)
                dst = torch.full((a.size + 40,), -7.0, dtype=src.dtype, device="cuda")
                H.B.jacobi_gather(r.plan, r.a.data_ptr(), dst[17 + off:].data_ptr(), stream)
                got = dst.cpu().numpy()
                assert np.array_equal(got[17 + off:17 + off + a.size], a.reshape(-1)), off
                assert np.all(got[:17 + off] == -7.0) and np.all(got[17 + off + a.size:] == -7.0), off
        finally:
            r.close()


def test_gather_ignores_the_copies_of_neighbours_cells(H):
    """Inter-tile halo cells may be stale: filled with NaN, they do not show in the gathered array."""
    import torch
    for dims, tiles in (((12, 20), (3, 5)), ((6, 8, 12), (2, 2, 3))):
        r = H.JacobiRun(dims, tiles)
        try:
            a = np.random.default_rng(4).uniform(-1, 1, [n + 2 for n in dims])
            r.load(a)
            lay = H.B.jacobi_get_layout(r.plan)
            g = r.a.view(torch.float64)
            raw = g.cpu().numpy().copy()
            for t in range(lay.ntiles):
                pos = (t // (lay.tiles[1] * lay.tiles[2]), t // lay.tiles[2] % lay.tiles[1], t % lay.tiles[2])
                n = lay.nplanes * (lay.tile[1] + 2)
                base = t * lay.tile_stride
                rows = raw[base:base + n * lay.pitch].reshape(lay.nplanes, lay.tile[1] + 2, lay.pitch)
                if lay.ndim == 3 and pos[0] > 0: rows[0] = np.nan
                if lay.ndim == 3 and pos[0] < lay.tiles[0] - 1: rows[-1] = np.nan
                if pos[1] > 0: rows[:, 0] = np.nan
                if pos[1] < lay.tiles[1] - 1: rows[:, -1] = np.nan
                if pos[2] > 0: raw[base + lay.xhalo_offset:][:n] = np.nan
                if pos[2] < lay.tiles[2] - 1: raw[base + lay.xhalo_offset + lay.xhalo_pitch:][:n] = np.nan
            g.copy_(torch.from_numpy(raw).cuda())
            assert np.array_equal(r.fetch(), a)
        finally:
            r.close()


def test_scatter_gather_of_more_tiles_than_one_launch_takes(H):
    """2^24 one-row tiles and some (15 GB): the scatter runs as two launches.  Out and back again, and a row of cells in between."""
    import torch
    n = (1 << 24) + 300
    r = H.JacobiRun((n, 3), (n, 1))
    try:
        stream = int(torch.cuda.current_stream().cuda_stream)
        a = torch.arange((n + 2) * 5, dtype=torch.float64, device="cuda").reshape(n + 2, 5)
        out = torch.zeros_like(a)
        H.B.jacobi_scatter(r.plan, a.data_ptr(), r.a.data_ptr(), stream)
        H.B.jacobi_gather(r.plan, r.a.data_ptr(), out.data_ptr(), stream)
        assert torch.equal(out, a)
        lay = H.B.jacobi_get_layout(r.plan)
        tiles = r.a.view(torch.float64)[:n * lay.tile_stride].view(n, lay.tile_stride)
        for k in range(3):                                   # the halo rows, too
            assert torch.equal(tiles[:, k * lay.pitch:k * lay.pitch + 3], a[k:k + n, 1:4])
    finally:
        r.close()


def test_gather_of_more_rows_than_one_launch_takes(H):
    """2^26 rows and some, a wavefront each (grid 8.7 GB): the gather runs as two launches, and rows on both sides of their seam arrive."""
    import torch
    n = (1 << 26) + 136
    r = H.JacobiRun((n, 3), (1000, 1))
    try:
        stream = int(torch.cuda.current_stream().cuda_stream)
        a = torch.arange((n + 2) * 5, dtype=torch.float64, device="cuda").reshape(n + 2, 5)
        out = torch.zeros_like(a)
        H.B.jacobi_scatter(r.plan, a.data_ptr(), r.a.data_ptr(), stream)
        H.B.jacobi_gather(r.plan, r.a.data_ptr(), out.data_ptr(), stream)
        assert torch.equal(out, a)
    finally:
        r.close()
