// Device code used only by the host API translation unit: the final stage of the residual
// reduction, halo / boundary face copies, scatter / gather, and the plain copy probe.
#pragma once
#include "jacobi_kernels.h"

namespace jk {

// Final stage of the residual: one workgroup adds the per-workgroup partials in a fixed
// order (thread t takes t, t+1024, ... into eight running sums by turns, so that eight loads are in
// flight instead of one - 32768 partials took 17-35 us with a single sum -; then a fixed tree over the
// eight, the shuffle tree and LDS) and writes the sqrt.
__global__ __launch_bounds__(1024) void residual_final_kernel(const double *__restrict__ partial,
                                                              long long n, double *__restrict__ result)
{
    __shared__ double red[16];
    constexpr int U = 8;
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.0;
    const long long step = blockDim.x;
    long long i = threadIdx.x;
    for (; i + (U - 1) * step < n; i += U * step) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = partial[i + u * step];
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] += v[u];
    }
#pragma unroll
    for (int u = 0; u < U - 1; ++u)                                   // fewer than U left
        if (i + u * step < n) acc[u] += partial[i + u * step];
    const double mine = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    const double tot = wg_sum(mine, red);
    if (threadIdx.x == 0) *result = sqrt(tot);
}

// ------------------------------------------------------------------------------------
// Boundary copy.  A face of a tile is one of its 2*ndim halo faces (0: x-, 1: x+, 2: y-, 3: y+, 4: z-,
// 5: z+).  For every face that lies on the domain boundary, the Dirichlet halo cells are copied from the
// `src` grid to the `dst` grid - the full padded extent of the face, with its edges and corners, so that
// the destination carries the complete ring.  Work item = (tile, face, chunk of 4*WG cells); workgroups
// stride over the item list.
// ------------------------------------------------------------------------------------
constexpr int FACE_CHUNK = 4 * WG;

template <typename T>
__global__ __launch_bounds__(WG) void boundary_copy_kernel(Geo g, const T *__restrict__ src, T *__restrict__ dst,
                                                           int chunks_per_face, long long nitems)
{
    const int nfaces = 2 * g.ndim;
    for (long long item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int chunk = (int)(item % chunks_per_face);
        const long long tf = item / chunks_per_face;
        const int face = (int)(tf % nfaces), t = (int)(tf / nfaces);
        const int axis = face >> 1, hi = face & 1;   // axis 0: x, 1: y, 2: z
        const int tz = t / (g.Ty * g.Tx), ty = (t / g.Tx) % g.Ty, tx = t % g.Tx;
        const int tc = axis == 0 ? tx : axis == 1 ? ty : tz;
        const int Tn = axis == 0 ? g.Tx : axis == 1 ? g.Ty : g.Tz;
        if (hi ? tc < Tn - 1 : tc > 0) continue;     // a neighbouring tile, not the boundary
        const long long tile = (long long)t * g.tile_stride;
        // face cells are indexed (a, b) with b fastest, over the padded extent
        const int nb = axis == 0 ? g.rows : g.tw;
        const int na = axis == 2 ? g.rows : g.nplanes;
        const long long n = (long long)na * nb;
        const long long base = (long long)chunk * FACE_CHUNK;
        for (int q = 0; q < 4; ++q) {
            const long long e = base + q * WG + threadIdx.x;
            if (e >= n) break;
            const int a = (int)(e / nb), b = (int)(e - (long long)a * nb);
            const long long off = axis == 0   ? (hi ? xp_off(g, a, b) : xm_off(g, a, b))      // (plane, row)
                                  : axis == 1 ? main_off(g, a, hi ? g.th + 1 : 0, b)          // (plane, column)
                                              : main_off(g, hi ? g.td + 1 : 0, a, b);         // (row, column)
            dst[tile + off] = src[tile + off];
        }
    }
}

// ------------------------------------------------------------------------------------
// Stand-alone halo exchange (paper Sec. VI-C: pack, transfer, unpack - one copy on one device): for every
// face of every tile that has a neighbour, halo cells <- the neighbour's edge cells, in place in one grid.
// y and z faces are rows of the neighbour (contiguous, cache-line aligned): copied as 16-byte vectors, whole
// vectors (the padding columns behind a row may hold anything and are overwritten with the source's).
// x faces, XSRC = 0: gathered from the neighbour's first / last column, one cell per row (one cell per cache
// line: 16 times the payload is read; always valid).  XSRC = 1: copied from the neighbour's dense x send
// arrays, which a FUSED_PACK update of that grid has just filled (dense to dense).
// Work item = (tile, face, chunk of 4*64 vectors or cells), one per WAVEFRONT (faces of small tiles are a few
// hundred bytes: a whole workgroup per face would idle most of its lanes); a lane issues its (up to) four
// loads before its stores.  Workgroups stride over the item list.
// ------------------------------------------------------------------------------------
constexpr int HALO_CHUNK = 4 * WAVE;

template <typename T, int XSRC>
__global__ __launch_bounds__(WG) void halo_exchange_kernel(Geo g, T *grid, int chunks_per_face, long long nitems)
{
    using V = typename Vec<T>::type;
    constexpr int NV = Vec<T>::N;
    const int nfaces = 2 * g.ndim;
    const int vrow = (g.tw + NV - 1) / NV;           // vectors per row (pitch is a multiple of NV)
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    for (long long item = (long long)blockIdx.x * WAVES_PER_WG + wave; item < nitems; item += (long long)gridDim.x * WAVES_PER_WG) {
        const int chunk = (int)(item % chunks_per_face);
        const long long tf = item / chunks_per_face;
        const int face = (int)(tf % nfaces), t = (int)(tf / nfaces);
        const int axis = face >> 1, hi = face & 1;   // axis 0: x, 1: y, 2: z
        const int tz = t / (g.Ty * g.Tx), ty = (t / g.Tx) % g.Ty, tx = t % g.Tx;
        const int tc = axis == 0 ? tx : axis == 1 ? ty : tz;
        const int Tn = axis == 0 ? g.Tx : axis == 1 ? g.Ty : g.Tz;
        if (!(hi ? tc < Tn - 1 : tc > 0)) continue;   // no neighbour on this side
        const long long tstep = axis == 0 ? 1 : axis == 1 ? g.Tx : (long long)g.Ty * g.Tx;
        const T *stile = grid + ((long long)t + (hi ? tstep : -tstep)) * g.tile_stride;
        T *dtile = grid + (long long)t * g.tile_stride;
        // offsets inside a tile fit 32 bits (a tile has fewer than 2^31 elements): keeps the index arithmetic cheap
        const unsigned base = (unsigned)chunk * HALO_CHUNK;
        unsigned dofs[4];
        constexpr unsigned NONE = 0xffffffffu;
        if (axis == 0) {
            // cells (plane a, row b), b fastest: consecutive lanes write consecutive halo entries
            const unsigned n = (unsigned)g.td * (unsigned)g.th;
            const unsigned s0 = XSRC ? (unsigned)(g.xsend + (hi ? 0 : g.hpitch)) : (hi ? 0u : (unsigned)(g.tw - 1));
            const unsigned d0 = (unsigned)(g.xoff + (hi ? g.hpitch : 0));
            T v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned e = base + q * WAVE + lane;
                dofs[q] = NONE;
                if (e >= n) continue;
                const unsigned a = e / (unsigned)g.th, b = e - a * (unsigned)g.th;
                const unsigned k = g.z0 + a, i = 1 + b;
                const unsigned entry = k * (unsigned)g.rows + i;
                // my x+ halo <- the right neighbour's first column; my x- halo <- the left neighbour's last column
                v[q] = stile[XSRC ? s0 + entry : entry * (unsigned)g.pitch + s0];
                dofs[q] = d0 + entry;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (dofs[q] != NONE) dtile[dofs[q]] = v[q];
        } else {
            // vectors (row a of the face, vector b of the row): y faces have one row per plane, z faces th rows
            const unsigned na = axis == 1 ? g.td : g.th;
            const unsigned n = na * (unsigned)vrow;
            // element offset of face row a: y faces step by a plane, z faces by a row
            const unsigned step = axis == 1 ? (unsigned)g.plane : (unsigned)g.pitch;
            const unsigned first = axis == 1 ? (unsigned)g.z0 * (unsigned)g.plane : (unsigned)g.pitch;
            const unsigned d0 = first + (axis == 1 ? (hi ? (unsigned)(g.th + 1) * g.pitch : 0u)
                                                   : (hi ? (unsigned)(g.td + 1) * (unsigned)g.plane : 0u));
            const unsigned s0 = first + (axis == 1 ? (hi ? 1u : (unsigned)g.th) * g.pitch
                                                   : (hi ? 1u : (unsigned)g.td) * (unsigned)g.plane);
            V v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned e = base + q * WAVE + lane;
                dofs[q] = NONE;
                if (e >= n) continue;
                const unsigned a = e / (unsigned)vrow, c = (e - a * (unsigned)vrow) * NV;
                v[q] = *(const V *)(stile + (s0 + a * step + c));
                dofs[q] = d0 + a * step + c;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (dofs[q] != NONE) *(V *)(dtile + dofs[q]) = v[q];
        }
    }
}

// ------------------------------------------------------------------------------------
// Scatter / gather between a padded global array and the tile-major grid.  Both are plain copies, so what counts
// is that every lane moves 16 bytes and that whole cache lines are written: each kernel walks its DESTINATION in
// vectors that are 16-byte aligned there, and reads the source with 16-byte loads that are only element-aligned
// (the tiles' rows start on cache lines, the global array's rows one ring cell off them).  Bound by HBM, which takes
// many short wavefronts best: a lane of a large grid moves ONE vector, so that a wavefront reads 1 KiB, writes it and is gone
// (four per lane, read then written: 5.4 - 5.6 TB/s; one: 5.7 - 6.4, 1.27 to 1.38 ns per workgroup).
// us, one cell per lane and load -> four vectors -> now:
//   16384^2 in 8 x 8 tiles:    scatter  893 ->  765 ->  720       gather  870 ->  776 ->  676
//   8192^2 in 64 x 64 tiles:            220 ->  178 ->  171               246 ->  176 ->  172
//   1024 x 1024 x 768, 6x8x8:          3033 -> 2330 -> 2210              3179 -> 2320 (four vectors still)
//   512^3, 4x4x4, fp32:                 431 ->  198 ->  186                460 ->  190 (three)
//   300^3, 30x30x30, fp32:             1059 ->  154 ->  156               1064 ->   90 (two)
// ------------------------------------------------------------------------------------
// Vectors per thread of the scatter, all loaded before the first is stored.  Grids that stay in the caches take two: 128^3 in one
// tile 6.9 us against 8.0 with one, larger ones the same.  Grids of 135 to 270 MB, which just do not, take one for what else is done with them: 256^3,
// fp64, 43.1 us with four, 42.2 with two, 46.5 with one if nothing but the scatter runs, again and again; 98.8, 97.8 and 101.9 with a gather between,
// 160.5, 159.3 and 158.5 with two updates; 300^3 62.9, 62.4, 67.0; 154, 148, 144; 271, 264, 260.
template <bool STREAM> constexpr int SC_VECS = STREAM ? 1 : 2;
constexpr int sc_unit(bool stream) { return (stream ? SC_VECS<true> : SC_VECS<false>) * WG; }      // vectors a workgroup copies (4 or 8 KiB)
constexpr int LINE_BYTES = 128;               // a cache line
constexpr int GATHER_VECS = 4;                // vectors per lane of the gather, at most

// Division of a 32-bit number by a divisor the host knows: a multiplication and two shifts (Granlund and
// Montgomery, "Division by invariant integers using multiplication", 1994).  Exact for every n.
struct FastDiv {
    unsigned m, sh1, sh2;
    __host__ void set(unsigned d)
    {
        unsigned l = 0;
        while (l < 32 && (1ull << l) < d) ++l;
        m = (unsigned)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
        sh1 = l < 1 ? l : 1;
        sh2 = l > 0 ? l - 1 : 0;
    }
    __host__ __device__ unsigned operator()(unsigned n) const
    {
        const unsigned t = (unsigned)(((unsigned long long)m * n) >> 32);
        return (t + ((n - t) >> sh1)) >> sh2;
    }
};

// Scatter: a workgroup fills sc_unit() consecutive vectors of one tile's rows - all padded rows, halo rows included -
// and the two x halo cells of the rows that begin among them (a run of consecutive entries of the dense arrays).
struct ScatterParams {
    long long GP, GQ;          // elements between rows / planes of the global array
    unsigned vrow;             // vectors per row: ceil(tw / NV)
    unsigned nvec;             // vectors of a tile: nplanes * rows * vrow
    unsigned wg_per_tile;
    FastDiv by_vrow, by_rows, by_wg_per_tile, by_layer, by_Tx;
    // workgroup order (see xcd_logical_wg; the host knows the sizes, so nothing is divided by a variable here)
    int xcd_chunk;
    unsigned first;            // workgroups of earlier launches
    unsigned in_groups;        // workgroups that lie in whole groups of NUM_XCD * xcd_chunk
    FastDiv by_group;
};

template <typename T, bool STREAM>
__global__ __launch_bounds__(WG) void scatter_kernel(Geo g, ScatterParams sp, const T *__restrict__ from, T *__restrict__ to)
{
    using V = typename Vec<T>::type;
    constexpr int NV = Vec<T>::N, VECS = SC_VECS<STREAM>, UNIT = sc_unit(STREAM);
    typedef T VU __attribute__((ext_vector_type(NV), aligned(sizeof(T))));
    unsigned lwg = blockIdx.x + sp.first;
    if (lwg < sp.in_groups) {
        const unsigned span = NUM_XCD * (unsigned)sp.xcd_chunk, first = sp.by_group(lwg) * span, within = lwg - first;
        lwg = first + within % NUM_XCD * (unsigned)sp.xcd_chunk + within / NUM_XCD;
    }
    const unsigned t = sp.by_wg_per_tile(lwg);
    const unsigned v0 = (lwg - t * sp.wg_per_tile) * UNIT;
    const unsigned tz = sp.by_layer(t), in_layer = t - tz * (unsigned)(g.Ty * g.Tx);
    const unsigned ty = sp.by_Tx(in_layer), tx = in_layer - ty * (unsigned)g.Tx;
    // the padded cell (plane 0, row 0, column 0) of the tile; column 0 is the cell right of the x- halo
    const T *corner = from + ((long long)tz * g.td * sp.GQ + (long long)ty * g.th * sp.GP + (long long)tx * g.tw + 1);
    T *tile = to + (long long)t * g.tile_stride;
    V v[VECS];
    unsigned dst[VECS];
#pragma unroll
    for (int q = 0; q < VECS; ++q) {
        const unsigned j = v0 + q * WG + threadIdx.x;
        v[q] = V(0);
        if (j >= sp.nvec) continue;
        const unsigned r = sp.by_vrow(j), c = (j - r * sp.vrow) * NV;      // row (all planes), first column
        const unsigned k = sp.by_rows(r), i = r - k * (unsigned)g.rows;
        const T *src = corner + ((long long)k * sp.GQ + (long long)i * sp.GP + c);
        dst[q] = r * (unsigned)g.pitch + c;
        if (c + NV <= (unsigned)g.tw) v[q] = *(const VU *)src;
        else {                                                            // the last vector of a row of ragged width
#pragma unroll
            for (int e = 0; e < NV - 1; ++e)
                if (c + e < (unsigned)g.tw) v[q][e] = src[e];
        }
    }
    const unsigned v1 = min(v0 + UNIT, sp.nvec);
    const unsigned r0 = sp.by_vrow(v0 + sp.vrow - 1), r1 = sp.by_vrow(v1 + sp.vrow - 1);
    for (unsigned r = r0 + threadIdx.x; r < r1; r += WG) {
        const unsigned k = sp.by_rows(r), i = r - k * (unsigned)g.rows;
        const T *src = corner + ((long long)k * sp.GQ + (long long)i * sp.GP);
        const T xm = src[-1], xp = src[g.tw];
        tile[g.xoff + r] = xm;
        tile[g.xoff + g.hpitch + r] = xp;
    }
#pragma unroll
    for (int q = 0; q < VECS; ++q)
        if (v0 + q * WG + threadIdx.x < sp.nvec) stv<STREAM>((V *)(tile + dst[q]), v[q]);
}

// Gather: a wavefront writes one padded row of the global array, or 64*Q vectors of a long one: the vectors that
// are aligned there, the first and last of a row partly (their other cells belong to the rows beside it).  Along a
// row the cells lie in Tx + 2 runs - the W ring cell, a row of every tile, the E ring cell; a vector inside one run is
// one load, one that crosses a seam is read cell by cell.  Everything that depends on the row alone is scalar.
// (Cutting the whole array into vectors regardless of rows, five divisions per vector, was bound by that arithmetic:
// 512^3 in fp32 387 us against 198 for the scatter.)
struct GatherParams {
    unsigned GP, plane_rows;   // cells per padded row; padded rows per plane
    unsigned shift;            // elements the array's first cell lies beyond a cache line
    unsigned nchunks, nitems;  // wavefronts per row; wavefronts in all
    unsigned first;            // workgroups of earlier launches
    FastDiv by_chunks, by_rows, by_td, by_th, by_tw;
};

template <typename T, bool STREAM, int Q>
__global__ __launch_bounds__(WG) void gather_kernel(Geo g, GatherParams gp, const T *__restrict__ from, T *__restrict__ to)
{
    using V = typename Vec<T>::type;
    constexpr int NV = Vec<T>::N;
    typedef T VU __attribute__((ext_vector_type(NV), aligned(sizeof(T))));
    const int lane = threadIdx.x % WAVE;
    const unsigned item = __builtin_amdgcn_readfirstlane((blockIdx.x + gp.first) * WAVES_PER_WG + threadIdx.x / WAVE);
    if (item >= gp.nitems) return;
    const unsigned row = gp.by_chunks(item), chunk = item - row * gp.nchunks;
    unsigned gk = 0, gi = row;
    if (g.ndim == 3) { gk = gp.by_rows(row); gi = row - gk * gp.plane_rows; }
    // ring planes and rows belong to the tiles next to them
    const int tz = g.ndim == 3 ? min((int)gp.by_td(max(gk, 1u) - 1), g.Tz - 1) : 0;
    const int ty = min((int)gp.by_th(max(gi, 1u) - 1), g.Ty - 1);
    const int k = (int)gk - tz * g.td, i = (int)gi - ty * g.th;
    const T *tiles = from + (long long)(tz * g.Ty + ty) * g.Tx * g.tile_stride;      // first tile of the row of tiles
    const long long first = main_off(g, k, i, 0);
    const T *w_ring = tiles + xm_off(g, k, i);
    const T *e_ring = tiles + ((long long)(g.Tx - 1) * g.tile_stride + xp_off(g, k, i));
    // run s of the row: 0 the W ring cell, 1 .. Tx the tiles, Tx + 1 the E ring cell
    auto run_start = [&](int s) -> const T * {
        return s == 0 ? w_ring : s > g.Tx ? e_ring : tiles + ((long long)(s - 1) * g.tile_stride + first);
    };
    const long long lin = (long long)row * gp.GP;
    // a wavefront's vectors start on a cache line: cells of the row's first line that belong to the row before
    const int lead = (int)((unsigned)(lin + gp.shift) % (LINE_BYTES / sizeof(T)));
    const int GP = (int)gp.GP;
    const unsigned first_vec = chunk * (Q * WAVE) + lane;
    V v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const long long at = (long long)(first_vec + q * WAVE) * NV - lead;  // first cell: padded column
        v[q] = V(0);
        if (at >= GP || at + NV <= 0) continue;
        const int gc = (int)max(at, 0ll);
        int s = 0, left = 1;
        const T *src = w_ring;
        if (gc > 0) {
            const int tx = min((int)gp.by_tw(gc - 1), g.Tx);       // Tx: the E ring cell
            const int c = gc - 1 - tx * g.tw;
            s = tx + 1;
            left = tx < g.Tx ? g.tw - c : 1;
            src = run_start(s) + c;
        }
        if (at >= 0 && left >= NV) {
            v[q] = *(const VU *)src;
            continue;
        }
        if (g.tw >= NV) {
            // at most one seam inside a vector: every cell from this run or the next, all loads at once
            const int skip = at < 0 ? (int)-at : 0;                // cells of the row before
            const T *next = run_start(min(s + 1, g.Tx + 1));
            T c[NV];
#pragma unroll
            for (int e = 0; e < NV; ++e) {
                const int x = max(e - skip, 0);
                const T *from_run = src + min(x, left - 1), *from_next = next + max(x - left, 0);
                c[e] = *(x < left || at + e >= GP ? from_run : from_next);
            }
#pragma unroll
            for (int e = 0; e < NV; ++e) v[q][e] = c[e];
            continue;
        }
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            if (at + e < 0 || at + e >= GP) continue;
            if (left == 0) {
                ++s;
                src = run_start(s);
                left = s <= g.Tx ? g.tw : 1;
            }
            v[q][e] = *src++;
            --left;
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const long long at = (long long)(first_vec + q * WAVE) * NV - lead;
        if (at >= 0 && at + NV <= GP) stv<STREAM>((V *)(to + (lin + at)), v[q]);
        else {
#pragma unroll
            for (int e = 0; e < NV; ++e)
                if (at + e >= 0 && at + e < GP) to[lin + at + e] = v[q][e];
        }
    }
}

// Plain streaming copy, 16 bytes per lane, one element per thread, workgroups in memory
// order (the fastest simple copy on this chip): the practical bandwidth ceiling the update
// kernel is compared with, and the known-size dispatch used to calibrate HBM counters.
__global__ __launch_bounds__(WG) void stream_copy_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                         long long n16)
{
    const long long i = (long long)blockIdx.x * WG + threadIdx.x;
    if (i < n16) dst[i] = src[i];
}

__global__ __launch_bounds__(WG) void clear_kernel(uint4 *p, long long n16)
{
    for (long long i = (long long)blockIdx.x * WG + threadIdx.x; i < n16; i += (long long)gridDim.x * WG) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

}  // namespace jk
