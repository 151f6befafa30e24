// Mid-sized 2-D grids: a whole jacobi_run in one launch, the grid in the registers of the chip.
//
// The domain is cut into nbx x nby blocks, one workgroup (8 wavefronts) each, at most one per CU.  A workgroup HOLDS
// 8*RW rows x 64*C columns: wavefront w rows [w*RW, (w+1)*RW), lane l columns [l*C, (l+1)*C).  The held ranges of
// neighbouring blocks overlap by 2d cells and more; each block OWNS the cells from d behind its held range's start to d
// behind the next one's.  Held ranges lie inside the domain and the outermost ones end where it ends, so the Dirichlet
// ring is never among the held cells: ring rows sit in LDS where the first / last wavefront finds the row next to its
// own, and a ring cell beside a row enters through the open end of the lane shift.  (Wanted: a domain wider than one
// block and at least as high, its width and d multiples of C.)
//
// Per iteration a wavefront publishes its first and last row in LDS (one barrier), and updates its rows in place,
// down and up by turns: the new row j goes into the registers of the row before (behind) it, whose last reader it
// is, so RW + 1 rows of registers hold RW rows and nothing is copied.
//
// What bounds it: per iteration the vector unit (3 additions, 1 product and 4 / C lane shifts per cell in fp64; 8 wavefronts
// of 8 rows x 128 columns 0.45 us, of which 0.39 are these instructions by their number; the vector units of a whole 1024^2 call
// are busy for 34 % of it), per exchange the latency of a message between two
// XCDs (0.5 - 0.6 us for one word per lane, 0.75 - 0.9 for 8 in a row, 1.1 - 1.2 for 16) and its bytes (2.5 us + 0.22 us per MB of all blocks' messages).  Eight
// wavefronts of many rows rather than sixteen of few: half the border rows through LDS and room for the whole state (16
// wavefronts of 4 rows: 0.93 against 0.74 us).  Measured, us per iteration, launches -> blocks, 100 iterations with the
// launch: 300^2 3.10 -> 0.69, 512^2 3.71 -> 0.79, 768^2 5.10 -> 0.98, 1024^2 5.42 -> 1.14, 1536^2 7.44 -> 1.88, 2048^2 11.5 -> 2.4;
// fp32 1500 x 1110 5.27 -> 1.11, 2048^2 6.08 -> 2.0.  256^2, 100 iterations and their norm: 99 -> 64 us against resident2d_kernel.
#pragma once
#include "blocks_common.h"

namespace jk {

constexpr int ROWS_AT_ONCE = 2;                // of an iteration, in the compiler's schedule (1, 4 and 8 run the same)

template <typename T, int C, int RW>
__global__ __launch_bounds__(BLK_WAVES * WAVE) void blocks2d_kernel(Geo g, Blocks2d p, T *ga, T *gb)
{
    typedef T VU __attribute__((ext_vector_type(C == 1 ? 2 : C), aligned(sizeof(T))));
    constexpr int HH = BLK_WAVES * RW, HW = WAVE * C;
    constexpr unsigned MB = MSG_BYTES<T>;
    // The plain path's code lies behind the others': 1024^2 128 -> 125 us per 100 iterations, 256^2 66.4 -> 63.8, 1536^2 268 -> 223, all
    // variants 0 to 15 % - but for fp32 with 4 x 12 cells per lane, which then spills elsewhere (2048^2 267 -> 380).
    // The rows' message offsets, constants of the run, take the registers of the grid (8 a row and more, in scratch memory where there
    // is no room); computed anew in every exchange the large variants run without most of that: us per iteration 2048^2 5.1 -> 2.1,
    // 2200^2 7.0 -> 3.2, 8000 x 500 6.0 -> 2.8, fp32 2048^2 2.1 -> 1.9, 2240^2 5.3 -> 4.1.  The others have the room, or lose more
    // by computing: 1536^2 1.71 -> 1.83, in fp32 1.01 -> 1.04.
    constexpr bool ANEW = C == 4 || (sizeof(T) == 8 && RW == 16);
    constexpr bool OUT_OF_THE_WAY = sizeof(T) == 8 || C != 4 || RW != 12;
    __shared__ T xch[2][BLK_WAVES][2][C][WAVE];    // [parity][wavefront][first / last row][component][lane]
    __shared__ T ring_row[2][C][WAVE];             // the Dirichlet rows above / below the domain
    __shared__ double red[BLK_WAVES];
    __shared__ int flag;

    const BlockRun &br = p.run;
    const int lane = threadIdx.x % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int nb = p.x.nb * p.y.nb;
    const int blk = block_of_workgroup(p.x.nb, p.y.nb, p.strip), by = blk / p.x.nb, bx = blk - by * p.x.nb;
    const unsigned epoch = agent_load(&br.sync->epoch);
    const unsigned max_exchanges = (unsigned)br.iters + (unsigned)br.norms + 2u;
    const int d = p.x.d;
    const int x0 = p.x.start(bx), y0 = p.y.start(by);
    const int xlo = p.x.own_lo(bx), xhi = p.x.own_hi(bx), ylo = p.y.own_lo(by), yhi = p.y.own_hi(by);
    const int col = x0 + lane * C;                 // first column of this lane
    const int row0 = y0 + wave * RW;               // first row of this wavefront
    const bool west = bx == 0, east = bx == p.x.nb - 1, north = by == 0, south = by == p.y.nb - 1;

    // this lane's cells in a row of tiles, for rows found by a RowWalk
    long long co[C];
    bool seam = false;
    auto find_cells = [&](int first_col) JK_INLINE {
        const int tx = first_col / g.tw;
        int c = first_col - tx * g.tw;
        long long off = (long long)tx * g.tile_stride + c;
#pragma unroll
        for (int e = 0; e < C; ++e) {
            co[e] = off;
            ++off;
            if (++c == g.tw) { c = 0; off += g.tile_stride - g.tw; }
        }
        seam = co[C - 1] - co[0] != C - 1;
    };
    find_cells(col);
    auto load_cells = [&](const T *rowp, T (&v)[C]) JK_INLINE {
        if (C > 1 && !seam) {
            const VU x = *(const VU *)(rowp + co[0]);
#pragma unroll
            for (int e = 0; e < C; ++e) v[e] = x[e];
        } else {
#pragma unroll
            for (int e = 0; e < C; ++e) v[e] = rowp[co[e]];
        }
    };

    // ---- the held cells; slots 1 .. RW of `a` (state S0), or 0 .. RW-1 after an odd number of steps
    T a[RW + 1][C];
    // Dirichlet cells beside the rows: in lane 0 of the blocks at the domain's west side, in lane 63 at the east side
    // (no block lies at both), zero elsewhere
    T ring[RW];
    {
        RowWalk row(g, row0);
        const bool ring_lane = west ? lane == 0 : east && lane == WAVE - 1;
        const long long ring_off = g.xoff + (west ? 0 : (long long)(g.Tx - 1) * g.tile_stride + g.hpitch);
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            load_cells(ga + (row.tile + row.i * (long long)g.pitch), a[j + 1]);
            ring[j] = T(0);
            if (ring_lane) ring[j] = ga[row.tile + ring_off + row.i];
            row.next(g);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int e = 0; e < C; ++e) a[0][e] = T(0);
    if (wave == 0 && north) {
        T v[C];
        load_cells(ga, v);                         // halo row 0 of the first row of tiles
#pragma unroll
        for (int e = 0; e < C; ++e) ring_row[0][e][lane] = v[e];
    }
    if (wave == BLK_WAVES - 1 && south) {
        T v[C];
        load_cells(ga + ((long long)(g.Ty - 1) * g.Tx * g.tile_stride + (long long)(g.th + 1) * g.pitch), v);
#pragma unroll
        for (int e = 0; e < C; ++e) ring_row[1][e][lane] = v[e];
    }
    // ---- the Dirichlet ring of the other grid: each side's cells shared out among the blocks along it
    {
        const int tid = threadIdx.x, nt = blockDim.x;
        if (north || south) {
            const int c0 = bx * p.x.n / p.x.nb, c1 = (bx + 1) * p.x.n / p.x.nb;
            for (int c = c0 + tid; c < c1; c += nt) {
                if (north) { const long long o = domain_cell_off(g, 0, -1, c); gb[o] = ga[o]; }
                if (south) { const long long o = domain_cell_off(g, 0, p.y.n, c); gb[o] = ga[o]; }
            }
        }
        if (west || east) {
            const int n = g.Ty * g.rows, r0 = by * n / p.y.nb, r1 = (by + 1) * n / p.y.nb;
            for (int r = r0 + tid; r < r1; r += nt) {
                const int ty = r / g.rows, i = r - ty * g.rows;
                const long long tile = (long long)ty * g.Tx * g.tile_stride;
                if (west) { const long long o = tile + xm_off(g, 0, i); gb[o] = ga[o]; }
                if (east) { const long long o = tile + (long long)(g.Tx - 1) * g.tile_stride + xp_off(g, 0, i); gb[o] = ga[o]; }
            }
        }
    }
    // Counted in once everything has been read: from the roll call on results may overwrite the source grid.
#pragma unroll
    for (int j = 0; j < RW; ++j) {
#pragma unroll
        for (int e = 0; e < C; ++e) arrived(a[j + 1][e]);
        arrived(ring[j]);
    }
    __syncthreads();
    unsigned ticket = 0;                           // looked at by thread 0 in the roll call, no sooner
    if (threadIdx.x == 0) ticket = agent_add(&br.sync->roll, 1u);

    // ---- one iteration.  UP = 0: rows from slots 1.. to slots 0..; UP = 1: back.  EDGE: 1 west, 2 east ring cells beside the rows
    int parity = 0;
    const bool at_north = north && wave == 0, at_south = south && wave == BLK_WAVES - 1;
    const int wave_up = max(wave - 1, 0), wave_dn = min(wave + 1, BLK_WAVES - 1);
    auto publish = [&](auto slot0) JK_INLINE {
        constexpr int S = decltype(slot0)::value;
#pragma unroll
        for (int e = 0; e < C; ++e) {
            xch[parity][wave][0][e][lane] = a[S][e];
            xch[parity][wave][1][e][lane] = a[S + RW - 1][e];
        }
        __syncthreads();
    };
    auto neighbours = [&](T (&above)[C], T (&below)[C]) JK_INLINE {
        const T(*up)[WAVE] = at_north ? ring_row[0] : xch[parity][wave_up][1];
        const T(*dn)[WAVE] = at_south ? ring_row[1] : xch[parity][wave_dn][0];
#pragma unroll
        for (int e = 0; e < C; ++e) {
            above[e] = up[e][lane];
            below[e] = dn[e][lane];
        }
    };
    auto step = [&](auto up_dir, auto edge) JK_INLINE {
        constexpr int UP = decltype(up_dir)::value, EDGE = decltype(edge)::value, S = UP ? 0 : 1;
        publish(std::integral_constant<int, S>{});
        T above[C], below[C];
        neighbours(above, below);
#pragma unroll
        for (int jj = 0; jj < RW; ++jj) {
            const int j = UP ? RW - 1 - jj : jj;
            const int s = S + j, to = UP ? j + 1 : j;
            T left, right;
            if constexpr (EDGE == 1) left = from_prev_lane_or(a[s][C - 1], ring[j]);
            else left = from_prev_lane_or_zero(a[s][C - 1]);
            if constexpr (EDGE == 2) right = from_next_lane_or(a[s][0], ring[j]);
            else right = from_next_lane_or_zero(a[s][0]);
            T v[C];
#pragma unroll
            for (int e = 0; e < C; ++e) {
                const T w = e > 0 ? a[s][e > 0 ? e - 1 : 0] : left;
                const T ea = e < C - 1 ? a[s][e < C - 1 ? e + 1 : e] : right;
                const T u = j > 0 ? a[j > 0 ? s - 1 : s][e] : above[e];
                const T dn = j < RW - 1 ? a[j < RW - 1 ? s + 1 : s][e] : below[e];
                v[e] = Coef<T>::quarter * ((w + ea) + (u + dn));
            }
#pragma unroll
            for (int e = 0; e < C; ++e) a[to][e] = v[e];
            // a few rows at a time: all at once would cost the registers that hold the grid
            if (jj % ROWS_AT_ONCE == ROWS_AT_ONCE - 1) __builtin_amdgcn_sched_barrier(0);
        }
        parity ^= 1;
    };
    auto iterate_edge = [&](int n, auto edge) JK_INLINE {
        for (int it = 0; it + 2 <= n; it += 2) {
            step(std::integral_constant<int, 0>{}, edge);
            step(std::integral_constant<int, 1>{}, edge);
        }
        if (n & 1) {
            step(std::integral_constant<int, 0>{}, edge);
#pragma unroll
            for (int j = RW; j >= 1; --j)
#pragma unroll
                for (int e = 0; e < C; ++e) a[j][e] = a[j - 1][e];
        }
    };
    auto iterate = [&](int n) JK_INLINE {
        if (east) iterate_edge(n, std::integral_constant<int, 2>{});
        else iterate_edge(n, std::integral_constant<int, 1>{});
    };

    // ---- exchange.  A block's message: rows [ylo, ylo+d), rows [yhi-d, yhi) (HW columns counted from xlo), then columns
    // [xlo, xlo+d), columns [xhi-d, xhi) (d cells per row, rows counted from ylo).  Inside a row of it the cells of the
    // lanes' first components come first, then those of the second, ...: every store and load is contiguous.  The offset
    // of a cell is a part that depends on the lane plus one that depends on the row; MSG_SKIP in either: nothing to send
    // or to receive.
    const bool own_col = col >= xlo && col < xhi;
    const bool ghost_w = !west && col >= xlo - d && col < xlo, ghost_e = !east && col >= xhi && col < xhi + d;
    const unsigned frame = blocks2d_frame(p.x, p.y) * MB;
    const unsigned bottom_part = (unsigned)(d * HW) * MB, left_part = 2u * bottom_part, right_part = left_part + (unsigned)(HH * d) * MB;
    const unsigned row_step = (unsigned)(HW / C) * MB, side_step = (unsigned)(d / C) * MB;      // from component to component
    unsigned send_row_ = MSG_SKIP, send_side_ = MSG_SKIP, recv_row_ = MSG_SKIP, recv_side_ = MSG_SKIP;
    if (own_col) {
        send_row_ = (unsigned)blk * frame + (unsigned)(col - xlo) / C * MB;
        recv_row_ = (unsigned)bx * frame + (unsigned)(col - xlo) / C * MB;
        if (!west && col < xlo + d) send_side_ = (unsigned)blk * frame + left_part + (unsigned)(col - xlo) / C * MB;
        if (!east && col >= xhi - d) send_side_ = (unsigned)blk * frame + right_part + (unsigned)(col - (xhi - d)) / C * MB;
    } else if (ghost_w) {
        recv_row_ = (unsigned)(bx - 1) * frame + (unsigned)(col - p.x.own_lo(bx - 1)) / C * MB;
        recv_side_ = (unsigned)(blk - 1) * frame + right_part + (unsigned)(col - (xlo - d)) / C * MB;
    } else if (ghost_e) {
        recv_row_ = (unsigned)(bx + 1) * frame + (unsigned)(col - xhi) / C * MB;
        recv_side_ = (unsigned)(blk + 1) * frame + left_part + (unsigned)(col - xhi) / C * MB;
    }
    unsigned send_row_y[RW], send_side_y[RW], recv_y[RW], recv_is_row[RW];
#pragma unroll
    for (int j = 0; j < RW; ++j) {
        const int y = row0 + j;
        const bool own = y >= ylo && y < yhi;
        const bool above = !north && y < ylo && y >= ylo - d, below = !south && y >= yhi && y < yhi + d;
        send_side_y[j] = own ? (unsigned)((y - ylo) * d) * MB : MSG_SKIP;
        send_row_y[j] = own && !north && y < ylo + d    ? (unsigned)((y - ylo) * HW) * MB
                        : own && !south && y >= yhi - d ? bottom_part + (unsigned)((y - (yhi - d)) * HW) * MB
                                                        : MSG_SKIP;
        recv_is_row[j] = above || below ? 0xffffffffu : 0u;
        recv_y[j] = above   ? (unsigned)((by - 1) * p.x.nb) * frame + bottom_part + (unsigned)((y - (ylo - d)) * HW) * MB
                    : below ? (unsigned)((by + 1) * p.x.nb) * frame + (unsigned)((y - yhi) * HW) * MB
                            : send_side_y[j];
    }
    unsigned exchanges = 0;
    bool healthy = true;
    auto exchange = [&]() JK_INLINE {
        ++exchanges;
        if (!healthy) return;
        const unsigned tag = epoch + exchanges;
        const __amdgpu_buffer_rsrc_t buf = buffer_of((char *)br.msg + (size_t)(exchanges & 1u) * br.msg_bytes, br.msg_bytes);
        const unsigned send_row = ANEW ? opaque_lane(send_row_) : send_row_, send_side = ANEW ? opaque_lane(send_side_) : send_side_;
        const unsigned recv_row = ANEW ? opaque_lane(recv_row_) : recv_row_, recv_side = ANEW ? opaque_lane(recv_side_) : recv_side_;
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            if (send_row_y[j] != MSG_SKIP) {                         // wave-uniform
#pragma unroll
                for (int e = 0; e < C; ++e) send_cell(a[j + 1][e], tag, buf, send_row + send_row_y[j] + e * row_step);
            }
            if (send_side_y[j] != MSG_SKIP) {
#pragma unroll
                for (int e = 0; e < C; ++e) send_cell(a[j + 1][e], tag, buf, send_side + send_side_y[j] + e * side_step);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ghost cells: a few rows at a time, each lane's until all of their words carry the tag
        // Blocks run level with each other, so asked at once the first question comes just too early and the answer to the second
        // one a way to memory and back later: 900 clocks first.  Us per 100 iterations with scatter and gather, at once -> so: 256^2 68.6
        // -> 65.5, 420^2 79.7 -> 71.2, 650^2 99.5 -> 93.7, fp32 420^2 64.7 -> 59.1, 650^2 79.6 -> 73.8; of 148 grids of one cell per lane none more than
        // 1 % longer, 20 % shorter at most.  One wait for all: 51 workgroups and fewer are 2 % slower with 20, from 180
        // on more would be better for some (of 64 clocks each, 14, 20, 24: 150 x 1800 77.5, 75.6, 75.2, fp32 650^2 73.8, 68.6, 67.5, but fp32 512^2
        // 58.5, 58.4, 59.2, 150 x 1800 61.4, 62.4, 63.4).  With more cells per lane the rows are asked for in portions, one after the
        // other, and a wait gives nothing (1024^2 129.2 -> 130.7 with 8, 1536^2 207.5 -> 206.1, 2048^2 the same).
        if constexpr (C == 1) __builtin_amdgcn_s_sleep(14);
        constexpr int CELLS = sizeof(T) == 8 ? 8 : 16, RB = C >= CELLS ? 1 : CELLS / C < RW ? CELLS / C : RW;
#pragma unroll
        for (int j0 = 0; j0 < RW; j0 += RB) {
            unsigned from[RB], step_e[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int j = j0 + b < RW ? j0 + b : RW - 1;
                from[b] = j0 + b < RW ? ((recv_row & recv_is_row[j]) | (recv_side & ~recv_is_row[j])) + recv_y[j] : MSG_SKIP;
                step_e[b] = (row_step & recv_is_row[j]) | (side_step & ~recv_is_row[j]);
            }
            for (unsigned n = 0;;) {
                Msg<T> m[RB][C];
#pragma unroll
                for (int b = 0; b < RB; ++b)
#pragma unroll
                    for (int e = 0; e < C; ++e) m[b][e].read(buf, from[b] + e * step_e[b]);
                bool waiting = false;
#pragma unroll
                for (int b = 0; b < RB; ++b) {
                    if (j0 + b >= RW) continue;
                    unsigned wrong = 0;
#pragma unroll
                    for (int e = 0; e < C; ++e) wrong |= m[b][e].wrong(tag);
                    const bool got = from[b] < MSG_SKIP && wrong == 0u;
#pragma unroll
                    for (int e = 0; e < C; ++e) a[j0 + b + 1][e] = got ? m[b][e].value() : a[j0 + b + 1][e];
                    from[b] = got ? MSG_SKIP : from[b];          // lanes that have theirs do not ask again
                    waiting = waiting || from[b] < MSG_SKIP;
                }
                if (!__any(waiting)) break;
                if (++n > br.spin_limit || ((n & 255u) == 0u && agent_load(&br.sync->failed) != 0u)) {
                    healthy = false;
                    break;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!healthy) agent_store(&br.sync->failed, 1u);
    };

    // ---- the norm of the grid as it is: the cells next to the owned ones are current
    auto norm_sum = [&]() JK_INLINE -> double {
        publish(std::integral_constant<int, 1>{});
        T above[C], below[C];
        neighbours(above, below);
        parity ^= 1;
        const int row_first = opaque(row0), col = x0 + opaque_lane(lane) * C;
        const bool own_col = col >= xlo && col < xhi;
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            const int y = row_first + j;
            if (y < ylo || y >= yhi) continue;
            const T left = from_prev_lane_or(a[j + 1][C - 1], west ? ring[j] : T(0));
            const T right = from_next_lane_or(a[j + 1][0], west ? T(0) : ring[j]);
#pragma unroll
            for (int e = 0; e < C; ++e) {
                const T w = e > 0 ? a[j + 1][e > 0 ? e - 1 : 0] : left;
                const T ea = e < C - 1 ? a[j + 1][e < C - 1 ? e + 1 : e] : right;
                const T u = j > 0 ? a[j][e] : above[e];
                const T dn = j < RW - 1 ? a[j < RW - 1 ? j + 2 : j + 1][e] : below[e];
                const T r = ((w + ea) + (u + dn)) - Coef<T>::four * a[j + 1][e];
                if (own_col) acc += (double)r * (double)r;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        return wg_sum(acc, red);                   // valid in thread 0
    };

    // ---- the run: stretches of at most d iterations with an exchange in between; a norm where one is due
    int it = 0, norm = 0, stale = 0;               // stale: iterations since the ghost cells were current
    bool norm_due = false;
    for (;;) {
        if (norm_due ? stale + 1 > d : stale > 0 && it < br.iters) {
            exchange();
            stale = 0;
        }
        if (norm_due) {
            const double tot = norm_sum();
            if (threadIdx.x == 0)
                __hip_atomic_store(&br.partial[(long long)norm * nb + blk], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ++norm;
            norm_due = false;
            continue;
        }
        if (it >= br.iters) break;
        const bool norm_ahead = br.norms > norm;
        const int target = norm_ahead ? (norm + 1) * br.every : br.iters;
        const int n = next_stretch(target - it, d, norm_ahead);
        iterate(n);
        stale = n;
        if (it == 0) {
            // is everybody there?  (the first exchange and the result wait for it)
            if (threadIdx.x == 0) roll_call(br.sync, (unsigned)nb, br.admitted, ticket, br.roll_limit, &flag);
            __syncthreads();
            if (OUT_OF_THE_WAY ? __builtin_expect(flag != ALL_PRESENT, 0) : flag != ALL_PRESENT) {
                if (flag >= 0) plain_path<T, 2>(g, br, ga, gb, red, &flag);
                block_epilogue(br, epoch, max_exchanges, red, &flag);
                return;
            }
        }
        it += n;
        norm_due = norm_ahead && it == target;
    }
    if (agent_load(&br.sync->failed) != 0u) healthy = false;
    T *fin = br.final_is_out ? gb : ga;
    {
        const int first_col = x0 + opaque_lane(lane) * C;
        find_cells(first_col);
        RowWalk row(g, y0 + opaque(wave) * RW);
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            const int y = row0 + j;
            T *rowp = fin + (row.tile + row.i * (long long)g.pitch);
            row.next(g);
            if (y < ylo || y >= yhi || first_col < xlo || first_col >= xhi) continue;
            T v[C];
#pragma unroll
            for (int e = 0; e < C; ++e) v[e] = healthy ? a[j + 1][e] : T(__builtin_nan(""));
            if (C > 1 && !seam) {
                VU x;
#pragma unroll
                for (int e = 0; e < C; ++e) x[e] = v[e];
                *(VU *)(rowp + co[0]) = x;
            } else {
#pragma unroll
                for (int e = 0; e < C; ++e) rowp[co[e]] = v[e];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    block_epilogue(br, epoch, max_exchanges, red, &flag);
}

}  // namespace jk
