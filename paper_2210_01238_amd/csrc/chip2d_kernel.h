// Large 2-D grids that the chip still holds: a whole jacobi_run in one launch, the grid in registers and LDS.
//
// The cut, the messages, the roll call and the run are those of the block kernels (blocks_common.h).  Unlike blocks2d_kernel a
// block holds NO ghost cells: every register goes to cells it owns, and the cells beside it come as messages in every iteration.
// A workgroup (8 wavefronts, one per CU) holds 8*RW rows x 64*C columns, C cells being 32 bytes; wavefront w holds rows
// [w*RW, (w+1)*RW): the first LT and the last LB of them in LDS, the RR in between in registers.  The held ranges are spread
// evenly over the domain; where they overlap both blocks compute the same bits.
//
// An iteration: the cells beside the block arrive (columns: one cell per lane, rows by the first and last wavefront) and are put
// into LDS, from where every row gets its W and E cell as a broadcast; then the rows are updated in place, down and up by turns -
// in registers the new row j goes where row j-1 (j+1) was, so RR + 1 rows of registers hold RR rows and nothing is copied; rows in
// LDS are read, kept for the row after them, and written back -; then the block's own border is sent.
//
// Eight wavefronts of up to 256 registers have all of a CU's 512 KB; 4096^2 in fp64 is 524288 bytes per CU, so that grid needs the
// LDS as well: 23 rows per wavefront in registers, 9 in LDS (144 KB), 64 registers for everything else.
//
// EVEN cuts (not RAGGED): the columns and rows that other blocks need are the first and last ones of lanes and wavefronts.  RAGGED ones
// - the width no multiple of C, or blocks that overlap by some rows - have them anywhere, which takes a third longer.
//
// What bounds it: of 4096^2's 11700 clocks per iteration (2 GHz) 9000 are the rows' update - 29 instructions per row and wavefront, 20
// of them the arithmetic and the lane shifts, two wavefronts per SIMD -, 2000 to 2700 the messages' way (sent 350, two hops of
// memory latency) and a barrier, which follow it: nothing is updated while they travel.  Measured, us per iteration with random cells,
// launches -> one launch, launch behind launch: fp64 2304^2 14.2 -> 2.4, 2560^2 16.9 -> 2.7, 3072 x 4096 31.8 -> 3.3, 4096^2 51.4 -> 4.7,
// ragged 1501^2 8.0 -> 2.6, 2601^2 17.6 -> 3.8, 4001^2 40.0 -> 6.4; fp32 3072^2 12.6 -> 2.5, 4096^2 20.5 -> 2.8, 5632^2 38.5 -> 4.8, ragged 5501^2
// 37.0 -> 6.3.  After an idle stretch 4096^2 takes 5.5 (1000 iterations and ten norms 5600 us, launch behind launch 4890).  A launch takes
// 16 us besides and 0.36 per MB of the grid, a norm 1.6 and 0.23 per row of a wavefront (fp32 1.5 and 0.35).
//
// Everything here is arranged around the registers; what spilled made an iteration three to six times as long.  So: arrays are
// indexed by constants and hold single cells (rows as vectors would need neighbouring registers), no branch stands between the rows
// of an iteration (where only some lanes or rows have something to write, the others write to a place where nobody looks), new cells are
// pinned where they are computed, and the loop over iterations holds nothing but two of them.  The largest variants do use scratch memory
// (bytes per lane: even fp64 192 with 24 rows and 188 with 23 + 9, fp32 88; ragged fp64 28 and 64, fp32 180 with 20 rows, 436 and 220), but
// not in that loop: what lies there is used once in a stretch, mostly by its last iteration if their number is odd, and by the norm.  Only the
// ragged fp32 ones feel it, 8 us in such a stretch and 27 with 24 rows.
#pragma once
#include "blocks_common.h"

namespace jk {

template <int I> using Int = std::integral_constant<int, I>;

// Where block b of a cut without ghost cells starts and ends.  (The cut's own members are not always inlined, and a call, even one that
// is never made, costs registers.)
__device__ __forceinline__ int start_of(const BlockCut &c, int b) { return (b * c.step + min(b, c.longer)) * c.unit; }
__device__ __forceinline__ int end_of(const BlockCut &c, int b) { return b == c.nb - 1 ? c.n : start_of(c, b + 1); }

template <typename T, int RR, int LT, int LB, bool RAGGED>
__global__ __launch_bounds__(BLK_WAVES * WAVE) void chip2d_kernel(Geo g, Chip2d p, T *ga, T *gb)
{
    constexpr int C = CHIP2D_LANE_BYTES / (int)sizeof(T), NV = 16 / (int)sizeof(T);
    constexpr int RW = LT + RR + LB, NL = LT + LB;
    constexpr int HH = BLK_WAVES * RW, HW = WAVE * C;
    constexpr bool IN_LDS = NL > 0;                 // then both ends of a wavefront's rows are there
    constexpr unsigned MB = MSG_BYTES<T>;
    static_assert(RW <= WAVE / 2 && (LT > 0) == (LB > 0), "");
    typedef T V16 __attribute__((ext_vector_type(NV)));
    struct Row { T c[C]; };
    auto each = [](auto f) JK_INLINE { static_for<C>(f); };         // a row's cells: rows are indexed by constants only
    typedef T RowU __attribute__((ext_vector_type(C), aligned(sizeof(T))));
    struct WE { T w, e; };
    // rows of the wavefronts: those kept in LDS, or copies of the first and the last one, two sets taking turns
    constexpr int SLOTS = IN_LDS ? NL : 2, SETS = IN_LDS ? 1 : 2;
    // (set, wavefront, slot), and behind them the rows above / below the block
    // and in RAGGED blocks a row on its way out (IN_LDS there is no room for two more, but there everybody has read the rows beside
    // the block before any wavefront can be as far as that, and what a block sends replaces no ring)
    constexpr int BEYOND = SETS * BLK_WAVES * SLOTS, STAGED = IN_LDS ? BEYOND : BEYOND + 2, NOWHERE = STAGED + 2;
    __shared__ V16 lds[RAGGED ? NOWHERE + 1 : BEYOND + 2][2][WAVE];
    __shared__ alignas(16) WE beside[BLK_WAVES * RW];           // the cells W and E of a row
    // on their way out: a wavefront's cells that the blocks beside it need; behind them the place for what the other lanes write
    constexpr int COLUMN = BLK_WAVES * 2 * RW;
    __shared__ T column[COLUMN + WAVE + RW];
    __shared__ double red[BLK_WAVES];
    __shared__ int flag;

    const BlockRun &br = p.run;
    const int lane = threadIdx.x % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int nbx = p.x.nb, nby = p.y.nb, nb = nbx * nby;
    const int blk = __builtin_amdgcn_readfirstlane(block_of_workgroup(nbx, nby, p.strip)), by = __builtin_amdgcn_readfirstlane(blk / nbx);
    const int bx = blk - by * nbx;
    const unsigned epoch = __builtin_amdgcn_readfirstlane(agent_load(&br.sync->epoch));
    const unsigned max_exchanges = (unsigned)br.iters + 2u;
    const int x0 = start_of(p.x, bx), y0 = start_of(p.y, by);
    const int row0 = y0 + wave * RW;               // first row of this wavefront
    const bool west = bx == 0, east = bx == nbx - 1, north = by == 0, south = by == nby - 1;

    long long co[C];                               // this lane's cells in a row of tiles, for rows found by a RowWalk
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
    auto row_from = [&](int row) JK_INLINE -> Row {
        const V16 x = lds[row][0][lane], y = lds[row][1][lane];
        Row v;
        each([&](auto e) JK_INLINE { v.c[e.value] = e.value < NV ? x[e.value % NV] : y[e.value % NV]; });
        return v;
    };
    auto row_to = [&](int row, Row v) JK_INLINE {
        V16 x, y;
        static_for<NV>([&](auto e) JK_INLINE { x[e.value] = v.c[e.value]; y[e.value] = v.c[NV + e.value]; });
        lds[row][0][lane] = x;
        lds[row][1][lane] = y;
    };
    auto slot = [&](int r) JK_INLINE -> int { return wave * SLOTS + (r < LT ? r : r - RR); };      // of a row of this wavefront kept in LDS
    const int beside_at = opaque_lane(wave * RW);   // (in a vector register: the address then needs no move for every row)
    int set = 0;                                    // of `lds` that holds the rows to read

    // ---- the held cells; register rows in slots 1 .. RR of `a`, between a step down and one up 0 .. RR-1
    // (Cell by cell, with constant indexes only: whole rows would have to lie in neighbouring registers.)
    T a[RR + 1][C];
    auto get = [&](auto j_) JK_INLINE -> Row {
        Row v;
        each([&](auto e) JK_INLINE { v.c[e.value] = a[decltype(j_)::value][e.value]; });
        return v;
    };
    auto put = [&](auto j_, Row v) JK_INLINE {
        each([&](auto e) JK_INLINE { a[decltype(j_)::value][e.value] = v.c[e.value]; });
    };
    find_cells(x0 + lane * C);
    {
        RowWalk row(g, row0);
        static_for<RW>([&](auto r_) JK_INLINE {
            constexpr int r = decltype(r_)::value;
            const T *rowp = ga + (row.tile + row.i * (long long)g.pitch);
            row.next(g);
            Row v;
            if (!seam) {
                const RowU x = *(const RowU *)(rowp + co[0]);
                each([&](auto e) JK_INLINE { v.c[e.value] = x[e.value]; });
            } else each([&](auto e) JK_INLINE { v.c[e.value] = rowp[co[e.value]]; });
            if constexpr (r >= LT && r < LT + RR) put(Int<1 + r - LT>{}, v);
            else row_to(slot(r), v);
            if constexpr (!IN_LDS && r == 0) row_to(wave * SLOTS, v);
            if constexpr (!IN_LDS && r == RW - 1) row_to(wave * SLOTS + 1, v);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    each([&](auto e) JK_INLINE { a[0][e.value] = T(0); });
    // the cells beside the block, ring or not (the ring's stay)
    if (const int r = lane % (WAVE / 2); r < RW) {
        const T v = ga[domain_cell_off(g, 0, row0 + r, lane < WAVE / 2 ? x0 - 1 : x0 + HW)];
        if (lane < WAVE / 2) beside[beside_at + r].w = v;
        else beside[beside_at + r].e = v;
    }
    if (wave == 0 || wave == BLK_WAVES - 1) {
        const int y = wave == 0 ? y0 - 1 : y0 + HH;
        Row v;
        each([&](auto e) JK_INLINE { v.c[e.value] = ga[domain_cell_off(g, 0, y, x0 + lane * C + e.value)]; });
        row_to(BEYOND + (wave == 0 ? 0 : 1), v);
    }
    // ---- the Dirichlet ring of the other grid: each side's cells shared out among the blocks along it
    {
        const int tid = threadIdx.x, nt = blockDim.x;
        if (north || south) {
            const int c0 = (int)((long long)bx * p.x.n / nbx), c1 = (int)((long long)(bx + 1) * p.x.n / nbx);
            for (int c = c0 + tid; c < c1; c += nt) {
                if (north) { const long long o = domain_cell_off(g, 0, -1, c); gb[o] = ga[o]; }
                if (south) { const long long o = domain_cell_off(g, 0, p.y.n, c); gb[o] = ga[o]; }
            }
        }
        if (west || east) {
            const int n = g.Ty * g.rows, r0 = (int)((long long)by * n / nby), r1 = (int)((long long)(by + 1) * n / nby);
            for (int r = r0 + tid; r < r1; r += nt) {
                const int ty = r / g.rows, i = r - ty * g.rows;
                const long long tile = (long long)ty * g.Tx * g.tile_stride;
                if (west) { const long long o = tile + xm_off(g, 0, i); gb[o] = ga[o]; }
                if (east) { const long long o = tile + (long long)(g.Tx - 1) * g.tile_stride + xp_off(g, 0, i); gb[o] = ga[o]; }
            }
        }
    }
    // Counted in once everything has been read: from the roll call on results may overwrite the source grid.  (What went to LDS
    // has been read.)
    static_for<RR * C>([&](auto k_) JK_INLINE { arrived(a[1 + decltype(k_)::value / C][decltype(k_)::value % C]); });
    __syncthreads();
    if (threadIdx.x == 0) roll_call(br.sync, (unsigned)nb, br.admitted, agent_add(&br.sync->roll, 1u), br.roll_limit, &flag);
    __syncthreads();
    if (__builtin_expect(flag != ALL_PRESENT, 0)) {
        if (flag >= 0) plain_path<T, 2>(g, br, ga, gb, red, &flag);
        block_epilogue(br, epoch, max_exchanges, red, &flag, CHIP2D_AREAS);
        return;
    }

    // ---- what other blocks need.  Columns, counted in this block: the one E of the block W of it, the one W of the block E of it (-1:
    // no such block; they lie in two lanes: plan_chip2d); rows of this wavefront: the one below the block above, the one above the block below.
    const int out_w = west ? -1 : start_of(p.x, bx - 1) + HW - x0, out_e = east ? -1 : start_of(p.x, bx + 1) - 1 - x0;
    const bool at_ends = (west || out_w % C == 0) && (east || out_e % C == C - 1);      // the first and the last cell of a lane
    const int lane_w = west ? -1 : out_w / C, lane_e = east ? -1 : out_e / C;
    const int out_n = north ? -1 : start_of(p.y, by - 1) + HH - y0 - wave * RW, out_s = south ? -1 : start_of(p.y, by + 1) - 1 - y0 - wave * RW;
    const int my_column = lane == lane_w ? wave * 2 * RW : lane == lane_e ? (wave * 2 + 1) * RW : COLUMN + lane;

    // ---- one iteration
    auto row_above = [&]() JK_INLINE -> Row { return row_from(opaque(wave == 0 ? BEYOND : (set * BLK_WAVES + wave - 1) * SLOTS + SLOTS - 1)); };
    auto row_below = [&]() JK_INLINE -> Row { return row_from(opaque(wave == BLK_WAVES - 1 ? BEYOND + 1 : (set * BLK_WAVES + wave + 1) * SLOTS)); };
    auto sums = [&](const WE &b, const Row &u, const Row &c, const Row &d) JK_INLINE -> Row {
        const T left = from_prev_lane(c.c[C - 1], b.w), right = from_next_lane(c.c[0], b.e);
        Row s;
        each([&](auto e_) JK_INLINE {
            constexpr int e = decltype(e_)::value;
            T w = left, ea = right;
            if constexpr (e > 0) w = c.c[e - 1];
            if constexpr (e < C - 1) ea = c.c[e + 1];
            s.c[e] = (w + ea) + (u.c[e] + d.c[e]);
        });
        return s;
    };
    WE ahead;                                       // the cells beside the next row, under way
    auto new_row = [&](int r, int next, const Row &u, const Row &c, const Row &d) JK_INLINE -> Row {
        const WE b = ahead;
        if (next >= 0 && next < RW) ahead = beside[beside_at + next];
        Row v = sums(b, u, c, d);
        each([&](auto e) JK_INLINE {
            v.c[e.value] = Coef<T>::quarter * v.c[e.value];
            arrived(v.c[e.value]);                 // computed here: the compiler would move it behind later branches, and the rows'
                                                   // shifted cells, which it cannot move, would fill the registers until then
        });
        column[my_column + r] = lane == lane_e ? v.c[C - 1] : v.c[0];
        return v;
    };
    auto down = [&]() JK_INLINE {                   // slots 1.. to 0..
        ahead = beside[beside_at];
        Row before = row_above(), cur, next, v, below;
        if constexpr (IN_LDS) below = row_below();
        if constexpr (IN_LDS) __syncthreads();      // everybody has read the rows at the ends
        if constexpr (IN_LDS) cur = row_from(slot(0));
        static_for<LT>([&](auto t_) JK_INLINE {
            constexpr int t = decltype(t_)::value;
            if constexpr (t + 1 < LT) next = row_from(slot(t + 1));
            else next = get(Int<1>{});
            v = new_row(t, t + 1, before, cur, next);
            row_to(slot(t), v);
            before = cur;
            cur = next;
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<RR>([&](auto j_) JK_INLINE {
            constexpr int j = decltype(j_)::value;
            if constexpr (j == RR - 1) {
                if constexpr (IN_LDS) next = row_from(slot(LT + RR));
                else next = row_below();            // the set stays as it is until the barrier behind this step
            } else next = get(Int<j + 2>{});
            if constexpr (j == 0) v = new_row(LT, LT + 1, before, get(Int<1>{}), next);
            else v = new_row(LT + j, LT + j + 1, get(Int<j>{}), get(Int<j + 1>{}), next);
            put(Int<j>{}, v);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (IN_LDS) {
            before = get(Int<RR>{});
            cur = next;
        }
        static_for<LB>([&](auto t_) JK_INLINE {
            constexpr int t = decltype(t_)::value;
            if constexpr (t + 1 < LB) next = row_from(slot(LT + RR + t + 1));
            else next = below;
            v = new_row(LT + RR + t, LT + RR + t + 1, before, cur, next);
            row_to(slot(LT + RR + t), v);
            before = cur;
            cur = next;
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto up = [&]() JK_INLINE {                     // slots 0.. to 1..
        ahead = beside[beside_at + RW - 1];
        Row after = row_below(), cur, next, v, above;
        if constexpr (IN_LDS) above = row_above();
        if constexpr (IN_LDS) __syncthreads();
        if constexpr (IN_LDS) cur = row_from(slot(RW - 1));
        static_for<LB>([&](auto t_) JK_INLINE {
            constexpr int t = LB - 1 - decltype(t_)::value;
            if constexpr (t > 0) next = row_from(slot(LT + RR + t - 1));
            else next = get(Int<RR - 1>{});
            v = new_row(LT + RR + t, LT + RR + t - 1, next, cur, after);
            row_to(slot(LT + RR + t), v);
            after = cur;
            cur = next;
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<RR>([&](auto j_) JK_INLINE {
            constexpr int j = RR - 1 - decltype(j_)::value;
            if constexpr (j == 0) {
                if constexpr (IN_LDS) next = row_from(slot(LT - 1));
                else next = row_above();
            } else next = get(Int<j - 1>{});
            if constexpr (j == RR - 1) v = new_row(LT + j, LT + j - 1, next, get(Int<j>{}), after);
            else v = new_row(LT + j, LT + j - 1, next, get(Int<j>{}), get(Int<j + 1>{}));
            put(Int<j + 1>{}, v);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (IN_LDS) {
            after = get(Int<0>{});
            cur = next;
        }
        static_for<LT>([&](auto t_) JK_INLINE {
            constexpr int t = LT - 1 - decltype(t_)::value;
            if constexpr (t > 0) next = row_from(slot(t - 1));
            else next = above;
            v = new_row(t, t - 1, next, cur, after);
            row_to(slot(t), v);
            after = cur;
            cur = next;
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ---- messages.  A block's: the column that the block W of it needs, the one E of it (a cell per held row), the row for the
    // one above, the one below (component by component).  Four areas take turns, for a row may be sent by another wavefront than the
    // one that receives the neighbour's: when one sends exchange x + 1 its neighbours have all of x - 3, which was in that area, behind them.
    constexpr unsigned FRAME = (2u * HH + 2u * HW) * MB, E_PART = HH * MB, N_PART = 2u * HH * MB, S_PART = N_PART + HW * MB;
    bool healthy = true;
    auto area = [&](int exchange) JK_INLINE {
        return buffer_of((char *)br.msg + (size_t)(exchange & (CHIP2D_AREAS - 1)) * br.msg_bytes, br.msg_bytes);
    };
    auto send = [&](int exchange, auto slot0) JK_INLINE {
        constexpr int S = decltype(slot0)::value;
        const unsigned tag = epoch + (unsigned)exchange;
        const __amdgpu_buffer_rsrc_t buf = area(exchange);
        const unsigned mine = (unsigned)opaque(blk) * FRAME;
        if (RAGGED && !at_ends)                    // widths that C does not divide: in two columns of blocks one of the cells is another one
            static_for<2>([&](auto side) JK_INLINE {
                const int c = side.value == 0 ? out_w : out_e, first = (wave * 2 + side.value) * RW;
                if (c < 0 || c % C == (side.value == 0 ? 0 : C - 1)) return;
                const int to = lane == c / C ? first : COLUMN + lane;
                static_for<RR>([&](auto j) JK_INLINE {
                    T v = a[S + j.value][0];
                    each([&](auto e) JK_INLINE { v = pick(c % C == e.value, a[S + j.value][e.value], v); });
                    column[to + LT + j.value] = v;
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (IN_LDS)
                    if (lane < RW && (lane < LT || lane >= LT + RR)) column[first + lane] = ((const T *)&lds[slot(lane)][c % C / NV][c / C])[c % NV];
            });
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        {
            const int l = opaque_lane(lane), side = l / (WAVE / 2), r = l % (WAVE / 2);
            const bool sends = r < RW && !(side ? east : west);
            T v = T(0);
            if (sends) v = column[(wave * 2 + side) * RW + r];
            send_cell(v, tag, buf, sends ? mine + (side ? E_PART : 0u) + (unsigned)(wave * RW + r) * MB : MSG_SKIP);
        }
        auto send_row = [&](auto side, const Row &v) JK_INLINE {
            const unsigned at = mine + (side.value == 0 ? N_PART : S_PART) + (unsigned)opaque_lane(lane) * MB;
            each([&](auto e) JK_INLINE {
                send_cell(v.c[e.value], tag, buf, at + e.value * (WAVE * MB));
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        static_for<2>([&](auto side) JK_INLINE {
            constexpr int end = side.value == 0 ? 0 : RW - 1;
            const int r = side.value == 0 ? out_n : out_s;
            if (RAGGED ? r < 0 || r >= RW : r != end) return;
            if (!RAGGED && !IN_LDS) send_row(side, get(Int<IN_LDS ? 0 : S + end>{}));
            else if (!RAGGED || (IN_LDS && (r < LT || r >= LT + RR))) send_row(side, row_from(slot(RAGGED ? r : end)));
            else {
                // one of the register rows: by way of LDS, all of them being written, the others to a place where nobody looks
                // (a branch per row costs the registers that hold the grid)
                static_for<RR>([&](auto j) JK_INLINE {
                    row_to(opaque(r == LT + j.value ? STAGED + side.value : NOWHERE), get(Int<S + j.value>{}));
                    __builtin_amdgcn_sched_barrier(0);
                });
                send_row(side, row_from(STAGED + side.value));
            }
        });
    };
    auto receive = [&](int exchange) JK_INLINE {
        if (!healthy) return;
        const unsigned tag = epoch + (unsigned)exchange;
        const __amdgpu_buffer_rsrc_t buf = area(exchange);
        const int l = opaque_lane(lane), r = l % (WAVE / 2);
        const bool w_half = l < WAVE / 2;
        const unsigned mine = (unsigned)opaque(blk) * FRAME;
        unsigned from = r < RW && !(w_half ? west : east)
                            ? (w_half ? mine - FRAME + E_PART : mine + FRAME) + (unsigned)(wave * RW + r) * MB : MSG_SKIP;
        const bool row_too = (wave == 0 && !north) || (wave == BLK_WAVES - 1 && !south);
        unsigned row_from_at = MSG_SKIP;
        if (row_too) row_from_at = (wave == 0 ? mine - (unsigned)nbx * FRAME + S_PART : mine + (unsigned)nbx * FRAME + N_PART) + (unsigned)l * MB;
        for (unsigned n = 0;;) {
            Msg<T> m, mr[C];
            m.read(buf, from);
            if (row_too) each([&](auto e) JK_INLINE { mr[e.value].read(buf, row_from_at + e.value * (WAVE * MB)); });
            if (from < MSG_SKIP && m.wrong(tag) == 0u) {
                if (w_half) beside[beside_at + r].w = m.value();
                else beside[beside_at + r].e = m.value();
                from = MSG_SKIP;
            }
            if (row_too && row_from_at < MSG_SKIP) {
                unsigned wrong = 0;
                each([&](auto e) JK_INLINE { wrong |= mr[e.value].wrong(tag); });
                if (wrong == 0u) {
                    Row v;
                    each([&](auto e) JK_INLINE { v.c[e.value] = mr[e.value].value(); });
                    row_to(BEYOND + (wave == 0 ? 0 : 1), v);
                    row_from_at = MSG_SKIP;
                }
            }
            if (!__any(from < MSG_SKIP || row_from_at < MSG_SKIP)) break;
            if (++n > br.spin_limit || ((n & 255u) == 0u && agent_load(&br.sync->failed) != 0u)) {
                healthy = false;
                agent_store(&br.sync->failed, 1u);
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    // after a step: the rows at the ends for the other wavefronts, the border for the other blocks
    auto publish = [&](int exchange, auto slot0) JK_INLINE {
        constexpr int S = decltype(slot0)::value;
        if constexpr (!IN_LDS) {
            set ^= 1;
            row_to((set * BLK_WAVES + wave) * SLOTS, get(slot0));
            row_to((set * BLK_WAVES + wave) * SLOTS + 1, get(Int<S + RR - 1>{}));
        }
        send(exchange, slot0);
        __syncthreads();
    };
    // ---- the norm of the grid as it is (register rows in slots 1 ..; the cells beside the block are current)
    auto norm_sum = [&]() JK_INLINE -> double {
        const Row above = row_above(), below = row_below();
        const int first_row = opaque(row0), first_col = x0 + opaque_lane(lane) * C;
        const int ylo = start_of(p.y, by), yhi = end_of(p.y, by), xlo = start_of(p.x, bx), xhi = end_of(p.x, bx);
        double acc = 0.0;
        auto add = [&](int r, const Row &u, const Row &c, const Row &d) JK_INLINE {
            if (first_row + r < ylo || first_row + r >= yhi) return;
            const Row s = sums(beside[beside_at + r], u, c, d);
            each([&](auto e) JK_INLINE {
                const T q = s.c[e.value] - Coef<T>::four * c.c[e.value];
                if (first_col + e.value >= xlo && first_col + e.value < xhi) acc += (double)q * (double)q;
            });
        };
        Row before = above, cur, next;
        if constexpr (IN_LDS) cur = row_from(slot(0));
        else cur = get(Int<1>{});
        static_for<RW>([&](auto r_) JK_INLINE {
            constexpr int r = decltype(r_)::value, n = r + 1;
            if constexpr (n == RW) next = below;
            else if constexpr (n >= LT && n < LT + RR) next = get(Int<1 + n - LT>{});
            else next = row_from(slot(n));
            add(r, before, cur, next);
            before = cur;
            cur = next;
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
        return wg_sum(acc, red);                   // valid in thread 0
    };

    // ---- the run: stretches of iterations, a norm between them.  Exchange k carries the grid that iteration k made; what the first
    // iteration needs came from memory.
    int it = 0;
    for (int norm = 0;;) {
        const bool norm_ahead = norm < br.norms;
        const int until = norm_ahead ? (norm + 1) * br.every : br.iters;
        while (it + 2 <= until) {
            down();
            publish(it + 1, Int<0>{});
            receive(it + 1);
            up();
            it += 2;
            publish(it, Int<1>{});
            if (it < br.iters || norm_ahead) receive(it);
        }
        if (it < until) {
            down();
            publish(++it, Int<0>{});
            static_for<RR>([&](auto j_) JK_INLINE { put(Int<RR - decltype(j_)::value>{}, get(Int<RR - 1 - decltype(j_)::value>{})); });
            if (it < br.iters || norm_ahead) receive(it);
        }
        if (!norm_ahead) break;
        const double tot = norm_sum();
        if (threadIdx.x == 0)
            __hip_atomic_store(&br.partial[(long long)norm * nb + blk], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ++norm;
    }
    if (agent_load(&br.sync->failed) != 0u) healthy = false;
    T *fin = br.final_is_out ? gb : ga;
    {
        const int first_col = x0 + opaque_lane(lane) * C;
        const int ylo = start_of(p.y, by), yhi = end_of(p.y, by), xlo = start_of(p.x, bx), xhi = end_of(p.x, bx);
        find_cells(first_col);
        const bool whole = !seam && first_col >= xlo && first_col + C <= xhi;
        RowWalk row(g, y0 + opaque(wave) * RW);
        static_for<RW>([&](auto r_) JK_INLINE {
            constexpr int r = decltype(r_)::value;
            const int y = row0 + r;
            T *rowp = fin + (row.tile + row.i * (long long)g.pitch);
            row.next(g);
            if (y < ylo || y >= yhi) return;
            Row v;
            if constexpr (r >= LT && r < LT + RR) v = get(Int<1 + r - LT>{});
            else v = row_from(slot(r));
            RowU x;
            each([&](auto e) JK_INLINE { x[e.value] = healthy ? v.c[e.value] : T(__builtin_nan("")); });
            if (whole) *(RowU *)(rowp + co[0]) = x;
            else
                each([&](auto e) JK_INLINE {
                    if (first_col + e.value >= xlo && first_col + e.value < xhi) rowp[co[e.value]] = x[e.value];
                });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    block_epilogue(br, epoch, max_exchanges, red, &flag, CHIP2D_AREAS);
}

}  // namespace jk
