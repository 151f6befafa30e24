// Small and mid-sized 3-D grids: a whole jacobi_run in one launch, the grid in the registers of the chip.
//
// The 3-D counterpart of blocks2d_kernel (cut, messages, roll call and run as there).  Blocks cut y and z only; a
// wavefront's lanes cover whole rows (64*C cells, Nx at most as many).  The 8 wavefronts of a workgroup form a 2 x 4 grid over
// the held rows: wavefront (wz, wy) keeps a patch of RZ x RY rows in registers.  Per iteration it publishes the rows at its
// patch's border in LDS, reads those next to it, and updates its rows plane by plane, upward and downward by turns: the
// new row (z, y) goes into the registers of the old row (z-1, y), whose last reader it is, so (RZ + 1) * RY rows of registers
// hold RZ * RY rows and nothing is copied.
//
// The Dirichlet rows and planes are held like any others (the cut counts them: n = N + 2 rows) and keep their values.  In x
// the W ring cell enters lane 0 through the open end of the lane shift, the E ring cell lane 63 where a row fills the
// wavefront (EXACT); otherwise it sits in the lane cell behind the row's last one and keeps its value there.
//
// What bounds it: latencies.  A message takes 0.5 - 0.9 us from XCD to XCD, and every one to three iterations all border rows
// have to go out, arrive and be taken apart: in fp64 with 4 x 2 rows of 64 cells per wavefront 2.75 us per iteration with an exchange
// after each, whatever the number of blocks.  Measured, us per iteration, launches -> blocks, calls
// of 100 iterations: 64^3 in eight tiles 5.91 -> 2.95, 96^3 8.01 -> 5.28, 108^3 7.31 -> 6.9; in fp32 64^3 5.78 -> 2.52, 96^3 7.97 ->
// 3.67, 128^3 6.69 -> 4.04.
#pragma once
#include "blocks_common.h"

namespace jk {

// rows of a patch that a neighbouring patch reads, numbered: planes 0 and RZ-1 whole, of the planes between them the ends
template <int RZ, int RY> struct PatchBorder {
    static constexpr int N = RZ == 1 ? RY : RY == 1 ? RZ : 2 * RY + (RZ - 2) * 2;
    static constexpr bool has(int z, int y) { return z == 0 || z == RZ - 1 || y == 0 || y == RY - 1; }
    static constexpr int index(int z, int y)
    {
        return z == 0 ? y : z == RZ - 1 ? RY + y : RY == 1 ? RY + RY + z - 1 : 2 * RY + (z - 1) * 2 + (y == 0 ? 0 : 1);
    }
};

template <typename T, int C, int RZ, int RY, bool EXACT>
__global__ __launch_bounds__(BLK_WAVES * WAVE) void blocks3d_kernel(Geo g, Blocks3d p, T *ga, T *gb)
{
    typedef T VU __attribute__((ext_vector_type(C == 1 ? 2 : C), aligned(sizeof(T))));
    constexpr int WY = 4, WZ = BLK_WAVES / WY;
    constexpr unsigned MB = MSG_BYTES<T>;
    constexpr unsigned ROW_BYTES = WAVE * C * MB;               // of a row's message
    using PB = PatchBorder<RZ, RY>;
    constexpr int NBUF = 2 * BLK_WAVES * PB::N * C * WAVE * (int)sizeof(T) <= 150 * 1024 ? 2 : 1;
    __shared__ T xch[NBUF][BLK_WAVES][PB::N][C][WAVE];          // [parity][wavefront][border row][component][lane]
    __shared__ double red[BLK_WAVES];
    __shared__ int flag;

    const BlockRun &br = p.run;
    const int lane = threadIdx.x % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int wz = wave / WY, wy = wave % WY;
    const int nb = p.y.nb * p.z.nb;
    const int blk = block_of_workgroup(p.y.nb, p.z.nb, p.strip), bz = blk / p.y.nb, by = blk - bz * p.y.nb;
    const unsigned epoch = agent_load(&br.sync->epoch);
    const unsigned max_exchanges = (unsigned)br.iters + (unsigned)br.norms + 2u;
    const int d = p.y.d, Nx = p.nx;
    const int z0 = p.z.start(bz) + wz * RZ, y0 = p.y.start(by) + wy * RY;        // first row of the patch (0: ring)
    const int zlo = p.z.own_lo(bz), zhi = p.z.own_hi(bz), ylo = p.y.own_lo(by), yhi = p.y.own_hi(by);

    // ---- this lane's cells in a row of tiles; cells Nx .. are not there (the first of them keeps the E ring value)
    long long co[C];
    bool whole = true;                             // all of them exist, in one tile
    auto find_cells = [&](int first) JK_INLINE {
        const int tx = min(first, Nx - 1) / g.tw;
        int c = first - tx * g.tw;
        long long off = (long long)tx * g.tile_stride + c;
#pragma unroll
        for (int e = 0; e < C; ++e) {
            co[e] = first + e < Nx ? off : -1;
            ++off;
            if (++c == g.tw) { c = 0; off += g.tile_stride - g.tw; }
        }
        whole = first + C <= Nx && co[C - 1] - co[0] == C - 1;
    };
    const int x0 = lane * C;
    find_cells(x0);
    // where row (z, y) of the padded rows is (z in [0, Nz+1], y in [0, Ny+1]): what the plane and what the row contribute to
    // the offsets of its cells and of its entries in the x halo arrays
    struct Part { long long cells, halo; };
    auto plane_part = [&](int z) JK_INLINE -> Part {
        const int tz = min(max(z - 1, 0) / g.td, g.Tz - 1), k = z - tz * g.td;
        const long long tile = (long long)tz * g.Ty * g.Tx * g.tile_stride;
        return {tile + k * g.plane, tile + (long long)k * g.rows + g.xoff};
    };
    auto row_part = [&](int y) JK_INLINE -> Part {
        const int ty = min(max(y - 1, 0) / g.th, g.Ty - 1), i = y - ty * g.th;
        const long long tile = (long long)ty * g.Tx * g.tile_stride;
        return {tile + (long long)i * g.pitch, tile + i};
    };
    const long long e_off = (long long)(g.Tx - 1) * g.tile_stride + g.hpitch;       // from a W halo entry to the E one

    // ---- the held rows; planes 1 .. RZ of `a` (state S0), or 0 .. RZ-1 after an odd number of steps
    T a[RZ + 1][RY][C];
    T ring_w[RZ][RY], ring_e[RZ][RY];              // in lane 0 / lane 63, zero elsewhere
    Part in_plane[RY], planes[RZ];
    static_for<RY>([&](auto y_) JK_INLINE { in_plane[decltype(y_)::value] = row_part(y0 + decltype(y_)::value); });
    static_for<RZ>([&](auto z_) JK_INLINE { planes[decltype(z_)::value] = plane_part(z0 + decltype(z_)::value); });
    static_for<RZ * RY>([&](auto j_) JK_INLINE {
        constexpr int J = decltype(j_)::value, z = J / RY, y = J % RY;
            const long long cells = planes[z].cells + in_plane[y].cells, halo = planes[z].halo + in_plane[y].halo;
            if (whole && C > 1) {
                const VU v = *(const VU *)(ga + (cells + co[0]));
#pragma unroll
                for (int e = 0; e < C; ++e) a[z + 1][y][e] = v[e];
            } else {
#pragma unroll
                for (int e = 0; e < C; ++e) a[z + 1][y][e] = co[e] >= 0 ? ga[cells + co[e]] : !EXACT && x0 + e == Nx ? ga[halo + e_off] : T(0);
            }
            ring_w[z][y] = lane == 0 ? ga[halo] : T(0);
            ring_e[z][y] = EXACT && lane == WAVE - 1 ? ga[halo + e_off] : T(0);
            __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int y = 0; y < RY; ++y)
#pragma unroll
        for (int e = 0; e < C; ++e) a[0][y][e] = T(0);
    // ---- the Dirichlet ring of the other grid: the cells beside every row by a thread per row, the ring rows by a
    // wavefront per row (the two ring planes, then the two ring rows of every plane between them)
    {
        const int Py = p.y.n, Pz = p.z.n, nrows = Pz * Py;
        for (int r = blk * (BLK_WAVES * WAVE) + (int)threadIdx.x; r < nrows; r += nb * (BLK_WAVES * WAVE)) {
            const int z = r / Py;
            const long long o = plane_part(z).halo + row_part(r - z * Py).halo;
            gb[o] = ga[o];
            gb[o + e_off] = ga[o + e_off];
        }
        for (int r = blk * BLK_WAVES + wave; r < 2 * Py + 2 * (Pz - 2); r += nb * BLK_WAVES) {
            const int q = r - 2 * Py;
            const int z = q < 0 ? (r < Py ? 0 : Pz - 1) : 1 + q / 2, y = q < 0 ? (r < Py ? r : r - Py) : (q & 1) * (Py - 1);
            const long long o = plane_part(z).cells + row_part(y).cells;
#pragma unroll
            for (int e = 0; e < C; ++e)
                if (co[e] >= 0) gb[o + co[e]] = ga[o + co[e]];
        }
    }
    // Counted in once everything has been read: from the roll call on results may overwrite the source grid.
    static_for<RZ * RY>([&](auto j_) JK_INLINE {
        constexpr int J = decltype(j_)::value, z = J / RY, y = J % RY;
#pragma unroll
            for (int e = 0; e < C; ++e) arrived(a[z + 1][y][e]);
            arrived(ring_w[z][y]);
            arrived(ring_e[z][y]);
    });
    __syncthreads();
    unsigned ticket = 0;                           // looked at by thread 0 in the roll call, no sooner
    if (threadIdx.x == 0) ticket = agent_add(&br.sync->roll, 1u);

    // ---- rows that keep their value: Dirichlet rows and planes
    unsigned frozen = 0;                           // bit z * RY + y
#pragma unroll
    for (int z = 0; z < RZ; ++z)
#pragma unroll
        for (int y = 0; y < RY; ++y)
            if (z0 + z == 0 || z0 + z == p.z.n - 1 || y0 + y == 0 || y0 + y == p.y.n - 1) frozen |= 1u << (z * RY + y);
    frozen = __builtin_amdgcn_readfirstlane(frozen);

    int parity = 0;
    const int w_ym = wy > 0 ? wave - 1 : wave, w_yp = wy < WY - 1 ? wave + 1 : wave;
    const int w_zm = wz > 0 ? wave - WY : wave, w_zp = wz < WZ - 1 ? wave + WY : wave;
    auto publish = [&](auto plane0) JK_INLINE {
        constexpr int S = decltype(plane0)::value;
        if constexpr (NBUF == 1) __syncthreads();                // the rows of the step before have been read
        static_for<RZ * RY>([&](auto j_) JK_INLINE {
            constexpr int z = decltype(j_)::value / RY, y = decltype(j_)::value % RY;
            if constexpr (PB::has(z, y))
#pragma unroll
                for (int e = 0; e < C; ++e) xch[parity][wave][PB::index(z, y)][e][lane] = a[S + z][y][e];
        });
        __syncthreads();
    };
    // the four rows around row J = z * RY + y of the state whose plane 0 is S; rows of other patches from LDS
    auto around = [&](auto plane0, auto j_, T (&ym)[C], T (&yp)[C], T (&zm)[C], T (&zp)[C]) JK_INLINE {
        constexpr int S = decltype(plane0)::value, z = decltype(j_)::value / RY, y = decltype(j_)::value % RY;
#pragma unroll
        for (int e = 0; e < C; ++e) {
            if constexpr (y > 0) ym[e] = a[S + z][y - 1][e]; else ym[e] = xch[parity][w_ym][PB::index(z, RY - 1)][e][lane];
            if constexpr (y < RY - 1) yp[e] = a[S + z][y + 1][e]; else yp[e] = xch[parity][w_yp][PB::index(z, 0)][e][lane];
            if constexpr (z > 0) zm[e] = a[S + z - 1][y][e]; else zm[e] = xch[parity][w_zm][PB::index(RZ - 1, y)][e][lane];
            if constexpr (z < RZ - 1) zp[e] = a[S + z + 1][y][e]; else zp[e] = xch[parity][w_zp][PB::index(0, y)][e][lane];
        }
    };
    auto step = [&](auto up_dir, auto freeze) JK_INLINE {
        constexpr int UP = decltype(up_dir)::value, S = UP ? 0 : 1;
        constexpr bool FREEZE = decltype(freeze)::value;
        publish(std::integral_constant<int, S>{});
        static_for<RZ * RY>([&](auto i_) JK_INLINE {
            constexpr int I = decltype(i_)::value, z = UP ? RZ - 1 - I / RY : I / RY, y = I % RY, J = z * RY + y, to = UP ? z + 1 : z;
            T ym[C], yp[C], zm[C], zp[C], v[C];
            around(std::integral_constant<int, S>{}, std::integral_constant<int, J>{}, ym, yp, zm, zp);
            const T left = from_prev_lane_or(a[S + z][y][C - 1], ring_w[z][y]);
            T right;
            if constexpr (EXACT) right = from_next_lane_or(a[S + z][y][0], ring_e[z][y]);
            else right = from_next_lane_or_zero(a[S + z][y][0]);
#pragma unroll
            for (int e = 0; e < C; ++e) {
                const T c = a[S + z][y][e];
                const T w = e > 0 ? a[S + z][y][e > 0 ? e - 1 : 0] : left;
                const T ea = e < C - 1 ? a[S + z][y][e < C - 1 ? e + 1 : e] : right;
                const T val = Coef<T>::sixth * (((w + ea) + (ym[e] + yp[e])) + (zm[e] + zp[e]));
                bool keep = false;
                if constexpr (!EXACT) keep = x0 + e == Nx;
                if constexpr (FREEZE) keep = keep || (frozen >> J & 1u);
                v[e] = !EXACT || FREEZE ? (keep ? c : val) : val;
            }
#pragma unroll
            for (int e = 0; e < C; ++e) a[to][y][e] = v[e];
            // a plane of the patch at a time, so that its rows' LDS reads are under way together
            if constexpr (y == RY - 1) __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (NBUF == 2) parity ^= 1;
    };
    auto iterate_rows = [&](int n, auto freeze) JK_INLINE {
        for (int it = 0; it + 2 <= n; it += 2) {
            step(std::integral_constant<int, 0>{}, freeze);
            step(std::integral_constant<int, 1>{}, freeze);
        }
        if (n & 1) {
            step(std::integral_constant<int, 0>{}, freeze);
            static_for<RZ * RY>([&](auto i_) JK_INLINE {
                constexpr int z = RZ - decltype(i_)::value / RY, y = decltype(i_)::value % RY;
#pragma unroll
                for (int e = 0; e < C; ++e) a[z][y][e] = a[z - 1][y][e];
            });
        }
    };
    auto iterate = [&](int n) JK_INLINE {
        if (frozen) iterate_rows(n, std::true_type{});
        else iterate_rows(n, std::false_type{});
    };

    // ---- exchange.  A block's message: its owned rows within d of a side, numbered: the d lowest planes, the d highest, of
    // those between them the d first and d last rows each.  A row's cells component by component.
    auto row_number = [&](int oz, int oy, int nz, int ny) JK_INLINE -> unsigned {         // (oz, oy) in a block of nz x ny owned rows
        return (unsigned)(oz < d         ? oz * ny + oy
                          : oz >= nz - d ? (oz - (nz - d) + d) * ny + oy
                                         : 2 * d * ny + (oz - d) * 2 * d + (oy < d ? oy : oy - (ny - d) + d));
    };
    const unsigned frame = (unsigned)p.frame_rows * ROW_BYTES;
    unsigned send_at[RZ * RY], recv_at[RZ * RY];
    static_for<RZ * RY>([&](auto j_) JK_INLINE {
        constexpr int J = decltype(j_)::value, z = J / RY, y = J % RY;
            const int gz = z0 + z, gy = y0 + y;
            const int sz = gz < zlo ? bz - 1 : gz >= zhi ? bz + 1 : bz, sy = gy < ylo ? by - 1 : gy >= yhi ? by + 1 : by;
            const bool mine = sz == bz && sy == by;
            const bool needed = sz >= 0 && sz < p.z.nb && sy >= 0 && sy < p.y.nb && gz >= zlo - d && gz < zhi + d && gy >= ylo - d && gy < yhi + d;
            const int lz = p.z.own_lo(sz), ly = p.y.own_lo(sy), nz = p.z.own_hi(sz) - lz, ny = p.y.own_hi(sy) - ly;
            const int oz = gz - lz, oy = gy - ly;
            const unsigned at = (unsigned)(sz * p.y.nb + sy) * frame + row_number(oz, oy, nz, ny) * ROW_BYTES;
            const bool sends = mine && ((bz > 0 && oz < d) || (bz < p.z.nb - 1 && oz >= nz - d) || (by > 0 && oy < d) || (by < p.y.nb - 1 && oy >= ny - d));
            send_at[z * RY + y] = sends ? at : MSG_SKIP;
            recv_at[z * RY + y] = !mine && needed ? at : MSG_SKIP;
    });
    unsigned exchanges = 0;
    bool healthy = true;
    auto exchange = [&]() JK_INLINE {
        ++exchanges;
        if (!healthy) return;
        const unsigned tag = epoch + exchanges;
        const __amdgpu_buffer_rsrc_t buf = buffer_of((char *)br.msg + (size_t)(exchanges & 1u) * br.msg_bytes, br.msg_bytes);
        // Computed anew in every exchange, but for patches that fit beside them: the rows' offsets take the registers of the grid (64^3 3.21
        // -> 2.75 us per iteration, 108^3 6.81 -> 6.58 and 44 -> 28 a launch, 128^3 in fp32 4.12 -> 3.56; 96^3 4.89 -> 4.95).
        const unsigned lane_at = (unsigned)(C == 2 && RZ == 4 ? lane : opaque_lane(lane)) * MB;
        static_for<RZ * RY>([&](auto j_) JK_INLINE {
            constexpr int J = decltype(j_)::value, z = J / RY, y = J % RY;
                if (send_at[z * RY + y] != MSG_SKIP) {                  // wave-uniform
#pragma unroll
                    for (int e = 0; e < C; ++e) send_cell(a[z + 1][y][e], tag, buf, lane_at + send_at[z * RY + y] + e * (WAVE * MB));
                }
                __builtin_amdgcn_sched_barrier(0);
        });
        // ghost rows, a few at a time, each until all of its words carry the tag
        constexpr int CELLS = sizeof(T) == 8 ? 8 : 16, RB = C >= CELLS ? 1 : CELLS / C < RZ * RY ? CELLS / C : RZ * RY;
        static_for<(RZ * RY + RB - 1) / RB>([&](auto g_) JK_INLINE {
            constexpr int J0 = decltype(g_)::value * RB, N = RZ * RY - J0 < RB ? RZ * RY - J0 : RB;
            unsigned waiting = 0;                                    // bit b: row J0 + b (wave-uniform)
            static_for<N>([&](auto b_) JK_INLINE { waiting |= recv_at[J0 + decltype(b_)::value] != MSG_SKIP ? 1u << decltype(b_)::value : 0u; });
            for (unsigned n = 0; waiting != 0u && healthy;) {
                Msg<T> m[N][C];
                static_for<N>([&](auto b_) JK_INLINE {
                    constexpr int b = decltype(b_)::value;
                    if (waiting >> b & 1u)
#pragma unroll
                        for (int e = 0; e < C; ++e) m[b][e].read(buf, lane_at + recv_at[J0 + b] + e * (WAVE * MB));
                });
                static_for<N>([&](auto b_) JK_INLINE {
                    constexpr int b = decltype(b_)::value, J = J0 + b;
                    if (!(waiting >> b & 1u)) return;
                    unsigned wrong = 0;
#pragma unroll
                    for (int e = 0; e < C; ++e) wrong |= m[b][e].wrong(tag);
                    if (__any(wrong != 0u)) return;
#pragma unroll
                    for (int e = 0; e < C; ++e) a[J / RY + 1][J % RY][e] = m[b][e].value();
                    waiting &= ~(1u << b);
                });
                if (waiting != 0u && (++n > br.spin_limit || ((n & 255u) == 0u && agent_load(&br.sync->failed) != 0u))) healthy = false;
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!healthy) agent_store(&br.sync->failed, 1u);
    };

    // ---- the norm of the grid as it is: the rows next to the owned ones are current
    auto norm_sum = [&]() JK_INLINE -> double {
        publish(std::integral_constant<int, 1>{});
        double acc = 0.0;
        const int first_z = opaque(z0), first_y = opaque(y0);
        static_for<RZ * RY>([&](auto j_) JK_INLINE {
            constexpr int J = decltype(j_)::value, z = J / RY, y = J % RY;
                const int gz = first_z + z, gy = first_y + y;
                if (gz < max(zlo, 1) || gz >= min(zhi, p.z.n - 1) || gy < max(ylo, 1) || gy >= min(yhi, p.y.n - 1)) return;
                T ym[C], yp[C], zm[C], zp[C];
                around(std::integral_constant<int, 1>{}, j_, ym, yp, zm, zp);
                const T left = from_prev_lane_or(a[z + 1][y][C - 1], ring_w[z][y]), right = from_next_lane_or(a[z + 1][y][0], ring_e[z][y]);
#pragma unroll
                for (int e = 0; e < C; ++e) {
                    const T w = e > 0 ? a[z + 1][y][e > 0 ? e - 1 : 0] : left;
                    const T ea = e < C - 1 ? a[z + 1][y][e < C - 1 ? e + 1 : e] : right;
                    const T r = (((w + ea) + (ym[e] + yp[e])) + (zm[e] + zp[e])) - Coef<T>::six * a[z + 1][y][e];
                    if (x0 + e < Nx) acc += (double)r * (double)r;
                }
                __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (NBUF == 2) parity ^= 1;
        __syncthreads();
        return wg_sum(acc, red);                   // valid in thread 0
    };

    // ---- the run: stretches of at most d iterations with an exchange in between; a norm where one is due
    int it = 0, norm = 0, stale = 0;               // stale: iterations since the ghost rows were current
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
            if (__builtin_expect(flag != ALL_PRESENT, 0)) {          // (64^3 365 -> 347 us per 100 iterations)
                if (flag >= 0) plain_path<T, 3>(g, br, ga, gb, red, &flag);
                block_epilogue(br, epoch, max_exchanges, red, &flag);
                return;
            }
        }
        it += n;
        norm_due = norm_ahead && it == target;
    }
    if (agent_load(&br.sync->failed) != 0u) healthy = false;
    T *fin = br.final_is_out ? gb : ga;
    find_cells(opaque_lane(lane) * C);
    const int first_z = opaque(z0), first_y = opaque(y0);
    static_for<RY>([&](auto y_) JK_INLINE { in_plane[decltype(y_)::value] = row_part(first_y + decltype(y_)::value); });
    static_for<RZ>([&](auto z_) JK_INLINE { planes[decltype(z_)::value] = plane_part(first_z + decltype(z_)::value); });
    static_for<RZ * RY>([&](auto j_) JK_INLINE {
        constexpr int J = decltype(j_)::value, z = J / RY, y = J % RY;
            const int gz = first_z + z, gy = first_y + y;
            if (gz < max(zlo, 1) || gz >= min(zhi, p.z.n - 1) || gy < max(ylo, 1) || gy >= min(yhi, p.y.n - 1)) return;
            const long long cells = planes[z].cells + in_plane[y].cells;
            T v[C];
#pragma unroll
            for (int e = 0; e < C; ++e) v[e] = healthy ? a[z + 1][y][e] : T(__builtin_nan(""));
            if (whole && C > 1) {
                VU x;
#pragma unroll
                for (int e = 0; e < C; ++e) x[e] = v[e];
                *(VU *)(fin + (cells + co[0])) = x;
            } else {
#pragma unroll
                for (int e = 0; e < C; ++e)
                    if (co[e] >= 0) fin[cells + co[e]] = v[e];
            }
            __builtin_amdgcn_sched_barrier(0);
    });
    block_epilogue(br, epoch, max_exchanges, red, &flag);
}

}  // namespace jk
