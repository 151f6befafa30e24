// 3-D grids that the chip holds: a whole jacobi_run in one launch, the grid in registers, without ghost cells.
//
// The messages, the roll call and the run are those of the block kernels (blocks_common.h).  A block is nz x ny whole rows in x.  Its
// wavefronts are a 2 x 2 x 2 grid (NXW = 2: a row lies in two wavefronts) or two blocks of 2 x 2 (NXW = 1: in one), and each
// counts planes, rows and cells FROM THE OUTSIDE of the block: its plane 0 lies at the block's z face, its row 0 at the y face, its cell 0
// (NXW = 2) at the domain's x face; the second wavefront of a pair counts backwards.  
// So all wavefronts run the same code: beyond index 0 is another block or the ring, beyond the last index the other wavefront of the
// pair.  A wavefront holds RZ planes of RY rows of 64*C cells in registers; where the block has one row less than 2*RY (one plane,
// any number of cells), both wavefronts of the pair hold the row in the middle and compute the same bits.
//
// (Sums and their products do not depend on which of two opposite neighbours comes first.)
//
// An iteration: the rows beyond plane 0 and row 0 arrive from the one wavefront of the block there that holds them, as messages, into
// registers; those beyond the last ones come from the pair's other wavefronts through LDS, as do the cells beyond the last cell; the rows
// are updated in place, plane by plane up and down by turns (the new row (z, y) goes where (z-1, y) was: (RZ + 1) * RY rows of registers
// hold RZ * RY rows); plane 0 and row 0 are sent.  Wavefronts answer each other in pairs, so two message areas are enough.
//
// What bounds it: small grids by the messages' way - 64^3 takes 3500 clocks an iteration, 500 of them for the rows, 2000 from the sent
// message to the received one, 700 in the barrier for the others' -, larger ones by the messages' bytes (0.15 us per MB of all blocks, beside
// what the rows take), which is why their tags are single bytes: with a tag behind every 4 bytes 64^3 takes 2.15 us instead of 1.78, 128^3
// 5.6 instead of 4.0, 210 x 198 x 250 in fp32 12.6 instead of 9.0.  Measured, us per iteration in long runs, launches or blocks3d_kernel -> here: fp64
// 48^3 2.6 -> 1.4, 64^3 3.2 -> 1.5, 96^3 4.9 -> 2.4, 108^3 6.8 -> 3.0, 128^3 7.8 -> 3.4, 160^3 14.4 -> 7.4; fp32 64^3 2.4 -> 1.3, 96^3 3.3 -> 1.8, 128^3 4.1 -> 2.4,
// 160^3 9.7 -> 3.9, 210 x 198 x 250 17.1 -> 5.0, 230 x 220 x 256 19.1 -> 5.7.  A launch takes 18 us besides, 0.55 per MB of the grid and 0.03
// per workgroup.  Larger patches than the compiled ones spill (fp64 2 cells x 6 x 6 rows: 8.2 us for 160^3).
#pragma once
#include "blocks_common.h"

namespace jk {

template <typename T, int C, int RZ, int RY, int NXW>
__global__ __launch_bounds__(BLK_WAVES * WAVE) void chip3d_kernel(Geo g, Chip3d p, T *ga, T *gb)
{
    constexpr int BW = 4 * NXW;                                               // wavefronts of a block
    constexpr int R = RZ * RY, N_OUT = RZ + RY;
    constexpr int NBUF = 2 * BLK_WAVES * N_OUT * C * WAVE * (int)sizeof(T) <= 128 * 1024 ? 2 : 1;
    static_assert(RZ >= 2 && RY >= 2, "");
    struct Row { T c[C]; };
    typedef T WE __attribute__((ext_vector_type(2)));
    __shared__ T xch[NBUF][BLK_WAVES][N_OUT][C][WAVE];          // rows for the pairs' other wavefronts: the last plane's, then the last rows
    // the cells beyond a row's first and last cell (W, E; two sets, by wavefront and row), and a place where nobody looks
    constexpr int NOWHERE = 2 * BLK_WAVES * R * 2;
    __shared__ alignas(16) T beside[NOWHERE + 2 * R + WAVE];
    __shared__ double red[BLK_WAVES];
    __shared__ int flag;

    const BlockRun &br = p.run;
    const int lane = threadIdx.x % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int wx = NXW == 2 ? wave & 1 : 0, wy = wave / NXW & 1, wz = wave / (2 * NXW) & 1;
    const int nb = p.y.nb * p.z.nb;
    const unsigned epoch = __builtin_amdgcn_readfirstlane(agent_load(&br.sync->epoch));
    // the blocks in the order in which the XCDs get runs of them: strips of p.strip blocks in y
    const int number = __builtin_amdgcn_readfirstlane(run_of_workgroup() * (BLK_WAVES / BW) + wave / BW);
    const bool there = number < nb;                // the last workgroup may have one block only
    int bz, by;
    {
        const int m = min(number, nb - 1), s = m / (p.strip * p.z.nb), in_strip = m - s * p.strip * p.z.nb, w = min(p.strip, p.y.nb - s * p.strip);
        bz = __builtin_amdgcn_readfirstlane(in_strip / w);
        by = __builtin_amdgcn_readfirstlane(s * p.strip + in_strip - bz * w);
    }
    const int Nx = p.nx;
    const int zs = p.z.start(bz), ze = p.z.start(bz + 1), ys = p.y.start(by), ye = p.y.start(by + 1);
    const bool short_z = ze - zs < 2 * RZ, short_y = ye - ys < 2 * RY;        // then by one
    // padded index (0: ring) of plane k, row j and cell i of this wavefront; -1: the one beyond
    auto at_z = [&](int k) JK_INLINE { return wz == 0 ? zs + 1 + k : ze - k; };
    auto at_y = [&](int j) JK_INLINE { return wy == 0 ? ys + 1 + j : ye - j; };
    auto at_x = [&](int i) JK_INLINE { return wx == 0 ? 1 + i : Nx - i; };
    auto cell = [&](int z, int y, int x) JK_INLINE { return domain_cell_off(g, z - 1, y - 1, x - 1); };        // of padded indexes
    // what the plane and what the row contribute to the offsets of a row's cells and of its entries in the x halo arrays
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
    auto x_part = [&](int x) JK_INLINE -> long long {           // of cell x of a row of tiles; -1: beyond its last one
        const int tx = (x - 1) / g.tw;
        return x > Nx ? -1 : (long long)tx * g.tile_stride + (x - 1 - tx * g.tw);
    };
    long long co[C];
    auto find_cells = [&](int l) JK_INLINE { static_for<C>([&](auto e) JK_INLINE { co[e.value] = x_part(at_x(l * C + e.value)); }); };
    find_cells(lane);
    auto row_of = [&](const Part &z, const Part &y) JK_INLINE -> Row {
        Row v;
        static_for<C>([&](auto e) JK_INLINE {
            const long long o = NXW == 1 && co[e.value] < 0 ? z.halo + y.halo + e_off : z.cells + y.cells + co[e.value];
            v.c[e.value] = ga[o];
        });
        return v;
    };

    // ---- the held rows: planes 1 .. RZ of `a`, or 0 .. RZ-1 between a step down and one up; the rows beyond plane 0 and beyond the rows 0
    T a[RZ + 1][RY][C], gz[RY][C], gy[RZ][C];
    auto put = [&](T(&to)[C], const Row &v) JK_INLINE { static_for<C>([&](auto e) JK_INLINE { to[e.value] = v.c[e.value]; }); };
    {
        Part rows[RY];
        const Part z_out = plane_part(at_z(-1)), y_out = row_part(at_y(-1));
        static_for<RY>([&](auto y) JK_INLINE {
            rows[y.value] = row_part(at_y(y.value));
            put(gz[y.value], row_of(z_out, rows[y.value]));
            put(a[0][y.value], Row{});
        });
        static_for<RZ>([&](auto z) JK_INLINE {
            const Part plane = plane_part(at_z(z.value));
            put(gy[z.value], row_of(plane, y_out));
            static_for<RY>([&](auto y) JK_INLINE { put(a[z.value + 1][y.value], row_of(plane, rows[y.value])); });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    static_assert(R <= WAVE, "");
    if (lane < R) {                                // the cells beside row `lane`
        const Part z = plane_part(at_z(lane / RY)), y = row_part(at_y(lane % RY));
        const long long halo = z.halo + y.halo, inner = NXW == 2 ? x_part(at_x(WAVE * C)) : -1;
        const bool whole = NXW == 1 || Nx == WAVE * C;           // the other end of the row, too: the ring on both sides
        const WE b = {ga[halo + (wx == 0 ? 0 : e_off)], ga[whole ? halo + (wx == 0 ? e_off : 0) : z.cells + y.cells + inner]};
        *(WE *)&beside[2 * (wave * R + lane)] = b;
        *(WE *)&beside[2 * ((BLK_WAVES + wave) * R + lane)] = b;
    }
    // ---- the Dirichlet ring of the other grid: the cells beside every row by a thread per row, the ring rows by a wavefront per
    // row (the two ring planes, then the two ring rows of every plane between them)
    {
        const int Py = p.y.n + 2, Pz = p.z.n + 2, nrows = Pz * Py, nwg = gridDim.x;
        for (int r = blockIdx.x * (BLK_WAVES * WAVE) + (int)threadIdx.x; r < nrows; r += nwg * (BLK_WAVES * WAVE)) {
            const int z = r / Py, y = r - z * Py;
            for (int x = 0; x <= Nx + 1; x += Nx + 1) { const long long o = cell(z, y, x); gb[o] = ga[o]; }
        }
        for (int r = blockIdx.x * BLK_WAVES + wave; r < 2 * Py + 2 * (Pz - 2); r += nwg * BLK_WAVES) {
            const int q = r - 2 * Py;
            const int z = q < 0 ? (r < Py ? 0 : Pz - 1) : 1 + q / 2, y = q < 0 ? (r < Py ? r : r - Py) : (q & 1) * (Py - 1);
            for (int x = 1 + lane; x <= Nx; x += WAVE) { const long long o = cell(z, y, x); gb[o] = ga[o]; }
        }
    }
    // ---- where this wavefront's messages are, and those of the two wavefronts that hold what lies beyond its plane 0 and its rows 0
    constexpr unsigned Z_BYTES = ByteTagged<T, RY * C>::BYTES, FRAME = Z_BYTES + ByteTagged<T, RZ * C>::BYTES;
    const bool z_out = there && (wz == 0 ? bz > 0 : bz < p.z.nb - 1), y_out = there && (wy == 0 ? by > 0 : by < p.y.nb - 1);
    auto frame_of = [&](int z, int y, int w) JK_INLINE { return (unsigned)((z * p.y.nb + y) * BW + w) * FRAME; };
    const int in_block = wave % BW;
    const unsigned mine = frame_of(bz, by, in_block);
    const unsigned from_z = frame_of(wz == 0 ? bz - 1 : bz + 1, by, in_block ^ (2 * NXW)), from_y = frame_of(bz, wy == 0 ? by - 1 : by + 1, in_block ^ NXW);
    // Tags of one byte come round, so what earlier launches left has to go before anybody looks: each wavefront clears what it will send.
    if (there)
        for (int exchange = 0; exchange < 2; ++exchange)
            for (unsigned at = (unsigned)lane * 16u; at < FRAME; at += WAVE * 16u)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, buffer_of((char *)br.msg + (size_t)exchange * br.msg_bytes, br.msg_bytes),
                                                       (int)(mine + at), 0, AUX_AGENT);
    // Counted in once everything has been read: from the roll call on results may overwrite the source grid.
    static_for<R * C>([&](auto k_) JK_INLINE {
        constexpr int k = decltype(k_)::value;
        arrived(a[1 + k / C / RY][k / C % RY][k % C]);
    });
    static_for<RY * C>([&](auto k) JK_INLINE { arrived(gz[k.value / C][k.value % C]); });
    static_for<RZ * C>([&](auto k) JK_INLINE { arrived(gy[k.value / C][k.value % C]); });
    stores_arrived();                              // the cleared messages of every wavefront
    __syncthreads();
    if (threadIdx.x == 0) roll_call(br.sync, gridDim.x, br.admitted, agent_add(&br.sync->roll, 1u), br.roll_limit, &flag);
    __syncthreads();
    if (__builtin_expect(flag != ALL_PRESENT, 0)) {
        if (flag >= 0) plain_path<T, 3>(g, br, ga, gb, red, &flag);
        block_epilogue(br, epoch, 0u, red, &flag);
        return;
    }

    // ---- what the pair's other wavefronts need: the last plane and the last rows, or the ones before where the block is short; the cell
    // that lies beyond the other one's last
    const int pair_x = wave ^ 1, pair_y = wave ^ NXW, pair_z = wave ^ (2 * NXW);
    const int out_x = Nx - 1 - WAVE * C;           // NXW = 2; counted as this wavefront counts; -1: the other one has the whole row
    const int beside_at = opaque_lane(2 * wave * R);
    const bool edge_lane = NXW == 2 && out_x >= 0 && lane == out_x / C;
    const bool keep_ring = NXW == 1 && Nx < WAVE * C;          // cells from Nx on keep their values: the ring's is the first
    int set = 0;
    auto publish = [&](auto plane0) JK_INLINE {
        constexpr int S = decltype(plane0)::value;
        if constexpr (NBUF == 1) __syncthreads();                // the rows of the step before have been read
        const int to = NBUF == 2 ? set ^ 1 : 0;
        static_for<RY>([&](auto y) JK_INLINE {
            static_for<C>([&](auto e) JK_INLINE {
                xch[to][wave][y.value][e.value][lane] = pick(short_z, a[S + RZ - 2][y.value][e.value], a[S + RZ - 1][y.value][e.value]);
            });
        });
        static_for<RZ>([&](auto z) JK_INLINE {
            static_for<C>([&](auto e) JK_INLINE {
                xch[to][wave][RY + z.value][e.value][lane] = pick(short_y, a[S + z.value][RY - 2][e.value], a[S + z.value][RY - 1][e.value]);
            });
        });
        if constexpr (NXW == 2) {
            const int cells = edge_lane ? 2 * ((set ^ 1) * BLK_WAVES + pair_x) * R + 1 : NOWHERE + lane;
            static_for<R>([&](auto r_) JK_INLINE {
                constexpr int z = decltype(r_)::value / RY, y = decltype(r_)::value % RY;
                T v = a[S + z][y][C - 1];
                if constexpr (C > 1)
                    static_for<C - 1>([&](auto e) JK_INLINE { v = pick(out_x % C == e.value, a[S + z][y][e.value], v); });
                beside[cells + 2 * decltype(r_)::value] = v;
            });
        }
    };
    // sum of the six neighbours of the row's cells
    auto sums = [&](auto plane0, auto r_, const WE &b) JK_INLINE -> Row {
        constexpr int S = decltype(plane0)::value, z = decltype(r_)::value / RY, y = decltype(r_)::value % RY;
        const T(&c)[C] = a[S + z][y];
        const int from = NBUF == 2 ? set : 0;
        const T left = from_prev_lane(c[C - 1], b[0]), right = from_next_lane(c[0], b[1]);
        Row s;
        static_for<C>([&](auto e_) JK_INLINE {
            constexpr int e = decltype(e_)::value;
            T w = left, ea = right, ym, yp, zm, zp;
            if constexpr (e > 0) w = c[e - 1];
            if constexpr (e < C - 1) ea = c[e + 1];
            if constexpr (y > 0) ym = a[S + z][y - 1][e]; else ym = gy[z][e];
            if constexpr (y < RY - 1) yp = a[S + z][y + 1][e]; else yp = xch[from][pair_y][RY + z][e][lane];
            if constexpr (z > 0) zm = a[S + z - 1][y][e]; else zm = gz[y][e];
            if constexpr (z < RZ - 1) zp = a[S + z + 1][y][e]; else zp = xch[from][pair_z][y][e][lane];
            s.c[e] = ((w + ea) + (ym + yp)) + (zm + zp);
        });
        return s;
    };
    auto step = [&](auto up_dir) JK_INLINE {
        constexpr int UP = decltype(up_dir)::value, S = UP ? 0 : 1;
        const int bs = beside_at + set * (2 * BLK_WAVES * R);
        WE ahead = *(const WE *)&beside[bs + 2 * (UP ? (RZ - 1) * RY : 0)];
        static_for<R>([&](auto i_) JK_INLINE {
            constexpr int I = decltype(i_)::value, z = UP ? RZ - 1 - I / RY : I / RY, y = I % RY, to = UP ? z + 1 : z;
            constexpr int nz = UP ? RZ - 1 - (I + 1) / RY : (I + 1) / RY, ny = (I + 1) % RY;
            const WE b = ahead;
            if constexpr (I + 1 < R) ahead = *(const WE *)&beside[bs + 2 * (nz * RY + ny)];
            Row v = sums(std::integral_constant<int, S>{}, std::integral_constant<int, z * RY + y>{}, b);
            static_for<C>([&](auto e) JK_INLINE {
                T x = Coef<T>::sixth * v.c[e.value];
                if constexpr (NXW == 1) x = pick(keep_ring && lane * C + e.value >= Nx, a[S + z][y][e.value], x);
                arrived(x);                        // computed here, not behind later branches
                v.c[e.value] = x;
            });
            put(a[to][y], v);
            if constexpr (I % 2 == 1 || y == RY - 1) __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ---- messages: a wavefront's plane 0 to one neighbour, its rows 0 to another
    constexpr int NZ = RY * C, NY = RZ * C;                      // cells per lane
    bool healthy = true;
    auto area = [&](int exchange) JK_INLINE {
        return buffer_of((char *)br.msg + (size_t)(exchange & 1) * br.msg_bytes, br.msg_bytes);
    };
    auto send = [&](int exchange, auto plane0) JK_INLINE {
        constexpr int S = decltype(plane0)::value;
        const unsigned tag = byte_tag(exchange);
        const __amdgpu_buffer_rsrc_t buf = area(exchange);
        if (z_out) ByteTagged<T, NZ>::send(tag, buf, mine, opaque_lane(lane), [&](auto k) JK_INLINE -> T { return a[S][k.value / C][k.value % C]; });
        if (y_out) ByteTagged<T, NY>::send(tag, buf, mine + Z_BYTES, opaque_lane(lane), [&](auto k) JK_INLINE -> T { return a[S + k.value / C][0][k.value % C]; });
    };
    auto receive = [&](int exchange) JK_INLINE {
        if (!healthy) return;
        const unsigned tag = byte_tag(exchange);
        const __amdgpu_buffer_rsrc_t buf = area(exchange);
        const int l = opaque_lane(lane);
        bool want_z = z_out, want_y = y_out;       // wave-uniform
        // Blocks run level with each other, so asked at once the first question would come just too early and the answer to the second
        // one a way to memory and back later.  A launch of few workgroups, and one whose wavefronts have many rows, ends an exchange sooner than
        // the wait does, or runs less level, and loses by it: so it depends on the rows, and on the workgroups from which on it measured faster.  Us per
        // 100 iterations with scatter and gather, at once -> after this wait (5 to 9 times 64 clocks; 3 more or less are up to 3 % slower or, 64^3 with
        // 8, 2 % faster):
        //   one cell, one wavefront to a row: 2 x 2 rows, 121 workgroups 180 -> 172, fp32 203 182 -> 167 (8: 123 -> 128, not told apart: the
        //     branch would cost the others as much); 3 x 3, 111: 210 -> 199 (63: 184 -> 189); 4 x 4, 115: 269 -> 261 (98: 248 -> 253, but 120: 249
        //     -> 255, too), fp32 209: 256 -> 241 (96: 197 -> 204); 6 x 6, 176: 470 -> 446 (120: 394 -> 399), fp32 181: 353 -> 323 (111: 283 -> 289)
        //   two wavefronts, fp64: 3 x 3 and 4 x 3, 176 to 255 workgroups 2 to 7 % faster (128: 135 -> 138); 4 x 4, 204 to 253 2 to 4 (182: 298 ->
        //     302); 5 x 5 from 0.8 % faster to 1.6 slower; 6 x 6 up to 2 % slower up to 208, then the same.  Two cells: 128^3 391 -> 378, but
        //     196 x 115 x 140 792 -> 801
        //   fp32, two wavefronts or more cells: up to 5 x 5, 176 to 256 1 to 9 % faster (80: 149 -> 158); more rows, 200 to 256 the same to 2 % faster
        //     (6 x 6, 176: 418 -> 426)
        constexpr bool F64 = sizeof(T) == 8;
        constexpr unsigned NEVER = ~0u, ROWS = RZ * RY;
        constexpr unsigned WAIT_FROM = C == 1 && NXW == 1 ? (RZ <= 2 || (RZ == 3 && !F64) ? 0 : RZ == 3 ? 70 : RZ == 4 || !F64 ? 112 : 176)
                                       : F64              ? (C > 1 || ROWS >= 25 ? NEVER : ROWS >= 16 ? 200 : 176)
                                                          : (ROWS > 25 ? 200 : 176);
        if constexpr (WAIT_FROM != NEVER)
            if (WAIT_FROM == 0 || gridDim.x >= WAIT_FROM) __builtin_amdgcn_s_sleep(F64 ? 5 : NXW == 1 && C == 1 ? 9 : 8);
        for (unsigned n = 0; want_z || want_y;) {
            ByteTagged<T, NZ> mz;
            ByteTagged<T, NY> my;
            if (want_z) mz.read(buf, from_z, l);
            if (want_y) my.read(buf, from_y + Z_BYTES, l);
            if (want_z && !__any(mz.wrong(tag))) {
                mz.take([&](auto k, T v) JK_INLINE { gz[k.value / C][k.value % C] = v; });
                want_z = false;
            }
            if (want_y && !__any(my.wrong(tag))) {
                my.take([&](auto k, T v) JK_INLINE { gy[k.value / C][k.value % C] = v; });
                want_y = false;
            }
            if ((want_z || want_y) && (++n > br.spin_limit || ((n & 255u) == 0u && agent_load(&br.sync->failed) != 0u))) {
                healthy = false;
                agent_store(&br.sync->failed, 1u);
                break;
            }
        }
    };
    auto finish_step = [&](int exchange, auto plane0) JK_INLINE {
        send(exchange, plane0);
        publish(plane0);
        set ^= 1;
        __syncthreads();
    };

    // ---- the norm of the grid as it is (planes 1 ..; the rows beyond are current)
    auto norm_sum = [&]() JK_INLINE -> double {
        double acc = 0.0;
        const int cells = NXW == 2 ? (wx == 0 ? WAVE * C : Nx - WAVE * C) : Nx, first = opaque_lane(lane) * C;
        const int planes = there ? wz == 1 && short_z ? RZ - 1 : RZ : 0, rows = wy == 1 && short_y ? RY - 1 : RY;
        static_for<R>([&](auto r_) JK_INLINE {
            constexpr int z = decltype(r_)::value / RY, y = decltype(r_)::value % RY;
            if (z >= planes || y >= rows) return;
            const Row s = sums(std::integral_constant<int, 1>{}, r_, *(const WE *)&beside[2 * ((set * BLK_WAVES + wave) * R + decltype(r_)::value)]);
            static_for<C>([&](auto e) JK_INLINE {
                const T q = s.c[e.value] - Coef<T>::six * a[z + 1][y][e.value];
                if (first + e.value < cells) acc += (double)q * (double)q;
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
        return wg_sum(acc, red);                   // valid in thread 0
    };

    // ---- the run: stretches of iterations, a norm between them.  Exchange k carries the grid that iteration k made; what the first
    // iteration needs of other blocks came from memory, of the other wavefronts through LDS.
    publish(std::integral_constant<int, 1>{});
    set ^= 1;
    __syncthreads();
    int it = 0;
    for (int norm = 0;;) {
        const bool norm_ahead = norm < br.norms;
        const int until = norm_ahead ? (norm + 1) * br.every : br.iters;
        while (it + 2 <= until) {
            step(std::integral_constant<int, 0>{});
            finish_step(it + 1, std::integral_constant<int, 0>{});
            receive(it + 1);
            step(std::integral_constant<int, 1>{});
            it += 2;
            finish_step(it, std::integral_constant<int, 1>{});
            if (it < br.iters || norm_ahead) receive(it);
        }
        if (it < until) {
            step(std::integral_constant<int, 0>{});
            finish_step(++it, std::integral_constant<int, 0>{});
            static_for<R * C>([&](auto k_) JK_INLINE {
                constexpr int k = decltype(k_)::value, z = RZ - k / C / RY, y = k / C % RY;
                a[z][y][k % C] = a[z - 1][y][k % C];
            });
            if (it < br.iters || norm_ahead) receive(it);
        }
        if (!norm_ahead) break;
        const double tot = norm_sum();
        if (threadIdx.x == 0)
            __hip_atomic_store(&br.partial[(long long)norm * gridDim.x + blockIdx.x], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ++norm;
    }
    if (agent_load(&br.sync->failed) != 0u) healthy = false;
    T *fin = br.final_is_out ? gb : ga;
    {
        const int cells = NXW == 2 ? (wx == 0 ? WAVE * C : Nx - WAVE * C) : Nx, first = opaque_lane(lane) * C;
        const int planes = there ? wz == 1 && short_z ? RZ - 1 : RZ : 0, rows = wy == 1 && short_y ? RY - 1 : RY;
        find_cells(opaque_lane(lane));
        static_for<RZ>([&](auto z) JK_INLINE {
            if (z.value >= planes) return;
            const long long plane = plane_part(opaque(at_z(z.value))).cells;
            static_for<RY>([&](auto y) JK_INLINE {
                if (y.value >= rows) return;
                const long long row = plane + row_part(opaque(at_y(y.value))).cells;
                static_for<C>([&](auto e) JK_INLINE {
                    if (first + e.value < cells) fin[row + co[e.value]] = healthy ? a[z.value + 1][y.value][e.value] : T(__builtin_nan(""));
                });
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    block_epilogue(br, epoch, 0u, red, &flag);
}

}  // namespace jk
