// What the block kernels (blocks2d_kernel.h, blocks3d_kernel.h, chip2d_kernel.h, chip3d_kernel.h) share: how the workgroups of a launch find out
// that they are all there, the messages they pass each other, the plain path they take if they are not, and how
// a launch ends.
//
// A block kernel runs ALL iterations of a jacobi_run in one launch: every workgroup keeps a block of the grid
// in registers, with `d` ghost cells around the part it owns, iterates `d` times without talking to anybody,
// and then exchanges the border of its block with its neighbours - with these alone, there is no barrier over
// the whole chip.
//
// Messages.  Every 8-byte word of a message carries 32 bits of payload and a 32-bit tag (the number of the
// exchange), so a word proves by itself that it has arrived: the receiver reads the cells it needs until all tags
// are right.  One store and one load are the whole transfer; no flag follows the data and no cache has to be
// written back or dropped (the accesses are agent-scope ones, which the XCDs' L2s pass through).  The
// price is twice the bytes, which are few.  Two message areas take turns: a workgroup writes exchange x + 2 into
// the area of exchange x only after it has read the neighbours' x + 1, which they sent after reading x.  Tags
// never repeat: a launch counts on from the plan's epoch, which the workgroup that finishes last moves on.
//
// Roll call.  Receiving means waiting, so the workgroups have to run at the same time.  They are at most one per
// CU, but other work may hold CUs - another plan's launch of this kind, too, which would wait in the same way.
// So nobody waits for a workgroup that may never start: each one counts itself in, and before its first exchange
// (or result) checks that all have; if one is missing for too long the roll is CLOSED.  Those that were counted
// then do the work together along the plain path - one iteration after the other through memory, a barrier among
// themselves in between - from the untouched source grid, and those that come later find the roll closed and
// leave.  Slower, but the same bits, and no launch depends on what else runs.
#pragma once
#include "launchers.h"
#include <utility>

// Lambdas that touch arrays kept in registers: one that the compiler does not inline puts them into memory.
#define JK_INLINE __attribute__((always_inline))

namespace jk {

constexpr unsigned ROLL_CLOSED = 1u << 30;

__device__ __forceinline__ unsigned agent_load(unsigned *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void agent_store(unsigned *p, unsigned v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned agent_add(unsigned *p, unsigned v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The same value, which the compiler cannot know to be the same: what is computed from it is computed again instead of
// kept in registers from the last time (row addresses, message offsets - the registers hold the grid).
__device__ __forceinline__ int opaque(int uniform) { uniform = __builtin_amdgcn_readfirstlane(uniform); asm volatile("" : "+s"(uniform)); return uniform; }
__device__ __forceinline__ int opaque_lane(int v) { asm volatile("" : "+v"(v)); return v; }

// Are all `expected` workgroups there?  *outcome: ALL_PRESENT, or TOO_LATE if the roll was closed before this workgroup
// counted itself in (it got `ticket`), or else this workgroup's number on the plain path.  Only the first `admitted` workgroups
// are let in: fewer than expected on request, as if the others had come too late.  One thread calls it.
constexpr int ALL_PRESENT = -1, TOO_LATE = -2;
__device__ __forceinline__ void roll_call(BlockSync *s, unsigned expected, unsigned admitted, unsigned ticket, unsigned limit, int *outcome)
{
    if (ticket >= admitted) { *outcome = TOO_LATE; return; }        // ROLL_CLOSED is beyond every number
    unsigned members = 0;
    for (unsigned n = 0; n <= limit; ++n) {
        const unsigned r = agent_load(&s->roll);
        if (r & ROLL_CLOSED) break;
        if (r >= admitted) {
            if (admitted == expected) members = expected;
            break;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    if (members == 0) {
        const unsigned before = __hip_atomic_fetch_or(&s->roll, ROLL_CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!(before & ROLL_CLOSED)) {
            members = min(before, admitted);
            agent_store(&s->participants, members);
            stores_arrived();                     // this workgroup's other wavefronts read it, too
        } else {
            // whoever closed it writes the number next: it runs, so this ends
            while ((members = agent_load(&s->participants)) == 0u) __builtin_amdgcn_s_sleep(1);
        }
    }
    *outcome = members == expected ? ALL_PRESENT : (int)ticket;
}

// A loaded value that has to be there before the program goes on.
template <typename T> __device__ __forceinline__ void arrived(T &v) { asm volatile("" : "+v"(v)); }

// One of two values - not one of two places: the arrays they come from stay in registers.
template <typename T> __device__ __forceinline__ T pick(bool first, T x, T y) { return first ? x : y; }

// f(0), f(1), ..., f(N-1) with compile-time indexes (integral_constant): arrays indexed by them stay in registers
// however much code a turn is.
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// Which block a workgroup takes.  The hardware deals workgroups out to the 8 XCDs in turn, and a message between two
// workgroups of one XCD stays in its L2 (one word per lane 0.44 us against 0.53 - 0.63, 16 in a row 0.77 against
// 1.1 - 1.2, and nothing on the way to memory), so each XCD gets a
// compact patch of blocks: the blocks are numbered strip by strip (`strip` blocks wide, rows of a strip one after the other)
// and every XCD takes a run of numbers.  strip = 0: as dealt.  Where a workgroup really runs does not matter for the result.
__device__ __forceinline__ int block_of_workgroup(int nbx, int nby, int strip)
{
    const int nb = nbx * nby, wg = blockIdx.x, xcd = wg % NUM_XCD;
    if (strip == 0) return wg;
    const int n = xcd * (nb / NUM_XCD) + min(xcd, nb % NUM_XCD) + wg / NUM_XCD;
    const int s = n / (strip * nby), in_strip = n - s * strip * nby, w = min(strip, nbx - s * strip);
    const int y = in_strip / w;
    return y * nbx + s * strip + in_strip - y * w;
}

// This workgroup's number when every XCD takes a run of consecutive ones.
__device__ __forceinline__ int run_of_workgroup()
{
    const int wg = blockIdx.x, n = gridDim.x, xcd = wg % NUM_XCD;
    return xcd * (n / NUM_XCD) + min(xcd, n % NUM_XCD) + wg / NUM_XCD;
}

// ---- messages -------------------------------------------------------------------------------------------
constexpr int AUX_AGENT = 16;               // sc1: agent scope, past the L2
constexpr int AUX_VOLATILE = (int)0x80000000u;
constexpr unsigned MSG_SKIP = 0x40000000u;  // an offset beyond every message area, also after another one has been added to it
template <typename T> constexpr int MSG_BYTES = 2 * (int)sizeof(T);      // of one cell

// One cell: its payload in 8-byte words, each with the tag behind it.
__device__ __forceinline__ void send_cell(double v, unsigned tag, __amdgpu_buffer_rsrc_t buf, unsigned off)
{
    const Int2 x = __builtin_bit_cast(Int2, v);
    const u32x4 m = {(unsigned)x.lo, tag, (unsigned)x.hi, tag};
    // No scalar offset: behind a 16-byte store with one the compiler lets the next vector instruction overwrite the
    // data registers at once, and on this chip the store then sent the new contents in some lanes (the low halves of
    // lanes 12 - 15 of every 16 here).  Without one it keeps them apart.
    __builtin_amdgcn_raw_buffer_store_b128(m, buf, (int)off, 0, AUX_AGENT);
}
__device__ __forceinline__ void send_cell(float v, unsigned tag, __amdgpu_buffer_rsrc_t buf, unsigned off)
{
    const u32x2 m = {__builtin_bit_cast(unsigned, v), tag};
    __builtin_amdgcn_raw_buffer_store_b64(m, buf, (int)off, 0, AUX_AGENT);
}
template <typename T> struct Msg;
template <> struct Msg<double> {
    u32x4 m;
    __device__ __forceinline__ void read(__amdgpu_buffer_rsrc_t buf, unsigned off)
    {
        m = __builtin_amdgcn_raw_buffer_load_b128(buf, (int)off, 0, AUX_AGENT | AUX_VOLATILE);
    }
    __device__ __forceinline__ unsigned wrong(unsigned tag) const { return (m[1] ^ tag) | (m[3] ^ tag); }      // 0: it is there
    __device__ __forceinline__ double value() const { return __builtin_bit_cast(double, Int2{(int)m[0], (int)m[2]}); }
};
template <> struct Msg<float> {
    u32x2 m;
    __device__ __forceinline__ void read(__amdgpu_buffer_rsrc_t buf, unsigned off)
    {
        m = __builtin_amdgcn_raw_buffer_load_b64(buf, (int)off, 0, AUX_AGENT | AUX_VOLATILE);
    }
    __device__ __forceinline__ unsigned wrong(unsigned tag) const { return m[1] ^ tag; }
    __device__ __forceinline__ float value() const { return __builtin_bit_cast(float, m[0]); }
};

// N cells per lane in 8-byte words with a tag of ONE byte each: the cells' 8-byte values (fp32: two cells each) with the highest byte
// replaced by the tag, and words of seven such bytes behind them.  9.1 to 12 bytes per fp64 cell instead of 16, 4.6 to 6 per fp32 cell
// instead of 8, for two or three more instructions on either side.  The tags come round after 255 exchanges, which is no
// matter as long as a word holds nothing older than the exchange before the one waited for: whoever sends clears its words at the
// start of a launch.  (Where the bytes are what an exchange costs: in 3-D.)
__device__ __forceinline__ unsigned byte_tag(int exchange) { return (unsigned)(exchange % 255 + 1) << 24; }
template <typename T, int N> struct ByteTagged {
    static constexpr int PER = 8 / (int)sizeof(T), M = (N + PER - 1) / PER, WORDS = M + (M + 6) / 7, PAIRS = WORDS / 2;
    static constexpr unsigned BYTES = byte_tagged_bytes(N, (int)sizeof(T));
    unsigned lo[WORDS], hi[WORDS];

    // word i of the message from its values' halves (get(item) -> Int2)
    template <int I, typename G> static __device__ __forceinline__ Int2 word(unsigned tag, G &&get)
    {
        if constexpr (I < M) {
            const Int2 v = get(std::integral_constant<int, I>{});
            return {v.lo, (int)(((unsigned)v.hi & 0xffffffu) | tag)};
        } else {
            constexpr int J = (I - M) * 7;
            unsigned l = 0, h = tag;
            static_for<7>([&](auto k) JK_INLINE {
                if constexpr (J + k.value < M) {
                    const unsigned top = (unsigned)get(std::integral_constant<int, J + k.value>{}).hi >> 24;
                    if constexpr (k.value < 4) l |= top << (8 * k.value);
                    else h |= top << (8 * (k.value - 4));
                }
            });
            return {(int)l, (int)h};
        }
    }
    template <typename F> static __device__ __forceinline__ void send(unsigned tag, __amdgpu_buffer_rsrc_t buf, unsigned at, int lane, F &&cell)
    {
        auto get = [&](auto i) JK_INLINE -> Int2 {
            if constexpr (PER == 1) return __builtin_bit_cast(Int2, cell(i));
            else {
                constexpr int K = 2 * decltype(i)::value;
                int h = 0;
                if constexpr (K + 1 < N) h = __builtin_bit_cast(int, cell(std::integral_constant<int, K + 1>{}));
                return {__builtin_bit_cast(int, cell(std::integral_constant<int, K>{})), h};
            }
        };
        static_for<PAIRS>([&](auto k) JK_INLINE {
            const Int2 x = word<2 * k.value>(tag, get), y = word<2 * k.value + 1>(tag, get);
            const u32x4 m = {(unsigned)x.lo, (unsigned)x.hi, (unsigned)y.lo, (unsigned)y.hi};
            __builtin_amdgcn_raw_buffer_store_b128(m, buf, (int)(at + (unsigned)lane * 16u + k.value * (WAVE * 16u)), 0, AUX_AGENT);      // (no scalar offset: see send_cell)
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (WORDS % 2 == 1) {
            const Int2 x = word<WORDS - 1>(tag, get);
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{(unsigned)x.lo, (unsigned)x.hi}, buf, (int)(at + (unsigned)lane * 8u + PAIRS * (WAVE * 16u)), 0, AUX_AGENT);
        }
    }
    __device__ __forceinline__ void read(__amdgpu_buffer_rsrc_t buf, unsigned at, int lane)
    {
        static_for<PAIRS>([&](auto k) JK_INLINE {
            const u32x4 m = __builtin_amdgcn_raw_buffer_load_b128(buf, (int)(at + (unsigned)lane * 16u + k.value * (WAVE * 16u)), 0, AUX_AGENT | AUX_VOLATILE);
            lo[2 * k.value] = m[0];
            hi[2 * k.value] = m[1];
            lo[2 * k.value + 1] = m[2];
            hi[2 * k.value + 1] = m[3];
        });
        if constexpr (WORDS % 2 == 1) {
            const u32x2 m = __builtin_amdgcn_raw_buffer_load_b64(buf, (int)(at + (unsigned)lane * 8u + PAIRS * (WAVE * 16u)), 0, AUX_AGENT | AUX_VOLATILE);
            lo[WORDS - 1] = m[0];
            hi[WORDS - 1] = m[1];
        }
    }
    __device__ __forceinline__ bool wrong(unsigned tag) const          // false: all of it is there
    {
        unsigned w = 0;
        static_for<WORDS>([&](auto i) JK_INLINE { w |= hi[i.value] ^ tag; });
        return w > 0xffffffu;
    }
    template <typename F> __device__ __forceinline__ void take(F &&put) const
    {
        static_for<M>([&](auto i_) JK_INLINE {
            constexpr int i = decltype(i_)::value, e = M + i / 7, k = i % 7;
            const unsigned top = (k < 4 ? lo[e] >> (8 * (k % 4)) : hi[e] >> (8 * (k % 4))) & 0xffu;
            const int l = (int)lo[i], h = (int)((hi[i] & 0xffffffu) | top << 24);
            if constexpr (PER == 1) put(i_, __builtin_bit_cast(T, Int2{l, h}));
            else {
                put(std::integral_constant<int, 2 * i>{}, __builtin_bit_cast(T, l));
                if constexpr (2 * i + 1 < N) put(std::integral_constant<int, 2 * i + 1>{}, __builtin_bit_cast(T, h));
            }
        });
    }
};

// A lane at the open end of a DPP wave shift receives zero; with these it receives `end`, which has to be zero in all
// other lanes (the OR and the shift are one instruction).
__device__ __forceinline__ float from_prev_lane_or(float v, float end)
{
    return __builtin_bit_cast(float, dpp_from_prev_z(__builtin_bit_cast(int, v)) | __builtin_bit_cast(int, end));
}
__device__ __forceinline__ float from_next_lane_or(float v, float end)
{
    return __builtin_bit_cast(float, dpp_from_next_z(__builtin_bit_cast(int, v)) | __builtin_bit_cast(int, end));
}
__device__ __forceinline__ double from_prev_lane_or(double v, double end)
{
    const Int2 a = __builtin_bit_cast(Int2, v), f = __builtin_bit_cast(Int2, end);
    return __builtin_bit_cast(double, Int2{dpp_from_prev_z(a.lo) | f.lo, dpp_from_prev_z(a.hi) | f.hi});
}
__device__ __forceinline__ double from_next_lane_or(double v, double end)
{
    const Int2 a = __builtin_bit_cast(Int2, v), f = __builtin_bit_cast(Int2, end);
    return __builtin_bit_cast(double, Int2{dpp_from_next_z(a.lo) | f.lo, dpp_from_next_z(a.hi) | f.hi});
}

// ---- cells of a grid by their place in the domain (-1 and N are the Dirichlet ring) ---------------------------
__device__ __forceinline__ long long domain_cell_off(const Geo &g, int z, int y, int x)
{
    const int tz = g.ndim == 3 ? min(max(z, 0) / g.td, g.Tz - 1) : 0;
    const int ty = min(max(y, 0) / g.th, g.Ty - 1), tx = min(max(x, 0) / g.tw, g.Tx - 1);
    const int k = g.ndim == 3 ? z - tz * g.td + 1 : 0, i = y - ty * g.th + 1, c = x - tx * g.tw;
    const long long tile = (((long long)tz * g.Ty + ty) * g.Tx + tx) * g.tile_stride;
    return tile + (c < 0 ? xm_off(g, k, i) : c == g.tw ? xp_off(g, k, i) : main_off(g, k, i, c));
}

// Consecutive rows y, y + 1, ... of the domain: the element offset of the first tile of the row of tiles (plane 0) and the
// row inside it.
struct RowWalk {
    long long tile;
    int i;
    __device__ __forceinline__ RowWalk(const Geo &g, int y)
    {
        const int ty = y / g.th;
        tile = (long long)ty * g.Tx * g.tile_stride;
        i = y - ty * g.th + 1;
    }
    __device__ __forceinline__ void next(const Geo &g)
    {
        if (++i > g.th) { i = 1; tile += (long long)g.Tx * g.tile_stride; }
    }
};

// ---- the schedule of a launch -----------------------------------------------------------------------------
// Barrier of the plain path among `members` workgroups; every thread calls it.  Returns false if it was given up.
__device__ __forceinline__ bool plain_barrier(const BlockRun &br, unsigned members, unsigned round, int *lds_flag)
{
    stores_arrived();                             // thread 0 then writes the L2 back for all of them
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        agent_add(&br.sync->barrier, 1u);
        bool ok = false;
        for (unsigned n = 0; n <= br.spin_limit; ++n) {
            if (agent_load(&br.sync->barrier) >= members * round) { ok = true; break; }
            if (agent_load(&br.sync->failed) != 0u) break;
            __builtin_amdgcn_s_sleep(2);
        }
        if (!ok) agent_store(&br.sync->failed, 1u);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *lds_flag = ok ? 1 : 0;
    }
    __syncthreads();
    return *lds_flag != 0;
}

// All iterations through memory, one after the other, by the workgroups that were counted in; *lds_flag: this one's
// number among them.  A thread per cell and iteration, cells addressed one by one.  `in` is untouched so far.  Same expressions, same bits.
template <typename T, int NDIM>
__device__ __forceinline__ void plain_path(const Geo &g, const BlockRun &br, T *in, T *out, double *red, int *lds_flag)
{
    const unsigned me = (unsigned)*lds_flag, members = agent_load(&br.sync->participants);
    __syncthreads();
    const unsigned Nz = NDIM == 3 ? g.Tz * g.td : 1, Ny = g.Ty * g.th, Nx = g.Tx * g.tw;
    const unsigned cells = Nz * Ny * Nx, first = me * blockDim.x + threadIdx.x, step = members * blockDim.x;   // far below 2^31
    T *src = in, *dst = out;
    unsigned round = 0;
    bool healthy = true;
    int norm = 0;
    for (int it = 0;; ++it) {
        const bool norm_here = br.norms > 0 && it > 0 && it % br.every == 0 && norm < br.norms;
        const bool copy_here = it == br.iters && (src != in) != (br.final_is_out != 0);    // the result lies in the other grid
        const bool update_here = it < br.iters;
        double acc = 0.0;
        for (unsigned w = first; w < cells; w += step) {
            const int row = (int)(w / Nx), x = (int)(w - row * Nx), z = NDIM == 3 ? row / (int)Ny : 0, y = row - z * (int)Ny;
            auto at = [&](int dz, int dy, int dx) JK_INLINE -> T {
                const int zz = z + dz, yy = y + dy, xx = x + dx;
                const bool ring = (NDIM == 3 && (unsigned)zz >= Nz) || (unsigned)yy >= Ny || (unsigned)xx >= Nx;
                return (ring ? in : src)[domain_cell_off(g, zz, yy, xx)];
            };
            const T c = at(0, 0, 0);
            T val = c;
            if (update_here || norm_here) {
                T sum = (at(0, 0, -1) + at(0, 0, 1)) + (at(0, -1, 0) + at(0, 1, 0));
                if constexpr (NDIM == 3) sum = sum + (at(-1, 0, 0) + at(1, 0, 0));
                val = (NDIM == 3 ? Coef<T>::sixth : Coef<T>::quarter) * sum;
                const double r = (double)(sum - (NDIM == 3 ? Coef<T>::six : Coef<T>::four) * c);
                acc += r * r;
            }
            if (update_here) dst[domain_cell_off(g, z, y, x)] = val;
            else if (copy_here) dst[domain_cell_off(g, z, y, x)] = c;
        }
        if (norm_here) {
            __syncthreads();
            const double tot = wg_sum(acc, red);
            if (threadIdx.x == 0) __hip_atomic_store(&br.partial[(long long)norm * gridDim.x + me], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            ++norm;
        }
        if (!update_here) break;
        if (healthy) healthy = plain_barrier(br, members, ++round, lds_flag);
        if (!healthy) break;
        T *t = src; src = dst; dst = t;
    }
    if (!healthy)                                   // given up: no plausible values
        for (unsigned w = first; w < cells; w += step) {
            const int row = (int)(w / Nx), z = NDIM == 3 ? row / (int)Ny : 0;
            (br.final_is_out ? out : in)[domain_cell_off(g, z, row - z * (int)Ny, (int)(w - row * Nx))] = T(__builtin_nan(""));
        }
}

// The end of a workgroup: the last one adds up the norms - one sum per workgroup that did the work: all of them, or those that
// were counted in when the roll was closed - and leaves the words as the next launch has to find them.
// `exchanges`: how many tags the launch has used at most; `areas`: of messages.  Every thread calls it.
__device__ __forceinline__ void block_epilogue(const BlockRun &br, unsigned epoch, unsigned exchanges, double *red, int *lds_flag, unsigned areas = 2u)
{
    // This workgroup's sums and its failure flag - any wavefront may have raised it - went out past the caches: they only have
    // to have arrived.  (An agent-scope release here would have every workgroup write back its XCD's whole L2.)
    stores_arrived();
    __syncthreads();
    if (threadIdx.x == 0) *lds_flag = agent_add(&br.sync->done, 1u) == gridDim.x - 1 ? 1 : 0;
    __syncthreads();
    if (!*lds_flag) return;
    const bool failed = agent_load(&br.sync->failed) != 0u;
    const unsigned counted = agent_load(&br.sync->participants), nsums = counted ? counted : gridDim.x;
    for (int k = 0; k < br.norms; ++k) {
        double v = 0.0;
        for (unsigned i = threadIdx.x; i < nsums; i += blockDim.x)
            v += __hip_atomic_load(&br.partial[(long long)k * gridDim.x + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double sum = wg_sum(v, red);
        if (threadIdx.x == 0) br.result[k] = failed ? __builtin_nan("") : sqrt(sum);
        __syncthreads();
    }
    unsigned next = epoch + exchanges;
    if (next > br.epoch_limit) {                 // by default once in some 2^31 exchanges
        u32x4 *m = (u32x4 *)br.msg;
        for (unsigned i = threadIdx.x; i < areas * (br.msg_bytes / 16u); i += blockDim.x) m[i] = u32x4{0u, 0u, 0u, 0u};
        next = 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        agent_store(&br.sync->roll, 0u);
        agent_store(&br.sync->participants, 0u);
        agent_store(&br.sync->done, 0u);
        agent_store(&br.sync->barrier, 0u);
        agent_store(&br.sync->failed, 0u);
        agent_store(&br.sync->epoch, next);
    }
}

// Iterations until the next exchange when `left` of them lead to the next norm or the end: as few stretches as
// possible, equally long, of at most d; before a norm one ghost cell has to be left over.
__device__ __forceinline__ int next_stretch(int left, int d, bool norm_due)
{
    const int m = max(1, (left + (norm_due && d > 1 ? 1 : 0) + d - 1) / d);
    return (left + m - 1) / m;
}

}  // namespace jk
