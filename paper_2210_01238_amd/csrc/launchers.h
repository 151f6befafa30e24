// Internal interface between the host API (jacobi.hip) and the translation units that hold
// the compiled variants of the update kernels.  The variants are spread over several files
// only so that they compile in parallel; each launcher picks the instantiation for its
// arguments, launches it and returns hipGetLastError() (hipErrorInvalidValue if the requested
// variant is not compiled).
#pragma once
#include "jacobi_kernels.h"
#include <mutex>

namespace jk {

struct LaunchArgs {
    unsigned nwg;        // workgroups (grid size); block size is always WG
    hipStream_t st;
    Geo g;
    StripParams sp;
    const void *src;     // element type is given by the f64 flag of the call
    void *dst;
    double *partial;     // per-workgroup partial sums (residual modes), else unused
    int aux = 0;         // kernel-specific extra (3-D blocked pass: row groups per tile)
    // Workgroup limit: `lds` bytes of dynamic LDS that nobody touches are requested with the launch so that at
    // most `per_cu` workgroups share a CU (0: no limit).  The request only goes out if the occupancy query
    // confirms that it has this effect for the kernel at hand (lds_for_launch); if not, the launch runs
    // without a limit and *limit_failed is set.
    unsigned lds = 0;
    int per_cu = 0;
    int64_t *limit_failed = nullptr;
};

// Dynamic LDS to pass to the launch of KERNEL (a __global__ function; the template argument makes the cache
// below one per compiled variant): a.lds if the runtime confirms that a workgroup of `block_threads` threads
// asking for it leaves room for at most a.per_cu workgroups on a CU, else 0.  Requests above 64 KiB are
// allowed for the kernel first (once per kernel and device).  Checked once per kernel, device and size.
template <auto KERNEL>
inline hipError_t lds_for_launch(const LaunchArgs &a, int block_threads, unsigned *lds)
{
    struct Cache { unsigned allowed = 65536, checked = 0; bool ok = false; };
    constexpr int MAX_DEV = 64;
    static Cache cache[MAX_DEV];
    static std::mutex lock;
    *lds = 0;
    if (a.lds == 0 || a.per_cu <= 0) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    bool ok = false;
    if (dev >= 0 && dev < MAX_DEV) {
        std::lock_guard<std::mutex> hold(lock);
        Cache &c = cache[dev];
        if (c.checked != a.lds) {
            if (a.lds > c.allowed) {
                e = hipFuncSetAttribute((const void *)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds);
                if (e != hipSuccess) return e;
                c.allowed = a.lds;
            }
            int nb = 0;
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, KERNEL, block_threads, a.lds);
            if (e != hipSuccess) (void)hipGetLastError();
            c.ok = e == hipSuccess && nb >= 1 && nb <= a.per_cu;
            c.checked = a.lds;
        }
        ok = c.ok;
    }
    if (ok) *lds = a.lds;
    else if (a.limit_failed) *a.limit_failed = 1;
    return hipSuccess;
}

// single-step update / residual (mode: Mode; unroll 1,2,4,8,16; nt: 0 or 2)
hipError_t launch_sweep2d_f64(int mode, int unroll, int nt, const LaunchArgs &a);
hipError_t launch_sweep2d_f32(int mode, int unroll, int nt, const LaunchArgs &a);
// rows_per_wave 1,2,4; unroll 1,2,4
hipError_t launch_sweep3d_f64(int mode, int rows_per_wave, int unroll, int nt, const LaunchArgs &a);
hipError_t launch_sweep3d_f32(int mode, int rows_per_wave, int unroll, int nt, const LaunchArgs &a);
// 2-D residual pass with the wavefronts of a workgroup stacked (rows 8 per wavefront, waves 4 or 8 per
// workgroup); a.nwg = work units (tile x band x column segment), a.sp.nblk = bands per tile
hipError_t launch_stack_f64(int rows, int waves, const LaunchArgs &a);
hipError_t launch_stack_f32(int rows, int waves, const LaunchArgs &a);
// two iterations per pass (8-row strips); mode MODE_UPDATE or MODE_BOTH
constexpr int T2_ROWS = 8;
hipError_t launch_t2(bool f64, int mode, const LaunchArgs &a);
// TP_MIN..TP_MAX iterations per pass, pipelined down tall strips (overlapped wavefronts)
constexpr int TP_MIN = 3, TP_MAX = 12;
hipError_t launch_tp_f64(int depth, int mode, const LaunchArgs &a);
hipError_t launch_tp_f32(int depth, int mode, const LaunchArgs &a);
// levels - 1 iterations and the norm of their result (MODE_AFTER, MODE_BOTH_AFTER); levels in TP_MIN+1..TP_MAX
hipError_t launch_tp_after_f64(int levels, int mode, const LaunchArgs &a);
hipError_t launch_tp_after_f32(int levels, int mode, const LaunchArgs &a);

// 3-D: passes of depth 2 (2 or 4 rows per wavefront) or 3 (2 rows), pipelined along z
constexpr int TP3D_MIN = 2, TP3D_MAX = 3;
hipError_t launch_tp3d_f64(int depth, int rows_per_wave, int mode, const LaunchArgs &a);
hipError_t launch_tp3d_f32(int depth, int rows_per_wave, int mode, const LaunchArgs &a);

// 3-D, workgroup-cooperative blocked passes: rows one wavefront holds at each depth (a workgroup stores
// TC3D_WAVES * rows - 2 * depth rows per plane)
constexpr int TC3D_MIN = 2, TC3D_MAX = 4;
constexpr int TC3D_WAVES = 8;   // wavefronts per workgroup (one workgroup per CU at 2 wavefronts per SIMD)
constexpr int tc3d_rows_per_wave(int depth) { return depth == 2 ? 8 : depth == 3 ? 6 : 5; }
hipError_t launch_tc3d_f64(int depth, int mode, const LaunchArgs &a);
hipError_t launch_tc3d_f32(int depth, int mode, const LaunchArgs &a);
// TC3D_MAX - 1 iterations and the norm of their result
hipError_t launch_tc3d_after_f64(const LaunchArgs &a);

// All iterations of a call in one launch (small 2-D grids; resident_kernel.h).  nseg 1 or 2 column segments per
// wavefront, 1..4 rows per wavefront.  With more than one workgroup a one-wavefront kernel that zeroes the
// barrier words is launched first.
constexpr int RES_WAVES = 16;                // wavefronts per workgroup (1024 threads: one workgroup per CU)
constexpr int RES_MAX_SEG = 2;               // column segments a wavefront holds (rows of at most 2 KiB)
constexpr int RES_MAX_RW = 4;                // rows per wavefront
struct ResidentParams {
    int B;                 // rows a workgroup owns
    int d;                 // ghost rows per side
    int nphase;            // phases; the first n_deep of them run depth + 1 iterations, the others depth
    int depth, n_deep;
    unsigned spin_limit;   // polls a workgroup waits at a grid barrier before it gives up
    unsigned *sync;        // [0]: arrivals, [1]: failure flag, [2]: workgroups that have finished.  All zero between
                           // launches (the last workgroup to finish clears them); unused with one workgroup
    int copy_ring;         // also carry the Dirichlet ring from the source grid to the other one
    double *partial;       // per-workgroup sums of the residual terms (one per workgroup; unused if residual is null)
    double *residual;      // if not null: the residual norm of the final grid goes here (then d > deepest phase)
};
struct ResidentLaunch {
    unsigned nwg;
    hipStream_t st;
    Geo g;
    ResidentParams rp;
    void *in, *out;
};
hipError_t launch_resident(bool f64, int nseg, int rows_per_wave, const ResidentLaunch &a);

// ---- mid-sized grids: a whole run in one launch, the grid in the registers of the chip (blocks_common.h) ------------
// Plan-owned words; all zero between launches except the epoch.
struct BlockSync {
    unsigned roll;            // workgroups counted in, ROLL_CLOSED
    unsigned participants;    // workgroups counted when the roll was closed (0: not yet known)
    unsigned done;            // workgroups that have finished
    unsigned barrier;         // plain path: arrivals
    unsigned failed;          // somebody gave up waiting: results are NaN
    unsigned epoch;           // number of the last exchange of all launches so far
};

// What one launch does.
struct BlockRun {
    int iters;             // iterations of the launch
    int every;             // norms of the grids after iterations every, 2*every, ... (0: none)
    int norms;             // how many of them (iters / every, or 0)
    int final_is_out;      // the result goes to the grid the launch does not start from
    unsigned roll_limit, spin_limit;   // polls before the roll is closed / before a wait is given up
    unsigned admitted;     // workgroups that may be counted in (all of them, unless a test wants the plain path)
    unsigned epoch_limit;  // an epoch beyond it has the messages cleared and starts at 0 again
    BlockSync *sync;
    void *msg;             // the message areas
    unsigned msg_bytes;    // of one of them
    double *partial;       // one sum per norm and workgroup
    double *result;        // the norms
};

// Cut of one dimension into blocks: held ranges of `held` cells start at start(b), multiples of `unit` evenly spread over
// the n cells; a block owns what lies d behind the start of its range up to d behind the start of the next one.
struct BlockCut {
    int n, held, nb, d, unit, step, longer;        // steps between starts in units: the first `longer` ones step + 1
    __host__ __device__ int start(int b) const { return (b * step + (b < longer ? b : longer)) * unit; }
    __host__ __device__ int own_lo(int b) const { return b == 0 ? 0 : start(b) + d; }
    __host__ __device__ int own_hi(int b) const { return b == nb - 1 ? n : start(b + 1) + d; }
};

struct Blocks2d {
    BlockCut x, y;
    int strip;             // width of the strips that the blocks are dealt out to the XCDs by
    BlockRun run;
};

constexpr int BLK_WAVES = 8;
// cells of a block's message: the d first and last rows (full held width), the d first and last columns
__host__ __device__ inline unsigned blocks2d_frame(const BlockCut &x, const BlockCut &y) { return 2u * x.d * (x.held + y.held); }

// Compiled variants: cells per lane, rows per wavefront, and what an exchange takes longer in fp64 / fp32 because the
// registers do not hold everything (us; measured; the cells themselves stay in registers).
#define JK_BLOCKS2D_VARIANTS(X)                                                                                              \
    X(1, 2, 0, 0) X(1, 4, 0, 0) X(1, 6, 0, 0) X(1, 8, 0, 0) X(1, 12, 0, 0) X(1, 16, 0, 0) X(2, 6, 0, 0) X(2, 8, 0, 0)        \
    X(2, 10, 0, 0) X(2, 12, 1.4, 0) X(2, 16, 20, 0) X(4, 8, 16, 1) X(4, 10, 25, 2) X(4, 12, 30, 5)
#define JK_BLOCKS2D_VARIANTS_F32(X) X(1, 24, 0, 0) X(2, 24, 0, 10.6)
struct Blocks2dLaunch {
    hipStream_t st;
    Geo g;
    Blocks2d p;
    void *in, *out;
};
hipError_t launch_blocks2d_f64(int c, int rw, const Blocks2dLaunch &a);
hipError_t launch_blocks2d_f32(int c, int rw, const Blocks2dLaunch &a);

// 2-D grids that fill the chip (chip2d_kernel.h): cuts without ghost cells (d = 0)
struct Chip2d {
    BlockCut x, y;
    int strip;
    BlockRun run;
};
constexpr int CHIP2D_AREAS = 4;                // message areas that take turns
constexpr int CHIP2D_LANE_BYTES = 32;          // of a row in a lane: 4 fp64, 8 fp32 cells
// Compiled variants: rows per wavefront in registers, in LDS above those, in LDS below; each for cuts that are even - the blocks' widths
// whole lanes, their heights not overlapping - and for the others.  Even fp64 cuts of 8 rows: blocks2d_kernel takes those grids.
#define JK_CHIP2D_VARIANTS(X) X(8, 0, 0) X(12, 0, 0) X(16, 0, 0) X(20, 0, 0) X(24, 0, 0) X(23, 4, 5)
__host__ __device__ constexpr bool chip2d_compiled(int rows_in_registers, bool f64, bool ragged) { return rows_in_registers != 8 || !f64 || ragged; }
struct Chip2dLaunch {
    hipStream_t st;
    Geo g;
    Chip2d p;
    void *in, *out;
};
hipError_t launch_chip2d_even_f64(int rows_in_registers, const Chip2dLaunch &a);
hipError_t launch_chip2d_even_f32(int rows_in_registers, const Chip2dLaunch &a);
hipError_t launch_chip2d_ragged_f64(int rows_in_registers, const Chip2dLaunch &a);
hipError_t launch_chip2d_ragged_f32(int rows_in_registers, const Chip2dLaunch &a);

// 3-D: cuts of the padded rows (n = N + 2) in z and y
struct Blocks3d {
    BlockCut z, y;
    int nx;
    int frame_rows;        // rows of a block's message at most
    int strip;
    BlockRun run;
};
// Compiled variants: cells per lane, rows in z and y a wavefront keeps (larger patches do not fit the registers), and what
// they cost in fp64 / fp32 (us; measured, see plan_blocks3d): an iteration and an exchange where the rows fill the wavefront, the
// same where they are shorter, and a launch besides its iterations.
#define JK_BLOCKS3D_VARIANTS(X)                                                                                              \
    X(1, 4, 2, (2.02, 1.09, 2.19, 1.02, 11), (0.66, 1.64, 0.62, 1.77, 12))                                                   \
    X(1, 6, 3, (1.36, 4.55, 1.85, 3.70, 36), (1.29, 2.98, 1.46, 3.54, 30))                                                   \
    X(2, 4, 2, (2.40, 1.44, 2.55, 1.43, 13), (1.00, 1.66, 1.17, 1.62, 15))                                                   \
    X(2, 5, 2, (3.14, 1.86, 2.32, 3.40, 19), (1.10, 2.04, 1.56, 3.27, 20))
#define JK_BLOCKS3D_VARIANTS_F32(X)                                                                                          \
    X(2, 6, 3, (0, 0, 0, 0, 0), (1.71, 4.22, 2.29, 4.02, 36))                                                                \
    X(4, 4, 2, (0, 0, 0, 0, 0), (2.11, 1.64, 2.44, 3.14, 19))                                                                \
    X(4, 5, 2, (0, 0, 0, 0, 0), (2.18, 4.02, 2.96, 3.99, 26))
// 3-D grids that fill the chip without ghost cells (chip3d_kernel.h): n cells in nb parts, which differ by one cell at most
struct EvenCut {
    int n, nb;
    __host__ __device__ __forceinline__ int start(int b) const { return (int)((long long)b * n / nb); }
};
// bytes of a wavefront's message of n cells per lane (ByteTagged): 8-byte words, seven bytes of each payload
__host__ __device__ constexpr unsigned byte_tagged_bytes(int n, int esize)
{
    const int items = (n * esize + 7) / 8, words = items + (items + 6) / 7;
    return ((unsigned)words * WAVE * 8u + 255u) / 256u * 256u;
}
struct Chip3d {
    EvenCut z, y;
    int nx;
    int strip;
    BlockRun run;
};
// Compiled variants: cells per lane, planes and rows a wavefront keeps, wavefronts a row lies in.
#define JK_CHIP3D_VARIANTS(X)                                                                                                \
    X(1, 2, 2, 1) X(1, 3, 3, 1) X(1, 4, 4, 1) X(1, 6, 6, 1) X(1, 3, 3, 2) X(1, 4, 3, 2) X(1, 4, 4, 2) X(1, 5, 5, 2)          \
    X(1, 6, 6, 2) X(2, 4, 4, 2) X(2, 5, 4, 2) X(2, 5, 5, 2)
#define JK_CHIP3D_VARIANTS_F32(X) X(2, 6, 6, 2) X(2, 7, 6, 2) X(2, 8, 7, 2) X(4, 4, 4, 2) X(4, 5, 5, 2)
struct Chip3dLaunch {
    hipStream_t st;
    Geo g;
    Chip3d p;
    void *in, *out;
};
hipError_t launch_chip3d_c1_f64(int rz, int ry, int nxw, const Chip3dLaunch &a);
hipError_t launch_chip3d_c1_f32(int rz, int ry, int nxw, const Chip3dLaunch &a);
hipError_t launch_chip3d_c2_f64(int rz, int ry, int nxw, const Chip3dLaunch &a);
hipError_t launch_chip3d_c2_f32(int rz, int ry, int nxw, const Chip3dLaunch &a);
hipError_t launch_chip3d_c4_f32(int rz, int ry, int nxw, const Chip3dLaunch &a);

struct Blocks3dLaunch {
    hipStream_t st;
    Geo g;
    Blocks3d p;
    void *in, *out;
};
hipError_t launch_blocks3d_f64(int c, int rz, int ry, const Blocks3dLaunch &a);
hipError_t launch_blocks3d_f32(int c, int rz, int ry, const Blocks3dLaunch &a);

}  // namespace jk
