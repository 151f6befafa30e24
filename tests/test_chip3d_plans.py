"""Which 3-D grids run without ghost cells (chip3d_kernel), and as what: planned on the CPU, with a stand-in for the HIP runtime (hip_stub)
that counts launches; the one-byte tags' packing against plain bytes; and the waits in the generated code."""
import os
import re
import subprocess

import pytest

import test_device_waits as waits
from test_block_plans import text
from test_chip3d_gpu import EVERY, ITERS, PLAIN, VARIANTS
from test_host_calls import ROOT, run, stub  # noqa: F401  (stub: a fixture)

HEAD = """
from numpy import float64, float32
def plan(dims, tiles, dtype):
    return J.jacobi_create(dims, tiles, J.JACOBI_F64 if dtype is float64 else J.JACOBI_F32)
def figures(p, *names):
    return tuple(J.jacobi_get_option(p, "chip_" + n) for n in names)
def grids(p, iters, every):
    "workgroups of the launches of a call"
    J.jacobi_prepare(p)
    J.jacobi_sweep(p, *GRIDS(p), 50)                     # the first one also clears the plan's words
    log()
    J.jacobi_run(p, *GRIDS(p), iters, every, 1 << 16) if every else J.jacobi_sweep(p, *GRIDS(p), iters)
    return [int(c[1]) for c in log() if c[0] == "hipLaunchKernel"]
"""


def test_every_compiled_variant_is_reached(stub):  # noqa: F811
    run(stub, HEAD + f"""
for want, cases in {text(VARIANTS)}.items():
    for dims, tiles, dtype in cases:
        p = plan(dims, tiles, dtype)
        assert figures(p, "cells_per_lane", "planes_per_wave", "rows_per_wave", "waves_per_row") == want, (dims, dtype, want)
        assert grids(p, {ITERS}, {EVERY}) == list(figures(p, "workgroups")), (dims, dtype, want, J.jacobi_get_option(p, "block_workgroups"))
        J.jacobi_destroy(p)
for dims, tiles, dtype in {text(PLAIN)}:
    p = plan(dims, tiles, dtype)
    assert grids(p, 30, 3) == grids(p, 23, 0) == list(figures(p, "workgroups")), (dims, dtype)
    J.jacobi_set_option(p, "chip", 0)
    assert J.jacobi_get_option(p, "block_workgroups") in (0, *grids(p, 23, 0))
    J.jacobi_destroy(p)
""")
    with open(os.path.join(ROOT, "paper_2210_01238_amd", "csrc", "launchers.h")) as f:
        src = f.read()
    tables = {k: {tuple(int(n) for n in v.split(",")) for v in re.findall(r"X\((\d[\d, ]*)\)", re.search(r"#define %s\(X\)((?:.*\\\n)*.*)" % k, src).group(1))}
              for k in ("JK_CHIP3D_VARIANTS", "JK_CHIP3D_VARIANTS_F32")}
    compiled = {(v, t) for v in tables["JK_CHIP3D_VARIANTS"] for t in ("float64", "float32")} | {(v, "float32") for v in tables["JK_CHIP3D_VARIANTS_F32"]}
    assert compiled == {(v, c[2].__name__) for v, cases in VARIANTS.items() for c in cases}


def test_cuts_cover_the_grid(stub):  # noqa: F811
    """Blocks of 2 * planes x 2 * rows or one fewer, two of one wavefront per row to a workgroup, at most as many workgroups as CUs."""
    run(stub, HEAD + """
import random
rng = random.Random(7)
seen = 0
for _ in range(3000):
    dtype = rng.choice((float64, float32))
    dims = tuple(int(2 ** rng.uniform(3, 8.3)) for _ in range(3))
    p = plan(dims, (1, 1, 1), dtype)
    wg, c, rz, ry, nxw = figures(p, "workgroups", "cells_per_lane", "planes_per_wave", "rows_per_wave", "waves_per_row")
    if wg:
        seen += 1
        nz, ny, nx = dims
        bz, by = -(-nz // (2 * rz)), -(-ny // (2 * ry))
        assert nz // bz >= 2 * rz - 1 and ny // by >= 2 * ry - 1
        assert wg == (bz * by if nxw == 2 else -(-bz * by // 2)) <= 256
        assert 64 * c < nx <= 128 * c if nxw == 2 else 8 <= nx <= 64 * c
        assert ny * nz >= (1000 if nxw == 2 else 256)
    J.jacobi_destroy(p)
assert seen > 500, seen
for dims in ((256, 256, 256), (7, 7, 64), (27, 29, 119), (512, 512, 512), (300, 300, 64)):
    p = plan(dims, (1, 1, 1), float64)
    assert figures(p, "workgroups") == (0,), dims
    J.jacobi_destroy(p)
""")


# Calls timed both ways (us, MI355X), chip = 0 (which run by launches: these grids have no cut with ghost cells) and chip = 1 forced
TIMED = [
    # dims, type, tblock, iterations, norm every, by launches, on the chip
    ((158, 82, 136), "float32", 4, 4, 0, 28.3, 39.2), ((124, 138, 152), "float32", 8, 4, 0, 34.4, 42.4),
    ((75, 156, 168), "float32", 8, 4, 4, 37.8, 43.0), ((145, 121, 176), "float32", 12, 5, 2, 49.4, 55.0), ((92, 164, 134), "float32", 4, 8, 0, 66.6, 55.6),
    ((120, 112, 184), "float64", 12, 10, 2, 111.3, 101.9), ((181, 196, 142), "float32", 1, 7, 2, 106.3, 91.2), ((181, 219, 172), "float32", 1, 7, 2, 114.7, 95.0),
]


def test_calls_take_the_faster_path(stub):  # noqa: F811
    """(A call on the chip is one launch.)"""
    run(stub, HEAD + f"""
wrong = []
for dims, dtype, tblock, iters, every, other, chip in {TIMED!r}:
    p = plan(dims, (1, 1, 1), float64 if dtype == "float64" else float32)
    J.jacobi_set_option(p, "tblock", tblock)
    if (len(grids(p, iters, every)) == 1) != (chip < other) or J.jacobi_get_option(p, "block_workgroups"):
        wrong.append((dims, dtype, tblock, iters, every, other, chip, J.jacobi_get_option(p, "block_workgroups")))
    J.jacobi_destroy(p)
assert not wrong, wrong
""")


PACKING = r"""
#include <cstdio>
#include <cstring>
#include <cstdlib>
// the message type of one lane, its buffer accesses replaced by an array of bytes
#define __device__
#define __forceinline__ inline
#define JK_INLINE
#include <type_traits>
#include <utility>
struct Int2 { int lo, hi; };
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
constexpr int WAVE = 64, AUX_AGENT = 0, AUX_VOLATILE = 0;
typedef unsigned char *__amdgpu_buffer_rsrc_t;
static void __builtin_amdgcn_raw_buffer_store_b128(u32x4 v, unsigned char *b, int at, int, int) { memcpy(b + at, &v, 16); }
static void __builtin_amdgcn_raw_buffer_store_b64(u32x2 v, unsigned char *b, int at, int, int) { memcpy(b + at, &v, 8); }
static u32x4 __builtin_amdgcn_raw_buffer_load_b128(unsigned char *b, int at, int, int) { u32x4 v; memcpy(&v, b + at, 16); return v; }
static u32x2 __builtin_amdgcn_raw_buffer_load_b64(unsigned char *b, int at, int, int) { u32x2 v; memcpy(&v, b + at, 8); return v; }
static void __builtin_amdgcn_sched_barrier(int) {}
template <typename F, int... I> inline void static_for_impl(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F> inline void static_for(F &&f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }
@BYTES@
@TYPE@
template <typename T, int N> int one()
{
    using M = ByteTagged<T, N>;
    static unsigned char area[M::BYTES + 64];
    memset(area, 0, sizeof area);
    memset(area + M::BYTES, 0xa5, 64);
    int bad = 0;
    for (int exchange = 1; exchange <= 600; ++exchange) {
        const unsigned tag = byte_tag(exchange), other = byte_tag(exchange - 2 < 0 ? 0 : exchange - 2);
        T v[WAVE][N];
        for (auto &row : v)
            for (T &x : row) {
                unsigned char b[sizeof(T)];
                for (auto &y : b) y = (unsigned char)(rand() >> 7);
                memcpy(&x, b, sizeof(T));
            }
        for (int lane = 0; lane < WAVE; ++lane) {
            M m;
            m.read(area, 0, lane);
            bad += !m.wrong(tag);                                  // nobody has sent yet
            M::send(tag, area, 0, lane, [&](auto k) -> T { return v[lane][k.value]; });
        }
        for (int lane = 0; lane < WAVE; ++lane) {
            M m;
            m.read(area, 0, lane);
            bad += m.wrong(tag) || !m.wrong(other);
            T got[N];
            m.take([&](auto k, T x) { memcpy(&got[k.value], &x, sizeof(T)); });
            bad += memcmp(got, v[lane], sizeof got) != 0;
            // any word that is late shows
            for (unsigned w = 0; w < M::WORDS; ++w) {
                M late = m;
                late.hi[w] = (late.hi[w] & 0xffffffu) | other;
                bad += !late.wrong(tag);
            }
        }
        for (int i = 0; i < 64; ++i) bad += area[M::BYTES + i] != 0xa5;
    }
    if (bad) printf("%d bytes, %d cells: %d\n", (int)sizeof(T), N, bad);
    return bad;
}
int main()
{
    return one<double, 2>() + one<double, 3>() + one<double, 4>() + one<double, 5>() + one<double, 6>() + one<double, 8>() + one<double, 10>() +
           one<float, 2>() + one<float, 3>() + one<float, 5>() + one<float, 6>() + one<float, 12>() + one<float, 14>() + one<float, 16>() + one<float, 20>() != 0;
}
"""


def test_one_byte_tags_carry_every_bit_and_show_every_late_word(tmp_path):
    """The packing, as it stands in the source, run on the CPU: every bit of any value arrives, and a message is complete only when
    each of its words is of this exchange."""
    src = {n: open(os.path.join(ROOT, "paper_2210_01238_amd", "csrc", n)).read() for n in ("blocks_common.h", "launchers.h")}
    size = re.search(r"constexpr unsigned byte_tagged_bytes\(.*?\n}\n", src["launchers.h"], re.S).group(0)
    kind = re.search(r"__device__ __forceinline__ unsigned byte_tag\(.*?\n};\n", src["blocks_common.h"], re.S).group(0)
    kind = kind.replace("byte_tagged_bytes", "byte_tagged_bytes").replace("static __device__ __forceinline__", "static inline")
    f = tmp_path / "pack.cpp"
    f.write_text(PACKING.replace("@BYTES@", size).replace("@TYPE@", kind))
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++20", "-O1", "-w", str(f), "-o", str(tmp_path / "pack")], check=True)
    r = subprocess.run([str(tmp_path / "pack")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """The instructions of one variant, in the order of the text."""
    from paper_2210_01238_amd import build
    d = tmp_path_factory.mktemp("asm")
    src, out = str(d / "one.hip"), str(d / "one.s")
    with open(src, "w") as f:
        f.write('#include "chip3d_kernel.h"\n'
                "template __global__ void jk::chip3d_kernel<float, 1, 2, 2, 1>(jk::Geo, jk::Chip3d, float *, float *);\n")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "-I", build.CSRC, "-I", os.path.join(ROOT, "include"),
                    "--cuda-device-only", "-S", src, "-o", out], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.STDOUT)
    found, inside = [], False
    for line in open(out):
        if re.match(r"_ZN2jk\d+chip3d_kernelI.*:", line):
            inside = True
        elif line.startswith(".Lfunc_end"):
            inside = False
        elif inside and line.startswith(".LBB"):
            found.append("label")
        elif inside and line.startswith("\t") and not line.lstrip().startswith((";", ".")):
            found.append(line.split(";")[0].strip())
    assert found
    return found


def test_end_of_a_workgroup_and_its_barriers_wait_for_every_wavefront(code):
    for pattern in (r"buffer_wbl2", r"global_atomic_add v.* offset:8 sc0"):
        bad, n = waits.unwaited(code, [i for i, x in enumerate(code) if re.match(pattern, x)])
        assert n >= 1 and not bad, (pattern, bad)


def test_messages_are_cleared_before_a_workgroup_is_counted_in(code):
    """Tags come round, so nobody may look at a message before its sender has cleared it: the count (the plan's first word, an atomic whose
    result is used) comes behind a barrier in front of which every wavefront has waited for its stores."""
    sites = [i for i, x in enumerate(code) if re.match(r"global_atomic_add v\d+, v\d+, v\d+, s\[[\d:]+\] sc0", x)]
    bad, n = waits.unwaited(code, sites)
    assert n >= 1 and not bad, bad
