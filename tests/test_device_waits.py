"""What one workgroup stores and another one reads: every wavefront's stores have to have arrived before the workgroup says
so.  __syncthreads() alone does not wait for them on this chip (wavefronts of a workgroup share their L1, so nothing
inside the workgroup needs it), and the wavefront that then does the signalling waits for its own stores only.  Such
a hole shows in results only by chance, so the generated code is looked at: one variant of each kernel, compiled here."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "blocks2d_kernel.h"
#include "blocks3d_kernel.h"
#include "resident_kernel.h"
template __global__ void jk::blocks2d_kernel<float, 1, 2>(jk::Geo, jk::Blocks2d, float *, float *);
template __global__ void jk::blocks3d_kernel<float, 2, 4, 2, true>(jk::Geo, jk::Blocks3d, float *, float *);
template __global__ void jk::resident2d_kernel<float, 1, 1>(jk::Geo, jk::ResidentParams, float *, float *);
"""
STORE = re.compile(r"(global|buffer|flat)_(store|atomic)")
EDGE = re.compile(r"label|s_c?branch")           # other ways lead here, or from here elsewhere
VMCNT0 = re.compile(r"s_waitcnt .*vmcnt\(0\)")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: its instructions, in the order of the text}"""
    from paper_2210_01238_amd import build
    d = tmp_path_factory.mktemp("asm")
    src, out = str(d / "one.hip"), str(d / "one.s")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "-I", build.CSRC, "-I", os.path.join(ROOT, "include"),
                    "--cuda-device-only", "-S", src, "-o", out], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.STDOUT)
    found, name = {}, None
    for line in open(out):
        m = re.match(r"_ZN2jk\d+(\w+?)I.*:", line)
        if m:
            name = m.group(1)
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line.startswith(".LBB"):
            found[name].append("label")
        elif name and line.startswith("\t") and not line.lstrip().startswith((";", ".")):
            found[name].append(line.split(";")[0].strip())
    assert set(found) == {"blocks2d_kernel", "blocks3d_kernel", "resident2d_kernel"}
    return found


def unwaited(code, sites):
    """Of the signals `sites` (indexes of instructions) those whose workgroup barrier some wavefront may pass with stores under way:
    no wait right in front of it, on every way to it.  A signal with a store of its own behind the barrier publishes that
    one, not what the others stored."""
    bad, looked_at = [], 0
    for i in sites:
        k = i - 1
        while k >= 0 and not code[k].startswith("s_barrier") and not STORE.match(code[k]):
            k -= 1
        if k < 0 or not code[k].startswith("s_barrier"):
            continue
        looked_at += 1
        k -= 1
        while k >= 0 and not VMCNT0.match(code[k]) and not STORE.match(code[k]) and not EDGE.match(code[k]):
            k -= 1
        if k < 0 or not VMCNT0.match(code[k]):
            bad.append(code[max(k, 0):i + 1])
    return bad, looked_at


@pytest.mark.parametrize("name", ["blocks2d_kernel", "blocks3d_kernel", "resident2d_kernel"])
def test_barrier_among_workgroups_waits_for_every_wavefront(kernels, name):
    """The write-back of the L2 comes after all stores of the workgroup."""
    code = kernels[name]
    bad, n = unwaited(code, [i for i, x in enumerate(code) if x.startswith("buffer_wbl2")])
    assert n >= 1 and not bad, bad


@pytest.mark.parametrize("name", ["blocks2d_kernel", "blocks3d_kernel"])
def test_end_of_a_workgroup_waits_for_every_wavefront(kernels, name):
    """Norms' sums and the failure flag come from any of them, and the workgroup that finishes last reads and clears them.  (The
    count of finished workgroups is the third word of the plan's.)"""
    code = kernels[name]
    bad, n = unwaited(code, [i for i, x in enumerate(code) if re.match(r"global_atomic_add v.* offset:8 sc0", x)])
    assert n >= 1 and not bad, bad


@pytest.mark.parametrize("name", ["blocks2d_kernel", "blocks3d_kernel"])
def test_number_of_participants_is_there_before_other_wavefronts_read_it(kernels, name):
    """The thread that closes the roll stores the number (the second word of the plan's), and the other wavefronts of its workgroup
    step through the cells by it: read as zero, their loop would not end."""
    code = kernels[name]
    reset = re.compile(r"global_store_dword v\d+, v\d+, s\[[\d:]+\] offset:8 sc1")       # the end of a launch clears word after word
    n = 0
    for i, x in enumerate(code):
        if not re.match(r"global_store_dword v\d+, v\d+, s\[[\d:]+\] offset:4 sc1", x) or reset.match(code[i + 1]):
            continue
        n += 1
        k = i + 1
        while not VMCNT0.match(code[k]) and not EDGE.match(code[k]) and not code[k].startswith("s_barrier"):
            k += 1
        assert VMCNT0.match(code[k]), code[i:k + 1]
    assert n >= 1
