"""The compiled gfx950 kernels keep every barrier loop uniform (CPU only: hipcc emits
the device assembly, nothing runs).

A workgroup barrier (s_barrier) inside a loop must be reached by every lane of every
wave on every trip. If a loop that holds a barrier leaves or repeats per lane (its
back edge lowered as an exec-mask update, `s_andn2_b64 exec, exec, ...`, rather than
a scalar branch), the lanes that leave early stop arriving at the barrier while the
others wait there: a hang. A copy loop written with thread-0 steps around its barrier
was compiled that way once. This test parses the loop nesting that LLVM writes into
the assembly comments and checks, for every kernel of the library, that no loop holding
a barrier has a per-lane back edge of its own (loops nested inside it, such as the
thread-0 polling of a ready flag, may be per lane as long as they hold no barrier).
"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2601_20595_amd import build as libbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNEL_SOURCES = ["chunk_gemm.hip", "chunk_attn.hip"]

_LABEL = re.compile(r"^(?:\.L(BB\d+_\d+)|; (%bb\.\d+)):")
_FUNC = re.compile(r"^(_Z\S+):")


def device_asm(src_path: str) -> str:
    """gfx950 assembly of one HIP source, with the library's own flags."""
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "k.s")
        cmd = [libbuild.hipcc()] + libbuild.compile_flags() + ["--cuda-device-only", "-S", "-x", "hip", src_path,
                                                               "-o", out]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        assert r.returncode == 0, r.stdout.decode(errors="replace")
        return open(out).read()


def divergent_barrier_loops(asm: str):
    """[(function, loop header)] of loops that hold an s_barrier (in their own blocks or
    nested loops) and whose own blocks take a per-lane back edge (s_andn2_b64 exec, exec)."""
    flagged = []
    funcs = []
    for line in asm.split("\n"):
        m = _FUNC.match(line)
        if m:
            funcs.append((m.group(1), []))
        elif funcs:
            funcs[-1][1].append(line)
    for fname, lines in funcs:
        blocks = []                  # [name, innermost loop header or None, [instructions]]
        parent = {}                  # loop header -> enclosing loop header (None at depth 1)
        cur = None
        pending = None               # annotations of the block being opened
        for line in lines:
            m = _LABEL.match(line)
            if m:
                cur = [m.group(1) or m.group(2), None, []]
                blocks.append(cur)
                pending = [line]
                continue
            if cur is None:
                continue
            stripped = line.strip()
            if pending is not None and stripped.startswith(";"):
                pending.append(line)
                continue
            if pending is not None:
                text = "\n".join(pending)
                parents = [(int(d), h) for h, d in re.findall(r"Parent Loop (BB\d+_\d+) Depth=(\d+)", text)]
                if "Loop Header" in text and cur[0].startswith("BB"):
                    cur[1] = cur[0]
                    if parents:
                        parent[cur[0]] = max(parents)[1]   # the deepest enclosing loop
                    else:
                        parent[cur[0]] = None
                else:
                    m2 = re.search(r"in Loop: Header=(BB\d+_\d+) Depth=\d+", text)
                    cur[1] = m2.group(1) if m2 else None
                pending = None
            cur[2].append(stripped)

        def chain(h):
            while h is not None:
                yield h
                h = parent.get(h)

        has_barrier, own_lane_exit = set(), set()
        for name, loop, insts in blocks:
            if loop is None:
                continue
            if any(i.startswith("s_barrier") for i in insts):
                has_barrier.update(chain(loop))
            if any(re.match(r"s_andn2_b64 exec, exec,", i) for i in insts):
                own_lane_exit.add(loop)
        for h in sorted(has_barrier & own_lane_exit):
            flagged.append((fname, h))
    return flagged


_BAD = r"""
#include <hip/hip_runtime.h>
// per-lane loop exit around a barrier: lanes leave at different trips
__global__ void per_lane_exit(const int* p, int* out) {
  int i = 0;
  for (;; ++i) {
    __syncthreads();
    if (p[threadIdx.x] <= i) break;
  }
  out[threadIdx.x] = i;
}
// the same loop with a workgroup-uniform exit: fine
__global__ void uniform_exit(const int* p, int* out) {
  __shared__ int s;
  int i = 0;
  for (;; ++i) {
    __syncthreads();
    if (threadIdx.x == 0) s = p[0] <= i;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s)) break;
  }
  out[threadIdx.x] = i;
}
"""


def test_checker_flags_a_per_lane_barrier_loop_and_passes_a_uniform_one():
    with tempfile.TemporaryDirectory() as d:
        src = os.path.join(d, "probe.hip")
        with open(src, "w") as f:
            f.write(_BAD)
        flagged = divergent_barrier_loops(device_asm(src))
    names = {f for f, _ in flagged}
    assert any("per_lane_exit" in f for f in names), flagged
    assert not any("uniform_exit" in f for f in names), flagged


@pytest.mark.parametrize("source", KERNEL_SOURCES)
def test_library_kernels_have_no_per_lane_barrier_loop(source):
    asm = device_asm(os.path.join(ROOT, "paper_2601_20595_amd", "csrc", source))
    kernels = re.findall(r"^(_Z\S+):", asm, re.M)
    assert kernels, "no kernels found in %s" % source
    assert divergent_barrier_loops(asm) == []


def wide_stores_with_offset_register(asm: str):
    """Buffer stores of 12 or 16 bytes per lane whose scalar offset (the operand after the
    resource) is anything but a literal constant."""
    bad = []
    for m in re.finditer(r"^\s*buffer_store_(?:dwordx[34]|format_xyzw?)\s+([^;\n]*)", asm, re.M):
        operands = [x.strip() for x in m.group(1).split(",")]
        if len(operands) < 4 or not re.fullmatch(r"-?(?:0x[0-9a-f]+|\d+)", (operands[3].split() or [""])[0]):
            bad.append(m.group(0).strip())
    return bad


def test_checker_flags_every_offset_register_of_a_wide_store():
    bad = ["buffer_store_dwordx4 v[0:3], v4, s[8:11], s20 offen", "buffer_store_dwordx4 v[0:3], v4, s[8:11], s20",
           "buffer_store_dwordx3 v[0:2], v4, s[8:11], vcc_lo offen sc0 sc1", "buffer_store_dwordx4 v[0:3], off, s[8:11], m0",
           "buffer_store_dwordx4 v[0:3], v4, s[8:11], ttmp3 offen offset:16",
           "buffer_store_dwordx4 a[0:3], v4, s[8:11], exec_hi offen", "buffer_store_dwordx4 v[0:3], v4, s[8:11]"]
    good = ["buffer_store_dwordx4 v[0:3], v4, s[8:11], 0 offen", "buffer_store_dwordx4 v[0:3], v4, s[8:11], 0",
            "buffer_store_dwordx3 v[0:2], off, s[8:11], 0 offset:4080 sc0 sc1 ; note, s3",
            "buffer_store_dwordx2 v[0:1], v4, s[8:11], s20 offen", "buffer_load_dwordx4 v[0:3], v4, s[8:11], s20 offen"]
    assert wide_stores_with_offset_register("".join("\t%s\n" % x for x in bad + good)) == bad


@pytest.mark.parametrize("source", KERNEL_SOURCES)
def test_no_wide_store_with_a_scalar_offset_register(source):
    """A buffer store of 12 or 16 bytes per lane reads its data registers for a few cycles
    after it has issued. The compiler protects them from the next VALU write only when the
    store's scalar offset is no register; with one, results were replaced by the next
    address now and then. Every such store must therefore have none."""
    asm = device_asm(os.path.join(ROOT, "paper_2601_20595_amd", "csrc", source))
    assert re.search(r"^\s*buffer_store_dwordx4 ", asm, re.M)
    assert wide_stores_with_offset_register(asm) == []
