"""Barriers in the gfx950 code of kernels whose blocks decide by a value that
another block or wave changes meanwhile (CPU: hipcc cross-compiles).

A block may act on such a value only if all its waves take the same one, so a
barrier has to lie between the one read and every use.  These tests follow
every path through a kernel's assembly; small kernels without the barrier show
that the search finds the fault."""

import functools
import os
import re
import subprocess

import pytest

from paper_1512_00066_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")


def kernels(text):
    """{name: [instruction or label, ...]} of the functions in hipcc -S output."""
    out, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = out.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None:
            ins = line.split(";")[0].strip()
            if ins and (re.match(r"^\.LBB\w+:$", ins) or not ins.startswith(".")):
                cur.append(ins)
    return out


def reaches(code, starts, target, through):
    """Whether some path from an instruction in `starts` meets one that matches
    `target` before any that matches `through`."""
    label = {ins[:-1]: k for k, ins in enumerate(code) if ins.endswith(":")}
    todo, seen = list(starts), set()
    while todo:
        k = todo.pop()
        if k in seen or k >= len(code):
            continue
        seen.add(k)
        ins = code[k]
        if re.match(target, ins):
            return True
        if re.match(through, ins) or ins.startswith("s_endpgm"):
            continue
        m = re.match(r"^s_c?branch\w*\s+(\.LBB\w+)", ins)
        assert not ins.startswith(("s_setpc", "s_swappc", "s_call")), ins
        if m:
            todo.append(label[m.group(1)])
        if not ins.startswith("s_branch"):
            todo.append(k + 1)
    return False


@functools.lru_cache(None)
def library_asm(source, folder):
    return kernels(open(B.device_asm(source, os.path.join(folder, source + ".s"))).read())


@pytest.fixture(scope="session")
def folder(tmp_path_factory):
    return str(tmp_path_factory.mktemp("asm"))


def small_asm(text, folder, name):
    src = os.path.join(folder, name + ".hip")
    open(src, "w").write("#include <hip/hip_runtime.h>\n" + text)
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    r = subprocess.run([B.HIPCC, *flags, "-x", "hip", "--cuda-device-only", "-S", src, "-o", src + ".s"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return kernels(open(src + ".s").read())


def leaves_before_barrier(code):
    return reaches(code, [0], r"s_endpgm", r"s_barrier")


def test_search_sees_a_wave_that_leaves_early(folder):
    body = """
extern "C" __global__ void __launch_bounds__(256) _Zstop(const int *done, const float *in, float *out) {
  __shared__ float part[256];
  %s
  part[threadIdx.x] = in[threadIdx.x];
  __syncthreads();
  out[threadIdx.x] = part[threadIdx.x ^ 128];
}
"""
    for name, head, bad in (("alone", "if (*done) return;", True),
                            ("block", "__shared__ int d; if (threadIdx.x == 0) d = *done; __syncthreads(); if (d) return;",
                             False)):
        (code,) = small_asm(body % head, folder, name).values()
        assert leaves_before_barrier(code) == bad


def test_jacobi_blocks_decide_to_stop_as_one(folder):
    """Block 0 sets the flag that ends the iteration while other blocks of the
    launch start: no wave of a step may leave by what it read of it alone."""
    steps = {n: c for n, c in library_asm("transform.hip", folder).items()
             if "jacobi_step" in n or "jacobi_slices" in n}
    assert len(steps) >= 14  # two types: five row widths and two slice layouts each
    bad = [n for n, c in steps.items() if leaves_before_barrier(c)]
    assert not bad, bad


def adds_after_own_look(code):
    looks = [k for k, ins in enumerate(code) if ins.startswith("ds_read")]
    return reaches(code, [k + 1 for k in looks], r"ds_or", r"s_barrier")


def test_search_sees_an_unguarded_look(folder):
    body = """
extern "C" __global__ void __launch_bounds__(256) _Zlong(const unsigned *in, unsigned *out, int n) {
  __shared__ unsigned found;
  if (threadIdx.x == 0) found = in[0];
  __syncthreads();
  unsigned f = found;
  if (f != 7u) {
    %s
    for (int p = threadIdx.x; p < n && f != 7u; p += 256) {
      atomicOr(&found, in[p]);
      __syncthreads();
      f = found;
      __syncthreads();
    }
  }
  out[threadIdx.x] = f;
}
"""
    for name, guard, bad in (("unguarded", "", True), ("guarded", "__syncthreads();", False)):
        (code,) = small_asm(body % guard, folder, name).values()
        assert any(ins.startswith("ds_or") for ins in code)
        assert adds_after_own_look(code) == bad


def test_bfs_waves_agree_on_a_long_row(folder):
    """The waves of a block add what they find of a long row to one word, and
    leave the row when the word is complete: a wave's look at the word has to
    lie a barrier before any wave's next addition."""
    (code,) = [c for n, c in library_asm("spmm.hip", folder).items() if "bfs_step_kernel" in n]
    assert any(ins.startswith("ds_or") for ins in code)
    assert not adds_after_own_look(code)
