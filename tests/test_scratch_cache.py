"""The scratch cache of a context without an allocator callback when device
memory runs out (CPU: the library's own code, with the HIP memory calls
replaced by the test program's)."""

import os
import subprocess

import pytest

import paper_1512_00066_amd as srtc
from paper_1512_00066_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include "internal.hpp"

static std::set<void *> held;       // device memory of the stand-in
static int refuse = 0;              // hipMalloc calls to refuse
static hipError_t last = hipSuccess;  // as the runtime keeps it: until it is read

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
  if (refuse > 0) return refuse--, last = hipErrorOutOfMemory;
  *p = malloc(n);
  held.insert(*p);
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (!held.erase(p)) return last = hipErrorInvalidValue;
  free(p);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}

#define CHECK(x) if (!(x)) return printf("line %d: %s\n", __LINE__, #x), 1
using namespace srtc;

static int live_blocks_stay() {
  Ctx c;
  void *used = c.raw_alloc(1000, SCRATCH), *idle = c.raw_alloc(5000, SCRATCH);
  c.raw_free(idle, SCRATCH);
  for (int kind : {(int)SCRATCH, (int)OUTPUT}) {
    refuse = 1;  // the first attempt; the second finds room
    void *p = c.raw_alloc(100000, kind);
    CHECK(p && held.count(p));
    CHECK(held.count(used));
    c.raw_free(p, kind);
  }
  c.raw_free(used, SCRATCH);
  CHECK(c.raw_alloc(1000, SCRATCH) == used);  // still the cache's
  void *big = c.raw_alloc(5000, SCRATCH);
  refuse = 2;
  bool failed = false;
  try { c.raw_alloc(1 << 20, SCRATCH); } catch (const Error &e) { failed = e.st == SRTC_ERR_OOM; }
  CHECK(failed && held.count(used) && held.count(big));
  c.raw_free(big, SCRATCH);
  c.release_cache();
  CHECK(held.empty());
  return 0;
}

static int error_is_read() {
  Ctx c;
  for (int kind : {(int)SCRATCH, (int)OUTPUT}) {
    refuse = 1;
    void *p = c.raw_alloc(3000, kind);
    CHECK(p && hipGetLastError() == hipSuccess);
    refuse = 2;
    try { c.raw_alloc(1 << 20, kind); } catch (const Error &e) { CHECK(e.st == SRTC_ERR_OOM); p = nullptr; }
    CHECK(!p && hipGetLastError() == hipSuccess);
  }
  // a callback that asks the runtime itself and is refused
  c.alloc = [](void *, size_t n) -> void * {
    void *p = nullptr;
    return hipMalloc(&p, n) == hipSuccess ? p : nullptr;
  };
  refuse = 1;
  void *p = &c;
  try { p = c.raw_alloc(100, SCRATCH); } catch (const Error &e) { CHECK(e.st == SRTC_ERR_OOM); p = nullptr; }
  CHECK(!p && hipGetLastError() == hipSuccess);
  return 0;
}

int main(int argc, char **argv) {
  (void)argc;
  return atoi(argv[1]) == 0 ? live_blocks_stay() : error_is_read();
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    srtc.lib()
    d = tmp_path_factory.mktemp("cache")
    (d / "cache.hip").write_text(PROGRAM)
    here = os.path.dirname(srtc.LIB_PATH)
    r = subprocess.run([B.HIPCC, "-std=c++17", f"--offload-arch={B.ARCH}", "-x", "hip", "-I", B.CSRC, "-Wno-unused-result",
                        str(d / "cache.hip"), "-x", "none", srtc.LIB_PATH, "-rdynamic", f"-Wl,-rpath,{here}", "-o",
                        str(d / "cache")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return str(d / "cache")


def run(program, which):
    r = subprocess.run([program, str(which)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_blocks_in_use_outlive_a_failed_allocation(program):
    run(program, 0)


def test_a_refusal_is_not_left_for_the_next_launch_check(program):
    run(program, 1)
