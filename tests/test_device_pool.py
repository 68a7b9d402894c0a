"""CPU: the pool that keeps device memory between block handles (csrc/device_pool.h), compiled with g++ against a runtime of
counters in place of HIP."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RUNTIME = r"""
#include "device_pool.h"
#include <cstdio>
#include <cstdlib>
static size_t g_limit, g_used;                 // bytes the "device" has, and how many are out
static hipError_t g_last = hipSuccess;         // as the runtime keeps it: set by a failure, read and cleared by hipGetLastError
struct Head { size_t n; };
extern "C" hipError_t hipMalloc(void **p, size_t n) {
  if (g_used + n > g_limit) return g_last = hipErrorOutOfMemory;
  Head *h = (Head *)malloc(sizeof(Head));      // (only the size is needed: the memory is never touched)
  h->n = n; g_used += n; *p = h;
  return hipSuccess;
}
extern "C" hipError_t hipFree(void *p) { g_used -= ((Head *)p)->n; free(p); return hipSuccess; }
extern "C" hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
"""
CASES = {
    # a build whose memory only exists once the pool has given its own back succeeds, and leaves no error behind
    "memory_held_by_the_pool": """
        g_limit = 48 << 20;
        size_t a, b, c;
        void *p = pool.take(0, 20 << 20, &a), *q = pool.take(0, 20 << 20, &b);
        CHECK(p && q);
        pool.give(0, p, a); pool.give(0, q, b);
        CHECK(g_used == (40u << 20));
        void *r = pool.take(0, 46 << 20, &c);
        CHECK(r && g_used == c);
        CHECK(hipGetLastError() == hipSuccess);""",
    # memory that does not exist is refused by the returned pointer alone: the next build reads no error of this one
    "no_memory_at_all": """
        g_limit = 1 << 20;
        size_t a;
        CHECK(!pool.take(0, 8 << 20, &a));
        CHECK(hipGetLastError() == hipSuccess && g_used == 0);
        CHECK(pool.take(0, 1 << 19, &a));
        CHECK(hipGetLastError() == hipSuccess);""",
    # bounded, per device, and a block comes back only for a request of a quarter of its size or more
    "bounds": """
        g_limit = (size_t)1 << 40;
        size_t got[20], n;
        void *p[20];
        for (int i = 0; i < 20; ++i) p[i] = pool.take(0, 4 << 20, &got[i]);
        for (int i = 0; i < 20; ++i) pool.give(0, p[i], got[i]);
        CHECK(g_used == (64u << 20));
        CHECK(pool.take(1, 4 << 20, &n) && g_used == (68u << 20));
        CHECK(pool.take(0, 1000, &n) && n == (1u << 16));
        CHECK(pool.take(0, 1 << 20, &n) && n == (4u << 20));""",
}


@pytest.mark.parametrize("name", CASES)
def test_device_pool(name, tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(RUNTIME + "int main() { DevicePool &pool = DevicePool::get(); " + CASES[name] + " return 0; }\n")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "paper_2505_17412_amd", "csrc"), "-o", str(exe), str(src), "-pthread"])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
