"""CPU check of the status-word pool (csrc/status_pool.h) against a stand-in
for the runtime whose clears, waits and device waits can be made to fail: a
slot whose clear failed is never handed out with the words it was left with."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_12805_amd", "csrc")

HIP = """
#pragma once
#include <cstddef>
#include <cstring>
typedef int hipError_t;
typedef void *hipStream_t;
constexpr hipError_t hipSuccess = 0;
extern int fail_memset, fail_sync, fail_device, calls;
inline hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) {
  calls++;
  if (fail_memset) return 1;
  memset(p, v, n);
  return 0;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { calls++; return fail_sync; }
inline hipError_t hipDeviceSynchronize() { calls++; return fail_device; }
"""

MAIN = r"""
#include "status_pool.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace pmklc;
int fail_memset, fail_sync, fail_device, calls;
static unsigned long long words[kStatusSlots * 4];
static StatusPool pool;
static hipError_t base(void **p) { *p = words; return hipSuccess; }
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)
static void zero(const StatusSlot &s) { for (int w = 0; w < 4; w++) CHECK(s.ptr[w] == 0); }
// a call that leaves its words dirty, its clear failing in the given way
static void failed_call(int memset_fails, int sync_fails) {
  StatusSlot s;
  CHECK(s.acquire(pool, nullptr, base) == hipSuccess);
  zero(s);
  for (int w = 0; w < 4; w++) s.ptr[w] = 7;
  fail_memset = memset_fails;
  fail_sync = sync_fails;
}
static void all_slots() {   // every slot at once, each with zero words
  std::vector<StatusSlot> all(kStatusSlots);
  for (auto &s : all) {
    CHECK(s.acquire(pool, nullptr, base) == hipSuccess);
    zero(s);
    s.clean = true;
  }
}
int main() {
  for (int how = 0; how < 3; how++) {
    failed_call(how != 1, how != 0);
    fail_memset = fail_sync = 0;
    { StatusSlot s; CHECK(s.acquire(pool, nullptr, base) == hipSuccess); zero(s); s.clean = true; }
    all_slots();
    all_slots();
  }
  // a clean call neither clears nor waits; another one clears its words
  calls = 0;
  { StatusSlot s; CHECK(s.acquire(pool, nullptr, base) == hipSuccess); s.clean = true; }
  CHECK(calls == 0);
  { StatusSlot s; CHECK(s.acquire(pool, nullptr, base) == hipSuccess); s.ptr[1] = 3; }
  CHECK(calls == 2);
  all_slots();
  CHECK(calls == 2);
  // a marked slot that cannot be cleared is refused, and is given back
  failed_call(1, 0);
  {
    std::vector<StatusSlot> others(kStatusSlots - 1);
    for (auto &s : others) { CHECK(s.acquire(pool, nullptr, base) == hipSuccess); zero(s); s.clean = true; }
    { StatusSlot s; CHECK(s.acquire(pool, nullptr, base) != hipSuccess); }
    fail_memset = 0;
    fail_device = 1;
    { StatusSlot s; CHECK(s.acquire(pool, nullptr, base) != hipSuccess); }
    fail_device = 0;
    { StatusSlot s; CHECK(s.acquire(pool, nullptr, base) == hipSuccess); zero(s); }
  }
  all_slots();
  CHECK(pool.busy == 0);
  printf("ok\n");
}
"""


def test_failed_clear_never_leaks(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "pool")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I", str(tmp_path), "-I", CSRC,
                           str(tmp_path / "main.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
