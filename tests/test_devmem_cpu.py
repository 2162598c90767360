"""CPU test of the device memory of a root pass (csrc/devmem.h, host code): the
header compiled against a counting stand-in for the device's allocator, over a
pass whose sub-networks want ever larger arrays, then smaller ones."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <map>
#include "devmem.h"

static std::map<void*, size_t> live;
static size_t held = 0, peak = 0, limit = ~(size_t)0;
static uintptr_t next_at = 1 << 20;  // (addresses only: nothing is written)
extern "C" hipError_t hipMalloc(void** p, size_t n) {
  if (held + n > limit) return hipErrorOutOfMemory;
  *p = reinterpret_cast<void*>(next_at);
  next_at += (n + 4095) & ~(size_t)4095;
  live[*p] = n;
  held += n;
  peak = peak > held ? peak : held;
  return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
  if (!live.count(p)) std::abort();
  held -= live[p];
  live.erase(p);
  return hipSuccess;
}
extern "C" hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" const char* hipGetErrorString(hipError_t) { return ""; }
int cvb::fail(int code, const char*, ...) { return code; }

using cvb::DevMem;
static const size_t kMB = 1 << 20;

// One pass: sub-network i wants small[i] arrays of 40 KB and the given large
// ones.  Returns the largest need of a sub-network; *rc the first failure.
static size_t pass(const std::vector<std::vector<size_t>>& large, int* rc) {
  DevMem mem, bm;
  size_t most = 0;
  *rc = 0;
  for (const auto& sizes : large) {
    DevMem a, b;
    a.take(mem);
    b.take(bm);
    b.keep = true;
    a.peer = &b;
    b.peer = &a;
    size_t need = 0;
    std::vector<std::pair<char*, size_t>> got;
    for (int t = 0; t < 30 && !*rc; ++t) {
      char* p;
      *rc = a.alloc(&p, 40000);
      got.push_back({p, 40000});
      need += 40960;
    }
    b.clear();
    for (size_t n : sizes) {
      char* p;
      if (!*rc) *rc = b.alloc(&p, n);
      got.push_back({p, n});
      need += n;
    }
    if (*rc) return most;
    for (auto& x : got)
      for (auto& y : got)
        if (&x != &y && x.first < y.first + y.second && y.first < x.first + x.second) std::abort();
    most = need > most ? need : most;
    mem.take(a);
    bm.take(b);
  }
  return most;
}

int main() {
  int rc;
  // growing by a fifth each time, so that no kept array serves the next one
  std::vector<std::vector<size_t>> grow, shrink;
  double n = 100.0 * kMB;
  for (int i = 0; i < 8; ++i, n *= 1.2) grow.push_back({(size_t)n, (size_t)n, (size_t)(n / 3)});
  shrink.assign(grow.rbegin(), grow.rend());
  for (auto* p : {&grow, &shrink}) {
    peak = held;
    const size_t most = pass(*p, &rc);
    std::printf("need %zu MB peak %zu MB\n", most / kMB, peak / kMB);
    if (rc || held) return 1;
    if (peak > most + 2 * DevMem::kKeep + 8 * kMB) return 2;
  }
  // a device that holds what the largest sub-network needs, and its rounding:
  // the pass fits, as it would without kept chunks
  std::vector<std::vector<size_t>> small = {{60 * kMB, 60 * kMB}, {72 * kMB, 72 * kMB}, {86 * kMB, 86 * kMB}};
  peak = held;
  const size_t most = pass(small, &rc);
  if (rc || held) return 3;
  limit = most + 8 * kMB;
  pass(small, &rc);
  if (rc || held) return 4;
  limit = most - 8 * kMB;
  pass(small, &rc);
  return rc == CV_ENOMEM && !held ? 0 : 5;
}
"""


@pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir("/opt/rocm/include/hip"), reason="no host toolchain")
def test_root_pass_memory_is_bounded(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    inc = os.path.join(ROOT, "paper_2103_06624_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", inc, str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, (r.returncode, r.stdout)
