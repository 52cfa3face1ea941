"""Scratch memory kept between synchronous calls: the bounds of what is kept and for
how long, on the CPU with a HIP runtime of a few lines that counts what it hands
out."""

import os
import shutil
import subprocess

import pytest

from paper_2507_18969_amd import build as B

HIP = r"""
#pragma once
#include <cstddef>
#include <cstdlib>
#include <map>
typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipMemcpyHostToDevice = 1 };
inline std::map<void*, size_t>& live() { static std::map<void*, size_t> m; return m; }
inline size_t& room() { static size_t r = (size_t)1 << 40; return r; }
inline size_t held() { size_t t = 0; for (auto& p : live()) t += p.second; return t; }
inline hipError_t hipMalloc(void** p, size_t b) {
  if (held() + b > room()) return hipErrorOutOfMemory;
  *p = malloc(1);
  live()[*p] = b;
  return hipSuccess;
}
inline hipError_t hipFree(void* p) { live().erase(p); free(p); return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipMemcpyAsync(void*, const void*, size_t, int, hipStream_t) { return hipSuccess; }
"""

MAIN = r"""
#include <cstdio>
#include <stdexcept>
#include "memory.h"
namespace edpc {
void hip_check(hipError_t e, const char* what) { if (e) throw std::runtime_error(what); }
}
using namespace edpc;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s (held %zu)\n", __LINE__, #x, held()); return 1; } } while (0)
int main() {
  const size_t M = (size_t)1 << 20;
  { Scratch a(32 * M, nullptr); }
  CHECK(held() == 32 * M);                               // kept
  { Scratch a(20 * M, nullptr); CHECK(held() == 32 * M); }  // taken again
  for (int i = 0; i < 70; ++i) Scratch a(24000, nullptr);
  CHECK(held() < M);                                     // small calls do not keep a large block alive
  { Scratch a(100, nullptr); CHECK(held() < M); }        // (they share small blocks)
  { Scratch a(40 * M, nullptr), b(30 * M, nullptr); }
  CHECK(held() <= 64 * M);                               // the bound on what is kept
  scratch_give_back();
  CHECK(held() == 0);
  { Scratch a(48 * M, nullptr); }
  room() = 60 * M;                                       // memory runs out: what is kept goes back
  {
    DeviceMemory m;
    CHECK(m.take<char>(40 * M) != nullptr);
    CHECK(held() == 40 * M);
  }
  CHECK(held() == 0);
  { Scratch a(48 * M, nullptr); }
  { Scratch a(50 * M, nullptr); CHECK(held() == 50 * M); }
  bool refused = false;
  try { device_malloc(61 * M); } catch (const std::runtime_error&) { refused = true; }
  CHECK(refused);
  printf("ok\n");
  return 0;
}
"""


def test_bounds(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "pool")
    src = os.path.join(B.CSRC, "memory.hip")
    r = subprocess.run([cxx, "-std=c++17", "-Wall", "-I", str(tmp_path), "-I", B.CSRC, "-x", "c++", src,
                        str(tmp_path / "main.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
