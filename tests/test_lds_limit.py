"""A kernel's limit of dynamic LDS belongs to a device: it is raised once on each, and
again where it failed.  On the CPU, with the two HIP calls counted."""

import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2507_18969_amd import build as B

HIP = r"""
#pragma once
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorUnknown = 999 };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
inline int& device() { static int d = 0; return d; }
inline int& calls() { static int c = 0; return c; }
inline int& answer() { static int a = 0; return a; }
inline hipError_t hipGetDevice(int* d) { *d = device(); return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { ++calls(); return answer(); }
"""

MAIN = r"""
#include <cstdio>
#include "lds_limit.h"
using namespace edpc;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s (%d calls)\n", __LINE__, #x, calls()); return 1; } } while (0)
int main() {
  LdsLimit a, b;
  for (int k = 0; k < 3; ++k) CHECK(a.raise(nullptr, 70000) == hipSuccess);
  CHECK(calls() == 1);
  CHECK(b.raise(nullptr, 70000) == hipSuccess && calls() == 2);
  device() = 5;
  for (int k = 0; k < 3; ++k) CHECK(a.raise(nullptr, 70000) == hipSuccess);
  CHECK(calls() == 3);
  device() = 63;
  answer() = hipErrorUnknown;
  CHECK(a.raise(nullptr, 70000) == hipErrorUnknown);
  answer() = hipSuccess;
  CHECK(a.raise(nullptr, 70000) == hipSuccess && a.raise(nullptr, 70000) == hipSuccess && calls() == 5);
  device() = 0;
  CHECK(a.raise(nullptr, 70000) == hipSuccess && calls() == 5);
  device() = 64;  // not counted: asked for every time
  CHECK(a.raise(nullptr, 70000) == hipSuccess && a.raise(nullptr, 70000) == hipSuccess && calls() == 7);
  printf("ok\n");
  return 0;
}
"""


def test_once_a_device(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "limit")
    r = subprocess.run([cxx, "-std=c++17", "-Wall", "-I", str(tmp_path), "-I", B.CSRC,
                        str(tmp_path / "main.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr


def test_every_launcher_goes_through_it():
    for p in glob.glob(os.path.join(B.CSRC, "*.hip")):
        src = open(p).read()
        for m in re.finditer(r"hipFuncSetAttribute", src):
            # or asks at every launch, under no switch
            assert not re.search(r"static bool \w+ = false", src[max(0, m.start() - 300):m.start()]), p
