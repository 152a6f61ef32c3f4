"""The library's memory that a call can do without (csrc/spare.cpp), compiled for the host
against a device of a given size made of malloc."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_02754_amd", "csrc")

DEVICE = r"""
#include <cassert>
#include <cstdio>
#include <cstdlib>
#include <map>
#include "spare.h"
static size_t g_total = 0, g_used = 0;
static int g_mallocs = 0, g_frees = 0, g_dev = 0;
static std::map<void*, size_t> g_live;
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  ++g_mallocs;
  if (g_used + n > g_total) return hipErrorOutOfMemory;
  *p = malloc(1);
  g_live[*p] = n;
  g_used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  assert(g_live.count(p));
  ++g_frees;
  g_used -= g_live[p];
  g_live.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = g_total - g_used; *t = g_total; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = g_dev; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
}
using namespace chfsi;
constexpr size_t MB = (size_t)1 << 20, GB = (size_t)1 << 30;
"""

GROWTH = r"""
int main() {
  g_total = 1000 * MB;
  {
    SpareBuf a;
    void* p = a.get(100 * MB);
    assert(p && a.get(50 * MB) == p && g_mallocs == 1);
    void* q = a.get(300 * MB);                       // grows: the old goes
    assert(q && a.bytes() == 300 * MB && g_used == 300 * MB && g_frees == 1);
    assert(!a.get(800 * MB));                        // not beside the old: the old stays
    assert(a.get(300 * MB) == q && g_used == 300 * MB && g_frees == 1);
    const int tries = g_mallocs;
    assert(!a.get(800 * MB) && !a.get(900 * MB) && g_mallocs == tries);   // remembered
    assert(a.get(200 * MB) == q);
    void* hog;
    assert(hipMalloc(&hog, 500 * MB) == hipSuccess && !a.get(400 * MB));
    hipFree(hog);
    assert(!a.get(400 * MB));
    a.retry();
    assert(a.get(400 * MB) && a.bytes() == 400 * MB);
  }
  assert(g_used == 0);
  puts("ok");
}
"""


def _run(tmp_path, body):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(DEVICE + body)
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src),
                    os.path.join(CSRC, "spare.cpp"), "-o", str(exe), "-lpthread"], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout == "ok\n"


def test_growth_and_failure(tmp_path):
    _run(tmp_path, GROWTH)
