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
#include <mutex>
#include "spare.h"
static size_t g_total = 0, g_used = 0;
static int g_mallocs = 0, g_frees = 0, g_dev = 0;
static std::mutex g_lock;
static std::map<void*, size_t> g_live;
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> lk(g_lock);
  ++g_mallocs;
  if (g_used + n > g_total) return hipErrorOutOfMemory;
  *p = malloc(1);
  g_live[*p] = n;
  g_used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> lk(g_lock);
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

BOUNDS = r"""
#include <memory>
#include <thread>
#include <vector>
#include "internal.h"
int main() {
  g_total = 288 * GB;
  {
    std::vector<std::unique_ptr<SpareBuf>> v;         // many owners: bounded together
    int got = 0;
    for (int i = 0; i < 50; ++i) {
      v.emplace_back(new SpareBuf);
      got += v.back()->get(GB) != nullptr;
    }
    assert(got == 8 && g_used == kSpareMax);
    assert(v[0]->get(GB / 2) && !v[1]->get(GB + 1));
    g_dev = 1;                                        // another device has its own share
    SpareBuf o;
    assert(o.get(2 * GB));
    g_dev = 0;
    v.clear();
    assert(g_used == 2 * GB);
  }
  {
    SpareBuf a, b;                                    // a sixteenth of the device stays free
    void* hog;
    assert(hipMalloc(&hog, 269 * GB) == hipSuccess);
    assert(!a.get(2 * GB) && a.get(GB) && !b.get(GB));
    SpareBuf s;                                       // (small ones are not asked about)
    assert(s.get(32 * MB) && !s.get(33 * MB));
    s.release();
    // an allocation that fails takes its context's back
    DevBuf<double> d;
    bool threw = false;
    try {
      d.alloc(19 * GB / 8);
    } catch (const Error& e) {
      threw = e.code == CHFSI_ENOMEM;
    }
    assert(threw && d.ptr == nullptr && a.bytes() == GB);
    d.spare = &a;
    d.alloc(19 * GB / 8);
    assert(d.ptr && a.bytes() == 0 && g_used == 288 * GB);
    hipFree(hog);
  }
  assert(g_used == 0);
  {
    std::vector<std::thread> t;                       // several threads
    for (int i = 0; i < 8; ++i)
      t.emplace_back([]() {
        for (int r = 0; r < 200; ++r) {
          SpareBuf s;
          s.get(64 * MB);
          s.get(128 * MB);
        }
      });
    for (auto& x : t) x.join();
    SpareBuf s;
    assert(s.get(kSpareMax));                         // all given back
  }
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


def test_bounds_and_giving_back(tmp_path):
    _run(tmp_path, BOUNDS)
