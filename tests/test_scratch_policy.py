"""The optional scratch's rules (csrc/scratch.h) on a model of a device's memory,
compiled with g++: what is optional stays within the room it is given, and on a
full device costs no allocation, no free and no wait."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include "scratch.h"
struct Mem {
  size_t left;
  int allocs = 0, frees = 0;
  std::map<void *, size_t> held;
  bool alloc(void **p, size_t n) {
    ++allocs;
    if (n > left) return false;
    *p = std::malloc(1);
    held[*p] = n;
    left -= n;
    return true;
  }
  void free(void *p) {
    ++frees;
    left += held.at(p);
    held.erase(p);
    std::free(p);
  }
  size_t available() { return left; }
};
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  const size_t M = 1 << 20, ALL = ~size_t(0) / 2;
  {  // grows, serves smaller calls without touching the device, is given back
    Mem mem{100 * M};
    sap::OptionalScratch<Mem> s;
    CHECK(s.reserve(mem, 10 * M, ALL) && s.reserve(mem, 3 * M, ALL) && s.reserve(mem, 10 * M, ALL));
    CHECK(mem.allocs == 1 && mem.frees == 0 && s.size >= 10 * M);
    CHECK(s.reserve(mem, 20 * M, ALL) && mem.held.size() == 1 && mem.left == 80 * M);
    s.release(mem);
    CHECK(mem.left == 100 * M && s.base == nullptr && s.size == 0);
  }
  {  // the budget: refused before the device is asked, and the buffer that is there stays
    Mem mem{100 * M};
    sap::OptionalScratch<Mem> s;
    CHECK(s.reserve(mem, 4 * M, 8 * M) && !s.reserve(mem, 9 * M, 8 * M));
    CHECK(mem.allocs == 1 && mem.frees == 0 && s.reserve(mem, 4 * M, 8 * M));
  }
  {  // a full device: asked once, then only after it reports room
    Mem mem{5 * M};
    sap::OptionalScratch<Mem> s;
    CHECK(s.reserve(mem, 2 * M, ALL) && !s.reserve(mem, 6 * M, ALL));
    const int allocs = mem.allocs, frees = mem.frees;
    for (int k = 0; k < 10; ++k) CHECK(!s.reserve(mem, 6 * M, ALL) && !s.reserve(mem, 7 * M, ALL));
    CHECK(mem.allocs == allocs && mem.frees == frees);
    CHECK(s.reserve(mem, 2 * M, ALL) && mem.allocs == allocs + 1);  // smaller calls are still served
    for (int k = 0; k < 10; ++k) CHECK(!s.reserve(mem, 6 * M, ALL) && s.reserve(mem, 2 * M, ALL));
    CHECK(mem.allocs == allocs + 1 && mem.frees == frees);
    mem.left += 4 * M;  // someone else gave memory back
    CHECK(s.reserve(mem, 6 * M, ALL));
    s.release(mem);
    CHECK(mem.held.empty());
  }
  return 0;
}
"""


def test_optional_scratch(tmp_path):
    src = tmp_path / "t.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "t"
    inc = os.path.join(ROOT, "paper_2506_03070_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-I", inc, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
