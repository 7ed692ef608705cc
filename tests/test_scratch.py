"""Growth of optional scratch (csrc/scratch.h) under a fake allocator: what is kept where memory is short, and
that other errors are not taken for a lack of memory.  Compiled with the host compiler; no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <cassert>
#include <cstdlib>
#include "scratch.h"

struct Buf { void* p = nullptr; size_t bytes = 0; };
static size_t room;       // what the fake device has left
static size_t size_of[64];
static int live, error;   // allocations alive; an error that every allocation meets
static int alloc_(size_t n, void** p) {
  if (error) return error;
  if (n > room) return -4;
  room -= n;
  *p = &size_of[live];
  size_of[live++] = n;
  return 0;
}
static int release_(void* p) { room += *(size_t*)p; return 0; }
static int grow(Buf& b, size_t want, size_t least) { return lsms::grow_scratch(b, want, least, -4, alloc_, release_); }

int main() {
  Buf b;
  room = 100;
  assert(grow(b, 40, 10) == 0 && b.bytes == 40 && room == 60);   // grown
  assert(grow(b, 30, 10) == 0 && b.bytes == 40 && room == 60);   // large enough already
  void* const kept = b.p;
  assert(grow(b, 90, 20) == 0 && b.bytes == 40 && b.p == kept);  // no room: what is there holds the least
  assert(grow(b, 90, 50) == 0 && b.bytes == 50 && room == 50);   // it does not: the least instead
  assert(grow(b, 90, 70) == 0 && b.bytes == 50 && room == 50);   // no room for that either: unchanged
  error = -3;
  assert(grow(b, 60, 20) == -3 && b.bytes == 50);                // not a lack of memory: reported
  assert(grow(b, 50, 20) == 0);                                  // nothing to allocate
  error = 0;
  Buf c;
  room = 5;
  assert(grow(c, 40, 10) == 0 && c.p == nullptr && c.bytes == 0);
  room = 15;
  assert(grow(c, 40, 10) == 0 && c.bytes == 10 && room == 5);
  return 0;
}
"""


def test_growth_with_too_little_memory(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-UNDEBUG", "-I",
                    os.path.join(ROOT, "paper_2311_12134_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
