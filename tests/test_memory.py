"""The setup's device-memory bookkeeping (memory.h), compiled for the host against a stand-in for the
runtime's allocation calls: a card of a given capacity that records the error of a refused request
until it is asked for."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, ROOT)

STUB = r"""
#pragma once
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <map>
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum hipMemcpyKind { hipMemcpyDeviceToDevice = 3 };
typedef void* hipStream_t;
namespace card {
inline size_t capacity = ~size_t(0), used = 0, calls = 0;
inline hipError_t pending = hipSuccess;
inline std::map<void*, size_t>& arrays() { static std::map<void*, size_t> a; return a; }
}  // namespace card
// the addresses alone matter for large arrays: nothing above 4 KB is read or written
inline hipError_t hipMalloc(void** p, size_t bytes) {
  ++card::calls;
  if (bytes > card::capacity - card::used) return card::pending = hipErrorOutOfMemory;
  static char* next = reinterpret_cast<char*>(size_t(1) << 40);
  *p = next;
  next += (bytes + 4095) / 4096 * 4096;
  card::used += bytes;
  card::arrays()[*p] = bytes;
  return hipSuccess;
}
template <typename T>
hipError_t hipMalloc(T** p, size_t bytes) { return hipMalloc(reinterpret_cast<void**>(p), bytes); }
inline hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = card::arrays().find(p);
  if (it == card::arrays().end()) std::abort();  // not an array of the card: freed twice or inside a slab
  card::used -= it->second;
  card::arrays().erase(it);
  return hipSuccess;
}
inline hipError_t hipGetLastError() { const hipError_t e = card::pending; card::pending = hipSuccess; return e; }
inline hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
"""

PROLOGUE = r"""
#include <cstdio>
#include "memory.h"
using namespace amgp;
constexpr size_t MB = size_t(1) << 20;
#define CHECK(c) do { if (!(c)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c); return 1; } } while (0)
"""

CASES = {
    # 40 MB lie idle and 20 MB are free: the idle ones go back for an array that the handle keeps
    "kept_array_from_idle_memory": r"""
int main() {
  Arena arena;
  {
    MemoryScope scope(&arena);
    card::capacity = 60 * MB;
    char *a, *b;
    CHECK(temp_malloc(&a, 40 * MB) == hipSuccess);
    dev_free(a);
    CHECK(card::used == 40 * MB);
    CHECK(keep_malloc(&b, 50 * MB) == hipSuccess);
    CHECK(hipGetLastError() == hipSuccess);
    dev_free(b);  // stays the arena's
    char* c;
    CHECK(keep_malloc(&c, 20 * MB) != hipSuccess);
  }
  CHECK(card::used == 50 * MB);
  arena.release();
  CHECK(card::used == 0);
}
""",
    # a small kept array where its whole slab no longer fits
    "slab_no_larger_than_what_is_left": r"""
int main() {
  Arena arena;
  {
    MemoryScope scope(&arena);
    card::capacity = 101 * MB;
    char *a, *b;
    CHECK(keep_malloc(&a, 100 * MB) == hipSuccess);
    CHECK(keep_malloc(&b, MB / 2) == hipSuccess);
    CHECK(hipGetLastError() == hipSuccess);
    CHECK(b >= a + 100 * MB || b + MB / 2 <= a);
    char* c;
    CHECK(keep_malloc(&c, MB) != hipSuccess);
  }
  arena.release();
  CHECK(card::used == 0);
}
""",
    # an array that outlives the setup gives back a block that is much too large for it, which then
    # serves the next temporary array; one of about its size, and one of the arena's, stay where they are
    "outgrown_blocks": r"""
int main() {
  Arena arena;
  char *a, *b, *c, *d;
  {
    MemoryScope scope(&arena);
    CHECK(temp_malloc(&a, 10 * MB) == hipSuccess);
    dev_free(a);
    CHECK(temp_malloc(&b, 8 * MB + MB / 2) == hipSuccess && b == a);
    CHECK(settle(nullptr, &b, 8 * MB + MB / 2) == hipSuccess);
    CHECK(b != a && arena.owns(b));
    CHECK(temp_malloc(&c, 10 * MB) == hipSuccess && c == a);
    CHECK(settle(nullptr, &c, 10 * MB) == hipSuccess && c == a && !arena.owns(c));
    CHECK(settle(nullptr, &b, 8 * MB) == hipSuccess && arena.owns(b));
    // no room for the move: the array stays in its block
    CHECK(temp_malloc(&d, 20 * MB) == hipSuccess);
    dev_free(d);
    CHECK(temp_malloc(&a, 18 * MB) == hipSuccess && a == d);
    card::capacity = card::used;
    CHECK(settle(nullptr, &a, 18 * MB) == hipSuccess && a == d);
    CHECK(hipGetLastError() == hipSuccess);
  }
  CHECK(card::arrays().count(a) && card::arrays().count(c));
  {
    MemoryScope scope(&arena);
    dev_free(a);
    dev_free(b);
    dev_free(c);
    arena.release();
  }
  CHECK(card::used == 0);
}
""",
    # arrays taken after a mark are given back, the room behind it is used again
    "marks": r"""
int main() {
  Arena arena;
  char *a, *b, *c, *d;
  {
    MemoryScope scope(&arena);
    CHECK(keep_malloc(&a, MB) == hipSuccess);
    const size_t held = card::used;
    const std::vector<size_t> mark = arena.mark();
    CHECK(keep_malloc(&b, MB / 2) == hipSuccess && card::used == held);
    CHECK(keep_malloc(&c, 30 * MB) == hipSuccess && card::used == held + 30 * MB);
    arena.rewind(mark);
    CHECK(card::used == held && arena.owns(a) && !arena.owns(c));
    CHECK(keep_malloc(&d, MB / 2) == hipSuccess && d == b);
  }
  arena.release();
  CHECK(card::used == 0);
}
""",
    # temporaries: one of about the size is taken again, all are returned with the scope
    "temporaries": r"""
int main() {
  Arena arena;
  {
    MemoryScope scope(&arena);
    char *a, *b, *c;
    CHECK(temp_malloc(&a, 10 * MB) == hipSuccess);
    dev_free(a);
    CHECK(temp_malloc(&b, 9 * MB) == hipSuccess && b == a);
    CHECK(temp_malloc(&c, 9 * MB) == hipSuccess && c != a);
    dev_free(b);
    dev_free(c);
    CHECK(card::calls == 2);
  }
  CHECK(card::used == 0);
}
""",
}


@pytest.mark.parametrize("name", list(CASES))
def test_memory(name, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    os.makedirs(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    src, exe = tmp_path / f"{name}.cpp", tmp_path / name
    src.write_text(PROLOGUE + CASES[name])
    csrc = os.path.join(ROOT, "paper_2407_09848_amd", "csrc")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", str(tmp_path), "-I", csrc,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr[-3000:]
