"""The pre-screen workspace's growth (csrc/morea_workspace.h) against an
allocator with a limit, on the CPU: what is asked of the allocator, what a call
gets, and that a refused growth is not asked for again by calls that the
workspace held has room for."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "morea_workspace.h"

static size_t g_limit;
static int g_allocs, g_frees;

static size_t call(morea::Workspace& w, size_t fixed, size_t smallest, size_t largest) {
  g_allocs = g_frees = 0;
  return morea::reserve_slab(
      w, fixed, 10, smallest, largest,
      [](size_t n) -> void* { g_allocs++; return n <= g_limit ? malloc(n) : nullptr; },
      [](void* p) { g_frees++; free(p); });
}

#define EXPECT(slab, allocs, frees, held)                                                              \
  do {                                                                                                 \
    if (got != (slab) || g_allocs != (allocs) || g_frees != (frees) || w.bytes != (held)) {            \
      printf("line %d: slab %zu, %d allocations, %d frees, %zu bytes\n", __LINE__, got, g_allocs,      \
             g_frees, w.bytes);                                                                        \
      return 1;                                                                                        \
    }                                                                                                  \
  } while (0)

int main() {
  morea::Workspace w;
  size_t got;
  g_limit = 1000000;
  got = call(w, 100, 64, 1000); EXPECT(1000u, 1, 0, 10100u);   // first
  got = call(w, 100, 64, 1000); EXPECT(1000u, 0, 0, 10100u);   // again
  got = call(w, 200, 64, 800); EXPECT(800u, 0, 0, 10100u);     // smaller
  got = call(w, 100, 64, 2000); EXPECT(2000u, 1, 1, 20100u);   // grows
  g_limit = 5000;
  got = call(w, 100, 64, 3000); EXPECT(64u, 2, 1, 740u);       // refused: the smallest slab
  got = call(w, 100, 64, 3000); EXPECT(64u, 0, 0, 740u);       // not asked for again
  got = call(w, 0, 64, 3000); EXPECT(64u, 0, 0, 740u);
  got = call(w, 100, 64, 20); EXPECT(20u, 0, 0, 740u);         // a small call has room
  got = call(w, 300, 64, 3000); EXPECT(64u, 2, 1, 940u);       // no room for the smallest: asked again
  got = call(w, 100, 64, 3000); EXPECT(64u, 0, 0, 940u);
  g_limit = 1000000;
  got = call(w, 600, 64, 3000); EXPECT(3000u, 1, 1, 30600u);   // granted
  got = call(w, 600, 64, 3100); EXPECT(3100u, 1, 1, 31600u);   // and grows as before
  g_limit = 900;
  got = call(w, 100, 64, 4000); EXPECT(64u, 2, 1, 740u);
  g_limit = 500;
  got = call(w, 400, 64, 64); EXPECT(0u, 1, 1, 0u);            // one size to ask for, no memory
  got = call(w, 400, 64, 3000); EXPECT(0u, 2, 0, 0u);
  got = call(w, 100, 64, 40); EXPECT(40u, 1, 0, 500u);
  // between: several slabs' room, held from a call with larger fixed parts
  g_limit = 3000;
  got = call(w, 2300, 64, 500); EXPECT(64u, 2, 1, 2940u);
  got = call(w, 100, 64, 500); EXPECT(256u, 0, 0, 2940u);
  free(w.data);
  return 0;
}
"""


def test_growth_and_refusal(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ is not installed")
    src, exe = tmp_path / "growth.cpp", tmp_path / "growth"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2303_04873_amd", "csrc"), "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
