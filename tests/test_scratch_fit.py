"""How kept scratch grows and falls back on a nearly full device
(csrc/scratch_fit.h), compiled with g++ against a memory of a few units.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_20728_amd", "csrc")

HEAD = r"""
#include <cstdio>
#include <vector>
#include "scratch_fit.h"
using namespace bsex;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x); return 1; } } while (0)
"""

GROW = r"""
int main() {
  const long M = 1L << 20;
  struct { long free, have, need, want; int rc; size_t tries; } t[] = {
      {100 * M, 0, 5 * M, 5 * M, BSE_OK, 1},         // the first one: as asked
      {100 * M, 3 * M, 4 * M, 6 * M, BSE_OK, 1},     // twice what there was
      {100 * M, 20 * M, 21 * M, 24 * M, BSE_OK, 1},  // at most 4 M more
      {100 * M, 3 * M, 9 * M, 9 * M, BSE_OK, 1},     // more than twice: as asked
      {22 * M, 20 * M, 21 * M, 21 * M, BSE_OK, 2},   // the longer one does not fit
      {20 * M, 20 * M, 21 * M, 0, BSE_ENOMEM, 2},    // nor does the one asked for
      {8 * M, 3 * M, 9 * M, 0, BSE_ENOMEM, 1}};
  for (auto& c : t) {
    std::vector<long> tries;
    long got = 0;
    const int rc = grow_scratch(c.have, c.need, [&](long n) {
      tries.push_back(n);
      if (n > c.free) return (int)BSE_ENOMEM;
      got = n;
      return (int)BSE_OK;
    });
    CHECK(rc == c.rc && got == c.want && tries.size() == c.tries && tries.back() >= c.need);
  }
  int n = 0;  // another error is passed on at once
  CHECK(grow_scratch(3 * M, 4 * M, [&](long) { ++n; return (int)BSE_EHIP; }) == BSE_EHIP && n == 1);
  return 0;
}
"""

# one call's buffers as the coupling's bands need them: pair grids of 10 units a
# set that stay when the second buffer, 4 a set, is out of memory
SETS = r"""
struct Mem {
  int free, grids = 0, rows = 0, tries = 0;
  int alloc(int sets) {
    ++tries;
    if (grids < sets) {
      free += 10 * grids;
      grids = 0;
      if (10 * sets > free) return BSE_ENOMEM;
      free -= 10 * (grids = sets);
    }
    if (rows < sets) {
      free += 4 * rows;
      rows = 0;
      if (4 * sets > free) return BSE_ENOMEM;
      free -= 4 * (rows = sets);
    }
    return BSE_OK;
  }
  void drop() {
    free += 10 * grids + 4 * rows;
    grids = rows = 0;
  }
};

int main() {
  struct { int free, want, sets, rc, limit; } t[] = {
      {200, 8, 8, BSE_OK, 0},      {112, 8, 8, BSE_OK, 0},      {111, 8, 1, BSE_OK, 1},
      {80, 8, 1, BSE_OK, 1},       {14, 8, 1, BSE_OK, 1},       {13, 8, 1, BSE_ENOMEM, 1},
      {14, 1, 1, BSE_OK, 0},       {13, 1, 1, BSE_ENOMEM, 0}};
  for (auto& c : t) {
    Mem m{c.free};
    int limit = 0, sets = 0;
    auto call = [&](int want) {
      return fit_sets(want, &limit, [&](int n) { return m.alloc(n); }, [&] { m.drop(); }, &sets);
    };
    CHECK(call(c.want) == c.rc && sets == c.sets && limit == c.limit);
    if (c.rc != BSE_OK) continue;
    // what one set does not need is free, and a later call does not try again
    CHECK(m.free == c.free - 14 * c.sets);
    const int tries = m.tries;
    CHECK(call(c.want) == BSE_OK && sets == c.sets && m.tries == tries + 1);
    CHECK(m.free == c.free - 14 * c.sets);
  }
  int limit = 0, sets = 0, n = 0, drops = 0;  // another error is passed on at once
  CHECK(fit_sets(8, &limit, [&](int) { ++n; return (int)BSE_EHIP; }, [&] { ++drops; }, &sets) ==
        BSE_EHIP);
  CHECK(n == 1 && drops == 0 && limit == 0);
  return 0;
}
"""


def _run(tmp_path, body):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is missing")
    src, exe = tmp_path / "fit.cpp", tmp_path / "fit"
    src.write_text(HEAD + body)
    p = subprocess.run([gxx, "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_workspace_growth(tmp_path):
    _run(tmp_path, GROW)


def test_sets_fall_back_to_one(tmp_path):
    _run(tmp_path, SETS)
