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
