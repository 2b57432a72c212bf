"""The parts of the host linear algebra (csrc/linalg_host.cpp) that are split over
its worker threads, at sizes where every one of them is: the eigensolver's
reduction, reflectors and rotations, the Cholesky factor and its inverse.

The source is compiled with g++ into a driver that reads the pool's own count
of split parts, so a threshold that keeps a part from the pool fails here:
below 260 rows a reduction step has 224 trailing rows or more, below 560 rows
a Cholesky column reaches its least work.  Results have to be bitwise those of
one thread, also when four callers use the pool at once (under ThreadSanitizer
and AddressSanitizer).
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_20728_amd", "csrc")

DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <thread>
#include <vector>
namespace bsex {
int host_syev(int n, double* A, double* w);
int host_cholesky(int n, double* A);
int host_trinv_lower(int n, double* L);
long host_pool_runs();
}
typedef std::vector<double> vec;

// what: 0 eigenproblem, 1 Cholesky factor, 2 its inverse too
static vec solve(int what, int n, unsigned seed) {
  std::mt19937_64 g(seed);
  std::normal_distribution<double> N(0.0, 1.0);
  vec A((size_t)n * n), w(n, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j <= i; ++j) A[(size_t)i * n + j] = A[(size_t)j * n + i] = N(g);
  if (what)
    for (int i = 0; i < n; ++i) A[(size_t)i * n + i] += 3.0 * n;
  int rc = what ? bsex::host_cholesky(n, A.data()) : bsex::host_syev(n, A.data(), w.data());
  if (!rc && what == 2) rc = bsex::host_trinv_lower(n, A.data());
  if (rc) exit(10);
  A.insert(A.end(), w.begin(), w.end());
  return A;
}

int main(int argc, char** argv) {
  const int what = atoi(argv[1]), n = atoi(argv[2]), callers = atoi(argv[3]);
  const long before = bsex::host_pool_runs();
  const vec ref = solve(what, n, 7);
  const long runs = bsex::host_pool_runs() - before;
  std::vector<int> bad(callers, 0);
  std::vector<std::thread> th;
  for (int c = 0; c < callers; ++c)
    th.emplace_back([&, c] {
      const vec x = solve(what, n, 7);
      bad[c] = memcmp(x.data(), ref.data(), sizeof(double) * x.size()) != 0;
    });
  for (auto& t : th) t.join();
  for (int c = 0; c < callers; ++c)
    if (bad[c]) return 11;
  uint64_t h = 1469598103934665603ull;
  for (double v : ref) {
    uint64_t b;
    memcpy(&b, &v, 8);
    h = (h ^ b) * 1099511628211ull;
  }
  std::printf("%ld %016llx\n", runs, (unsigned long long)h);
  return 0;
}
"""


def _build(d, flags):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("g++ or the ROCm headers are missing")
    src, exe = d / "driver.cpp", d / "driver"
    src.write_text(DRIVER)
    cmd = [gxx, "-std=c++17", "-pthread", *flags, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I", CSRC, str(src), os.path.join(CSRC, "linalg_host.cpp"), "-o", str(exe)]
    p = subprocess.run(cmd, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    return exe


def _run(exe, what, n, threads, callers=0):
    env = dict(os.environ, BSEX_HOST_THREADS=str(threads),
               TSAN_OPTIONS="halt_on_error=1 second_deadlock_stack=1",
               ASAN_OPTIONS="detect_leaks=0 halt_on_error=1")
    p = subprocess.run([str(exe), str(what), str(n), str(callers)], env=env, capture_output=True,
                       text=True, timeout=300)
    assert p.returncode == 0, (p.returncode, (p.stdout + p.stderr)[-3000:])
    assert "WARNING: ThreadSanitizer" not in p.stderr, p.stderr[-3000:]
    runs, bits = p.stdout.split()
    return int(runs), bits


@pytest.fixture(scope="module")
def plain(tmp_path_factory):
    return _build(tmp_path_factory.mktemp("pool"), ["-O2"])


# least split parts: the reduction steps with 224 trailing rows or more, the
# reflectors and the rotations; a column of the factor; the inverse
@pytest.mark.parametrize("what,n,least", [(0, 90, 1), (0, 140, 2), (0, 259, 37), (0, 273, 51),
                                          (1, 560, 1), (1, 600, 100), (2, 215, 1), (2, 289, 1)])
def test_split_parts(plain, what, n, least):
    one, bits1 = _run(plain, what, n, 1)
    four, bits4 = _run(plain, what, n, 4)
    assert one == 0 and four >= least, (one, four)
    assert bits4 == bits1


@pytest.mark.parametrize("san", ["thread", "address"])
def test_concurrent_callers(tmp_path, san):
    exe = _build(tmp_path, ["-O1", "-g", f"-fsanitize={san}"])
    for what, n in ((0, 250), (1, 570), (2, 240)):
        runs, bits = _run(exe, what, n, 4, callers=4)
        assert runs > 0
        assert bits == _run(exe, what, n, 1)[1]
