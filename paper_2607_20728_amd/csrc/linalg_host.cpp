// Small dense symmetric eigensolver and Cholesky on the host (FP64).
//
// Eigensolver: Householder reduction to tridiagonal form T = Q^T A Q, then
// implicit symmetric QR steps with the Wilkinson shift, chasing the bulge
// with plane rotations and deflating negligible off-diagonal entries (the
// method of Golub and Van Loan, "Matrix Computations", Sec. 8.3).  Used for
// the Rayleigh-Ritz and Gram problems of the Davidson and ground-state
// subspace solvers (n up to several hundred).
//
// The O(n^3) parts work on 16 independent values side by side (four vector
// registers), laid out so that the sums that belong to one value stay in one
// lane, in the order of the scalar algorithm, and nothing is contracted: the
// result does not depend on the vector width.  An eigenproblem of 73 took
// 0.25 ms on 16 threads and takes 0.21 on one (of 200: 2.6 and now 1.8, of
// 300: 6.2 and 6.4 ms), a Cholesky factor of 200 with its inverse 0.43 and now
// 0.20 ms.  From about 200 rows on the parts are split over a small pool of
// host threads; below that the work is shorter than waking them, which on a
// busy host takes milliseconds.
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <cstdlib>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

#include "common.h"

namespace bsex {

namespace {

// Host worker threads.  The caller takes part as worker 0; idle workers spin
// for a short while, then sleep on a condition variable.  A call made while
// another thread holds the pool runs its parts one after another instead.
class Workers {
 public:
  static Workers& get() {
    static Workers* w = new Workers(count());  // kept until the process ends
    return *w;
  }
  int size() const { return n_; }
  void run(const std::function<void(int, int)>& fn) {
    std::unique_lock<std::mutex> own(run_mx_, std::try_to_lock);
    if (n_ == 1 || !own.owns_lock()) {
      for (int t = 0; t < n_; ++t) fn(t, n_);
      return;
    }
    job_ = &fn;
    left_.store(n_ - 1, std::memory_order_relaxed);
    {
      std::lock_guard<std::mutex> g(mx_);
      gen_.fetch_add(1, std::memory_order_release);
    }
    cv_.notify_all();
    fn(0, n_);
    while (left_.load(std::memory_order_acquire) != 0) relax();
  }

 private:
  explicit Workers(int n) : n_(n) {
    for (int t = 1; t < n_; ++t) std::thread([this, t] { loop(t); }).detach();
  }
  // threads: BSEX_HOST_THREADS, else the CPUs this process may run on, at most 16
  static int count() {
    int n = 1;
    if (const char* s = std::getenv("BSEX_HOST_THREADS")) {
      n = std::atoi(s);
    } else {
      cpu_set_t set;
      CPU_ZERO(&set);
      n = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set)
                                                        : (int)std::thread::hardware_concurrency();
      n = std::min(n, 16);
    }
    return std::max(1, std::min(n, 64));
  }
  static void relax() { __builtin_ia32_pause(); }
  void loop(int t) {
    unsigned seen = 0;
    for (;;) {
      unsigned g;
      int spins = 0;
      while ((g = gen_.load(std::memory_order_acquire)) == seen) {
        if (++spins < (1 << 14)) {
          relax();
          continue;
        }
        std::unique_lock<std::mutex> lk(mx_);
        cv_.wait(lk, [&] { return gen_.load(std::memory_order_acquire) != seen; });
      }
      seen = g;
      (*job_)(t, n_);
      left_.fetch_sub(1, std::memory_order_acq_rel);
    }
  }
  const int n_;
  std::mutex run_mx_, mx_;
  std::condition_variable cv_;
  std::atomic<unsigned> gen_{0};
  std::atomic<int> left_{0};
  const std::function<void(int, int)>* job_ = nullptr;
};

// fn(lo, hi) over [0, m) in contiguous parts; one part when the work is
// below `least` operations
template <class F>
void split_range(int m, double flops, double least, F&& fn) {
  Workers& w = Workers::get();
  if (w.size() == 1 || flops < least) {
    fn(0, m);
    return;
  }
  w.run([&](int t, int nt) {
    const int lo = (int)((long)m * t / nt), hi = (int)((long)m * (t + 1) / nt);
    if (hi > lo) fn(lo, hi);
  });
}

// least work worth handing out: within a sequence of parts, whose workers are
// awake (15 us on one thread; from 7e4 on, 200 rows took 2.2 ms for 1.8 and 300
// rows 9.3 for 6.4), and for a part by itself
constexpr double kSplitStep = 1.5e5, kSplitOnce = 8.0e6;

struct Rot {
  int k;
  double c, s;
};

// ---- lane kernels -----------------------------------------------------------------
// A block of kL columns; the matrices are padded so that whole blocks that
// begin at any column can be read and written.
constexpr int kL = 16;
typedef double v4 __attribute__((vector_size(32), aligned(8)));
// Each kernel is compiled for the baseline and for AVX2 (without FMA) and
// picks by the CPU.
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
bool wide() {
  static const bool w = __builtin_cpu_supports("avx2");
  return w;
}
#define LANES_WIDE __attribute__((target("avx2")))
#else
bool wide() { return false; }
#define LANES_WIDE
#endif
#define LANES __attribute__((always_inline)) inline
#define LANES_PICK(name, params, args)         \
  LANES_WIDE void name##_wide params { name##_body args; } \
  void name##_base params { name##_body args; }            \
  inline void name params { wide() ? name##_wide args : name##_base args; }

int padded(int n) { return (n + kL - 1) / kL * kL + kL; }

// p[i] = b (sum_j B[j][i] v[j]), even and odd j summed apart; blocks [b0, b1)
// of i < m
LANES void symv_block_body(int b0, int b1, int m, const double* B, int ld, const double* v,
                           double b, double* p) {
#pragma clang fp contract(off)
  for (int q = b0; q < b1; ++q) {
    const double* x = B + q * kL;
    v4 s[4] = {}, t[4] = {};
    int j = 0;
    for (; j + 1 < m; j += 2, x += 2 * (size_t)ld)
      for (int l = 0; l < 4; ++l) {
        s[l] += *(const v4*)(x + 4 * l) * v[j];
        t[l] += *(const v4*)(x + ld + 4 * l) * v[j + 1];
      }
    if (j < m)
      for (int l = 0; l < 4; ++l) s[l] += *(const v4*)(x + 4 * l) * v[j];
    for (int l = 0; l < 4; ++l) *(v4*)(p + q * kL + 4 * l) = b * (s[l] + t[l]);
  }
}
LANES_PICK(symv_block,
           (int b0, int b1, int m, const double* B, int ld, const double* v, double b, double* p),
           (b0, b1, m, B, ld, v, b, p))

// columns [b0, b1) (blocks) of B -= v w^T + w v^T, m rows.  Split like
// symv_block, so a worker reads what it wrote.
LANES void rank2_block_body(int b0, int b1, int m, double* B, int ld, const double* v,
                            const double* w) {
#pragma clang fp contract(off)
  const int c0 = b0 * kL, c1 = b1 * kL < m ? b1 * kL : m;
  for (int i = 0; i < m; ++i) {
    double* x = B + (size_t)i * ld;
    const double vi = v[i], wi = w[i];
    int j = c0;
    for (; j + 4 <= c1; j += 4) *(v4*)(x + j) -= vi * *(const v4*)(w + j) + wi * *(const v4*)(v + j);
    for (; j < c1; ++j) x[j] -= vi * w[j] + wi * v[j];
  }
}
LANES_PICK(rank2_block,
           (int b0, int b1, int m, double* B, int ld, const double* v, const double* w),
           (b0, b1, m, B, ld, v, w))

// columns [b0, b1) (blocks) of X <- (1 - b v v^T) X, m rows
LANES void reflect_block_body(int b0, int b1, int m, double* X, int ld, const double* v, double b) {
#pragma clang fp contract(off)
  for (int q = b0; q < b1; ++q) {
    double* x = X + q * kL;
    v4 s[4] = {};
    for (int i = 0; i < m; ++i)
      for (int l = 0; l < 4; ++l) s[l] += v[i] * *(const v4*)(x + (size_t)i * ld + 4 * l);
    for (int l = 0; l < 4; ++l) s[l] *= b;
    for (int i = 0; i < m; ++i)
      for (int l = 0; l < 4; ++l) *(v4*)(x + (size_t)i * ld + 4 * l) -= s[l] * v[i];
  }
}
LANES_PICK(reflect_block,
           (int b0, int b1, int m, double* X, int ld, const double* v, double b),
           (b0, b1, m, X, ld, v, b))

// the rotations on the rows of a dense block of kL columns; the row that two
// successive rotations share stays in registers
LANES void rotate_block_body(const Rot* rots, size_t nrot, double* band) {
#pragma clang fp contract(off)
  v4 c[4];
  int held = -1;
  for (size_t q = 0; q < nrot; ++q) {
    const Rot r = rots[q];
    double* x = band + (size_t)r.k * kL;
    if (held != r.k) {
      if (held >= 0)
        for (int l = 0; l < 4; ++l) *(v4*)(band + (size_t)held * kL + 4 * l) = c[l];
      for (int l = 0; l < 4; ++l) c[l] = *(const v4*)(x + 4 * l);
    }
    for (int l = 0; l < 4; ++l) {
      const v4 y = *(const v4*)(x + kL + 4 * l);
      *(v4*)(x + 4 * l) = r.c * c[l] + r.s * y;
      c[l] = -r.s * c[l] + r.c * y;
    }
    held = r.k + 1;
  }
  if (held >= 0)
    for (int l = 0; l < 4; ++l) *(v4*)(band + (size_t)held * kL + 4 * l) = c[l];
}
LANES_PICK(rotate_block, (const Rot* rots, size_t nrot, double* band), (rots, nrot, band))

// t[i] = a[i] - sum_{k < m} f[k] X[k][i], k ascending, one block of i
LANES void fold_block_body(int m, const double* f, const double* X, int ld, double* t) {
#pragma clang fp contract(off)
  v4 s[4];
  for (int l = 0; l < 4; ++l) s[l] = *(const v4*)(t + 4 * l);
  for (int k = 0; k < m; ++k) {
    const double fk = f[k];
    for (int l = 0; l < 4; ++l) s[l] -= *(const v4*)(X + (size_t)k * ld + 4 * l) * fk;
  }
  for (int l = 0; l < 4; ++l) *(v4*)(t + 4 * l) = s[l];
}
LANES_PICK(fold_block,
           (int m, const double* f, const double* X, int ld, double* t),
           (m, f, X, ld, t))

// A <- Q^T A Q tridiagonal (A symmetric, rows ld apart).  Reflector k,
// I - beta_k v_k v_k^T acting on indices k+1..n-1, is kept in row k of V
// (columns k+1..n-1).
void householder_tridiag(int n, int ld, std::vector<double>& A, std::vector<double>& V,
                         std::vector<double>& beta, std::vector<double>& d,
                         std::vector<double>& e) {
  auto a = [&](int i, int j) -> double& { return A[(size_t)i * ld + j]; };
  std::vector<double> p(ld), w(ld);
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1;  // length of the column below the diagonal
    double* v = &V[(size_t)k * ld + k + 1];
    double nrm2 = 0.0;
    for (int i = 0; i < m; ++i) {
      v[i] = a(k + 1 + i, k);
      nrm2 += v[i] * v[i];
    }
    const double tail = nrm2 - v[0] * v[0];
    beta[k] = 0.0;
    if (tail <= 0.0) continue;  // already tridiagonal in this column
    const double nrm = std::sqrt(nrm2);
    const double alpha = v[0] > 0 ? -nrm : nrm;
    v[0] -= alpha;
    const double bk = 2.0 / (v[0] * v[0] + tail);
    beta[k] = bk;
    double* B = &a(k + 1, k + 1);  // the trailing block
    // p = beta B v
    split_range((m + kL - 1) / kL, 2.0 * m * m, kSplitStep,
                [&](int lo, int hi) { symv_block(lo, hi, m, B, ld, v, bk, p.data()); });
    double pv = 0.0;
    for (int i = 0; i < m; ++i) pv += p[i] * v[i];
    const double K = 0.5 * bk * pv;
    for (int i = 0; i < m; ++i) w[i] = p[i] - K * v[i];
    split_range((m + kL - 1) / kL, 4.0 * m * m, 2 * kSplitStep,
                [&](int lo, int hi) { rank2_block(lo, hi, m, B, ld, v, w.data()); });
    a(k + 1, k) = a(k, k + 1) = alpha;
    for (int i = 1; i < m; ++i) a(k + 1 + i, k) = a(k, k + 1 + i) = 0.0;
  }
  for (int i = 0; i < n; ++i) d[i] = a(i, i);
  for (int i = 0; i + 1 < n; ++i) e[i] = a(i + 1, i);
  e[n - 1] = 0.0;
}

// Q = H_0 H_1 ... H_{n-3}: the reflectors applied to the unit vectors, column
// j of Q, from the last to the first (H_k leaves e_j alone for k >= j).
void form_q(int n, int ld, const std::vector<double>& V, const std::vector<double>& beta,
            std::vector<double>& Q) {
  for (int j = 0; j < n; ++j) Q[(size_t)j * ld + j] = 1.0;
  for (int k = n - 3; k >= 0; --k) {
    if (beta[k] == 0.0) continue;
    const int m = n - k - 1;
    double* X = &Q[(size_t)(k + 1) * ld + k + 1];
    const double* v = &V[(size_t)k * ld + k + 1];
    split_range((m + kL - 1) / kL, 4.0 * m * m, 2 * kSplitStep,
                [&](int lo, int hi) { reflect_block(lo, hi, m, X, ld, v, beta[k]); });
  }
}

// apply recorded plane rotations to the rows of Qt (rows ld apart), a dense
// copy of one block of columns at a time
void apply_rotations(int n, const std::vector<Rot>& rots, double* Qt, int ld) {
  if (rots.empty()) return;
  split_range((n + kL - 1) / kL, 6.0 * (double)rots.size() * n, kSplitOnce, [&](int lo, int hi) {
    std::vector<double> band((size_t)n * kL);
    for (int q = lo; q < hi; ++q) {
      double* x = Qt + q * kL;
      for (int r = 0; r < n; ++r)
        std::copy(x + (size_t)r * ld, x + (size_t)r * ld + kL, &band[(size_t)r * kL]);
      rotate_block(rots.data(), rots.size(), band.data());
      for (int r = 0; r < n; ++r)
        std::copy(&band[(size_t)r * kL], &band[(size_t)r * kL] + kL, x + (size_t)r * ld);
    }
  });
}

// One implicit Wilkinson-shifted QR step on the unreduced block [lo, hi] of
// the tridiagonal (d, e); the rotations are appended to rots.  The entries
// that two successive rotations share are carried in registers: a rotation is
// a chain of a square root, a division and a few products, and took nearly
// twice as long with a store and a load in it.
void qr_step(int lo, int hi, double* d, double* e, std::vector<Rot>& rots) {
  const double a = d[hi - 1], b = e[hi - 1], c = d[hi];
  const double delta = 0.5 * (a - c);
  const double rad = std::hypot(delta, b);
  const double mu = c - b * b / (delta + (delta >= 0 ? rad : -rad));
  double x = d[lo] - mu, z = e[lo];
  double akk = d[lo], ak1 = e[lo];
  const size_t q0 = rots.size();
  rots.resize(q0 + (hi - lo));
  Rot* out = rots.data() + q0;
  for (int k = lo; k < hi; ++k) {
    double r = std::sqrt(x * x + z * z);
    if (!(r > 1e-150 && r < 1e150)) r = std::hypot(x, z);  // squares out of range
    double cs = 1.0, sn = 0.0;
    if (r > 0.0) {
      cs = x / r;
      sn = z / r;
    }
    if (k > lo) e[k - 1] = r;
    const double a11 = d[k + 1];
    d[k] = cs * cs * akk + 2 * cs * sn * ak1 + sn * sn * a11;
    x = cs * sn * (a11 - akk) + (cs * cs - sn * sn) * ak1;
    akk = sn * sn * akk - 2 * cs * sn * ak1 + cs * cs * a11;
    if (k + 1 < hi) {
      const double e1 = e[k + 1];
      z = sn * e1;
      ak1 = cs * e1;
    }
    *out++ = Rot{k, cs, sn};
  }
  e[hi - 1] = x;
  d[hi] = akk;
}

}  // namespace

int host_syev(int n, double* Ain, double* w) {
  if (n <= 0) return 0;
  const int ld = padded(n);
  std::vector<double> A((size_t)(n + 1) * ld, 0.0), V((size_t)(n + 1) * ld, 0.0), beta(n, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j)
      A[(size_t)i * ld + j] = 0.5 * (Ain[(size_t)i * n + j] + Ain[(size_t)j * n + i]);
  std::vector<double> d(n), e(n);
  householder_tridiag(n, ld, A, V, beta, d, e);
  std::fill(V.begin() + (size_t)(n > 2 ? n - 2 : 0) * ld, V.end(), 0.0);
  std::fill(A.begin(), A.end(), 0.0);
  form_q(n, ld, V, beta, A);
  std::vector<double>& Qv = V;  // the eigenvectors' rows, from Q^T
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) Qv[(size_t)i * ld + j] = A[(size_t)j * ld + i];
  double* Qt = Qv.data();
  std::vector<Rot> rots;
  const size_t flush_at = (size_t)1 << 20;
  rots.reserve(std::min(flush_at, (size_t)n * n));
  int hi = n - 1, guard = 0;
  const double eps = 2.220446049250313e-16;
  while (hi > 0) {
    if (std::fabs(e[hi - 1]) <= eps * (std::fabs(d[hi - 1]) + std::fabs(d[hi]))) {
      e[hi - 1] = 0.0;
      --hi;
      continue;
    }
    int lo = hi - 1;
    while (lo > 0 && std::fabs(e[lo - 1]) > eps * (std::fabs(d[lo - 1]) + std::fabs(d[lo]))) --lo;
    if (lo > 0) e[lo - 1] = 0.0;
    qr_step(lo, hi, d.data(), e.data(), rots);
    if (rots.size() >= flush_at) {
      apply_rotations(n, rots, Qt, ld);
      rots.clear();
    }
    if (++guard > 60 * n + 100) return 1;
  }
  apply_rotations(n, rots, Qt, ld);
  std::vector<int> idx(n);
  for (int i = 0; i < n; ++i) idx[i] = i;
  std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return d[x] < d[y]; });
  for (int j = 0; j < n; ++j) {
    w[j] = d[idx[j]];
    for (int i = 0; i < n; ++i) Ain[(size_t)i * n + j] = Qt[(size_t)idx[j] * ld + i];
  }
  return 0;
}

int host_cholesky(int n, double* A) {
  // column by column, the factor held by columns: U[j][i] = L_ij
  const int ld = padded(n);
  std::vector<double> U((size_t)(n + 1) * ld, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j <= i; ++j) U[(size_t)j * ld + i] = A[(size_t)i * n + j];
  for (int j = 0; j < n; ++j) {
    double* x = &U[(size_t)j * ld + j];  // rows j.. of column j
    const int m = n - j;
    split_range((m + kL - 1) / kL, 2.0 * m * (double)j, kSplitStep, [&](int lo, int hi) {
      std::vector<double> f(j);
      for (int k = 0; k < j; ++k) f[k] = U[(size_t)k * ld + j];
      for (int q = lo; q < hi; ++q) fold_block(j, f.data(), &U[j + q * kL], ld, x + q * kL);
    });
    if (!(x[0] > 0.0)) return 1;
    const double r = std::sqrt(x[0]);
    x[0] = r;
    for (int i = 1; i < m; ++i) x[i] /= r;
  }
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) A[(size_t)i * n + j] = j <= i ? U[(size_t)j * ld + i] : 0.0;
  return 0;
}

int host_trinv_lower(int n, double* L) {
  for (int i = 0; i < n; ++i) {
    const double d = L[(size_t)i * n + i];
    if (!(d != 0.0) || !std::isfinite(d)) return 1;
  }
  // M = L^{-1} by forward substitution, M_ij = (delta_ij - sum_{j<=k<i} L_ik
  // M_kj) / L_ii, a block of columns at a time (its sums begin at its first
  // column: M_kj = 0 above the diagonal adds nothing)
  const int ld = padded(n);
  std::vector<double> M((size_t)(n + 1) * ld, 0.0);
  split_range((n + kL - 1) / kL, (double)n * n * n / 3, kSplitOnce, [&](int lo, int hi) {
    for (int q = lo; q < hi; ++q) {
      const int j0 = q * kL;
      for (int i = j0; i < n; ++i) {
        double* x = &M[(size_t)i * ld + j0];
        if (i < j0 + kL) x[i - j0] = 1.0;
        fold_block(i - j0, L + (size_t)i * n + j0, &M[(size_t)j0 * ld + j0], ld, x);
        const double d = L[(size_t)i * n + i];
        for (int l = 0; l < kL && j0 + l <= i; ++l) x[l] /= d;
      }
    }
  });
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) L[(size_t)i * n + j] = M[(size_t)i * ld + j];
  return 0;
}

}  // namespace bsex
