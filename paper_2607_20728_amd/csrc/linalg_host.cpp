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
// result does not depend on the vector width.  Matrices are held in blocks of
// 16 columns, each contiguous and always with the same worker.  On 16 threads
// (EPYC), against the scalar form split by rows: an eigenproblem of 73 0.29 ms
// and now 0.24 (one thread), of 100 0.53 and 0.50, of 200 3.0 and 1.95, of 300
// 6.5 and 4.9, of 400 11.7 and 8.9, of 800 51 and 38; a Cholesky factor of 200
// with its inverse 0.51 and 0.21, of 600 5.4 and 4.1.
//
// A part is split over a small pool of host threads from the work on that
// pays for waking them: the rotations from about 85 rows, the reflectors' product
// from 131, the inverse from 208, a reduction step from 224 trailing rows, a
// Cholesky column from about 550 rows.
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
  long runs() const { return runs_.load(std::memory_order_relaxed); }
  void run(const std::function<void(int, int)>& fn) {
    std::unique_lock<std::mutex> own(run_mx_, std::try_to_lock);
    if (n_ == 1 || !own.owns_lock()) {
      for (int t = 0; t < n_; ++t) fn(t, n_);
      return;
    }
    runs_.fetch_add(1, std::memory_order_relaxed);
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
  std::atomic<long> runs_{0};
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

// fn(q) for the blocks [q0, q1), block q always on the same worker
template <class F>
void deal_blocks(int q0, int q1, double flops, double least, F&& fn) {
  Workers& w = Workers::get();
  if (w.size() == 1 || flops < least) {
    for (int q = q0; q < q1; ++q) fn(q);
    return;
  }
  w.run([&](int t, int nt) {
    for (int q = q0 + (t - q0 % nt + nt) % nt; q < q1; q += nt) fn(q);
  });
}

// Least work worth handing out: a step of the reduction and a column of the
// Cholesky factor (with workers that are awake from the step before), and a
// part by itself.  Eigenproblems of 100 / 160 / 240 take 0.54 / 1.31 / 2.95 ms with
// 3e5 and 8e6, 0.50 / 1.20 / 2.88 with 3e5 and 3e6, 0.46 / 1.20 / 2.93 with 3e5 and
// 1e6 (but inverses of 160 and 200 0.07 and 0.11 ms for 0.05 and 0.09), 0.50 / 1.21 /
// 2.95 with 6e5 and 3e6; a Cholesky factor of 800 takes 4.8 ms from 1.5e5 on
// and 6.8 from 3e5 on.
constexpr double kSplitReduce = 3.0e5, kSplitColumn = 1.5e5, kSplitOnce = 3.0e6;

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

int blocks(int n) { return (n + kL - 1) / kL; }
int padded(int n) { return blocks(n) * kL + kL; }

// One step of the reduction on a block x of kL columns (rows kL apart), rows
// [i0, n): the rank-2 update x -= v w^T + w v^T of the step before, where v is
// given (vj, wj: v and w at the block's columns), and with the rows so updated
// p = b x^T u, even and odd rows summed apart.
LANES void reduce_block_body(int i0, int n, double* x, const double* v, const double* w,
                             const double* vj, const double* wj, const double* u, double b,
                             double* p) {
#pragma clang fp contract(off)
  v4 s[4] = {}, t[4] = {}, cv[4], cw[4];
  if (v)
    for (int l = 0; l < 4; ++l) {
      cv[l] = *(const v4*)(vj + 4 * l);
      cw[l] = *(const v4*)(wj + 4 * l);
    }
  auto row = [&](int i, v4* sum) __attribute__((always_inline)) {
    double* r = x + (size_t)i * kL;
    for (int l = 0; l < 4; ++l) {
      v4 y = *(const v4*)(r + 4 * l);
      if (v) {
        y -= v[i] * cw[l] + w[i] * cv[l];
        *(v4*)(r + 4 * l) = y;
      }
      sum[l] += y * u[i];
    }
  };
  int i = i0;
  for (; i + 1 < n; i += 2) {
    row(i, s);
    row(i + 1, t);
  }
  if (i < n) row(i, s);
  for (int l = 0; l < 4; ++l) *(v4*)(p + 4 * l) = b * (s[l] + t[l]);
}
LANES_PICK(reduce_block,
           (int i0, int n, double* x, const double* v, const double* w, const double* vj,
            const double* wj, const double* u, double b, double* p),
           (i0, n, x, v, w, vj, wj, u, b, p))

// rows [i0, n) of a block x of kL columns <- (1 - b v v^T) x
LANES void reflect_block_body(int i0, int n, double* x, const double* v, double b) {
#pragma clang fp contract(off)
  v4 s[4] = {};
  for (int i = i0; i < n; ++i)
    for (int l = 0; l < 4; ++l) s[l] += v[i] * *(const v4*)(x + (size_t)i * kL + 4 * l);
  for (int l = 0; l < 4; ++l) s[l] *= b;
  for (int i = i0; i < n; ++i)
    for (int l = 0; l < 4; ++l) *(v4*)(x + (size_t)i * kL + 4 * l) -= s[l] * v[i];
}
LANES_PICK(reflect_block, (int i0, int n, double* x, const double* v, double b), (i0, n, x, v, b))

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

// T = Q^T A Q tridiagonal (d, e), A symmetric in blocks of kL columns, [n][kL]
// each (overwritten).  Reflector k, I - beta_k v_k v_k^T acting on indices
// k+1..n-1, is kept in row k of V (rows ld apart, zero up to column k).
// A block belongs to one worker from the first step to the last and is read
// and written once a step, the update of a step together with the product of
// the next: with blocks that began at the step's own column, and two visits, a
// line changed hands at every row of every step, and an eigenproblem of 400
// took 17.7 ms.
void householder_tridiag(int n, int ld, std::vector<double>& A, std::vector<double>& V,
                         std::vector<double>& beta, std::vector<double>& d,
                         std::vector<double>& e) {
#pragma clang fp contract(off)
  const int nq = blocks(n);
  std::vector<double> p(ld, 0.0), w(ld, 0.0);
  const double* v0 = nullptr;  // the reflector whose update is still to be made
  // column k from row k on, with that update
  auto entry = [&](int i, int k) {
    const double x = A[((size_t)(k / kL) * n + i) * kL + k % kL];
    return v0 ? x - (v0[i] * w[k] + w[i] * v0[k]) : x;
  };
  for (int k = 0; k + 2 < n; ++k) {
    const int i0 = k + 1;
    double* v = &V[(size_t)k * ld];
    d[k] = entry(k, k);
    double nrm2 = 0.0;
    for (int i = i0; i < n; ++i) {
      v[i] = entry(i, k);
      nrm2 += v[i] * v[i];
    }
    const double tail = nrm2 - v[i0] * v[i0];
    beta[k] = 0.0;
    e[k] = v[i0];
    const bool skip = tail <= 0.0;  // already tridiagonal in this column
    if (!skip) {
      const double nrm = std::sqrt(nrm2);
      e[k] = v[i0] > 0 ? -nrm : nrm;
      v[i0] -= e[k];
      beta[k] = 2.0 / (v[i0] * v[i0] + tail);
    }
    if (!skip || v0)
      deal_blocks(i0 / kL, nq, 6.0 * (n - i0) * (n - i0), kSplitReduce, [&](int q) {
        reduce_block(i0, n, &A[(size_t)q * n * kL], v0, w.data(), v0 ? v0 + q * kL : nullptr,
                     &w[q * kL], v, beta[k], &p[q * kL]);
      });
    v0 = nullptr;
    if (skip) continue;
    double pv = 0.0;
    for (int i = i0; i < n; ++i) pv += p[i] * v[i];
    const double K = 0.5 * beta[k] * pv;
    w[k] = 0.0;
    for (int i = i0; i < n; ++i) w[i] = p[i] - K * v[i];
    v0 = v;
  }
  if (n > 1) {
    d[n - 2] = entry(n - 2, n - 2);
    e[n - 2] = entry(n - 1, n - 2);
  }
  d[n - 1] = entry(n - 1, n - 1);
  e[n - 1] = 0.0;
}

// Q^T in blocks of kL columns, [n][kL] each (element (r, c) of Q^T at row r of
// block c / kL), Q = H_0 H_1 ... H_{n-3}: the reflectors applied to the unit
// vectors, column j of Q, from the last to the first (H_k leaves e_j alone for
// k >= j), kL columns at a time.
void form_qt(int n, int ld, const std::vector<double>& V, const std::vector<double>& beta,
             std::vector<double>& Qt) {
  const int nq = blocks(n);
  deal_blocks(0, nq, 4.0 / 3.0 * n * (double)n * n, kSplitOnce, [&](int q) {
    std::vector<double> x((size_t)nq * kL * kL, 0.0);
    for (int l = 0; l < kL && q * kL + l < n; ++l) x[(size_t)(q * kL + l) * kL + l] = 1.0;
    for (int k = std::min(q * kL + kL - 2, n - 3); k >= 0; --k)
      if (beta[k] != 0.0) reflect_block(k + 1, n, x.data(), &V[(size_t)k * ld], beta[k]);
    for (int b = 0; b < nq; ++b)
      for (int l = 0; l < kL && q * kL + l < n; ++l)
        for (int i = 0; i < kL; ++i)
          Qt[((size_t)b * n + q * kL + l) * kL + i] = x[(size_t)(b * kL + i) * kL + l];
  });
}

// apply recorded plane rotations to the rows of Qt, a block of columns at a time
void apply_rotations(int n, const std::vector<Rot>& rots, std::vector<double>& Qt) {
  if (rots.empty()) return;
  deal_blocks(0, blocks(n), 6.0 * (double)rots.size() * n, kSplitOnce,
              [&](int q) { rotate_block(rots.data(), rots.size(), &Qt[(size_t)q * n * kL]); });
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

long host_pool_runs() { return Workers::get().runs(); }

int host_syev(int n, double* Ain, double* w) {
  if (n <= 0) return 0;
  const int nq = blocks(n), ld = nq * kL;
  std::vector<double> A((size_t)nq * n * kL, 0.0), V((size_t)n * ld, 0.0), beta(n, 0.0);
  for (int q = 0; q < nq; ++q)
    for (int i = 0; i < n; ++i)
      for (int j = q * kL; j < std::min(n, (q + 1) * kL); ++j)
        A[((size_t)q * n + i) * kL + j % kL] = 0.5 * (Ain[(size_t)i * n + j] + Ain[(size_t)j * n + i]);
  std::vector<double> d(n), e(n);
  householder_tridiag(n, ld, A, V, beta, d, e);
  std::vector<double>& Qt = A;
  form_qt(n, ld, V, beta, Qt);
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
      apply_rotations(n, rots, Qt);
      rots.clear();
    }
    if (++guard > 60 * n + 100) return 1;
  }
  apply_rotations(n, rots, Qt);
  std::vector<int> idx(n);
  for (int i = 0; i < n; ++i) idx[i] = i;
  std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return d[x] < d[y]; });
  for (int j = 0; j < n; ++j) w[j] = d[idx[j]];
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j)
      Ain[(size_t)i * n + j] = Qt[((size_t)(i / kL) * n + idx[j]) * kL + i % kL];
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
    split_range((m + kL - 1) / kL, 2.0 * m * (double)j, kSplitColumn, [&](int lo, int hi) {
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
