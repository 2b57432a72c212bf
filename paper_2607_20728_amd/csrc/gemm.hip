// FP64 and FP32 GEMMs on the CDNA matrix cores (v_mfma_f64_16x16x4f64,
// v_mfma_f32_16x16x4f32).
//
// Workgroup tile BM x 64, K steps of 16 (32 in FP32) through two LDS buffers
// (the next step's tiles are held in registers meanwhile), four waves.  BM = 64:
// the waves own 32 x 32 quarters as 2 x 2 MFMA tiles.  BM = 16, for outputs
// of at most 16 rows (the solvers' products of a few vectors with a whole
// subspace): the waves own the four 16 x 16 tiles side by side, so no matrix
// core work or LDS is spent on 48 rows of zeros.  Operand layout of the
// 16x16x4 instructions: A[i][k] and B[k][j] from lane i + 16 k (i, j < 16,
// k < 4); the four accumulator values of lane j + 16 q are C[q + 4 t][j]
// (f64) and C[4 q + t][j] (f32), t < 4 (both checked on the device).
//
// The tall variant splits a long K across workgroups (C = A B^T with small
// M, N) and sums the partial tiles in a fixed order, so results repeat
// bitwise.
#include <algorithm>

#include "common.h"

namespace bsex {

namespace {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int BN = 64;
// K step: 1024 cycles of a wave's matrix work in a 64 x 64 tile
template <typename T>
constexpr int bk_full() {
  return sizeof(T) == 8 ? 16 : 32;
}
constexpr int BK = bk_full<double>();

// rows of the workgroup tile for an M-row output
inline int bm_for(long M) { return M <= 16 ? 16 : 64; }

// A launch of few workgroups waits for its loads: each K step ends at a
// barrier behind the next step's tiles.  Such launches take K steps of 64
// (and 32 x 32 tiles instead of 64 x 64, four times as many workgroups), so
// there are a quarter of the waits.  Every output element still sums its K
// in the same order, so results do not change.
constexpr int BKF = 64, BMF = 32;

template <typename T>
struct MfmaOf;
template <>
struct MfmaOf<double> {
  typedef double4_t acc_t;
  static __device__ __forceinline__ acc_t step(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of accumulator value t of lane group q
  static __device__ __forceinline__ int row(int q, int t) { return q + 4 * t; }
};
template <>
struct MfmaOf<float> {
  typedef float4_t acc_t;
  static __device__ __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q, int t) { return 4 * q + t; }
};

// one workgroup tile of C = alpha op(A) op(B) + beta C (in T, accumulated in T)
template <typename T, int TA, int TB, int BM, int BN, int BK>
__device__ __forceinline__ void gemm_tile(long M, long N, long K, T alpha,
                                          const T* __restrict__ A, long lda,
                                          const T* __restrict__ B, long ldb, T beta,
                                          const T* Cin, T* __restrict__ C, long ldc,
                                          long k_chunk, long c_split_stride, int ntn,
                                          int by_row) {
  typedef MfmaOf<T> MF;
  constexpr int WGM = BM >= 32 ? 2 : 1;  // waves along M
  constexpr int WGN = 4 / WGM;           // waves along N
  constexpr int TM = BM / (16 * WGM);    // MFMA tiles per wave along M
  constexpr int TN = BN / (16 * WGN);    // and along N
  // padded rows: 8-byte values need an odd stride, 4-byte ones one that keeps
  // the four k rows of an operand read and the 32 of a write on banks apart
  constexpr int PAD = sizeof(T) == 8 ? 1 : 17;
  constexpr int NBUF = BK == BKF ? 1 : 2;
  __shared__ T As[NBUF][BK][BM + PAD];
  __shared__ T Bs[NBUF][BK][BN + PAD];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  long mt;
  int nt;
  if (by_row) {  // a row of tiles on one XCD, which reads its A rows once
    xcd_item(blockIdx.x, ntn, true, mt, nt);
    if (mt * BM >= M) return;
  } else {  // tile columns spread over the XCDs, each reading its B columns
    mt = blockIdx.x / ntn;
    nt = (int)(blockIdx.x % ntn);
  }
  const long m0 = mt * BM;
  const long n0 = (long)nt * BN;
  const long kb = (long)blockIdx.z * k_chunk;
  const long ke = min(K, kb + k_chunk);
  typename MF::acc_t acc[TM][TN];
  for (int a = 0; a < TM; ++a)
    for (int b = 0; b < TN; ++b)
      for (int t = 0; t < 4; ++t) acc[a][b][t] = 0;

  // element e of a thread's share of the A tile is (m, k) = a_mk(e), of the
  // B tile (n, k) = b_nk(e); the next K step's tiles are loaded into
  // registers while the matrix cores work on the current one.  Each element
  // has a pointer that a step advances, and rows past the edge of op(A) or
  // op(B) read the last one (their products reach no stored element), so only
  // a last, partial K step tests anything: with an address and two tests per
  // element and step, the vector units were busy for half as long as the
  // matrix cores (FP32, 3,400 x 256 x 60,000: 2.07 ms, now 1.74; FP64, split
  // 3,470 x 320 x 34,000: 1.33, now 1.22).  The FP64 form of few workgroups
  // runs a few steps only and keeps the tests: setting up 16 pointers took
  // longer (8.0 us against 7.4 for a product of one coupling column).
  constexpr bool PTR = BK != BKF || sizeof(T) == 4;
  constexpr int NA = BM * BK / 256, NB = BN * BK / 256;
  auto a_mk = [&](int e, int& m, int& k) {
    if (TA) {  // A[k][m], m contiguous
      m = e % BM;
      k = e / BM;
    } else {   // A[m][k], k contiguous
      k = e % BK;
      m = e / BK;
    }
  };
  auto b_nk = [&](int e, int& n, int& k) {
    if (TB) {  // B[n][k], k contiguous
      k = e % BK;
      n = e / BK;
    } else {   // B[k][n], n contiguous
      n = e % BN;
      k = e / BN;
    }
  };
  T ra[NA], rb[NB];
  const T* pa[PTR ? NA : 1];
  const T* pb[PTR ? NB : 1];
#pragma unroll
  for (int q = 0; PTR && q < NA; ++q) {
    int m, k;
    a_mk(tid + 256 * q, m, k);
    const unsigned gm = (unsigned)min(m0 + m, M - 1);
    pa[q] = TA ? A + (kb + k) * lda + gm : A + (unsigned long)gm * lda + kb + k;
  }
#pragma unroll
  for (int q = 0; PTR && q < NB; ++q) {
    int n, k;
    b_nk(tid + 256 * q, n, k);
    const unsigned gn = (unsigned)min(n0 + n, N - 1);
    pb[q] = TB ? B + (unsigned long)gn * ldb + kb + k : B + (kb + k) * ldb + gn;
  }
  const long da = TA ? BK * lda : BK, db = TB ? BK : BK * ldb;
  auto fetch = [&](long k0) {
    if constexpr (!PTR) {
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        int m, k;
        a_mk(tid + 256 * q, m, k);
        const long gm = m0 + m, gk = k0 + k;
        ra[q] = (gm < M && gk < ke) ? (TA ? A[gk * lda + gm] : A[gm * lda + gk]) : (T)0;
      }
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        int n, k;
        b_nk(tid + 256 * q, n, k);
        const long gn = n0 + n, gk = k0 + k;
        rb[q] = (gn < N && gk < ke) ? (TB ? B[gn * ldb + gk] : B[gk * ldb + gn]) : (T)0;
      }
      return;
    }
    if (k0 + BK <= ke) {
#pragma unroll
      for (int q = 0; q < NA; ++q) ra[q] = *pa[q];
#pragma unroll
      for (int q = 0; q < NB; ++q) rb[q] = *pb[q];
    } else {
#pragma unroll
      for (int q = 0; q < NA; ++q) {
        int m, k;
        a_mk(tid + 256 * q, m, k);
        ra[q] = k0 + k < ke ? *pa[q] : (T)0;
      }
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        int n, k;
        b_nk(tid + 256 * q, n, k);
        rb[q] = k0 + k < ke ? *pb[q] : (T)0;
      }
    }
#pragma unroll
    for (int q = 0; q < NA; ++q) pa[q] += da;
#pragma unroll
    for (int q = 0; q < NB; ++q) pb[q] += db;
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      int m, k;
      a_mk(tid + 256 * q, m, k);
      As[buf][k][m] = ra[q];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      int n, k;
      b_nk(tid + 256 * q, n, k);
      Bs[buf][k][n] = rb[q];
    }
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int kr = kk + (lane >> 4);
      T a[TM], b[TN];
#pragma unroll
      for (int t = 0; t < TM; ++t) a[t] = As[buf][kr][wm * 16 * TM + t * 16 + (lane & 15)];
#pragma unroll
      for (int t = 0; t < TN; ++t) b[t] = Bs[buf][kr][wn * 16 * TN + t * 16 + (lane & 15)];
#pragma unroll
      for (int ta = 0; ta < TM; ++ta)
#pragma unroll
        for (int tb = 0; tb < TN; ++tb)
          acc[ta][tb] = MF::step(a[ta], b[tb], acc[ta][tb]);
    }
  };
  if (kb < ke) {
    fetch(kb);
    if constexpr (NBUF == 2) {
      // one barrier a step: the next tiles go to the other buffer
      stage(0);
      if (kb + BK < ke) fetch(kb + BK);
      __syncthreads();
      int buf = 0;
      for (long k0 = kb; k0 < ke; k0 += BK, buf ^= 1) {
        multiply(buf);
        if (k0 + BK < ke) {
          stage(buf ^ 1);
          if (k0 + 2 * BK < ke) fetch(k0 + 2 * BK);
        }
        __syncthreads();
      }
    } else {
      for (long k0 = kb; k0 < ke; k0 += BK) {
        stage(0);
        __syncthreads();
        if (k0 + BK < ke) fetch(k0 + BK);
        multiply(0);
        __syncthreads();
      }
    }
  }
  // the beta term's values are read together: one at a time, each between two
  // stores that may alias it, they took the latency of 16 reads in a row
  T* Cz = C + (long)blockIdx.z * c_split_stride;
  const long cm = m0 + wm * 16 * TM, cn = n0 + wn * 16 * TN + (lane & 15);
  T old[TM][TN][4];
  if (beta != (T)0) {
    const T* Co = Cin ? Cin : Cz;
#pragma unroll
    for (int ta = 0; ta < TM; ++ta)
#pragma unroll
      for (int tb = 0; tb < TN; ++tb)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const long gm = cm + ta * 16 + MF::row(lane >> 4, t), gn = cn + tb * 16;
          old[ta][tb][t] = gm < M && gn < N ? Co[gm * ldc + gn] : (T)0;
        }
  }
#pragma unroll
  for (int ta = 0; ta < TM; ++ta)
#pragma unroll
    for (int tb = 0; tb < TN; ++tb)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const long gm = cm + ta * 16 + MF::row(lane >> 4, t), gn = cn + tb * 16;
        if (gm < M && gn < N) {
          T v = alpha * acc[ta][tb][t];
          if (beta != (T)0) v += beta * old[ta][tb][t];
          Cz[gm * ldc + gn] = v;
        }
      }
}

template <int TA, int TB, int BM, int BN, int BK>
__global__ __launch_bounds__(256) void k_dgemm(long M, long N, long K, double alpha,
                                               const double* __restrict__ A, long lda,
                                               const double* __restrict__ B, long ldb,
                                               double beta, const double* Cin,
                                               double* __restrict__ C, long ldc, long k_chunk,
                                               long c_split_stride, int ntn, int by_row) {
  gemm_tile<double, TA, TB, BM, BN, BK>(M, N, K, alpha, A, lda, B, ldb, beta, Cin, C, ldc, k_chunk,
                                        c_split_stride, ntn, by_row);
}

template <int TA, int TB, int BM, int BN, int BK>
__global__ __launch_bounds__(256) void k_sgemm(long M, long N, long K, float alpha,
                                               const float* __restrict__ A, long lda,
                                               const float* __restrict__ B, long ldb,
                                               float beta, const float* Cin,
                                               float* __restrict__ C, long ldc, long k_chunk,
                                               long c_split_stride, int ntn, int by_row) {
  gemm_tile<float, TA, TB, BM, BN, BK>(M, N, K, alpha, A, lda, B, ldb, beta, Cin, C, ldc, k_chunk,
                                       c_split_stride, ntn, by_row);
}

// C = alpha * sum_z P[z] + beta * C, z ascending.  ZL > 1: ZL threads load an
// element's partials, ZL of them at a time each, into LDS, and one sums them
// there (one thread that loaded and added 512 in turn took 10 us and more).
template <int ZL>
__global__ __launch_bounds__(256) void k_reduce_split(long M, long N, int nz,
                                                      const double* __restrict__ P, long pstride,
                                                      double alpha, double beta,
                                                      double* __restrict__ C, long ldc) {
  constexpr int NE = 256 / ZL;
  const int el = threadIdx.x % NE, zl = threadIdx.x / NE;
  const long e = (long)blockIdx.x * NE + el;
  double s = 0.0;
  if constexpr (ZL == 1) {
    if (e < M * N) {
#pragma unroll 8
      for (int z = 0; z < nz; ++z) s += P[z * pstride + e];
    }
  } else {
    __shared__ double red[ZL * ZL][NE];
    for (int z0 = 0; z0 < nz; z0 += ZL * ZL) {
      double v[ZL];
#pragma unroll
      for (int q = 0; q < ZL; ++q) {
        const int z = z0 + q * ZL + zl;
        v[q] = z < nz && e < M * N ? P[z * pstride + e] : 0.0;
      }
      if (z0 > 0) __syncthreads();
#pragma unroll
      for (int q = 0; q < ZL; ++q) red[q * ZL + zl][el] = v[q];
      __syncthreads();
      const int n = min(ZL * ZL, nz - z0);
      if (zl == 0) {
#pragma unroll 8
        for (int z = 0; z < n; ++z) s += red[z][el];
      }
    }
    if (zl > 0) return;
  }
  if (e >= M * N) return;
  const long m = e / N, n = e % N;
  double v = alpha * s;
  if (beta != 0.0) v += beta * C[m * ldc + n];
  C[m * ldc + n] = v;
}

void reduce_split(long M, long N, int nz, const double* P, double alpha, double beta, double* C,
                  long ldc, hipStream_t st) {
  const long tot = M * N;
  if (nz > 16)
    hipLaunchKernelGGL(k_reduce_split<16>, dim3((unsigned)((tot + 15) / 16)), dim3(256), 0, st, M,
                       N, nz, P, tot, alpha, beta, C, ldc);
  else
    hipLaunchKernelGGL(k_reduce_split<1>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, M,
                       N, nz, P, tot, alpha, beta, C, ldc);
}

}  // namespace

namespace {

// the tiles of a launch with s K splits: 64 x 64 (16 x 64 up to 16 rows) in K
// steps of 16, or the latency forms when that gives fewer than `few` workgroups
struct Tiling {
  int bm, bn, bk;
  long mt, nt;
};
Tiling tiling(long M, long N, long K, long s, long few) {
  Tiling t{M <= 16 ? 16 : 64, BN, BK, 0, 0};
  t.mt = (M + t.bm - 1) / t.bm;
  t.nt = (N + t.bn - 1) / t.bn;
  if (t.mt * t.nt * s < few && K >= 2 * BKF) {
    t.bk = BKF;
    if (t.bm == 64) t.bm = t.bn = BMF;
    t.mt = (M + t.bm - 1) / t.bm;
    t.nt = (N + t.bn - 1) / t.bn;
  }
  return t;
}

template <typename T, int TA, int TB, int BM, int BN_, int BK_, typename... Args>
void launch_tile(dim3 grid, hipStream_t st, Args... args) {
  if constexpr (sizeof(T) == 8)
    hipLaunchKernelGGL((k_dgemm<TA, TB, BM, BN_, BK_>), grid, dim3(256), 0, st, args...);
  else
    hipLaunchKernelGGL((k_sgemm<TA, TB, BM, BN_, BK_>), grid, dim3(256), 0, st, args...);
}

template <typename T, int TA, int TB, typename... Args>
void launch_form(const Tiling& t, dim3 grid, hipStream_t st, Args... args) {
  if (t.bm == 16)
    t.bk == BKF ? launch_tile<T, TA, TB, 16, BN, BKF>(grid, st, args...)
                : launch_tile<T, TA, TB, 16, BN, bk_full<T>()>(grid, st, args...);
  else
    t.bk == BKF ? launch_tile<T, TA, TB, BMF, BMF, BKF>(grid, st, args...)
                : launch_tile<T, TA, TB, 64, BN, bk_full<T>()>(grid, st, args...);
}

// few: below this many workgroups the latency forms serve.  FP64 fills a
// CU's matrix units from one workgroup, FP32 (half the time per instruction)
// needs more in flight: 3,400 x 256 x 60,000 in 212 full tiles takes 2.00 ms,
// in 848 small ones 1.73.
template <typename T>
int launch(int ta, int tb, long M, long N, long K, T alpha, const T* A, long lda, const T* B,
           long ldb, T beta, const T* Cin, T* C, long ldc, long kc, long cstride, long s,
           hipStream_t st) {
  const Tiling t = tiling(M, N, K, s, sizeof(T) == 8 ? 256 : 512);
  const int by_row = t.nt < t.mt && xcd_group_on() ? 1 : 0;
  const long nwg = (by_row ? round8(t.mt) : t.mt) * t.nt;
  if (nwg > 0x7fffffffL || M > 0xffffffffL || N > 0xffffffffL || s > 65535)
    return fail(BSE_EINVAL, "gemm: output too large for the grid");
  const dim3 grid((unsigned)nwg, 1, (unsigned)s);
  const int ntn = (int)t.nt;
#define GO(TA_, TB_)                                                                             \
  launch_form<T, TA_, TB_>(t, grid, st, M, N, K, alpha, A, lda, B, ldb, beta, Cin, C, ldc, kc, \
                           cstride, ntn, by_row)
  if (!ta && !tb)
    GO(0, 0);
  else if (!ta && tb)
    GO(0, 1);
  else if (ta && !tb)
    GO(1, 0);
  else
    GO(1, 1);
#undef GO
  BSE_HIP(hipGetLastError());
  return BSE_OK;
}

long tiles_of(long M, long N) {
  const long bm = bm_for(M);
  return ((M + bm - 1) / bm) * ((N + BN - 1) / BN);
}

}  // namespace

int dgemm(int ta, int tb, long M, long N, long K, double alpha, const double* A, long lda,
          const double* B, long ldb, double beta, double* C, long ldc, hipStream_t st) {
  return dgemm_from(ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, nullptr, C, ldc, st);
}

int sgemm(int ta, int tb, long M, long N, long K, float alpha, const float* A, long lda,
          const float* B, long ldb, float beta, float* C, long ldc, hipStream_t st) {
  if (M <= 0 || N <= 0) return BSE_OK;
  if (K <= 0) alpha = 0.0f;
  return launch<float>(ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, nullptr, C, ldc,
                       K > 0 ? K : 1, 0L, 1, st);
}

int dgemm_from(int ta, int tb, long M, long N, long K, double alpha, const double* A, long lda,
               const double* B, long ldb, double beta, const double* Cin, double* C, long ldc,
               hipStream_t st) {
  if (M <= 0 || N <= 0) return BSE_OK;
  if (K <= 0) alpha = 0.0;
  return launch<double>(ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, Cin, C, ldc, K > 0 ? K : 1,
                        0L, 1, st);
}

// K splits that raise `s` splits of `tiles` output tiles to about 1024
// workgroups (4 per CU) with chunks of at least KMIN: the products of small
// systems have few tiles and a short K, and run for as long as one
// workgroup's walk over its chunk.
// Chunks of at least 1024 only took 49 us for 16 x 80 x 1503, now 7; 61 us for
// 48 x 160 x 3695, now 13; 78 us for 96 x 96 x 6979, now 20.
constexpr long KMIN = 128;
static long fill_splits(long tiles, long s, long K) {
  if (tiles * s >= 1024) return s;
  return std::max(s, std::min(1024 / tiles, K / KMIN));
}

// split-K factor for an op(A) op(B) product whose tile grid is small: aim at
// ~4096 workgroups (16 per CU, so global-load latency is hidden by occupancy)
// with K chunks of at least 1024, at 1024 workgroups with shorter ones
static long k_splits(long M, long N, long K, bool fill) {
  const long tiles = tiles_of(M, N);
  if (tiles >= 2048) return 1;
  const long s = K < 2048 ? 1 : std::min((K + 1023) / 1024, std::max(1L, 4096 / tiles));
  return std::max(fill ? fill_splits(tiles, s, K) : s, 1L);
}

long dgemm_work(long M, long N, long K, bool fill) {
  const long s = k_splits(M, N, K, fill);
  return s > 1 ? s * M * N : 0;
}

int dgemm_ws(int ta, int tb, long M, long N, long K, double alpha, const double* A, long lda,
             const double* B, long ldb, double beta, double* C, long ldc, double* work,
             long work_len, hipStream_t st, bool fill) {
  long s = k_splits(M, N, K, fill);
  if (s <= 1 || !work || s * M * N > work_len)
    return dgemm(ta, tb, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, st);
  long kc = (K + s - 1) / s;
  kc = ((kc + BK - 1) / BK) * BK;
  s = (K + kc - 1) / kc;
  BSE_TRY(launch<double>(ta, tb, M, N, K, 1.0, A, lda, B, ldb, 0.0, nullptr, work, N, kc, M * N, s,
                         st));
  reduce_split(M, N, (int)s, work, alpha, beta, C, ldc, st);
  BSE_HIP(hipGetLastError());
  return BSE_OK;
}

// K splits of a product with a long K: about TALL_TARGET workgroups in all,
// K chunks of at least 1024
constexpr long TALL_TARGET = 1024;
static long tall_splits(long M, long N, long K, bool fill) {
  const long tiles = tiles_of(M, N);
  long s = TALL_TARGET / (tiles > 0 ? tiles : 1);
  const long maxs = (K + 1023) / 1024;
  if (s > maxs) s = maxs;
  if (fill) s = fill_splits(tiles > 0 ? tiles : 1, s, K);
  return std::max(s, 1L);
}

long dgemm_tall_work(long M, long N, long K, bool fill) {
  return tall_splits(M, N, K, fill) * M * N;
}

int dgemm_tall(long M, long N, long K, double alpha, const double* A, long lda, const double* B,
               long ldb, double beta, double* C, long ldc, double* work, long work_len,
               hipStream_t st, bool fill) {
  if (M <= 0 || N <= 0) return BSE_OK;
  long s = tall_splits(M, N, K, fill);
  if (s * M * N > work_len) return fail(BSE_EINVAL, "dgemm_tall: work buffer too small");
  long kc = (K + s - 1) / s;
  kc = ((kc + BK - 1) / BK) * BK;
  if (kc < BK) kc = BK;
  s = (K + kc - 1) / kc;
  if (s < 1) s = 1;
  BSE_TRY(launch<double>(0, 1, M, N, K, 1.0, A, lda, B, ldb, 0.0, nullptr, work, N, kc, M * N, s,
                         st));
  reduce_split(M, N, (int)s, work, alpha, beta, C, ldc, st);
  BSE_HIP(hipGetLastError());
  return BSE_OK;
}

}  // namespace bsex
