// One-time FP64 factorizations.
//
// Preconditioner P = (S + T/tau)^-1 (Sec. 2.4, Eq. 17): a blocked symmetric sweep. The paper inverts
// once per MD step with a library LU, since P need not be positive definite (Sec. 3.1); here each
// block column costs one pivot-block inversion plus two MFMA GEMMs. Step for pivot block K (width
// b), with A the current matrix (symmetric throughout):
//   U = A[:, K] with its rows of K zero                             (column panel copy)
//   W = A_KK^-1                                                     (one workgroup, in registers)
//   V = U W                                                         (n x b GEMM)
//   A -= V U^T                                                      (rank-b update, upper half)
//   A[:, K] = V, A[K, :] = V^T, A_KK = -W
// After the last block A holds minus the inverse. The pivot block is inverted by Gauss-Jordan with
// partial (row) pivoting inside the block, so an indefinite S + T/tau whose diagonal entries
// vanish or change sign along the sweep is handled as long as each pivot block is
// nonsingular; the blocks themselves are not exchanged. A singular pivot block or a non-finite
// value is reported, and inverse_residual() measures ||A P X - X|| on probe vectors so that a
// caller can reject an inaccurate inverse instead of using it.
//
// Cholesky flavour: S = L L^T and L^-1, block column by block column.
#include <math.h>

#include <type_traits>

#include "omm_internal.h"

namespace omm {
namespace {

constexpr int NB = 128;
constexpr int PROBES = 16;  // probe rows of inverse_residual

// U = A[:, k0:k0+b] (ld b) with zeros in the rows of the block, W = A[k0:k0+b, k0:k0+b].
__global__ void k_panel(const double* A, int64_t n, int64_t k0, int b, double* U, double* W) {
  const int64_t total = n * b;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * 256) {
    const int64_t i = e / b;
    const int j = (int)(e % b);
    const double v = A[i * n + k0 + j];
    const bool diag_blk = i >= k0 && i < k0 + b;
    U[e] = diag_blk ? 0.0 : v;
    if (diag_blk) W[(i - k0) * b + j] = v;
  }
}

// A[:, k0:k0+b] = V and A[k0:k0+b, :] = V^T outside the block, A_KK = -(W + W^T) / 2; 32 x 32 tiles
// of V (rows blockIdx.x, columns blockIdx.y), transposed through LDS.
__global__ __launch_bounds__(256) void k_sweep_write(double* A, int64_t n, int64_t k0, int b,
                                                     const double* V, const double* W) {
  __shared__ double t[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t i0 = (int64_t)blockIdx.x * 32;
  const int j0 = blockIdx.y * 32;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = i0 + r;
    const int j = j0 + tx;
    if (i < n && j < b) {
      const bool diag_blk = i >= k0 && i < k0 + b;
      const int64_t p = i - k0;
      const double v = diag_blk ? -0.5 * (W[p * b + j] + W[j * b + p]) : V[i * b + j];
      t[r][tx] = v;
      A[i * n + k0 + j] = v;
    }
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = i0 + tx;
    const int j = j0 + r;
    if (i < n && j < b && !(i >= k0 && i < k0 + b)) A[(k0 + j) * n + i] = t[tx][r];
  }
}

// The b x b blocks (b <= NB = 128) below are worked by 512 threads in registers: thread (ti, tj) holds
// the 8 x 4 elements of rows ti + 16 a and columns tj + 32 c. The elimination is a chain of b
// dependent steps, so what counts is the latency of one: LDS carries a step's pivot column (COL_LD
// doubles per ti: 16-byte aligned, on different banks) and row, the register indices are known at
// compile time, the next pivot column is updated and published before the rest, and reciprocals
// are two Newton steps on the hardware's estimate (full FP64 accuracy, a third of the latency of a
// division).
constexpr int COL_LD = 10;

__device__ __forceinline__ double recip(double d) {
  double x = __builtin_amdgcn_rcp(d);
  x = fma(x, fma(-d, x, 1.0), x);
  return fma(x, fma(-d, x, 1.0), x);
}
// 1 / sqrt(d) and sqrt(d)
__device__ __forceinline__ double recip_sqrt(double d, double* root) {
  double x = __builtin_amdgcn_rsq(d);
  x = fma(0.5 * x, fma(-d * x, x, 1.0), x);
  x = fma(0.5 * x, fma(-d * x, x, 1.0), x);
  const double r = d * x;
  *root = fma(fma(-r, r, d), 0.5 * x, r);
  return x;
}

template <int N>
__device__ __forceinline__ void read_pairs(double (&v)[N], const double* src) {
#pragma unroll
  for (int k = 0; k < N; k += 2) {
    const double2 q = *reinterpret_cast<const double2*>(src + k);
    v[k] = q.x;
    v[k + 1] = q.y;
  }
}

// Largest value over the 16 lanes of a DPP row, in every lane of it.
__device__ __forceinline__ unsigned row16_max(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));  // row_ror:8
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
  return v;
}

// In-place inverse of W by Gauss-Jordan with partial row pivoting. Step p eliminates column p with
// the row r of largest |W[r][p]| (to 13 bits of the mantissa) among the rows not used yet; no row
// is moved: row r of the eliminated matrix is row p of the inverse, and its column q is column
// r_q. Two barriers a step: the pivot column with the row its 16 owners chose, and the pivot row. A
// zero or non-finite pivot sets *bad.
// 128 x 128: 138 us (five barriers a step and exchanged rows took 560 us).
__global__ __launch_bounds__(512) void k_small_gj(double* W, int b, int* bad) {
  __shared__ __attribute__((aligned(16))) double colp[16 * COL_LD], rowp[NB];
  __shared__ int pivot;
  __shared__ int row_of[NB], step_of[NB];  // pivot row of a step, step of a row
  const int tid = threadIdx.x, ti = tid & 15, tj = tid >> 4;
  double w[8][4];
  unsigned used = 0;  // bit a: row ti + 16 a is not a candidate
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    if (ti + 16 * a >= b) used |= 1u << a;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti + 16 * a, j = tj + 32 * c;
      w[a][c] = i < b && j < b ? W[i * b + j] : 0.0;
    }
  }
  // the owners of a column (16 lanes, all rows) publish it and its pivot row
  auto publish_column = [&](auto cc) __attribute__((always_inline)) {
    constexpr int C = decltype(cc)::value;
    unsigned key = 0;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      colp[ti * COL_LD + a] = w[a][C];
      const unsigned hi = (unsigned)__double2hiint(w[a][C]) & 0x7fffff80u;
      key = max(key, (used >> a & 1) ? 0u : (0x80000000u | hi | (unsigned)(127 - (ti + 16 * a))));
    }
    key = row16_max(key);
    if (ti == 0) pivot = 127 - (int)(key & 127u);
  };
  if (tj == 0) publish_column(std::integral_constant<int, 0>{});
  auto columns = [&](auto cc) __attribute__((always_inline)) {
    constexpr int C = decltype(cc)::value, CN = C < 3 ? C + 1 : C;
    for (int s = 0; s < 32; ++s) {
      const int p = 32 * C + s;
      if (p >= b) break;
      __syncthreads();
      const int r = __builtin_amdgcn_readfirstlane(pivot), tr = r & 15;
      const double d = colp[tr * COL_LD + (r >> 4)];
      double ca[8];
      read_pairs<8>(ca, colp + ti * COL_LD);
      // the pivot row goes out and its elements become 0 - (-1) (row / d)
      auto publish_row = [&](auto ac) __attribute__((always_inline)) {
        constexpr int A = decltype(ac)::value;
        if (ti == tr) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            rowp[tj * 4 + k] = w[A][k];
            w[A][k] = 0.0;
          }
          ca[A] = -1.0;
          used |= 1u << A;
        }
        asm volatile("; rows 16 * %0" ::"n"(A));  // keeps the cases apart: merged, they index w at run time
      };
      switch (r >> 4) {
        case 0: publish_row(std::integral_constant<int, 0>{}); break;
        case 1: publish_row(std::integral_constant<int, 1>{}); break;
        case 2: publish_row(std::integral_constant<int, 2>{}); break;
        case 3: publish_row(std::integral_constant<int, 3>{}); break;
        case 4: publish_row(std::integral_constant<int, 4>{}); break;
        case 5: publish_row(std::integral_constant<int, 5>{}); break;
        case 6: publish_row(std::integral_constant<int, 6>{}); break;
        default: publish_row(std::integral_constant<int, 7>{}); break;
      }
      const double ip = recip(d);
      if (tid == 0) {
        row_of[p] = r;
        step_of[r] = p;
        if (!(fabs(d) > 0.0) || !isfinite(ip)) atomicOr(bad, 1);
      }
      __syncthreads();
      double rr[4];
      read_pairs<4>(rr, rowp + tj * 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) rr[k] *= ip;
      if (tj == s) {  // the pivot column: 0 - c_i / d
        rr[C] = ip;
#pragma unroll
        for (int a = 0; a < 8; ++a) w[a][C] = 0.0;
      }
      auto eliminate = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 8; ++a) w[a][k] = fma(-ca[a], rr[k], w[a][k]);
      };
      eliminate(C);
      if (CN != C) eliminate(CN);
      if (s < 31) {
        if (tj == s + 1) publish_column(std::integral_constant<int, C>{});
      } else if (CN != C) {
        if (tj == 0) publish_column(std::integral_constant<int, CN>{});
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k != C && k != CN) eliminate(k);
    }
  };
  columns(std::integral_constant<int, 0>{});
  columns(std::integral_constant<int, 1>{});
  columns(std::integral_constant<int, 2>{});
  columns(std::integral_constant<int, 3>{});
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti + 16 * a, j = tj + 32 * c;
      if (i < b && j < b) W[step_of[i] * b + row_of[j]] = w[a][c];
    }
}

// Probe vectors for inverse_residual: X[r][i] = +-1 from an integer hash of (r, i).
__global__ void k_probe(double* X, int64_t n, int rows) {
  const int64_t total = n * rows;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * 256) {
    uint64_t h = (uint64_t)e * 0x9E3779B97F4A7C15ull + 0x632BE59BD9B4E019ull;
    h ^= h >> 31;
    h *= 0xD6E8FEB86659FD93ull;
    h ^= h >> 32;
    X[e] = (h & 1) ? 1.0 : -1.0;
  }
}

// *out = max |Z| over `total` elements (one workgroup).
__global__ __launch_bounds__(1024) void k_maxabs(const double* Z, int64_t total, double* out) {
  __shared__ double m[1024];
  double v = 0.0;
  for (int64_t e = threadIdx.x; e < total; e += 1024) v = fmax(v, fabs(Z[e]));
  m[threadIdx.x] = v;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) m[threadIdx.x] = fmax(m[threadIdx.x], m[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = (isfinite(m[0]) ? m[0] : INFINITY);
}

// Cholesky factorization of the b x b diagonal block at (k0, k0) of A: writes L_KK to the same place
// of L (zero above the diagonal) and its inverse to Linv and to W (b x b, lower). Right looking, with the
// elimination of the unit matrix alongside (row j of x becomes row j of the inverse in step j); one
// barrier a step, the published column and row being double-buffered. Entries of a column above
// its diagonal are published as zeros, so finished rows and columns take no updates. A pivot that is
// not positive and finite sets *bad (the block is then garbage, never used).
// 128 x 128: 86 us (the factorization in LDS and a forward substitution through memory took 1104).
__global__ __launch_bounds__(512) void k_chol_block(const double* A, double* L, double* Linv, int64_t n,
                                                    int64_t k0, int b, double* W, int* bad) {
  __shared__ __attribute__((aligned(16))) double colp[2][16 * COL_LD], rowx[2][NB];
  const int tid = threadIdx.x, ti = tid & 15, tj = tid >> 4;
  double l[8][4], x[8][4];
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti + 16 * a, j = tj + 32 * c;
      l[a][c] = i < b && j < b ? A[(k0 + i) * n + k0 + j] : 0.0;
      x[a][c] = i == j ? 1.0 : 0.0;
    }
  // column j of the remaining matrix and row j of x, j = 16 O + s
  auto publish = [&](auto oc, int s, int buf) __attribute__((always_inline)) {
    constexpr int O = decltype(oc)::value;
    const int j = 16 * O + s;
    if (tj == (j & 31))
#pragma unroll
      for (int a = 0; a < 8; ++a) colp[buf][ti * COL_LD + a] = ti + 16 * a >= j ? l[a][O / 2] : 0.0;
    if (ti == s)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        rowx[buf][tj * 4 + c] = x[O][c];
        x[O][c] = 0.0;
      }
  };
  publish(std::integral_constant<int, 0>{}, 0, 0);
  auto steps = [&](auto oc) __attribute__((always_inline)) {
    constexpr int O = decltype(oc)::value, C = O / 2, ON = O < 7 ? O + 1 : O;
    for (int s = 0; s < 16; ++s) {
      const int j = 16 * O + s, buf = s & 1;
      if (j >= b) break;
      __syncthreads();
      double ca[8], cb[4], xr[4];
      double d = colp[buf][s * COL_LD + O];
      read_pairs<8>(ca, colp[buf] + ti * COL_LD);
#pragma unroll
      for (int c = 0; c < 4; ++c) cb[c] = colp[buf][(tj & 15) * COL_LD + (tj >> 4) + 2 * c];
      read_pairs<4>(xr, rowx[buf] + tj * 4);
      if (!(d > 0.0) || !isfinite(d)) {
        if (tid == 0) atomicOr(bad, 1);
        d = 1.0;
      }
      double p;
      const double ip = recip_sqrt(d, &p);
#pragma unroll
      for (int k = 0; k < 8; ++k) ca[k] *= ip;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        cb[k] *= ip;
        xr[k] *= ip;
      }
      const double co = ti == s ? -1.0 : ca[O];  // row j of x: 0 - (-1) (row / p)
      auto update_l = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int a = O; a < 8; ++a) l[a][c] = fma(-ca[a], cb[c], l[a][c]);
      };
      auto update_x = [&](int a) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c <= C; ++c) x[a][c] = fma(a == O ? -co : -ca[a], xr[c], x[a][c]);
      };
      // what step j + 1 needs first
      update_l(C);
      if (ON / 2 != C) update_l(ON / 2);
      update_x(O);
      if (ON != O) update_x(ON);
      if (tj == (j & 31))  // column j of L
#pragma unroll
        for (int a = 0; a < 8; ++a) l[a][C] = ti + 16 * a == j ? p : ca[a];
      if (s < 15) publish(std::integral_constant<int, O>{}, s + 1, buf ^ 1);
      else if (ON != O) publish(std::integral_constant<int, ON>{}, 0, buf ^ 1);
#pragma unroll
      for (int c = C + 1; c < 4; ++c)
        if (c != ON / 2) update_l(c);
#pragma unroll
      for (int a = O + 2; a < 8; ++a) update_x(a);
    }
  };
  steps(std::integral_constant<int, 0>{});
  steps(std::integral_constant<int, 1>{});
  steps(std::integral_constant<int, 2>{});
  steps(std::integral_constant<int, 3>{});
  steps(std::integral_constant<int, 4>{});
  steps(std::integral_constant<int, 5>{});
  steps(std::integral_constant<int, 6>{});
  steps(std::integral_constant<int, 7>{});
#pragma unroll
  for (int a = 0; a < 8; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti + 16 * a, j = tj + 32 * c;
      if (i < b && j < b) {
        L[(k0 + i) * n + k0 + j] = j <= i ? l[a][c] : 0.0;
        W[i * b + j] = Linv[(k0 + i) * n + k0 + j] = j <= i ? x[a][c] : 0.0;
      }
    }
}

__global__ void k_zero(double* A, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256)
    A[e] = 0.0;
}

__global__ void k_nonfinite(const double* A, int64_t n, int* bad) {
  int f = 0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256)
    if (!isfinite(A[e])) f = 1;
  if (f) atomicOr(bad, 1);
}

// A = -A, with the check of k_nonfinite
__global__ void k_negate(double* A, int64_t n, int* bad) {
  int f = 0;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
    const double v = A[e];
    if (!isfinite(v)) f = 1;
    A[e] = -v;
  }
  if (f) atomicOr(bad, 1);
}

dim3 ew_grid(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return dim3((unsigned)(b < 1 ? 1 : b > 8192 ? 8192 : b));
}

// C = alpha A B + beta X (X nullable) in FP64, small tiles.
hipError_t product(int M, int N, int K, const double* A, int64_t lda, int la, const double* B, int64_t ldb,
                   int lb, double* C, int64_t ldc, double alpha, const double* X, double beta, int tri,
                   int kcut, hipStream_t s) {
  GemmDesc d{CF64, T_F64, T_F64, T_F64, T_F64, la, lb, 0, 1};
  GemmOp op{};
  op.M = M; op.N = N; op.nseg = 1;
  op.A[0] = A; op.lda[0] = lda;
  op.B[0] = B; op.ldb[0] = ldb;
  op.K[0] = K;
  op.C = C; op.ldc = ldc;
  op.X = X; op.ldx = X ? ldc : 0;
  op.alpha = alpha; op.beta = beta;
  op.tri = tri;
  op.kcut = kcut;
  direct_choose(d, &op, 1);
  return gemm_launch(d, &op, 1, nullptr, nullptr, 0, s);
}

hipError_t read_flag(const int* flag, hipStream_t s, int* out) {
  const hipError_t e = hipMemcpyAsync(out, flag, sizeof(int), hipMemcpyDeviceToHost, s);
  return e != hipSuccess ? e : hipStreamSynchronize(s);
}

}  // namespace

#define TRYHIP(x)                          \
  do {                                     \
    const hipError_t e_ = (x);             \
    if (e_ != hipSuccess) return e_;       \
  } while (0)

size_t invert_work_doubles(int64_t n) {
  // U, V (n x NB), W (NB x NB), flag word
  return (size_t)n * NB * 2 + (size_t)NB * NB + 8;
}

hipError_t invert_symmetric(double* A, int64_t n, double* work, hipStream_t s, int* bad_host) {
  double* U = work;
  double* V = U + (size_t)n * NB;
  double* W = V + (size_t)n * NB;
  int* flag = reinterpret_cast<int*>(W + (size_t)NB * NB);
  const int N = (int)n;
  TRYHIP(hipMemsetAsync(flag, 0, sizeof(int), s));
  for (int64_t k0 = 0; k0 < n; k0 += NB) {
    const int b = (int)((n - k0) < NB ? (n - k0) : NB);
    hipLaunchKernelGGL(k_panel, ew_grid(n * b), dim3(256), 0, s, A, n, k0, b, U, W);
    hipLaunchKernelGGL(k_small_gj, dim3(1), dim3(512), 0, s, W, b, flag);
    TRYHIP(hipGetLastError());
    if (n > b) {
      TRYHIP(product(N, b, b, U, b, KC, W, b, RC, V, b, 1.0, nullptr, 0.0, 0, 0, s));    // V = U W
      TRYHIP(product(N, N, b, V, b, KC, U, b, KC, A, n, -1.0, A, 1.0, 1, 0, s));  // A -= V U^T
    }
    hipLaunchKernelGGL(k_sweep_write, dim3((unsigned)((n + 31) / 32), (b + 31) / 32), dim3(256), 0, s, A,
                       n, k0, b, V, W);
    TRYHIP(hipGetLastError());
  }
  hipLaunchKernelGGL(k_negate, ew_grid(n * n), dim3(256), 0, s, A, n * n, flag);
  TRYHIP(hipGetLastError());
  return read_flag(flag, s, bad_host);
}

size_t inverse_residual_work_doubles(int64_t n) { return (size_t)3 * PROBES * n + 8; }

// max_ij |(X P A)_ij - X_ij| for PROBES rows X of +-1 entries, with A = S + (1/tau) T (T null:
// A = S): X P A = X exactly when P = A^-1, and the residual of a backward-stable inverse is
// ~ eps times the growth of the elimination. P, S, T are symmetric, so every product reads
// its operator k-contiguous.
hipError_t inverse_residual(const double* P, const double* S, const double* T, double inv_tau,
                            int64_t n, double* work, hipStream_t s, double* res_host) {
  double* X = work;
  double* Y = X + (size_t)PROBES * n;
  double* Z = Y + (size_t)PROBES * n;
  double* out = Z + (size_t)PROBES * n;
  const int64_t total = (int64_t)PROBES * n;
  int blocks = (int)((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_probe, dim3(blocks), dim3(256), 0, s, X, n, PROBES);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int N = (int)n;
  auto mul = [&](const double* A, const double* B, double* C, const double* Xa, double alpha, double beta) {
    return product(PROBES, N, N, A, n, KC, B, n, KC, C, n, alpha, Xa, beta, 0, 0, s);
  };
  TRYHIP(mul(X, P, Y, nullptr, 1.0, 0.0));       // Y = X P
  TRYHIP(mul(Y, S, Z, X, 1.0, -1.0));            // Z = Y S - X
  if (T) TRYHIP(mul(Y, T, Z, Z, inv_tau, 1.0));  // Z += (1/tau) Y T
  hipLaunchKernelGGL(k_maxabs, dim3(1), dim3(1024), 0, s, Z, total, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(res_host, out, sizeof(double), hipMemcpyDeviceToHost, s)) != hipSuccess)
    return e;
  return hipStreamSynchronize(s);
}

size_t cholesky_work_doubles(int64_t n) { return (size_t)n * NB + (size_t)NB * NB + 8; }

// S = L L^T and L^-1, both lower with zeros above (n x n, row-major), from A = S, which is overwritten.
// For each block column K (width b <= 128): factor A_KK and invert its triangle in one workgroup
// (W = L_KK^-1), L_IK = A_IK W^T for the rows below, A_II -= L_IK L_IK^T on the trailing square
// (upper half, mirrored), and row block K of the inverse from those above it,
// L^-1_K = -W (L_K,<K L^-1_<K), whose inner product skips the zeros of L^-1.
hipError_t cholesky_and_inverse(double* A, double* L, double* Linv, int64_t n, double* work, hipStream_t s,
                                int* bad_host) {
  double* T = work;  // b x k0
  double* W = T + (size_t)n * NB;
  int* flag = reinterpret_cast<int*>(W + (size_t)NB * NB);
  TRYHIP(hipMemsetAsync(flag, 0, sizeof(int), s));
  hipLaunchKernelGGL(k_zero, ew_grid(n * n), dim3(256), 0, s, L, n * n);
  hipLaunchKernelGGL(k_zero, ew_grid(n * n), dim3(256), 0, s, Linv, n * n);
  for (int64_t k0 = 0; k0 < n; k0 += NB) {
    const int b = (int)((n - k0) < NB ? (n - k0) : NB);
    hipLaunchKernelGGL(k_chol_block, dim3(1), dim3(512), 0, s, A, L, Linv, n, k0, b, W, flag);
    TRYHIP(hipGetLastError());
    if (k0 > 0) {
      const int K = (int)k0;
      TRYHIP(product(b, K, K, L + k0 * n, n, KC, Linv, n, RC, T, K, 1.0, nullptr, 0.0, 0, KCUT_B_FROM_N, s));
      TRYHIP(product(b, K, b, W, b, KC, T, K, RC, Linv + k0 * n, n, -1.0, nullptr, 0.0, 0, 0, s));
    }
    const int64_t r0 = k0 + b;
    const int R = (int)(n - r0);
    if (R <= 0) break;
    double* LI = L + r0 * n + k0;
    double* AI = A + r0 * n + r0;
    TRYHIP(product(R, b, b, A + r0 * n + k0, n, KC, W, b, KC, LI, n, 1.0, nullptr, 0.0, 0, 0, s));
    TRYHIP(product(R, R, b, LI, n, KC, LI, n, KC, AI, n, -1.0, AI, 1.0, 1, 0, s));
  }
  hipLaunchKernelGGL(k_nonfinite, ew_grid(n * n), dim3(256), 0, s, L, n * n, flag);
  hipLaunchKernelGGL(k_nonfinite, ew_grid(n * n), dim3(256), 0, s, Linv, n * n, flag);
  TRYHIP(hipGetLastError());
  return read_flag(flag, s, bad_host);
}

}  // namespace omm
