// Memory-bound stages of one CG line search (Sec. 2.3 of the paper): FP64 reductions for the
// Polak-Ribiere coefficient and the quartic coefficients (Eq. 13), the device-side line
// minimum, and the updates of Eq. 16. All reductions are two-pass with a fixed grid, so a rerun
// is bitwise identical. The scalar state of a minimization lives in device memory (DevState);
// no stage needs the host.
#include <math.h>

#include <algorithm>

#include "omm_internal.h"

namespace omm {
namespace {

constexpr int NT = 256;
// block-reduction scratch: up to NCOEF values at once (block_sums), one slot per wave each
constexpr int SH_SUMS = NCOEF * (NT / 64);

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// Sum over the wave (fixed order), in every lane: rotations within the rows of 16 lanes, then the four
// row sums. Register moves only (a shuffle down goes through LDS twice per step).
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0x121>(v);
  v = dpp_add<0x122>(v);
  v = dpp_add<0x124>(v);
  v = dpp_add<0x128>(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Sum of `v` over the block (FP64, fixed order). Result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) t += sh[i];
  return t;
}

// block_sum of W values at once (each in block_sum's order: the same results), with one pair of
// barriers instead of W; sh holds W * NT / 64 doubles. Results valid in thread 0.
template <int W>
__device__ __forceinline__ void block_sums(double (&v)[W], double* sh) {
#pragma unroll
  for (int k = 0; k < W; ++k) v[k] = wave_sum(v[k]);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < W; ++k) sh[k * (NT / 64) + w] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < W; ++k) {
      double t = 0.0;
      for (int i = 0; i < NT / 64; ++i) t += sh[k * (NT / 64) + i];
      v[k] = t;
    }
}

// Fixed-order sum over nb partial rows (stride w) of column c, by the whole block; result in
// thread 0. Each thread sums a strided subset in index order, then block_sum combines them.
__device__ __forceinline__ double sum_partials(const double* partials, int nb, int w, int c,
                                               double* sh) {
  double v = 0.0;
  for (int b = threadIdx.x; b < nb; b += NT) v += partials[b * w + c];
  return block_sum(v, sh);
}

// sum_partials of columns 0..W-1 of rows of width W, in the same per-column order, with the
// loads of all columns in flight together.
template <int W>
__device__ __forceinline__ void sum_partials_all(const double* partials, int nb, double* sh,
                                                 double (&out)[W]) {
  double v[W];
#pragma unroll
  for (int k = 0; k < W; ++k) v[k] = 0.0;
  for (int b = threadIdx.x; b < nb; b += NT)
#pragma unroll
    for (int k = 0; k < W; ++k) v[k] += partials[b * W + k];
  block_sums<W>(v, sh);
#pragma unroll
  for (int k = 0; k < W; ++k) out[k] = v[k];
}

int red_blocks(int64_t n) {
  int64_t b = (n + NT - 1) / NT;
  if (b > RED_BLOCKS) b = RED_BLOCKS;
  if (b < 1) b = 1;
  return (int)b;
}

__global__ void k_shift(const double* H, const double* S, double eta, double* Hs, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT)
    Hs[i] = H[i] - eta * S[i];
}

template <typename A, typename B>
__global__ void k_convert(const A* src, B* dst, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT)
    dst[i] = (B)src[i];
}

__device__ __forceinline__ unsigned short bf16_bits(float f) {
  unsigned int u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

// hi/lo bf16 planes of src (rows x cols, contiguous) into rows of length ld >= cols (ld a
// multiple of 4): rows blockIdx.y, blockIdx.y + gridDim.y, .., 4 elements per thread (8-byte
// stores).
template <typename T>
__global__ void k_split(const T* src, unsigned short* hi, unsigned short* lo, int64_t rows,
                        int64_t cols, int64_t ld, const DevState* st) {
  if (st && st->done) return;
  typedef unsigned short us4 __attribute__((ext_vector_type(4)));
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
    const T* srow = src + r * cols;
    for (int64_t c4 = ((int64_t)blockIdx.x * NT + threadIdx.x) * 4; c4 < cols;
         c4 += (int64_t)gridDim.x * NT * 4) {
      if (c4 + 4 <= cols) {
        us4 h, l;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double v = (double)srow[c4 + u];
          const unsigned short hb = bf16_bits((float)v);
          h[u] = hb;
          l[u] = bf16_bits((float)(v - (double)__uint_as_float(((unsigned int)hb) << 16)));
        }
        *reinterpret_cast<us4*>(hi + r * ld + c4) = h;
        *reinterpret_cast<us4*>(lo + r * ld + c4) = l;
      } else {
        for (int64_t c = c4; c < cols; ++c) {
          const double v = (double)srow[c];
          const unsigned short hb = bf16_bits((float)v);
          hi[r * ld + c] = hb;
          lo[r * ld + c] = bf16_bits((float)(v - (double)__uint_as_float(((unsigned int)hb) << 16)));
        }
      }
    }
  }
}

// Transposing split through a 32 x 33 LDS tile: dst (cols x rows, row length ld) = planes of
// src^T.
template <typename T>
__global__ void k_split_t(const T* src, unsigned short* hi, unsigned short* lo, int rows, int cols,
                          int64_t ld, const DevState* st) {
  if (st && st->done) return;
  __shared__ T t[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int gr = r0 + r, gc = c0 + tx;
    t[r][tx] = (gr < rows && gc < cols) ? src[(int64_t)gr * cols + gc] : (T)0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int oc = c0 + r, orow = r0 + tx;  // output row oc (a source column), column orow
    if (oc < cols && orow < rows) {
      const double v = (double)t[tx][r];
      const unsigned short hb = bf16_bits((float)v);
      const int64_t o = (int64_t)oc * ld + orow;
      hi[o] = hb;
      lo[o] = bf16_bits((float)(v - (double)__uint_as_float(((unsigned int)hb) << 16)));
    }
  }
}

int ew_blocks(int64_t n) {
  int64_t b = (n + NT - 1) / NT;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return (int)b;
}

// flags[0] |= non-finite entry, flags[1] |= |a_ij - a_ji| > rtol * max(1, |a_ij|, |a_ji|).
__global__ void k_validate(const double* A, int64_t n, double rtol, int* flags) {
  __shared__ double t[32][33];
  const int64_t bi = (int64_t)blockIdx.y * 32, bj = (int64_t)blockIdx.x * 32;
  if (bj < bi) return;  // upper block triangle (incl. diagonal blocks) covers every pair
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bj + r, j = bi + tx;  // transposed tile (bj, bi)
    t[r][tx] = (i < n && j < n) ? A[i * n + j] : 0.0;
  }
  __syncthreads();
  int bad_f = 0, bad_s = 0;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi + r, j = bj + tx;
    if (i < n && j < n) {
      const double a = A[i * n + j], b = t[tx][r];
      if (!isfinite(a)) bad_f = 1;
      const double m = fmax(1.0, fmax(fabs(a), fabs(b)));
      if (!(fabs(a - b) <= rtol * m)) bad_s = 1;
    }
  }
  if (bad_f) atomicOr(&flags[0], 1);
  if (bad_s) atomicOr(&flags[1], 1);
}

// Up to three symmetric inputs (blockIdx.z) on their way into a context: the checks of k_validate
// (flags[2 z] non-finite, flags[2 z + 1] asymmetric) and, for those with a stored copy, flags[6] = 1 when
// the symmetrized input differs from it bit for bit. Reads each input once and the upper half of
// each stored copy (exactly symmetric); writes nothing.
__global__ __launch_bounds__(NT) void k_check_inputs(SymInputs in, int64_t n, double rtol, int* flags) {
  __shared__ double t[32][33];
  const int64_t bi = (int64_t)blockIdx.y * 32, bj = (int64_t)blockIdx.x * 32;
  const double* A = in.src[blockIdx.z];
  const double* P = in.compare[blockIdx.z];
  if (bj < bi || !A) return;  // the upper block triangle (incl. diagonal blocks) covers every pair
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bj + r, j = bi + tx;
    t[r][tx] = (i < n && j < n) ? A[i * n + j] : 0.0;
  }
  __syncthreads();
  bool bad_f = false, bad_s = false, changed = false;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi + r, j = bj + tx;
    if (i >= n || j >= n) continue;
    const double a = A[i * n + j], b = t[tx][r];
    bad_f |= !isfinite(a) || !isfinite(b);
    bad_s |= !(fabs(a - b) <= rtol * fmax(1.0, fmax(fabs(a), fabs(b))));
    if (P && j >= i)
      changed |= __double_as_longlong(0.5 * (a + b)) != __double_as_longlong(P[i * n + j]);
  }
  // One relaxed store a wave (an atomic from every wave would queue on the address). The stores queue
  // too where S and T have changed and nearly every wave raises flags[6]: 50 us at 717 orbitals and 394 at
  // 2301, whose bytes take about 4 and 40; unchanged, 40 us at 2048 and 130 at 4096.
  auto raise = [&](bool c, int* f) {
    if (__any(c) && (threadIdx.x & 63) == 0)
      __hip_atomic_store(f, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  raise(bad_f, flags + 2 * blockIdx.z);
  raise(bad_s, flags + 2 * blockIdx.z + 1);
  raise(changed, flags + 6);
}

// dst = (src + src^T) / 2 of up to three inputs (blockIdx.z), each pair of elements from one load.
__global__ __launch_bounds__(NT) void k_store_inputs(SymInputs in, int64_t n) {
  __shared__ double t[32][33], u[32][33];
  const int64_t bi = (int64_t)blockIdx.y * 32, bj = (int64_t)blockIdx.x * 32;
  const double* A = in.src[blockIdx.z];
  double* D = in.dst[blockIdx.z];
  if (bj < bi || !A) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bj + r, j = bi + tx;
    t[r][tx] = (i < n && j < n) ? A[i * n + j] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi + r, j = bj + tx;
    if (i >= n || j >= n) continue;
    const double v = 0.5 * (A[i * n + j] + t[tx][r]);
    D[i * n + j] = v;
    u[r][tx] = v;
  }
  if (bi == bj) return;  // a diagonal block holds both halves
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bj + r, j = bi + tx;
    if (i < n && j < n) D[i * n + j] = u[tx][r];
  }
}

// A <- (A + A^T) / 2; one thread per unordered pair.
__global__ void k_symmetrize(double* A, int64_t n) {
  __shared__ double t[32][33];
  const int64_t bi = (int64_t)blockIdx.y * 32, bj = (int64_t)blockIdx.x * 32;
  if (bj < bi) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  // load transposed tile (bj, bi) and this tile (bi, bj); write both halves
  __shared__ double u[32][33];
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bj + r, j = bi + tx;
    t[r][tx] = (i < n && j < n) ? A[i * n + j] : 0.0;
    const int64_t i2 = bi + r, j2 = bj + tx;
    u[r][tx] = (i2 < n && j2 < n) ? A[i2 * n + j2] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = bi + r, j = bj + tx;
    if (i < n && j < n) {
      if (bi == bj && j < i) continue;  // diagonal block: each pair once (j >= i)
      const double v = 0.5 * (u[r][tx] + t[tx][r]);
      A[i * n + j] = v;
      A[j * n + i] = v;
    }
  }
}

// ---- energy of (HW, SW): Eq. 8 -----------------------------------------------------------------
__device__ __forceinline__ void b_energy_partials(const double* HW, const double* SW, int M, double* partials, int bid, int nb) {
  __shared__ double sh[SH_SUMS];
  const int64_t n = (int64_t)M * M;
  double tr = 0.0, f = 0.0, trs = 0.0;
  for (int64_t i = (int64_t)bid * NT + threadIdx.x; i < n; i += (int64_t)nb * NT) {
    const int r = (int)(i / M), c = (int)(i % M);
    const double h = HW[i], s = SW[i];
    f += s * h;
    if (r == c) { tr += h; trs += s; }
  }
  double v3[3] = {tr, f, trs};
  block_sums<3>(v3, sh);
  const double a = v3[0], b = v3[1], c = v3[2];
  if (threadIdx.x == 0) {
    partials[bid * 3 + 0] = a;
    partials[bid * 3 + 1] = b;
    partials[bid * 3 + 2] = c;
  }
}

__global__ void k_energy_partials(const double* HW, const double* SW, int M, double* partials) {
  b_energy_partials(HW, SW, M, partials, blockIdx.x, gridDim.x);
}

__device__ __forceinline__ void f_energy_init_final(const double* partials, int nb, DevState* st, double* trace) {
  __shared__ double sh[SH_SUMS];
  const double tr = sum_partials(partials, nb, 3, 0, sh);
  const double f = sum_partials(partials, nb, 3, 1, sh);
  if (threadIdx.x != 0) return;
  const double E = 4.0 * tr - 2.0 * f;
  st->E = E;
  st->E_prev = E;
  if (trace) trace[0] = E;
  if (!isfinite(E)) st->done = -5;
}

__global__ void k_energy_init_final(const double* partials, int nb, DevState* st, double* trace) {
  f_energy_init_final(partials, nb, st, trace);
}

// ---- Polak-Ribiere coefficient and direction ----------------------------------------------------
template <typename T, typename TP = T>
__device__ __forceinline__ void b_pr_partials(const T* G, const TP* PG, const T* Gp, int64_t n, int first,
                              double* partials, const DevState* st, int bid, int nb) {
  if (st->done) return;
  __shared__ double sh[SH_SUMS];
  double s1 = 0.0, s2 = 0.0;
  for (int64_t i = (int64_t)bid * NT + threadIdx.x; i < n; i += (int64_t)nb * NT) {
    const double pg = (double)PG[i];
    s1 += pg * (double)G[i];
    if (!first) s2 += pg * (double)Gp[i];
  }
  double v2[2] = {s1, s2};
  block_sums<2>(v2, sh);
  const double a = v2[0], b = v2[1];
  if (threadIdx.x == 0) {
    partials[bid * 2 + 0] = a;
    partials[bid * 2 + 1] = b;
  }
}

template <typename T, typename TP>
__global__ void k_pr_partials(const T* G, const TP* PG, const T* Gp, int64_t n, int first,
                              double* partials, const DevState* st) {
  b_pr_partials(G, PG, Gp, n, first, partials, st, blockIdx.x, gridDim.x);
}

// The same sums four elements per load (arrays 4-element aligned; the tail past the last full
// group of four is added by block 0), two groups in flight per thread.
template <typename TG, typename TP>
__global__ void k_pr_partials4(const TG* G, const TP* PG, const TG* Gp, int64_t n, int first,
                               double* partials, const DevState* st) {
  if (st->done) return;
  typedef TG G4 __attribute__((ext_vector_type(4)));
  typedef TP P4 __attribute__((ext_vector_type(4)));
  __shared__ double sh[SH_SUMS];
  const int64_t n4 = n / 4, stride = (int64_t)gridDim.x * NT;
  const G4* g4 = reinterpret_cast<const G4*>(G);
  const G4* q4 = reinterpret_cast<const G4*>(Gp);
  const P4* p4 = reinterpret_cast<const P4*>(PG);
  double s1 = 0.0, s2 = 0.0;
  int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
  for (; i + stride < n4; i += 2 * stride) {
    const P4 pa = p4[i], pb = p4[i + stride];
    const G4 ga = g4[i], gb = g4[i + stride];
    s1 += (double)pa.x * ga.x + (double)pa.y * ga.y + (double)pa.z * ga.z + (double)pa.w * ga.w;
    s1 += (double)pb.x * gb.x + (double)pb.y * gb.y + (double)pb.z * gb.z + (double)pb.w * gb.w;
    if (!first) {
      const G4 qa = q4[i], qb = q4[i + stride];
      s2 += (double)pa.x * qa.x + (double)pa.y * qa.y + (double)pa.z * qa.z + (double)pa.w * qa.w;
      s2 += (double)pb.x * qb.x + (double)pb.y * qb.y + (double)pb.z * qb.z + (double)pb.w * qb.w;
    }
  }
  if (i < n4) {
    const P4 pa = p4[i];
    const G4 ga = g4[i];
    s1 += (double)pa.x * ga.x + (double)pa.y * ga.y + (double)pa.z * ga.z + (double)pa.w * ga.w;
    if (!first) {
      const G4 qa = q4[i];
      s2 += (double)pa.x * qa.x + (double)pa.y * qa.y + (double)pa.z * qa.z + (double)pa.w * qa.w;
    }
  }
  if (blockIdx.x == 0)
    for (int64_t j = 4 * n4 + threadIdx.x; j < n; j += NT) {
      s1 += (double)PG[j] * (double)G[j];
      if (!first) s2 += (double)PG[j] * (double)Gp[j];
    }
  double v2[2] = {s1, s2};
  block_sums<2>(v2, sh);
  const double a = v2[0], b = v2[1];
  if (threadIdx.x == 0) {
    partials[blockIdx.x * 2 + 0] = a;
    partials[blockIdx.x * 2 + 1] = b;
  }
}

// Polak-Ribiere beta from the partial sums, in every thread (each block sums them itself, in the same
// order: a launch of its own for this took 4.5 us of every line search). One block (`writer`) keeps it
// in the state, with <PG, G>, whose two slots alternate so that no block reads what another
// writes.
__device__ __forceinline__ double beta_of(const double* partials, int nb, int first, int parity,
                                          DevState* st, bool writer) {
  __shared__ double sh[SH_SUMS];
  __shared__ double shared_beta;
  double v[2];
  sum_partials_all<2>(partials, nb, sh, v);
  if (threadIdx.x == 0) {
    double beta = 0.0;
    if (!first) {
      beta = (v[0] - v[1]) / st->pg_g[parity ^ 1];
      if (!isfinite(beta)) beta = 0.0;
    }
    shared_beta = beta;
    if (writer) {
      st->beta = beta;
      st->pg_g[parity] = v[0];
    }
  }
  __syncthreads();
  return shared_beta;
}

template <typename T, typename TP = T>
__device__ __forceinline__ void b_direction(const TP* PG, T* D, int64_t n, int first, double beta, int bid, int nb) {
  for (int64_t i = (int64_t)bid * NT + threadIdx.x; i < n; i += (int64_t)nb * NT) {
    const double d = first ? -(double)PG[i] : -(double)PG[i] + beta * (double)D[i];
    D[i] = (T)d;
  }
}

// One block per (K block, column tile): does the SPARSE_BN x SPARSE_BK sub-matrix hold a
// non-zero?
__global__ void k_block_pattern(const double* B, int64_t n, unsigned char* flags) {
  const int kb = blockIdx.x, t = blockIdx.y;
  const int nkb = gridDim.x;
  int nz = 0;
  for (int e = threadIdx.x; e < SPARSE_BN * SPARSE_BK; e += NT) {
    const int64_t r = (int64_t)t * SPARSE_BN + e / SPARSE_BK;
    const int64_t k = (int64_t)kb * SPARSE_BK + e % SPARSE_BK;
    if (r < n && k < n && B[r * n + k] != 0.0) nz = 1;
  }
  nz = __syncthreads_or(nz);
  if (threadIdx.x == 0) flags[(int64_t)t * nkb + kb] = (unsigned char)nz;
}

template <typename T, typename TP>
__global__ __launch_bounds__(NT) void k_direction(const TP* PG, T* D, int64_t n, int first, int parity,
                                                 const double* partials, int np, DevState* st) {
  if (st->done) return;
  const double beta = beta_of(partials, np, first, parity, st, blockIdx.x == 0);
  b_direction(PG, D, n, first, beta, blockIdx.x, gridDim.x);
}

// The same direction rounded to bf16: D keeps the rounded values (exact in T) and `hi` their bf16
// bits (rows of length ld), so the products with D need no lo plane and the CG update moves along
// exactly this D. One row of D (rows x cols) per blockIdx.y.
template <typename T, typename TP>
__global__ __launch_bounds__(NT) void k_direction_bf16(const TP* PG, T* D, unsigned short* hi, int64_t rows,
                                                      int64_t cols, int64_t ld, int first, int parity,
                                                      const double* partials, int np, DevState* st) {
  if (st->done) return;
  const double beta = beta_of(partials, np, first, parity, st, blockIdx.x == 0 && blockIdx.y == 0);
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y)
    for (int64_t c = (int64_t)blockIdx.x * NT + threadIdx.x; c < cols;
         c += (int64_t)gridDim.x * NT) {
      const int64_t i = r * cols + c, q = r * ld + c;
      // the previous direction is exact in bf16: read back from its plane
      const double d =
          first ? -(double)PG[i]
                : -(double)PG[i] + beta * (double)__uint_as_float(((unsigned int)hi[q]) << 16);
      const unsigned short hb = bf16_bits((float)d);
      hi[q] = hb;
      if (D) D[i] = (T)__uint_as_float(((unsigned int)hb) << 16);
    }
}

// The same, four columns per thread (cols and ld multiples of 4, aligned rows) and four rows per
// block, all loads of a block's rows issued before its stores.
template <typename T, typename TP>
__global__ __launch_bounds__(NT) void k_direction_bf16x4(const TP* PG, T* D, unsigned short* hi,
                                                        int64_t rows, int64_t cols, int64_t ld,
                                                        int first, int parity, const double* partials,
                                                        int np, DevState* st) {
  if (st->done) return;
  typedef TP P4 __attribute__((ext_vector_type(4)));
  typedef unsigned short U4 __attribute__((ext_vector_type(4)));
  constexpr int RB = 4;
  const double beta = beta_of(partials, np, first, parity, st, blockIdx.x == 0 && blockIdx.y == 0);
  const int64_t c = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (4 * c >= cols) return;
  for (int64_t r0 = (int64_t)blockIdx.y * RB; r0 < rows; r0 += (int64_t)gridDim.y * RB) {
    P4 pg[RB];
    U4 hv[RB];
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int64_t r = r0 + k;
      if (r < rows) {
        pg[k] = *reinterpret_cast<const P4*>(PG + r * cols + 4 * c);
        if (!first) hv[k] = *reinterpret_cast<const U4*>(hi + r * ld + 4 * c);
      }
    }
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int64_t r = r0 + k;
      if (r >= rows) continue;
      U4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double prev = first ? 0.0 : (double)__uint_as_float(((unsigned int)hv[k][e]) << 16);
        const double d = first ? -(double)pg[k][e] : -(double)pg[k][e] + beta * prev;
        h[e] = bf16_bits((float)d);
      }
      *reinterpret_cast<U4*>(hi + r * ld + 4 * c) = h;
      if (D)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          D[r * cols + 4 * c + e] = (T)__uint_as_float(((unsigned int)h[e]) << 16);
    }
  }
}

// ---- quartic coefficients (Eq. 13) --------------------------------------------------------------
// Sums (index order used by the finalizer):
//  0 Tr HW   1 Tr H'   2 Tr H''
//  3 <SW,HW> 4 <S',HW> 5 <SW,H'> 6 <S'',HW> 7 <SW,H''> 8 sum S'_ij H'_ji 9 <S',H'>
//  10 <S'',H'> 11 <S',H''> 12 <S'',H''>
// With HW, SW, H'', S'' symmetric, Tr{A B} = <A, B> whenever A or B is symmetric; only
// Tr{S' H'} needs the transposed access.
__device__ __forceinline__ void b_coef_partials(const double* HW, const double* SW, const double* H1,
                                const double* S1, const double* H2, const double* S2, int M,
                                double* partials, const DevState* st, int bid, int nb) {
  if (st->done) return;
  __shared__ double t[32][33];
  __shared__ double sh[SH_SUMS];
  double acc[NCOEF];
#pragma unroll
  for (int k = 0; k < NCOEF; ++k) acc[k] = 0.0;
  const int tb = (M + 31) / 32;
  const int ntiles = tb * tb;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int tile = bid; tile < ntiles; tile += nb) {
    const int bi = (tile / tb) * 32, bj = (tile % tb) * 32;
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = bj + r, j = bi + tx;
      t[r][tx] = (i < M && j < M) ? H1[(int64_t)i * M + j] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = bi + r, j = bj + tx;
      if (i < M && j < M) {
        const int64_t e = (int64_t)i * M + j;
        const double hw = HW[e], sw = SW[e], h1 = H1[e], s1 = S1[e], h2 = H2[e], s2 = S2[e];
        const double h1t = t[tx][r];  // H'_ji
        if (i == j) { acc[0] += hw; acc[1] += h1; acc[2] += h2; }
        acc[3] += sw * hw;
        acc[4] += s1 * hw;
        acc[5] += sw * h1;
        acc[6] += s2 * hw;
        acc[7] += sw * h2;
        acc[8] += s1 * h1t;
        acc[9] += s1 * h1;
        acc[10] += s2 * h1;
        acc[11] += s1 * h2;
        acc[12] += s2 * h2;
      }
    }
  }
  block_sums<NCOEF>(acc, sh);
  if (threadIdx.x == 0)
    for (int k = 0; k < NCOEF; ++k) partials[bid * NCOEF + k] = acc[k];
}

// Pair p of the tile pairs (bi <= bj) of a T x T tiling.
__device__ __forceinline__ void tile_pair(int p, int T, int& bi, int& bj) {
  bi = 0;
  while (p >= T - bi) {
    p -= T - bi;
    ++bi;
  }
  bj = bi + p;
}

// The same sums for one system over pairs of 32 x 32 tiles: HW, SW, H'' and S'' are symmetric and only
// their upper halves are read, H' and S' wholly, the mirror tile through LDS.
__global__ __launch_bounds__(NT) void k_coef_sym(Subspace m, double* partials, const DevState* st) {
  if (st->done) return;
  __shared__ double th[32][33], ts[32][33];
  __shared__ double sh[SH_SUMS];
  double acc[NCOEF];
#pragma unroll
  for (int k = 0; k < NCOEF; ++k) acc[k] = 0.0;
  const int M = m.M, T = (M + 31) / 32, npairs = T * (T + 1) / 2;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int p = blockIdx.x; p < npairs; p += gridDim.x) {
    int bi, bj;
    tile_pair(p, T, bi, bj);
    const int i0 = bi * 32, j0 = bj * 32;
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = j0 + r, j = i0 + tx;
      const bool in = i < M && j < M;
      th[r][tx] = in ? m.H1[(int64_t)i * M + j] : 0.0;
      ts[r][tx] = in ? m.S1[(int64_t)i * M + j] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = i0 + r, j = j0 + tx;
      if (i >= M || j >= M || i > j) continue;
      const int64_t e = (int64_t)i * M + j;
      const double hw = m.HW[e], sw = m.SW[e], h2 = m.H2[e], s2 = m.S2[e];
      const double h1 = m.H1[e], s1 = m.S1[e];
      if (i == j) {
        acc[0] += hw; acc[1] += h1; acc[2] += h2;
        acc[3] += sw * hw; acc[4] += s1 * hw; acc[5] += sw * h1; acc[6] += s2 * hw; acc[7] += sw * h2;
        acc[8] += s1 * h1; acc[9] += s1 * h1; acc[10] += s2 * h1; acc[11] += s1 * h2; acc[12] += s2 * h2;
      } else {
        const double h1t = th[tx][r], s1t = ts[tx][r];  // H'_ji, S'_ji
        const double h1s = h1 + h1t, s1s = s1 + s1t;
        acc[3] += 2.0 * sw * hw;
        acc[4] += s1s * hw;
        acc[5] += sw * h1s;
        acc[6] += 2.0 * s2 * hw;
        acc[7] += 2.0 * sw * h2;
        acc[8] += s1 * h1t + s1t * h1;
        acc[9] += s1 * h1 + s1t * h1t;
        acc[10] += s2 * h1s;
        acc[11] += s1s * h2;
        acc[12] += 2.0 * s2 * h2;
      }
    }
  }
  block_sums<NCOEF>(acc, sh);
  if (threadIdx.x == 0)
    for (int k = 0; k < NCOEF; ++k) partials[blockIdx.x * NCOEF + k] = acc[k];
}

// Line minimum of q(x) = sum_k a_k x^k: the first local minimum met going downhill from x = 0
// (the functional has no lower bound, so the lowest of two minima may lie beyond the basin).
// Descent side x > 0 if a1 < 0 (x < 0 if a1 > 0; a1 = 0 gives x = 0). Candidates are real roots
// of q' on that side (closed-form cubic, two Newton steps) with q'' > 0; the smallest |x| wins.
// a4 (then a3) is dropped when negligible against |a1|+|a2|+|a3|+|a4|.
__device__ double dq(const double* a, double x) {
  return a[1] + 2.0 * a[2] * x + 3.0 * a[3] * x * x + 4.0 * a[4] * x * x * x;
}
__device__ double d2q(const double* a, double x) {
  return 2.0 * a[2] + 6.0 * a[3] * x + 12.0 * a[4] * x * x;
}

__device__ int cubic_roots(double a, double b, double c, double d, double* r) {
  const double A = b / a, B = c / a, Cc = d / a;
  const double p = B - A * A / 3.0;
  const double q = 2.0 * A * A * A / 27.0 - A * B / 3.0 + Cc;
  const double sh = -A / 3.0;
  const double disc = (q / 2.0) * (q / 2.0) + (p / 3.0) * (p / 3.0) * (p / 3.0);
  if (disc > 0.0) {
    const double u = cbrt(-q / 2.0 - copysign(sqrt(disc), q));
    r[0] = u - p / (3.0 * u) + sh;
    return 1;
  }
  if (p == 0.0) {
    r[0] = sh;
    return 1;
  }
  const double m = 2.0 * sqrt(-p / 3.0);
  const double arg = fmin(1.0, fmax(-1.0, 3.0 * q / (p * m)));
  const double phi = acos(arg) / 3.0;
  const double two_pi_3 = 2.0 * M_PI / 3.0;
  for (int k = 0; k < 3; ++k) r[k] = m * cos(phi - two_pi_3 * k) + sh;
  return 3;
}

__device__ int line_minimum(const double* a, double* xout) {
  if (a[1] == 0.0) { *xout = 0.0; return 1; }
  const double side = a[1] < 0.0 ? 1.0 : -1.0;
  const double scale = fabs(a[1]) + fabs(a[2]) + fabs(a[3]) + fabs(a[4]);
  const double tiny = 1e-14 * scale;
  double roots[3];
  int nr = 0;
  if (fabs(a[4]) > tiny) {
    nr = cubic_roots(4.0 * a[4], 3.0 * a[3], 2.0 * a[2], a[1], roots);
  } else if (fabs(a[3]) > tiny) {
    const double qa = 3.0 * a[3], qb = 2.0 * a[2], qc = a[1];
    const double disc = qb * qb - 4.0 * qa * qc;
    if (disc >= 0.0) {
      const double s = -0.5 * (qb + copysign(sqrt(disc), qb));
      if (s != 0.0) roots[nr++] = qc / s;
      roots[nr++] = s / qa;
    }
  } else {
    if (a[2] > 0.0) { *xout = -a[1] / (2.0 * a[2]); return 1; }
    return 0;
  }
  int found = 0;
  double best = 0.0;
  for (int k = 0; k < nr; ++k) {
    double x = roots[k];
    for (int it = 0; it < 2; ++it) {
      const double h = d2q(a, x);
      if (h == 0.0) break;
      const double step = dq(a, x) / h;
      if (!isfinite(step)) break;
      x -= step;
    }
    if (!isfinite(x) || side * x <= 0.0 || !(d2q(a, x) > 0.0)) continue;
    if (!found || fabs(x) < fabs(best)) {
      best = x;
      found = 1;
    }
  }
  *xout = best;
  return found;
}

// The quartic of the line search from the partial sums of its 13 terms and its minimum x, in every thread
// of the block (false: none). Wave w sums columns w, w + 4, ..; the same sums in every block that
// calls this, so that a kernel may find x for itself; one block (`writer`) keeps the result, or the
// error code, in the state. It does not set `done`: the waves of a launch test that as they start, and
// a block of which some waves saw it set in mid-launch would go on without them (thread 0 of a
// launch of one block, or the next launch, sets it from line_code).
__device__ __forceinline__ bool line_x(const double* partials, int nb, DevState* st, bool writer,
                                       double* xout) {
  __shared__ double s[NCOEF];
  __shared__ double xs;
  __shared__ int found;
  const int lane = threadIdx.x & 63;
  for (int c = threadIdx.x >> 6; c < NCOEF; c += NT / 64) {
    double v = 0.0;
    for (int r = lane; r < nb; r += 64) v += partials[r * NCOEF + c];
    v = wave_sum(v);
    if (lane == 0) s[c] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a[5];
    a[0] = 4.0 * s[0] - 2.0 * s[3];
    a[1] = 8.0 * s[1] - 4.0 * s[4] - 4.0 * s[5];
    a[2] = 4.0 * s[2] - 2.0 * s[6] - 2.0 * s[7] - 4.0 * s[8] - 4.0 * s[9];
    a[3] = -4.0 * s[10] - 4.0 * s[11];
    a[4] = -2.0 * s[12];
    int code = 0;
    for (int k = 0; k < 5; ++k)
      if (!isfinite(a[k])) code = -5;
    double x = 0.0;
    if (code == 0 && !line_minimum(a, &x)) code = -7;
    if (writer) {
      for (int k = 0; k < 5; ++k) st->alpha[k] = a[k];
      st->line_code = code;
      if (!code) st->x = x;
    }
    xs = x;
    found = code == 0;
  }
  __syncthreads();
  *xout = xs;
  return found != 0;
}

__global__ __launch_bounds__(NT) void k_line_final(const double* partials, int nb, DevState* st) {
  if (st->done) return;
  double x;
  if (!line_x(partials, nb, st, true, &x) && threadIdx.x == 0) st->done = st->line_code;
}

// ---- updates (Eq. 16 and the footnote of Sec. 2.3) ----------------------------------------------
template <typename T, typename TD = T>
__device__ __forceinline__ void b_update_mn(T* C, const T* D, T* HC, const TD* HD, T* SC, const TD* SD, int64_t n,
                            double x, int bid, int nb) {
  for (int64_t i = (int64_t)bid * NT + threadIdx.x; i < n; i += (int64_t)nb * NT) {
    C[i] = (T)((double)C[i] + x * (double)D[i]);
    HC[i] = (T)((double)HC[i] + x * (double)HD[i]);
    SC[i] = (T)((double)SC[i] + x * (double)SD[i]);
  }
}

template <typename T, typename TD>
__global__ void k_update_mn(T* C, const T* D, T* HC, const TD* HD, T* SC, const TD* SD, int64_t n,
                            const DevState* st) {
  if (st->done) return;
  b_update_mn(C, D, HC, HD, SC, SD, n, st->x, blockIdx.x, gridDim.x);
}

__device__ __forceinline__ void split_store(double v, unsigned short* hi, unsigned short* lo,
                                            int64_t e) {
  const unsigned short hb = bf16_bits((float)v);
  hi[e] = hb;
  lo[e] = bf16_bits((float)(v - (double)__uint_as_float(((unsigned int)hb) << 16)));
}

// Eq. 16 for C, HC, SC (rows x cols) with the bf16 planes of the new HC and SC, row-major and
// transposed (through a 32 x 33 LDS tile), one 32 x 32 tile per block.
__device__ __forceinline__ float bf16_value(unsigned short b) {
  return __uint_as_float(((unsigned int)b) << 16);
}

template <typename T, typename TD>
__global__ void k_update_split_mn(T* C, const unsigned short* Dh, int64_t ldd, T* HC, const TD* HD,
                                  T* SC, const TD* SD, int rows, int cols, StatePlanes p,
                                  const DevState* st) {
  if (st->done) return;
  __shared__ T th[32][33], ts[32][33];
  const double x = st->x;
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int gr = r0 + r, gc = c0 + tx;
    T h = (T)0, v = (T)0;
    if (gr < rows && gc < cols) {
      const int64_t e = (int64_t)gr * cols + gc;
      const double d = (double)bf16_value(Dh[(int64_t)gr * ldd + gc]);
      C[e] = (T)((double)C[e] + x * d);
      h = (T)((double)HC[e] + x * (double)HD[e]);
      v = (T)((double)SC[e] + x * (SD ? (double)SD[e] : d));
      HC[e] = h;
      SC[e] = v;
      const int64_t q = (int64_t)gr * p.ld + gc;
      split_store((double)h, p.hc_hi, p.hc_lo, q);
      split_store((double)v, p.sc_hi, p.sc_lo, q);
    }
    th[r][tx] = h;
    ts[r][tx] = v;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int oc = c0 + r, orow = r0 + tx;  // output row oc (a source column), column orow
    if (oc < cols && orow < rows) {
      const int64_t o = (int64_t)oc * p.ldt + orow;
      split_store((double)th[tx][r], p.hct_hi, p.hct_lo, o);
      split_store((double)ts[tx][r], p.sct_hi, p.sct_lo, o);
    }
  }
}

// The same for an even number of columns (8-byte aligned rows), one 64 x 64 tile per block:
// each thread takes two adjacent columns, so the T arrays move in 16-byte and the planes in
// 4-byte (two bf16) accesses, and every plane row segment a block writes (also transposed) is
// one 128-byte line. The transpose goes through LDS as packed (hi | lo << 16) words. Every store
// is non-temporal (see stream_store).
__device__ __forceinline__ unsigned split_word(double v) {
  const unsigned hb = bf16_bits((float)v);
  const unsigned lb = bf16_bits((float)(v - (double)__uint_as_float(hb << 16)));
  return hb | (lb << 16);
}

// Two bf16 values as one 4-byte store that bypasses the caches' normal retention: everything
// the update writes is next read a whole line search later, long after it would have left L2.
__device__ __forceinline__ void stream_store(unsigned w, unsigned short* dst) {
  __builtin_nontemporal_store(w, reinterpret_cast<unsigned*>(dst));
}

typedef unsigned PlaneTile[64][65];

template <typename T, typename TD>
__device__ __forceinline__ void b_update_split_mn2(T* C, const unsigned short* Dh, int64_t ldd, T* HC,
                                                   const TD* HD, T* SC, const TD* SD, int rows, int cols,
                                                   const StatePlanes& p, double x, int bx, int by,
                                                   PlaneTile& th, PlaneTile& ts) {
  typedef T T2 __attribute__((ext_vector_type(2)));
  typedef TD TD2 __attribute__((ext_vector_type(2)));
  const int c0 = bx * 64, r0 = by * 64;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 column pairs x 8 rows
  const int gc = c0 + 2 * tx;
  // rows ty + 8 k, four at a time: all loads of a batch are issued before its stores
  constexpr int RB = 4;
#pragma unroll
  for (int b = 0; b < 8; b += RB) {
    T2 c[RB], hc[RB], sc[RB];
    TD2 hd[RB], sd[RB];
    unsigned dw[RB];  // two bf16 directions
    bool in[RB];
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int gr = r0 + ty + 8 * (b + k);
      in[k] = gr < rows && gc < cols;  // cols even: gc + 1 < cols as well
      if (in[k]) {
        const int64_t e = (int64_t)gr * cols + gc;
        c[k] = *reinterpret_cast<const T2*>(C + e);
        dw[k] = *reinterpret_cast<const unsigned*>(Dh + (int64_t)gr * ldd + gc);
        hc[k] = *reinterpret_cast<const T2*>(HC + e);
        hd[k] = *reinterpret_cast<const TD2*>(HD + e);
        sc[k] = *reinterpret_cast<const T2*>(SC + e);
        if (SD) sd[k] = *reinterpret_cast<const TD2*>(SD + e);
      }
    }
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int r = ty + 8 * (b + k), gr = r0 + r;
      unsigned wh0 = 0, wh1 = 0, ws0 = 0, ws1 = 0;
      if (in[k]) {
        const int64_t e = (int64_t)gr * cols + gc;
        const double d0 = (double)__uint_as_float(dw[k] << 16);
        const double d1 = (double)__uint_as_float(dw[k] & 0xffff0000u);
        T2 cn, h, v;
        cn.x = (T)((double)c[k].x + x * d0);
        cn.y = (T)((double)c[k].y + x * d1);
        h.x = (T)((double)hc[k].x + x * (double)hd[k].x);
        h.y = (T)((double)hc[k].y + x * (double)hd[k].y);
        v.x = (T)((double)sc[k].x + x * (SD ? (double)sd[k].x : d0));
        v.y = (T)((double)sc[k].y + x * (SD ? (double)sd[k].y : d1));
        __builtin_nontemporal_store(cn, reinterpret_cast<T2*>(C + e));
        __builtin_nontemporal_store(h, reinterpret_cast<T2*>(HC + e));
        __builtin_nontemporal_store(v, reinterpret_cast<T2*>(SC + e));
        wh0 = split_word((double)h.x);
        wh1 = split_word((double)h.y);
        ws0 = split_word((double)v.x);
        ws1 = split_word((double)v.y);
        const int64_t q = (int64_t)gr * p.ld + gc;
        stream_store((wh0 & 0xffffu) | (wh1 << 16), p.hc_hi + q);
        stream_store((wh0 >> 16) | (wh1 & 0xffff0000u), p.hc_lo + q);
        stream_store((ws0 & 0xffffu) | (ws1 << 16), p.sc_hi + q);
        stream_store((ws0 >> 16) | (ws1 & 0xffff0000u), p.sc_lo + q);
      }
      th[r][2 * tx] = wh0;
      th[r][2 * tx + 1] = wh1;
      ts[r][2 * tx] = ws0;
      ts[r][2 * tx + 1] = ws1;
    }
  }
  __syncthreads();
  // transposed: output row oc = c0 + j (a source column), output columns r0 + 2 tx, r0 + 2 tx + 1
  const int orow = r0 + 2 * tx;
  for (int j = ty; j < 64; j += 8) {
    const int oc = c0 + j;
    if (oc >= cols || orow >= rows) continue;
    const unsigned a0 = th[2 * tx][j], b0 = ts[2 * tx][j];
    const int64_t o = (int64_t)oc * p.ldt + orow;
    if (orow + 1 < rows) {
      const unsigned a1 = th[2 * tx + 1][j], b1 = ts[2 * tx + 1][j];
      stream_store((a0 & 0xffffu) | (a1 << 16), p.hct_hi + o);
      stream_store((a0 >> 16) | (a1 & 0xffff0000u), p.hct_lo + o);
      stream_store((b0 & 0xffffu) | (b1 << 16), p.sct_hi + o);
      stream_store((b0 >> 16) | (b1 & 0xffff0000u), p.sct_lo + o);
    } else {
      p.hct_hi[o] = (unsigned short)(a0 & 0xffffu);
      p.hct_lo[o] = (unsigned short)(a0 >> 16);
      p.sct_hi[o] = (unsigned short)(b0 & 0xffffu);
      p.sct_lo[o] = (unsigned short)(b0 >> 16);
    }
  }
}

template <typename T, typename TD>
__global__ __launch_bounds__(NT) void k_update_split_mn2(T* C, const unsigned short* Dh,
                                                         int64_t ldd, T* HC, const TD* HD, T* SC,
                                                         const TD* SD, int rows, int cols,
                                                         StatePlanes p, const DevState* st) {
  if (st->done) return;
  __shared__ PlaneTile th, ts;
  b_update_split_mn2(C, Dh, ldd, HC, HD, SC, SD, rows, cols, p, st->x, blockIdx.x, blockIdx.y, th, ts);
}

// HW += x (H' + H'^T) + x^2 H'', SW likewise; partial sums of Tr HW, <SW, HW>, Tr SW.
__device__ __forceinline__ void b_update_mm(double* HW, double* SW, const double* H1, const double* S1,
                            const double* H2, const double* S2, int M, double* partials,
                            const DevState* st, int bid, int nb) {
  if (st->done) return;
  __shared__ double th[32][33], ts[32][33];
  __shared__ double sh[SH_SUMS];
  const double x = st->x;
  double tr = 0.0, f = 0.0, trs = 0.0;
  const int tb = (M + 31) / 32;
  const int ntiles = tb * tb;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int tile = bid; tile < ntiles; tile += nb) {
    const int bi = (tile / tb) * 32, bj = (tile % tb) * 32;
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = bj + r, j = bi + tx;
      const bool in = i < M && j < M;
      th[r][tx] = in ? H1[(int64_t)i * M + j] : 0.0;
      ts[r][tx] = in ? S1[(int64_t)i * M + j] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = bi + r, j = bj + tx;
      if (i < M && j < M) {
        const int64_t e = (int64_t)i * M + j;
        const double hw = HW[e] + x * H1[e] + x * th[tx][r] + x * x * H2[e];
        const double sw = SW[e] + x * S1[e] + x * ts[tx][r] + x * x * S2[e];
        HW[e] = hw;
        SW[e] = sw;
        f += sw * hw;
        if (i == j) { tr += hw; trs += sw; }
      }
    }
  }
  double v3[3] = {tr, f, trs};
  block_sums<3>(v3, sh);
  const double a = v3[0], b = v3[1], c = v3[2];
  if (threadIdx.x == 0) {
    partials[bid * 3 + 0] = a;
    partials[bid * 3 + 1] = b;
    partials[bid * 3 + 2] = c;
  }
}

// The same update for one system, using that HW, SW, H'' and S'' are symmetric: each block takes a
// pair of 32 x 32 tiles (bi, bj), bi <= bj, computes the upper one from the upper tiles of HW,
// SW, H'', S'' and both tiles of H', S' (the mirror one transposed through LDS), and writes the
// result to both (on a diagonal tile, its upper triangle to both halves), with its bf16 planes if
// there are any. HW and SW come out exactly symmetric; every element of H', S' and of the upper halves
// is read once.
typedef double MMTile[32][33];

__device__ __forceinline__ void mm_store(const Subspace& m, int i, int j, double hw, double sw) {
  const int64_t e = (int64_t)i * m.M + j;
  m.HW[e] = hw;
  m.SW[e] = sw;
  if (m.hw_hi) {
    const int64_t q = (int64_t)i * m.ldp + j;
    split_store(hw, m.hw_hi, m.hw_lo, q);
    split_store(sw, m.sw_hi, m.sw_lo, q);
  }
}

__device__ __forceinline__ void b_update_mm_sym(const Subspace& m, double x, double* partials, int bid, int nb,
                                                MMTile (&t)[4]) {
  __shared__ double sh[SH_SUMS];
  MMTile &th = t[0], &ts = t[1], &oh = t[2], &os = t[3];
  double tr = 0.0, f = 0.0, trs = 0.0;
  const int M = m.M, T = (M + 31) / 32, npairs = T * (T + 1) / 2;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int p = bid; p < npairs; p += nb) {
    int bi, bj;
    tile_pair(p, T, bi, bj);
    const int i0 = bi * 32, j0 = bj * 32;
    const bool diag = bi == bj;
    __syncthreads();
    // th[c][r] = H'[j0 + c][i0 + r], the transposed partner of output (i0 + r, j0 + c)
    for (int rr = ty; rr < 32; rr += 8) {
      const int i = j0 + rr, j = i0 + tx;
      const bool in = i < M && j < M;
      th[rr][tx] = in ? m.H1[(int64_t)i * M + j] : 0.0;
      ts[rr][tx] = in ? m.S1[(int64_t)i * M + j] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
      const int i = i0 + r, j = j0 + tx;
      if (i < M && j < M && (!diag || r <= tx)) {
        const int64_t e = (int64_t)i * M + j;
        const double hw = m.HW[e] + x * m.H1[e] + x * th[tx][r] + x * x * m.H2[e];
        const double sw = m.SW[e] + x * m.S1[e] + x * ts[tx][r] + x * x * m.S2[e];
        mm_store(m, i, j, hw, sw);
        oh[r][tx] = hw;
        os[r][tx] = sw;
        if (diag && r == tx) {
          tr += hw;
          trs += sw;
          f += sw * hw;
        } else {
          f += 2.0 * sw * hw;
        }
      }
    }
    __syncthreads();
    // mirror: element (j0 + rr, i0 + tx) = output (i0 + tx, j0 + rr)
    for (int rr = ty; rr < 32; rr += 8) {
      const int i = j0 + rr, j = i0 + tx;
      if (i < M && j < M && (!diag || tx < rr)) mm_store(m, i, j, oh[tx][rr], os[tx][rr]);
    }
  }
  double v3[3] = {tr, f, trs};
  block_sums<3>(v3, sh);
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k) partials[bid * 3 + k] = v3[k];
}

__global__ __launch_bounds__(NT) void k_update_mm_sym(Subspace m, double* partials, const DevState* st) {
  if (st->done) return;
  __shared__ MMTile t[4];
  b_update_mm_sym(m, st->x, partials, blockIdx.x, gridDim.x, t);
}

// Small systems: the line minimum and both updates in one launch. Every block finds x itself; the
// first nmm then update HW and SW, the others C, HC, SC. `lpart` (np rows of the quartic's terms)
// and `epart` (the energy's) are different arrays, since some blocks still read one while others
// write the other.
template <typename T, typename TD>
__global__ __launch_bounds__(NT) void k_update_line(T* C, const T* D, T* HC, const TD* HD, T* SC, const TD* SD,
                                                    int64_t n, Subspace m, int nmm, const double* lpart,
                                                    int np, double* epart, DevState* st) {
  if (st->done) return;
  __shared__ MMTile t[4];
  double x;
  if (!line_x(lpart, np, st, blockIdx.x == 0, &x)) return;
  const int bid = blockIdx.x;
  if (bid < nmm) b_update_mm_sym(m, x, epart, bid, nmm, t);
  else b_update_mn(C, D, HC, HD, SC, SD, n, x, bid - nmm, gridDim.x - nmm);
}

template <typename T, typename TD>
__global__ __launch_bounds__(NT) void k_update_split_line(T* C, const unsigned short* Dh, int64_t ldd, T* HC,
                                                          const TD* HD, T* SC, const TD* SD, int rows,
                                                          int cols, StatePlanes p, Subspace m, int nmm,
                                                          const double* lpart, int np, double* epart,
                                                          DevState* st) {
  if (st->done) return;
  __shared__ union {
    MMTile t[4];
    PlaneTile u[2];
  } lds;
  double x;
  if (!line_x(lpart, np, st, blockIdx.x == 0, &x)) return;
  const int bid = blockIdx.x, tile = bid - nmm, bx = (cols + 63) / 64;
  if (bid < nmm) b_update_mm_sym(m, x, epart, bid, nmm, lds.t);
  else b_update_split_mn2(C, Dh, ldd, HC, HD, SC, SD, rows, cols, p, x, tile % bx, tile / bx, lds.u[0], lds.u[1]);
}

__device__ __forceinline__ void f_update_final(const double* partials, int nb, int M, DevState* st,
                               double* trace) {
  if (st->done) return;
  if (st->line_code) {  // the line minimum of the launch before found none: nothing was updated
    if (threadIdx.x == 0) st->done = st->line_code;
    return;
  }
  __shared__ double sh[SH_SUMS];
  double s3[3];
  sum_partials_all<3>(partials, nb, sh, s3);
  const double tr = s3[0], f = s3[1], trs = s3[2];
  if (threadIdx.x != 0) return;
  const double E_new = 4.0 * tr - 2.0 * f;
  const double E_old = st->E;
  const double diff = fabs(2.0 * (E_new - E_old)), sum = fabs(E_new + E_old);
  st->E_prev = E_old;
  st->E = E_new;
  st->iter += 1;
  st->rel_change = sum > 0.0 ? diff / sum : diff;
  if (trace) trace[st->iter] = E_new;
  if (!isfinite(E_new)) { st->done = -5; return; }
  if (trs > 16.0 * (double)M) { st->done = -8; return; }
  if (diff <= st->tol * sum) { st->done = 1; return; }
  if (st->iter >= st->max_iter) st->done = 2;
}

__global__ void k_update_final(const double* partials, int nb, int M, DevState* st,
                               double* trace) {
  f_update_final(partials, nb, M, st, trace);
}

__global__ void k_identity_minus(const double* SW, double* out, int M, double diag, double scale) {
  const int64_t n = (int64_t)M * M;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
    const int r = (int)(i / M), c = (int)(i % M);
    out[i] = scale * ((r == c ? diag : 0.0) - SW[i]);
  }
}

__global__ void k_axpby(const double* a, const double* b, double* out, double ca, double cb,
                        int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT)
    out[i] = ca * a[i] + cb * b[i];
}

// ---- grouped kernels (blockIdx.y = system) -----------------------------------------------------
__global__ void g_energy_partials(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  b_energy_partials(d.HW, d.SW, d.M, d.partials, blockIdx.x, gridDim.x);
}
__global__ void g_energy_init_final(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  f_energy_init_final(d.partials, GROUP_BLOCKS, d.st, d.trace);
}
template <typename T>
__device__ __forceinline__ void g_pr_partials_t(const SysDev& d, int parity, int first) {
  const T* G = static_cast<const T*>(parity ? d.G1 : d.G0);
  const T* Gp = static_cast<const T*>(parity ? d.G0 : d.G1);
  const T* PG = d.precon ? static_cast<const T*>(d.PG) : G;
  b_pr_partials<T>(G, PG, Gp, (int64_t)d.M * d.N, first, d.partials, d.st, blockIdx.x, gridDim.x);
}
__global__ void g_pr_partials(const SysDev* sys, int parity, int first) {
  const SysDev& d = sys[blockIdx.y];
  if (d.f64) g_pr_partials_t<double>(d, parity, first);
  else g_pr_partials_t<float>(d, parity, first);
}
template <typename T>
__device__ __forceinline__ void g_direction_t(const SysDev& d, int parity, int first) {
  const T* G = static_cast<const T*>(parity ? d.G1 : d.G0);
  const T* PG = d.precon ? static_cast<const T*>(d.PG) : G;
  const double beta = beta_of(d.partials, GROUP_BLOCKS, first, parity, d.st, blockIdx.x == 0);
  b_direction<T>(PG, static_cast<T*>(d.D), (int64_t)d.M * d.N, first, beta, blockIdx.x, gridDim.x);
}
__global__ void g_direction(const SysDev* sys, int parity, int first) {
  const SysDev& d = sys[blockIdx.y];
  if (d.st->done) return;
  if (d.f64) g_direction_t<double>(d, parity, first);
  else g_direction_t<float>(d, parity, first);
}
__global__ void g_coef_partials(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  b_coef_partials(d.HW, d.SW, d.H1, d.S1, d.H2, d.S2, d.M, d.partials, d.st, blockIdx.x, gridDim.x);
}
__global__ void g_line_final(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  if (d.st->done) return;
  double x;
  if (!line_x(d.partials, GROUP_BLOCKS, d.st, true, &x) && threadIdx.x == 0) d.st->done = d.st->line_code;
}
template <typename T>
__device__ __forceinline__ void g_update_mn_t(const SysDev& d) {
  b_update_mn<T>(static_cast<T*>(d.C), static_cast<const T*>(d.D), static_cast<T*>(d.HC),
                 static_cast<const T*>(d.HD), static_cast<T*>(d.SC), static_cast<const T*>(d.SD),
                 (int64_t)d.M * d.N, d.st->x, blockIdx.x, gridDim.x);
}
__global__ void g_update_mn(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  if (d.st->done) return;
  if (d.f64) g_update_mn_t<double>(d);
  else g_update_mn_t<float>(d);
}
__global__ void g_update_mm(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  b_update_mm(d.HW, d.SW, d.H1, d.S1, d.H2, d.S2, d.M, d.partials, d.st, blockIdx.x, gridDim.x);
}
__global__ void g_update_final(const SysDev* sys) {
  const SysDev& d = sys[blockIdx.y];
  f_update_final(d.partials, GROUP_BLOCKS, d.M, d.st, d.trace);
}

int pair_blocks(int M) {
  const int T = (M + 31) / 32, n = T * (T + 1) / 2;
  return n < RED_BLOCKS ? n : RED_BLOCKS;
}

}  // namespace

hipError_t shift_hamiltonian(const double* H, const double* S, double eta, double* Hs, int64_t n,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_shift, dim3(ew_blocks(n)), dim3(NT), 0, s, H, S, eta, Hs, n);
  return hipGetLastError();
}

hipError_t convert_f64_f32(const double* src, float* dst, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((k_convert<double, float>), dim3(ew_blocks(n)), dim3(NT), 0, s, src, dst, n);
  return hipGetLastError();
}

namespace {
dim3 split_grid(int64_t rows, int64_t cols) {
  int64_t bx = (cols + 4 * NT - 1) / (4 * NT);
  if (bx < 1) bx = 1;
  return dim3((unsigned)bx, (unsigned)(rows < 65535 ? rows : 65535));
}
}  // namespace

hipError_t split_bf16(const float* src, unsigned short* hi, unsigned short* lo, int64_t rows,
                      int64_t cols, int64_t ld, const DevState* st, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ld < cols || ld % 4 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split<float>, split_grid(rows, cols), dim3(NT), 0, s, src, hi, lo, rows, cols,
                     ld, st);
  return hipGetLastError();
}

hipError_t split_bf16(const double* src, unsigned short* hi, unsigned short* lo, int64_t rows,
                      int64_t cols, int64_t ld, const DevState* st, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ld < cols || ld % 4 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split<double>, split_grid(rows, cols), dim3(NT), 0, s, src, hi, lo, rows,
                     cols, ld, st);
  return hipGetLastError();
}

hipError_t split_bf16_t(const float* src, unsigned short* hi, unsigned short* lo, int rows,
                        int cols, int64_t ld, const DevState* st, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ld < rows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split_t<float>, dim3((cols + 31) / 32, (rows + 31) / 32), dim3(NT), 0, s, src,
                     hi, lo, rows, cols, ld, st);
  return hipGetLastError();
}

hipError_t split_bf16_t(const double* src, unsigned short* hi, unsigned short* lo, int rows,
                        int cols, int64_t ld, const DevState* st, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ld < rows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split_t<double>, dim3((cols + 31) / 32, (rows + 31) / 32), dim3(NT), 0, s,
                     src, hi, lo, rows, cols, ld, st);
  return hipGetLastError();
}

hipError_t convert_f32_f64(const float* src, double* dst, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((k_convert<float, double>), dim3(ew_blocks(n)), dim3(NT), 0, s, src, dst, n);
  return hipGetLastError();
}

// dst = src; *diff = 1 if any element changes (bit pattern), else *diff is left as it was
__global__ void k_copy_compare(const double* src, double* dst, int64_t n, int* diff) {
  bool changed = false;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
    const double v = src[i];
    changed |= __double_as_longlong(v) != __double_as_longlong(dst[i]);
    dst[i] = v;
  }
  // one store a wave, and none once another wave's is seen: atomics on one address from every wave
  // took 66 us at 717 orbitals, 260 us at 2301
  if (__any(changed) && (threadIdx.x & 63) == 0 && __hip_atomic_load(diff, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
    __hip_atomic_store(diff, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

hipError_t copy_compare_f64(const double* src, double* dst, int64_t n, int* diff, hipStream_t s) {
  hipLaunchKernelGGL(k_copy_compare, dim3(ew_blocks(n)), dim3(NT), 0, s, src, dst, n, diff);
  return hipGetLastError();
}

hipError_t copy_f64(const double* src, double* dst, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL((k_convert<double, double>), dim3(ew_blocks(n)), dim3(NT), 0, s, src, dst, n);
  return hipGetLastError();
}

hipError_t validate_symmetric(const double* A, int64_t n, double rtol, int* flags, hipStream_t s) {
  const int tb = (int)((n + 31) / 32);
  hipLaunchKernelGGL(k_validate, dim3(tb, tb), dim3(NT), 0, s, A, n, rtol, flags);
  return hipGetLastError();
}

hipError_t check_inputs(const SymInputs& in, int64_t n, double rtol, int* flags, hipStream_t s) {
  const int tb = (int)((n + 31) / 32);
  hipLaunchKernelGGL(k_check_inputs, dim3(tb, tb, 3), dim3(NT), 0, s, in, n, rtol, flags);
  return hipGetLastError();
}

hipError_t store_inputs(const SymInputs& in, int64_t n, hipStream_t s) {
  const int tb = (int)((n + 31) / 32);
  hipLaunchKernelGGL(k_store_inputs, dim3(tb, tb, 3), dim3(NT), 0, s, in, n);
  return hipGetLastError();
}

hipError_t symmetrize(double* A, int64_t n, hipStream_t s) {
  const int tb = (int)((n + 31) / 32);
  hipLaunchKernelGGL(k_symmetrize, dim3(tb, tb), dim3(NT), 0, s, A, n);
  return hipGetLastError();
}

hipError_t energy_init(const double* HW, const double* SW, int M, double* partials, DevState* st,
                       double* trace, hipStream_t s) {
  const int nb = red_blocks((int64_t)M * M);
  hipLaunchKernelGGL(k_energy_partials, dim3(nb), dim3(NT), 0, s, HW, SW, M, partials);
  hipLaunchKernelGGL(k_energy_init_final, dim3(1), dim3(NT), 0, s, partials, nb, st, trace);
  return hipGetLastError();
}

hipError_t block_pattern(const double* B, int64_t n, unsigned char* flags, hipStream_t s) {
  const int nkb = (int)((n + SPARSE_BK - 1) / SPARSE_BK);
  const int nt = (int)((n + SPARSE_BN - 1) / SPARSE_BN);
  hipLaunchKernelGGL(k_block_pattern, dim3(nkb, nt), dim3(NT), 0, s, B, n, flags);
  return hipGetLastError();
}

template <typename T, typename TP, typename TG>
hipError_t beta_and_direction(const TG* G, const TP* PG, const TG* Gprev, T* D, int64_t n, int k,
                              double* partials, DevState* st, hipStream_t s, unsigned short* hi,
                              int64_t cols, int64_t ld) {
  if (!hi && !D) return hipErrorInvalidValue;
  const int first = k == 0 ? 1 : 0, parity = k & 1;
  const int nb = red_blocks(n);
  // each direction block first sums the partials: no more blocks than run at once
  constexpr int64_t DIR_BLOCKS = 2048;
  const bool vec = ((uintptr_t)G | (uintptr_t)Gprev) % (4 * sizeof(TG)) == 0 &&
                   (uintptr_t)PG % (4 * sizeof(TP)) == 0;
  if (vec)
    hipLaunchKernelGGL((k_pr_partials4<TG, TP>), dim3(nb), dim3(NT), 0, s, G, PG, Gprev, n, first,
                       partials, st);
  else
    hipLaunchKernelGGL((k_pr_partials<TG, TP>), dim3(nb), dim3(NT), 0, s, G, PG, Gprev, n, first,
                       partials, st);
  if (hi) {
    if (cols <= 0 || n % cols != 0 || ld < cols) return hipErrorInvalidValue;
    const int64_t rows = n / cols;
    const bool vec4 = cols % 4 == 0 && ld % 4 == 0 && (uintptr_t)PG % (4 * sizeof(TP)) == 0 &&
                      (uintptr_t)hi % 8 == 0;
    const int64_t bx = (cols / (vec4 ? 4 : 1) + NT - 1) / NT;
    const int64_t by = std::min<int64_t>(vec4 ? (rows + 3) / 4 : rows,
                                         std::max<int64_t>(1, DIR_BLOCKS / bx));
    const dim3 grid((unsigned)bx, (unsigned)by);
    if (vec4)
      hipLaunchKernelGGL((k_direction_bf16x4<T, TP>), grid, dim3(NT), 0, s, PG, D, hi, rows, cols, ld,
                         first, parity, partials, nb, st);
    else
      hipLaunchKernelGGL((k_direction_bf16<T, TP>), grid, dim3(NT), 0, s, PG, D, hi, rows, cols, ld, first,
                         parity, partials, nb, st);
  } else {
    hipLaunchKernelGGL((k_direction<T, TP>), dim3(std::min<int64_t>(ew_blocks(n), DIR_BLOCKS)), dim3(NT),
                       0, s, PG, D, n, first, parity, partials, nb, st);
  }
  return hipGetLastError();
}
#define OMM_BETA_DIRECTION(T, TP, TG)                                                            \
  template hipError_t beta_and_direction<T, TP, TG>(const TG*, const TP*, const TG*, T*, int64_t, \
                                                    int, double*, DevState*, hipStream_t,         \
                                                    unsigned short*, int64_t, int64_t);
OMM_BETA_DIRECTION(double, double, double)
OMM_BETA_DIRECTION(float, float, float)
OMM_BETA_DIRECTION(double, float, double)
OMM_BETA_DIRECTION(double, float, float)
#undef OMM_BETA_DIRECTION

// With at most 256 blocks of partial sums a block can sum them in about a microsecond itself, and the
// line minimum, the update of C, HC, SC and that of HW, SW are one launch: 17.8 us instead of 27.0 (6.5 +
// 12.1 + 8.4) at 2048 x 384 in the BF16 scheme. Beyond, the sums (106 KB for 1024 blocks) would be
// re-read by every block.
bool line_fused(int M) { return pair_blocks(M) <= 256; }

hipError_t line_search(const Subspace& m, double* partials, DevState* st, bool fused, hipStream_t s) {
  const int nb = pair_blocks(m.M);
  hipLaunchKernelGGL(k_coef_sym, dim3(nb), dim3(NT), 0, s, m, partials, st);
  if (!fused) hipLaunchKernelGGL(k_line_final, dim3(1), dim3(NT), 0, s, partials, nb, st);
  return hipGetLastError();
}

template <typename T, typename TD>
hipError_t update_coefficients(T* C, const T* D, T* HC, const TD* HD, T* SC, const TD* SD,
                               int64_t n, const DevState* st, hipStream_t s) {
  hipLaunchKernelGGL((k_update_mn<T, TD>), dim3(ew_blocks(n)), dim3(NT), 0, s, C, D, HC, HD, SC, SD,
                     n, st);
  return hipGetLastError();
}
#define OMM_UPDATE(T, TD)                                                                        \
  template hipError_t update_coefficients<T, TD>(T*, const T*, T*, const TD*, T*, const TD*,     \
                                                 int64_t, const DevState*, hipStream_t);
OMM_UPDATE(double, double)
OMM_UPDATE(float, float)
OMM_UPDATE(double, float)
#undef OMM_UPDATE

namespace {
// Whether k_update_split_mn2 may take the arrays: an even number of columns, aligned pairs.
template <typename T, typename TD>
bool split_wide(const T* C, const unsigned short* Dh, int64_t ldd, const T* HC, const TD* HD, const T* SC,
                const TD* SD, int cols, const StatePlanes& p) {
  return cols % 2 == 0 && p.ld % 2 == 0 && p.ldt % 2 == 0 && ldd % 2 == 0 && (uintptr_t)Dh % 4 == 0 &&
         ((uintptr_t)C | (uintptr_t)HC | (uintptr_t)SC) % (2 * sizeof(T)) == 0 &&
         ((uintptr_t)HD | (uintptr_t)SD) % (2 * sizeof(TD)) == 0;
}
}  // namespace

template <typename T, typename TD>
hipError_t update_coefficients_split(T* C, const unsigned short* Dh, int64_t ldd, T* HC,
                                     const TD* HD, T* SC, const TD* SD, int rows, int cols,
                                     const StatePlanes& p, const DevState* st, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (!Dh || ldd < cols || p.ld < cols || p.ldt < rows) return hipErrorInvalidValue;
  if (split_wide<T, TD>(C, Dh, ldd, HC, HD, SC, SD, cols, p))
    hipLaunchKernelGGL((k_update_split_mn2<T, TD>), dim3((cols + 63) / 64, (rows + 63) / 64),
                       dim3(NT), 0, s, C, Dh, ldd, HC, HD, SC, SD, rows, cols, p, st);
  else
    hipLaunchKernelGGL((k_update_split_mn<T, TD>), dim3((cols + 31) / 32, (rows + 31) / 32),
                       dim3(NT), 0, s, C, Dh, ldd, HC, HD, SC, SD, rows, cols, p, st);
  return hipGetLastError();
}
#define OMM_UPDATE_SPLIT(T, TD)                                                                  \
  template hipError_t update_coefficients_split<T, TD>(T*, const unsigned short*, int64_t, T*,   \
                                                       const TD*, T*, const TD*, int, int,       \
                                                       const StatePlanes&, const DevState*,      \
                                                       hipStream_t);
OMM_UPDATE_SPLIT(double, double)
OMM_UPDATE_SPLIT(float, float)
OMM_UPDATE_SPLIT(double, float)
#undef OMM_UPDATE_SPLIT

hipError_t update_subspace(const Subspace& m, double* partials, DevState* st, double* trace, hipStream_t s) {
  const int nb = pair_blocks(m.M);
  hipLaunchKernelGGL(k_update_mm_sym, dim3(nb), dim3(NT), 0, s, m, partials, st);
  hipLaunchKernelGGL(k_update_final, dim3(1), dim3(NT), 0, s, partials, nb, m.M, st, trace);
  return hipGetLastError();
}

template <typename T, typename TD>
hipError_t update_line(T* C, const T* D, T* HC, const TD* HD, T* SC, const TD* SD, int64_t n,
                       const Subspace& m, const double* lpart, double* epart, DevState* st,
                       double* trace, hipStream_t s) {
  const int nmm = pair_blocks(m.M);
  const int nmn = (int)std::min<int64_t>((n + NT - 1) / NT, 512);
  hipLaunchKernelGGL((k_update_line<T, TD>), dim3(nmm + nmn), dim3(NT), 0, s, C, D, HC, HD, SC, SD, n, m,
                     nmm, lpart, nmm, epart, st);
  hipLaunchKernelGGL(k_update_final, dim3(1), dim3(NT), 0, s, epart, nmm, m.M, st, trace);
  return hipGetLastError();
}
#define OMM_UPDATE_LINE(T, TD)                                                                   \
  template hipError_t update_line<T, TD>(T*, const T*, T*, const TD*, T*, const TD*, int64_t,    \
                                         const Subspace&, const double*, double*, DevState*,     \
                                         double*, hipStream_t);
OMM_UPDATE_LINE(double, double)
OMM_UPDATE_LINE(float, float)
OMM_UPDATE_LINE(double, float)
#undef OMM_UPDATE_LINE

template <typename T, typename TD>
hipError_t update_split_line(T* C, const unsigned short* Dh, int64_t ldd, T* HC, const TD* HD, T* SC,
                             const TD* SD, int rows, int cols, const StatePlanes& p, const Subspace& m,
                             const double* lpart, double* epart, DevState* st, double* trace,
                             hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (!split_wide<T, TD>(C, Dh, ldd, HC, HD, SC, SD, cols, p)) {
    hipLaunchKernelGGL(k_line_final, dim3(1), dim3(NT), 0, s, lpart, pair_blocks(m.M), st);
    const hipError_t e = update_coefficients_split<T, TD>(C, Dh, ldd, HC, HD, SC, SD, rows, cols, p, st, s);
    return e != hipSuccess ? e : update_subspace(m, epart, st, trace, s);
  }
  if (!Dh || ldd < cols || p.ld < cols || p.ldt < rows) return hipErrorInvalidValue;
  const int nmm = pair_blocks(m.M), tiles = ((cols + 63) / 64) * ((rows + 63) / 64);
  hipLaunchKernelGGL((k_update_split_line<T, TD>), dim3(nmm + tiles), dim3(NT), 0, s, C, Dh, ldd, HC, HD, SC,
                     SD, rows, cols, p, m, nmm, lpart, nmm, epart, st);
  hipLaunchKernelGGL(k_update_final, dim3(1), dim3(NT), 0, s, epart, nmm, m.M, st, trace);
  return hipGetLastError();
}
#define OMM_UPDATE_SPLIT_LINE(T, TD)                                                             \
  template hipError_t update_split_line<T, TD>(T*, const unsigned short*, int64_t, T*, const TD*, T*, \
                                               const TD*, int, int, const StatePlanes&,          \
                                               const Subspace&, const double*, double*,          \
                                               DevState*, double*, hipStream_t);
OMM_UPDATE_SPLIT_LINE(double, double)
OMM_UPDATE_SPLIT_LINE(float, float)
OMM_UPDATE_SPLIT_LINE(double, float)
#undef OMM_UPDATE_SPLIT_LINE

hipError_t group_energy_init(const SysDev* d_sys, int nsys, hipStream_t s) {
  hipLaunchKernelGGL(g_energy_partials, dim3(GROUP_BLOCKS, nsys), dim3(NT), 0, s, d_sys);
  hipLaunchKernelGGL(g_energy_init_final, dim3(1, nsys), dim3(NT), 0, s, d_sys);
  return hipGetLastError();
}

hipError_t group_direction(const SysDev* d_sys, int nsys, int parity, int first, hipStream_t s) {
  hipLaunchKernelGGL(g_pr_partials, dim3(GROUP_BLOCKS, nsys), dim3(NT), 0, s, d_sys, parity, first);
  hipLaunchKernelGGL(g_direction, dim3(4 * GROUP_BLOCKS, nsys), dim3(NT), 0, s, d_sys, parity, first);
  return hipGetLastError();
}

hipError_t group_line_search(const SysDev* d_sys, int nsys, hipStream_t s) {
  hipLaunchKernelGGL(g_coef_partials, dim3(GROUP_BLOCKS, nsys), dim3(NT), 0, s, d_sys);
  hipLaunchKernelGGL(g_line_final, dim3(1, nsys), dim3(NT), 0, s, d_sys);
  return hipGetLastError();
}

hipError_t group_update(const SysDev* d_sys, int nsys, hipStream_t s) {
  hipLaunchKernelGGL(g_update_mn, dim3(4 * GROUP_BLOCKS, nsys), dim3(NT), 0, s, d_sys);
  hipLaunchKernelGGL(g_update_mm, dim3(GROUP_BLOCKS, nsys), dim3(NT), 0, s, d_sys);
  hipLaunchKernelGGL(g_update_final, dim3(1, nsys), dim3(NT), 0, s, d_sys);
  return hipGetLastError();
}

hipError_t identity_minus(const double* SW, double* out, int M, double diag, double scale,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_identity_minus, dim3(ew_blocks((int64_t)M * M)), dim3(NT), 0, s, SW, out, M,
                     diag, scale);
  return hipGetLastError();
}

hipError_t axpby_f64(const double* a, const double* b, double* out, double ca, double cb, int64_t n,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_axpby, dim3(ew_blocks(n)), dim3(NT), 0, s, a, b, out, ca, cb, n);
  return hipGetLastError();
}

}  // namespace omm
