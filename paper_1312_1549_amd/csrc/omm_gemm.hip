// GEMM launcher: picks the instantiation for a descriptor, sizes the grid (XCD-remapped tile
// ids, split-K along y, up to 4 same-shape products along z) and reduces split-K partials in a
// fixed order.
#include <math.h>

#include <algorithm>

#include "omm_gemm_impl.h"

namespace omm {
namespace gemm_detail {
gemm_fn pick_f64(const GemmDesc& d);
gemm_fn pick_f32(const GemmDesc& d);
gemm_fn pick_bf16x3(const GemmDesc& d);
gemm_fn pick_bf16x2(const GemmDesc& d);
sk_fn pick_sk_bf16x3(const GemmDesc& d);
sk_fn pick_sk_bf16x2(const GemmDesc& d);
grouped_fn pick_grouped_f32(const GemmDesc& d);
grouped_fn pick_grouped_f64(const GemmDesc& d);

namespace {
// Sums the split-K partials (type TP: that of the accumulators) in split order, FP64, and applies the
// epilogue: four columns per thread, rows blockIdx.y, blockIdx.y + gridDim.y, ..
template <typename TC, typename TX, typename TP>
__global__ __launch_bounds__(256) void splitk_reduce(GemmBatch batch, const int* done, int nsplit,
                                                     const TP* ws) {
  if (done && *done) return;
  typedef TP P4 __attribute__((ext_vector_type(4)));
  const GemmOp& op = batch.op[blockIdx.z];
  const int64_t mn = (int64_t)op.M * op.N, step = mn * gridDim.z;
  const int c0 = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c0 >= op.N) return;
  const bool whole = op.N % 4 == 0;  // rows of partials start on 4-element boundaries
  for (int row = blockIdx.y; row < op.M; row += gridDim.y) {
    if (op.tri && row > c0 + 3) continue;  // below the diagonal: its tile may not have run
    const TP* p = ws + (int64_t)blockIdx.z * mn + (int64_t)row * op.N + c0;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int sp = 0; sp < nsplit; ++sp, p += step) {
      if (whole) {
        const P4 v = *reinterpret_cast<const P4*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += (double)v[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c0 + e < op.N) s[e] += (double)p[e];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int col = c0 + e;
      if (col >= op.N || (op.tri && row > col)) continue;
      double v = op.alpha * s[e];
      if (op.X) v += op.beta * (double)ldg<TX>(op.X, (int64_t)row * op.ldx + col);
      store_out<TC>(op, row, col, v);
    }
  }
}
// C[i][j] = C[j][i] for i > j of every symmetric (tri) product: 32 x 32 blocks on and below the
// diagonal, each read transposed through LDS from its mirror block.
template <typename TC>
__global__ __launch_bounds__(256) void mirror_lower(GemmBatch batch, const int* done) {
  if (done && *done) return;
  const GemmOp& op = batch.op[blockIdx.z];
  if (op.tri != 1) return;
  const int bi = blockIdx.y * 32, bj = blockIdx.x * 32;  // destination block (rows bi, cols bj)
  if (bj > bi || bi >= op.M) return;
  __shared__ TC t[32][33];
  TC* C = static_cast<TC*>(op.C);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {  // source block: rows bj, cols bi
    const int i = bj + r, j = bi + tx;
    if (i < op.M && j < op.N) t[r][tx] = C[(int64_t)i * op.ldc + j];
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int i = bi + r, j = bj + tx;
    if (i < op.M && j < op.N && i > j) C[(int64_t)i * op.ldc + j] = t[tx][r];
  }
}
// The second half of the rows of every paired product (see GemmOp) and of its planes, from the first: a
// pass of its own for the staged and BF16 tiles (in their epilogue it costs the direct-to-LDS tile
// registers: 292 -> 361 us for the block-sparse [HD | SD] of 6500 orbitals).
template <typename TC>
__global__ __launch_bounds__(256) void pair_fill(GemmBatch batch, const int* done) {
  if (done && *done) return;
  const GemmOp& op = batch.op[blockIdx.z];
  if (!op.pair_rows) return;
  const int half = op.N >> 1, c = blockIdx.x * 256 + threadIdx.x;
  if (c >= op.N) return;
  const bool neg = c < half;
  const int src = neg ? c + half : c - half;
  const unsigned short sgn = neg ? 0x8000 : 0;  // bf16 rounding is symmetric in the sign
  TC* C = static_cast<TC*>(op.C);
  unsigned short* planes[2] = {static_cast<unsigned short*>(op.Chi), static_cast<unsigned short*>(op.Clo)};
  for (int r = blockIdx.y; r < op.M; r += gridDim.y) {
    const TC v = C[(int64_t)r * op.ldc + src];
    C[(int64_t)(r + op.pair_rows) * op.ldc + c] = neg ? -v : v;
    for (unsigned short* p : planes)
      if (p) p[(int64_t)(r + op.pair_rows) * op.ldp + c] = p[(int64_t)r * op.ldp + src] ^ sgn;
  }
}
}  // namespace
}  // namespace gemm_detail

using namespace gemm_detail;

namespace {
// split-K partials in the accumulators' type
size_t splitk_ws_bytes(const GemmDesc& d, const GemmOp* ops, int nops) {
  if (d.splitk <= 1) return 0;
  return (size_t)d.splitk * nops * (size_t)ops[0].M * ops[0].N * (d.compute == CF64 ? sizeof(double) : sizeof(float));
}
}  // namespace

size_t gemm_ws_bytes(const GemmDesc& d, const GemmOp* ops, int nops) {
  if (d.tile == 6) return (size_t)2 * SK_GRID * DMA_BM * DMA_BN * sizeof(float);
  return splitk_ws_bytes(d, ops, nops);
}

int gemm_num_tiles() { return NTILES; }

// Which small tile an FP64 / FP32 launch takes. A CU works on one tile's MFMAs at a time, so the
// launch lasts about ceil(tiles / 256) rounds of one tile's MFMAs, at the rate the tile's shape
// reaches, plus what a round exposes of its first loads and its sum over the waves (more for the
// larger tiles, of which fewer share a CU); the least of that wins, the larger tile on a tie (fewer
// operand bytes). Rates relative to 72 (FP64) and 154 (FP32) TFLOP/s and the exposed times are
// measured. FP64 384 x 2048 x 2048 (rule / measured, us): 16x32 73 / 75, 32x32 55 / 55, 48x48 76 / 74,
// 48x64 53 / 54, 64x64 68 / 66, 64x96 98 / 96; two FP32 768 x 4096 x 4096: 32x32 556 / 541, 48x64 460 /
// 448, 64x64 454 / 439.
//
// 32 x 32 asks for the most operand bytes per flop that still pays, and two corrections stand for that.
// Times below are whole launches (us), 32x32 against the best other tile; A of M x K, B of N x K, both
// k-contiguous.
//  * Under three rounds its rate counts 0.75: the four projections of 384 x 384 x 2048 in FP64 (two of
//    them symmetric) take 52 with it, 45 with 48x48. Two of 256 x 1024 x 1024 go the other way (19.6
//    against 27.7), but there it is chosen all the same, the others needing as many rounds.
//  * From three rounds on, in FP32 up to K = 1024, its rate counts 0.75 instead of 0.62. Four of 256 x 2048 x K, against 64x64: K =
//    512 22.8 / 23.2, 768 31.7 / 30.6, 1024 38.5 / 37.5, 1152 42.3 / 40.8, 1536 56.8 / 51.3, 2048 74.0 /
//    65.3. Four of 384 x 2048 x K, against 48x64: 512 33.2 / 34.2, 1024 57.8 / 54.7, 1152 63.5 / 60.4,
//    1536 84.1 / 76.4. The two cross between 512 and 768, and up to the line the choice is within 6 % of
//    the best; batches whose systems' K runs from 256 to 1024 share one tile (101 us a launch with 32x32,
//    105 to 135 with the others), which is why the line lies beyond the crossing.
// Of 126 FP64 and FP32 products with 256 to 4096 columns the choice is within 7 % of the fastest tile in
// 113. The others are FP32: two rounds of 32x32 with K >= 1000 (two of 256 x 1024 x 2048 take 28.0, 20.2
// with 32x32; two of 192 x 1024 x 1024 14.3, 11.6) and five rounds (four of 160 x 2048 x 1024 take 32.5,
// 28.8 with 48x64).
void direct_choose(GemmDesc& d, const GemmOp* ops, int nops) {
  static const double rate64[NDIRECT] = {0.64, 0.85, 0.93, 0.90, 0.94, 0.97};
  static const double rate32[NDIRECT] = {0.45, 0.62, 0.75, 0.77, 0.78, 0.85};
  static const double exposed[NDIRECT] = {0.5, 0.6, 2.0, 3.0, 4.0, 6.0};  // us per round
  const bool f64 = d.compute == CF64;
  const double fma_us = (f64 ? 72e6 : 154e6) / 2 / 256;  // multiply-adds per CU and us
  double kmax = 1.0;
  auto k_of = [](const GemmOp& op) { return (double)op.K[0] + (op.nseg > 1 ? op.K[1] : 0); };
  for (int o = 0; o < nops; ++o) kmax = std::max(kmax, k_of(ops[o]));
  double best = 0.0;
  for (int i = 0; i < NDIRECT; ++i) {
    const int bm = DIRECT_BM[i], bn = DIRECT_BN[i];
    double tiles = 0.0;  // weighted by K (the products of a grouped launch differ)
    for (int o = 0; o < nops; ++o) {
      const double tm = (ops[o].M + bm - 1) / bm, tn = (ops[o].N + bn - 1) / bn;
      // a symmetric product computes the tiles that reach the diagonal
      tiles += (ops[o].tri ? tm * tn / 2 + std::max(tm, tn) / 2 : tm * tn) * k_of(ops[o]) / kmax;
    }
    const double rounds = ceil(tiles / 256.0);
    double rate = f64 ? rate64[i] : rate32[i];
    if (i == 1 && rounds < 3) rate *= 0.75;
    else if (i == 1 && !f64 && kmax <= 1024) rate = 0.75;
    const double cost = rounds * (bm * bn * kmax / (rate * fma_us) + exposed[i]);
    if (i == 0 || cost <= best) {
      best = cost;
      d.tile = DIRECT_TILE0 + i;
    }
  }
  d.splitk = 1;
}

namespace {
// Preconditions of the direct-to-LDS tile: 16-byte aligned planes, leading dimensions that are
// multiples of 8, and K-segment boundaries on 8-element boundaries.
bool dma_ok(const GemmDesc& d, const GemmOp* ops, int nops) {
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  for (int i = 0; i < nops; ++i) {
    const GemmOp& op = ops[i];
    if (op.nseg == 2 && op.K[0] % 8 != 0) return false;
    for (int g = 0; g < op.nseg; ++g) {
      if (op.lda[g] % 8 != 0 || op.ldb[g] % 8 != 0) return false;
      // lane addresses are 32-bit byte offsets from the plane base
      constexpr int64_t lim = (int64_t)1 << 31;
      if ((int64_t)op.M * op.lda[g] >= lim || (int64_t)op.N * op.ldb[g] >= lim) return false;
      if (!al(op.A[g]) || !al(op.B[g])) return false;
      if (!one_plane_a(d.compute) && !al(op.Alo[g])) return false;
      if (!one_plane_b(d.compute) && !al(op.Blo[g])) return false;
    }
  }
  return true;
}
}  // namespace

namespace {
sk_fn pick_sk(const GemmDesc& d) {
  if (d.compute == CBF16X3) return pick_sk_bf16x3(d);
  if (d.compute == CBF16X2A || d.compute == CBF16X2B || d.compute == CBF16X1)
    return pick_sk_bf16x2(d);
  return nullptr;
}
}  // namespace

bool gemm_supported(const GemmDesc& d) {
  if (d.tile < 0 || d.tile >= NTILES) return false;
  if (d.tile == 6) return d.splitk <= 1 && pick_sk(d) != nullptr;
  if (tile_direct(d.tile) && d.splitk > 1) return false;
  if (d.compute == CF64) return pick_f64(d) != nullptr;
  if (d.compute == CF32) return pick_f32(d) != nullptr;
  if (d.compute == CBF16X3) return pick_bf16x3(d) != nullptr;
  if (d.compute == CBF16X2A || d.compute == CBF16X2B || d.compute == CBF16X1)
    return pick_bf16x2(d) != nullptr;
  return false;
}

hipError_t gemm_grouped_launch(const GemmDesc& d, const GemmOp* d_ops, const int* d_tile_start,
                               const int* const* d_done, int nops, int tiles, hipStream_t s) {
  if ((d.compute != CF32 && d.compute != CF64) || nops < 1 || tiles < 1 || !tile_direct(d.tile))
    return hipErrorInvalidValue;
  grouped_fn fn = d.compute == CF64 ? pick_grouped_f64(d) : pick_grouped_f32(d);
  if (!fn) return hipErrorInvalidValue;
  GroupedArgs g{d_ops, d_tile_start, d_done, nops};
  hipLaunchKernelGGL(fn, dim3(deal_grid(tiles)), dim3(tile_threads(d.tile, d.compute)), 0,
                     s, g);
  return hipGetLastError();
}

int gemm_tile_rows(int tile, int mode) { return tile_bm(tile, mode); }
int gemm_tile_cols(int tile, int mode) { return tile_bn(tile, mode); }

namespace {
hipError_t launch_products(const GemmDesc& d, const GemmOp* ops, int nops, const int* done,
                           double* ws, size_t ws_bytes, hipStream_t s) {
  if (nops < 1 || nops > 4) return hipErrorInvalidValue;
  GemmBatch b;
  for (int i = 0; i < nops; ++i) {
    b.op[i] = ops[i];
    if (ops[i].M != ops[0].M || ops[i].N != ops[0].N) return hipErrorInvalidValue;
    if (ops[i].nseg < 1 || ops[i].nseg > 2) return hipErrorInvalidValue;
  }
  const int M = ops[0].M, N = ops[0].N;
  if (M <= 0 || N <= 0) return hipSuccess;
  if (d.tile < 0 || d.tile >= NTILES) return hipErrorInvalidValue;
  GemmDesc dd = d;
  bool sparse = false;
  for (int i = 0; i < nops; ++i) sparse |= ops[i].kptr != nullptr;
  if (sparse) {
    // block-sparse B lists are read over the whole K range: BF16 modes by the direct-to-LDS
    // tile (which stages a column tile's list in LDS), FP64/FP32 by the register tiles (whose
    // column tiles, 64 to 256 wide, lie within one 256-column list tile)
    for (int i = 0; i < nops; ++i)
      if (ops[i].nseg != 1 || !ops[i].kidx) return hipErrorInvalidValue;
    if (is_bf16_mode(dd.compute)) {
      for (int i = 0; i < nops; ++i)
        if ((ops[i].K[0] + SPARSE_BK - 1) / SPARSE_BK > SPARSE_KL_MAX) return hipErrorInvalidValue;
      if (!dma_ok(dd, ops, nops)) return hipErrorInvalidValue;
      dd.tile = 5;
    } else if (dd.tile > 4) {
      return hipErrorInvalidValue;
    }
    dd.splitk = 1;
  }
  if (dd.tile == 6) {
    if (dma_ok(dd, ops, nops)) {
      sk_fn fn = pick_sk(dd);
      if (!fn || dd.splitk > 1) return hipErrorInvalidValue;
      if (!ws || ws_bytes < gemm_ws_bytes(dd, ops, nops)) return hipErrorInvalidValue;
      int tiles = 0;  // tile-ops over all products
      for (int i = 0; i < nops; ++i) tiles += op_tiles(ops[i], DMA_BM, DMA_BN);
      const int ktot = ops[0].K[0] + (ops[0].nseg > 1 ? ops[0].K[1] : 0);
      for (int i = 1; i < nops; ++i)
        if (ops[i].nseg != ops[0].nseg || ops[i].K[0] != ops[0].K[0] ||
            (ops[0].nseg > 1 && ops[i].K[1] != ops[0].K[1]))
          return hipErrorInvalidValue;  // one K schedule for every product of the launch
      SkArgs a;
      a.T = tiles;
      a.nops = nops;
      a.nk = (ktot + DMA_BK - 1) / DMA_BK;
      a.R = a.T / SK_GRID;
      a.W = (int64_t)(a.T - a.R * SK_GRID) * a.nk;
      float* parts = reinterpret_cast<float*>(ws);
      hipLaunchKernelGGL(fn, dim3(SK_GRID), dim3(512), 0, s, b, done, a, parts);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess || a.W == 0) return e;
      sk_fixup_fn fx = dd.tc == T_F64   ? gemm_sk_fixup<double, double>
                       : dd.tx == T_F64 ? gemm_sk_fixup<float, double>
                                        : gemm_sk_fixup<float, float>;
      if (dd.tc == T_F64 && dd.tx != T_F64) return hipErrorInvalidValue;
      hipLaunchKernelGGL(fx, dim3(a.T - a.R * SK_GRID, SK_FIX_CHUNKS), dim3(256), 0, s, b, done, a,
                         SK_GRID, (const float*)parts);
      return hipGetLastError();
    }
    dd.tile = 4;  // same 256 x 256 tile on the register path, one workgroup per tile
    dd.splitk = 1;
  }
  if (tile_direct(dd.tile) && dd.splitk > 1) return hipErrorInvalidValue;
  if (dd.tile == 5 && !dma_ok(dd, ops, nops)) dd.tile = 4;  // same 256 x 256 tile, register path
  gemm_fn fn = nullptr;
  if (dd.compute == CF64) fn = pick_f64(dd);
  else if (dd.compute == CF32) fn = pick_f32(dd);
  else if (dd.compute == CBF16X3) fn = pick_bf16x3(dd);
  else if (dd.compute == CBF16X2A || dd.compute == CBF16X2B || dd.compute == CBF16X1)
    fn = pick_bf16x2(dd);
  if (!fn) return hipErrorInvalidValue;
  const int bm = tile_bm(dd.tile, dd.compute), bn = tile_bn(dd.tile, dd.compute);
  const int tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  const int per = (tiles + 7) / 8;
  const int splitk = dd.splitk > 1 ? dd.splitk : 1;
  if (splitk > 1 && (!ws || ws_bytes < splitk_ws_bytes(dd, ops, nops)))
    return hipErrorInvalidValue;
  // small tiles of symmetric or triangular products are dealt in short runs
  bool dealt = false;
  for (int i = 0; i < nops; ++i) dealt |= ops[i].tri || ops[i].kcut;
  dim3 grid(tile_direct(dd.tile) && dealt ? std::max(deal_grid(tiles), 8 * per) : 8 * per, splitk, nops);
  hipLaunchKernelGGL(fn, grid, dim3(tile_threads(dd.tile, dd.compute)), 0, s, b, done, splitk, ws);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || splitk == 1) return e;
  // blocks of 1024 columns, rows dealt so that a few thousand blocks run
  const int bx = (N + 1023) / 1024;
  const dim3 rgrid(bx, std::min(M, std::max(1, 4096 / (bx * nops))), nops);
  auto reduce = [&](auto* partials) {
    typedef typename std::remove_pointer<decltype(partials)>::type TP;
    void (*red)(GemmBatch, const int*, int, const TP*) =
        dd.tc == T_F64 ? (dd.tx == T_F64 ? splitk_reduce<double, double, TP> : splitk_reduce<double, float, TP>)
                       : (dd.tx == T_F64 ? splitk_reduce<float, double, TP> : splitk_reduce<float, float, TP>);
    hipLaunchKernelGGL(red, rgrid, dim3(256), 0, s, b, done, splitk, (const TP*)partials);
  };
  if (dd.compute == CF64) reduce(ws);
  else reduce(reinterpret_cast<float*>(ws));
  return hipGetLastError();
}
}  // namespace

hipError_t gemm_launch(const GemmDesc& d, const GemmOp* ops, int nops, const int* done, double* ws,
                       size_t ws_bytes, hipStream_t s) {
  if (nops < 1 || nops > 4) return hipErrorInvalidValue;
  bool tri = false;
  for (int i = 0; i < nops; ++i) {
    // the small tiles store the rotated rows of C alone
    if (ops[i].pair_rows && ops[i].Chi && tile_direct(d.tile)) return hipErrorInvalidValue;
    if (!ops[i].tri) continue;
    if (ops[i].M != ops[i].N || ops[i].Chi || ops[i].kptr) return hipErrorInvalidValue;
    tri |= ops[i].tri == 1;
  }
  hipError_t e = launch_products(d, ops, nops, done, ws, ws_bytes, s);
  // the small tiles write both halves of symmetric and paired results themselves
  if (e != hipSuccess || ops[0].M <= 0 || tile_direct(d.tile)) return e;
  GemmBatch b;
  bool pairs = false;
  for (int i = 0; i < nops; ++i) {
    b.op[i] = ops[i];
    pairs |= ops[i].pair_rows != 0;
  }
  if (tri) {
    const int nb = (ops[0].M + 31) / 32;
    hipLaunchKernelGGL(d.tc == T_F64 ? mirror_lower<double> : mirror_lower<float>, dim3(nb, nb, nops),
                       dim3(256), 0, s, b, done);
  }
  if (pairs) {
    const dim3 grid((ops[0].N + 255) / 256, std::min(ops[0].M, 4096), nops);
    hipLaunchKernelGGL(d.tc == T_F64 ? pair_fill<double> : pair_fill<float>, grid, dim3(256), 0, s, b, done);
  }
  return hipGetLastError();
}

}  // namespace omm
