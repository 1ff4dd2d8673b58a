// FP64 / FP32 MFMA products in small tiles without workgroup staging.
//
// An FP64 (FP32) 16x16x4 MFMA keeps its SIMD busy for 64 (32) cycles, so at these types a wave
// needs few operand bytes per cycle, and what costs time is a tile grid that leaves CUs idle, a
// barrier per K step and scattered operand loads. Here the four waves of a workgroup share one
// output tile of (TM 16) x (TN 16), each taking every WK-th K step on its own (no barriers); their
// partial sums meet in LDS at the end, in FP64 and in wave order. A CU then works on one small
// tile at a time and direct_choose picks the shape that divides the product best.
//
// Operands. A K step is 64 bytes of every operand row: KS = 8 (FP64) or 16 (FP32) k, lane group
// kq = l / 16 taking the 16-byte chunk kq (VM elements, one per MFMA). (The order of k within a step
// is a free choice as long as A and B agree.)
//  * r-contiguous (RC): adjacent lanes hold adjacent rows, so fragments are loaded from memory
//    straight into registers, two rows per lane: fragments 2p and 2p + 1 hold the even and odd
//    rows of 32 (frag_row).
//  * k-contiguous (KC): the fragment layout puts adjacent lanes on different rows, and the address
//    unit coalesces adjacent lanes only (16-byte loads of such fragments ran at one lane per
//    cycle, 15 bytes per cycle and CU, whatever the cache held). So each wave brings its rows in
//    by direct-to-LDS loads, four lanes to a 64-byte row chunk, into a private ring of NB steps
//    (vmcnt waits, no barrier) and reads its fragments from there, one step ahead. The chunks of a
//    row are rotated by row / 2, which puts the 16 lanes an LDS read serves per clock on distinct
//    banks.
// Symmetric operands (Hs, S, P, HW, SW) can be read either way; RC is the cheaper one.
//
// Measured against the staged tiles of omm_gemm_impl.h (64 x 64 or 128 x 128, whichever was faster),
// one launch: FP64 131 x 717 x 717 58 -> 7.4 us, 384 x 2048 x 2048 150 -> 54 us (60 TFLOP/s), four
// 384 x 384 x 2048 148 -> 45 us, 2000 x 13000 x 13000 14.0 -> 10.4 ms (65 TFLOP/s); FP32 two 768 x
// 4096 x 4096 652 -> 439 us (117 TFLOP/s). What is left at the large sizes is the operand traffic
// from L2 (pinning every load to one step takes the RC form from 59 to 70 TFLOP/s, the rate of
// the library's 8192^3 FP64 product).
//
// Bounds. Rows past the edge are clamped to the last row (their outputs are never stored); the
// part of K past the last whole step is read element by element with zeros outside.
#pragma once

#include "omm_gemm_impl.h"

namespace omm {
namespace gemm_detail {

constexpr int WK = 4;  // waves of a workgroup, sharing the K steps of one tile

// Row (or column) within the tile of MFMA row rr of fragment f: pairs of fragments interleave for
// an r-contiguous operand.
template <int LAYOUT, int TF>
__device__ __forceinline__ int frag_row(int f, int rr) {
  if constexpr (LAYOUT == RC && TF % 2 == 0) return (f >> 1) * 32 + 2 * rr + (f & 1);
  else return f * 16 + rr;
}

// s_waitcnt vmcnt <= n only
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | (((N >> 4) & 3) << 14));
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void wait_lgkm0() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
  __builtin_amdgcn_sched_barrier(0);
}

template <typename mt, typename T, int LAYOUT, int TF, int NB>
struct DirectOperand {
  static constexpr bool LDS = LAYOUT == KC;
  static constexpr bool PAIR = LAYOUT == RC && TF % 2 == 0;
  static constexpr int VM = 16 / sizeof(mt);  // k of one lane and step, consecutive
  static constexpr int KS = 4 * VM;           // k of a step
  static_assert(!LDS || sizeof(T) == sizeof(mt), "k-contiguous operands have the MFMA's type");
  // memory instructions of one step
  static constexpr int NLOAD = LDS ? TF : PAIR ? TF / 2 * VM : TF * VM;
  static constexpr int RING = LDS ? NB * TF * 1024 : 0;  // LDS bytes of one wave
  typedef T pair_t __attribute__((ext_vector_type(2), aligned(sizeof(T))));
  typedef mt lvec_t __attribute__((ext_vector_type(VM)));
  struct Regs {
    T v[TF][VM];  // converted to the MFMA type where they are used
  };

  const char* base;  // element (r0, 0)
  int64_t ld;
  unsigned off[TF];  // RC: byte offset of this lane's row of fragment f at its first k;
                     // KC: of the row and chunk this lane fetches in load j
  __amdgpu_buffer_rsrc_t rs;
  char* ring;
  int lds0;  // KC: byte offset of this lane's chunk of fragment 0 within a step of the ring
  Regs r[LDS ? 2 : NB];

  __device__ __forceinline__ void init(const void* X, int64_t ld_, int r0, int rmax, int lane,
                                       char* ring_) {
    ld = ld_;
    const int li = lane & 15, kq = lane >> 4;
    base = static_cast<const char*>(X) + (LDS ? (int64_t)r0 * ld : (int64_t)r0) * sizeof(T);
    if constexpr (LDS) {
      ring = ring_;
      const int64_t bytes = (int64_t)(rmax - r0) * ld * sizeof(T);
      rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), (short)0,
                                             (int)(unsigned)min(bytes, (int64_t)0xffffffff),
                                             0x00020000);
      const int lrow = lane >> 2, chunk = ((lane & 3) - (lane >> 3)) & 3;
#pragma unroll
      for (int j = 0; j < TF; ++j)
        off[j] = (unsigned)((min(r0 + 16 * j + lrow, rmax - 1) - r0) * ld * (int)sizeof(T)) + 16 * chunk;
      lds0 = li * 64 + ((kq + (li >> 1)) & 3) * 16;
    } else {
#pragma unroll
      for (int f = 0; f < TF; ++f) {
        // a pair load reads rows r and r + 1: past an even rmax it starts at rmax - 2
        const int row = min(r0 + frag_row<LAYOUT, TF>(f, li),
                            PAIR && f % 2 == 0 ? (rmax - 1) & ~1 : rmax - 1);
        off[f] = (unsigned)((kq * VM * ld + row - r0) * (int)sizeof(T));
      }
    }
  }

  // the whole step at k0: into step q of the ring, or into register buffer q
  __device__ __forceinline__ void issue(int q, int k0) {
    if constexpr (LDS) {
#pragma unroll
      for (int j = 0; j < TF; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rs, reinterpret_cast<__attribute__((address_space(3))) void*>(
                    (__attribute__((address_space(3))) char*)(ring + (q * TF + j) * 1024)),
            16, off[j], k0 * (int)sizeof(T), 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < VM; ++e) {
        const char* p = base + (int64_t)(k0 + e) * ld * sizeof(T);
        if constexpr (PAIR) {
#pragma unroll
          for (int f = 0; f < TF; f += 2) {
            const pair_t x = *reinterpret_cast<const pair_t*>(p + off[f]);
            r[q].v[f][e] = x[0];
            r[q].v[f + 1][e] = x[1];
          }
        } else {
#pragma unroll
          for (int f = 0; f < TF; ++f) r[q].v[f][e] = *reinterpret_cast<const T*>(p + off[f]);
        }
      }
    }
  }

  // KC: fragments of step q of the ring into register buffer d
  __device__ __forceinline__ void fetch(int d, int q) {
    if constexpr (LDS) {
#pragma unroll
      for (int f = 0; f < TF; ++f) {
        const lvec_t x = *reinterpret_cast<const lvec_t*>(ring + (q * TF + f) * 1024 + lds0);
#pragma unroll
        for (int e = 0; e < VM; ++e) r[d].v[f][e] = x[e];
      }
    }
  }

  // partial step at k0 straight into register buffer 0: k < K only, zeros past K
  __device__ __forceinline__ void load_tail(int k0, int K, int r0, int rmax, int lane) {
    const int li = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int e = 0; e < VM; ++e) {
      const int k = k0 + kq * VM + e;
#pragma unroll
      for (int f = 0; f < TF; ++f) {
        const int row = min(r0 + frag_row<LAYOUT, TF>(f, li), rmax - 1) - r0;
        const char* p = base + (LDS ? row * ld + k : k * ld + row) * (int64_t)sizeof(T);
        r[0].v[f][e] = k < K ? *reinterpret_cast<const T*>(p) : (T)0;
      }
    }
  }
};

// Linear tile index -> (tm, tn) in bands of four tile columns, columns fastest: the 32 tiles an
// XCD works on at a time are then 8 x 4 (24 operand panels for 32 tiles, against 33 down a single
// column).
__device__ __forceinline__ void band_tile(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int band = t / (tiles_m * 4);
  const int c0 = band * 4, w = min(4, tiles_n - c0);
  const int r = t - band * tiles_m * 4;
  tm = r / w;
  tn = c0 + r % w;
}

// LDS of one workgroup: the operand rings of its waves, reused for the partial sums.
template <typename OA, typename OB>
constexpr int direct_lds() {
  constexpr int ring = WK * (OA::RING + OB::RING), red = WK * WK * 2048;
  return ring > red ? ring : red;
}

// The output tile (tm, tn) of op, by the WK waves of a workgroup. USER: a value for each calling kernel; where
// both call the same instantiation, the compiler's host pass rejects the second call ("substitution
// failure").
template <int MODE, typename TA, typename TB, typename TC, typename TX, int LA, int LB, int TM,
          int TN, int NB, int USER>
__device__ __forceinline__ void direct_tile(const GemmOp& op, int tm, int tn) {
  typedef typename std::conditional<MODE == CF64, double, float>::type mt;
  typedef typename AccT<MODE>::type acc_t;
  typedef DirectOperand<mt, TA, LA, TM, NB> OA;
  typedef DirectOperand<mt, TB, LB, TN, NB> OB;
  constexpr int VM = OA::VM, KS = OA::KS, NV = OA::NLOAD + OB::NLOAD;
  constexpr bool LDS = OA::LDS || OB::LDS;
  static_assert(NB % 2 == 0, "fragment buffers alternate");
  __shared__ __attribute__((aligned(16))) char smem[direct_lds<OA, OB>()];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = tm * TM * 16, n0 = tn * TN * 16;
  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
  int first = w;  // this wave's first step of the segment (the segments' steps go round robin)
  for (int seg = 0; seg < op.nseg; ++seg) {
    const int K = op.K[seg];
    // A pair load in the last row of an odd-sized r-contiguous operand reads one element past it:
    // into the next k row, which the last k row does not have, so that row goes to the tail.
    const bool odd = (OA::PAIR && op.M % 2 != 0) || (OB::PAIR && op.N % 2 != 0);
    // the K range of the tile, without the known zeros of a triangular operand (tile origins are
    // multiples of KS, so the range starts on a whole step)
    const int kb = op.kcut & KCUT_B_FROM_N ? n0 : 0;
    int ke = K;
    if (op.kcut & KCUT_A_TO_M) ke = min(ke, m0 + TM * 16);
    if (op.kcut & KCUT_B_TO_N) ke = min(ke, n0 + TN * 16);
    const int nfull = ((odd && ke == K ? K - 1 : ke) - kb) / KS;
    OA oa;
    OB ob;
    oa.init(op.A[seg], op.lda[seg], m0, op.M, lane, smem + w * (OA::RING + OB::RING));
    ob.init(op.B[seg], op.ldb[seg], n0, op.N, lane, smem + w * (OA::RING + OB::RING) + OA::RING);
    // MFMAs of elements E0 .. E1 - 1 of a step
    auto compute = [&](int da, int db, auto E0, auto E1) {
#pragma unroll
      for (int e = E0; e < E1; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = mfma4((mt)oa.r[da].v[i][e], (mt)ob.r[db].v[j][e], acc[i][j]);
    };
    constexpr std::integral_constant<int, 0> e0{};
    constexpr std::integral_constant<int, VM / 2> eh{};
    constexpr std::integral_constant<int, VM> e1{};
    const int cnt = first < nfull ? (nfull - first + WK - 1) / WK : 0;
    if (cnt > 0) {
      // k of this wave's step i (past the end: the last one again, unused)
      auto kof = [&](int i) { return kb + (first + min(i, cnt - 1) * WK) * KS; };
      // Ring step p holds step i with i % NB == p. Loads into the ring run NB steps ahead of the
      // MFMAs and their fragments are read one step ahead; register loads run NB - 1 ahead.
      auto issue = [&](int q, int i) {  // q = i % NB, known at compile time
        if constexpr (OA::LDS) oa.issue(q, kof(i));
        else oa.issue((q + NB - 1) % NB, kof(i - 1));
        if constexpr (OB::LDS) ob.issue(q, kof(i));
        else ob.issue((q + NB - 1) % NB, kof(i - 1));
      };
      auto regs_a = [](int q) { return OA::LDS ? q % 2 : q; };
      auto regs_b = [](int q) { return OB::LDS ? q % 2 : q; };
      static_for<NB>([&](auto q) {
        if constexpr (q == 0) {
          if constexpr (OA::LDS) oa.issue(0, kof(0));
          if constexpr (OB::LDS) ob.issue(0, kof(0));
        } else {
          issue(q, q);
        }
        __builtin_amdgcn_sched_barrier(0);  // the vmcnt waits count on this order
      });
      if constexpr (LDS) {
        wait_vm<(NB - 1) * NV>();
        oa.fetch(0, 0);
        ob.fetch(0, 0);
      }
      int it = 0;
      for (; it + NB <= cnt; it += NB)
        static_for<NB>([&](auto q) {
          // loads in the first half of the step's MFMAs, fragment reads in the second: left to
          // itself the scheduler sinks both behind the MFMAs and every step waits for them
          constexpr int NR = (OA::LDS ? TM : 0) + (OB::LDS ? TN : 0), NM = VM / 2 * TM * TN;
          // the ring step about to be refilled has been read
          if constexpr (LDS) wait_lgkm0();
          issue(q, it + q + NB);
          compute(regs_a(q), regs_b(q), e0, eh);
          static_for<NV>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NM / NV > 0 ? NM / NV : 1, 0);
          });
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (LDS) {
            wait_vm<(NB - 1) * NV>();
            oa.fetch((q + 1) % 2, (q + 1) % NB);
            ob.fetch((q + 1) % 2, (q + 1) % NB);
          }
          compute(regs_a(q), regs_b(q), eh, e1);
          if constexpr (LDS)
            static_for<NR>([&](auto) {
              __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x008, NM / (NR > 0 ? NR : 1) > 0 ? NM / (NR > 0 ? NR : 1) : 1, 0);
            });
          __builtin_amdgcn_sched_barrier(0);
        });
      static_for<NB - 1>([&](auto q) {
        if (it + q < cnt) {
          if constexpr (LDS) {
            wait_vm<0>();
            oa.fetch((q + 1) % 2, (q + 1) % NB);
            ob.fetch((q + 1) % 2, (q + 1) % NB);
          }
          compute(regs_a(q), regs_b(q), e0, e1);
        }
      });
      if constexpr (LDS) wait_vm<0>();  // nothing lands in the ring after this
    }
    const int kt = kb + nfull * KS;
    if (ke > kt && (nfull % WK) == first) {
      oa.load_tail(kt, ke, m0, op.M, lane);
      ob.load_tail(kt, ke, n0, op.N, lane);
      compute(0, 0, e0, e1);
    }
    first = (first + 1) % WK;
  }
  // Partial sums of the WK waves: WK fragments at a time through LDS; wave w adds up (in wave order)
  // and stores fragment c + w.
  double* red = reinterpret_cast<double*>(smem);
  constexpr int NF = TM * TN;
#pragma unroll
  for (int c = 0; c < NF; c += WK) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < WK; ++q)
      if (c + q < NF)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[((w * WK + q) * 4 + r) * 64 + lane] = (double)acc[(c + q) / TN][(c + q) % TN][r];
    __syncthreads();
    const int f = c + w;
    if (f >= NF) continue;
    const int i = f / TN, j = f % TN;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < WK; ++q) s += red[((q * WK + w) * 4 + r) * 64 + lane];
      const int rr = MODE == CF64 ? (lane >> 4) + 4 * r : 4 * (lane >> 4) + r;
      const int row = m0 + frag_row<LA, TM>(i, rr), col = n0 + frag_row<LB, TN>(j, lane & 15);
      if (row < op.M && col < op.N) {
        double v = op.alpha * s;
        if (op.X) v += op.beta * (double)ldg<TX>(op.X, (int64_t)row * op.ldx + col);
        if (!op.tri || row <= col) store_out<TC>(op, row, col, v);
        if (op.pair_rows) {  // the pair rotation's element (see GemmOp), in place of a separate pass
          const int half = op.N >> 1;
          const TC c = (TC)v;
          static_cast<TC*>(op.C)[(int64_t)(row + op.pair_rows) * op.ldc +
                                 (col < half ? col + half : col - half)] = col < half ? c : -c;
        }
        // symmetric result: the mirror element too, in place of a separate mirror pass
        if (op.tri == 1 && row < col) store_out<TC>(op, col, row, v);
      }
    }
  }
}

// Workgroup -> tile in runs of consecutive tiles per XCD, dealt in turn. The grid is whole rounds of 8
// runs (deal_grid).
__device__ __forceinline__ int dealt_tile(int bid, int total) {
  const int run = deal_run(total), x = bid & 7, y = bid >> 3;
  return (y / run) * (8 * run) + x * run + y % run;
}

// Up to 4 same-shape products (blockIdx.z). Each XCD gets one contiguous run of tiles, except where the
// work of a tile depends on its place (symmetric results, triangular operands): there short runs
// are dealt to the XCDs in turn, from the end with the long K ranges and the columns that reach
// furthest above the diagonal (one run each left the last XCD with twice the average: 477 instead
// of 256 us for a symmetric 4096 x 4096 x 768).
template <int MODE, typename TA, typename TB, typename TC, typename TX, int LA, int LB, int TM,
          int TN, int NB, int OCC>
__global__ __launch_bounds__(WK * 64, OCC) void gemm_direct_kernel(GemmBatch batch,
                                                                   const int* done, int, double*) {
  if (done && *done) return;
  const GemmOp& op = batch.op[blockIdx.z];
  constexpr int BM = TM * 16, BN = TN * 16;
  const int tiles_m = (op.M + BM - 1) / BM, tiles_n = (op.N + BN - 1) / BN;
  const int total = tiles_m * tiles_n, per = (total + 7) >> 3;
  int t;
  if (op.tri || op.kcut) {
    t = dealt_tile(blockIdx.x, total);
    if (!(op.kcut & KCUT_B_FROM_N)) t = total - 1 - t;
  } else {
    t = (int)(blockIdx.x >> 3) < per ? (blockIdx.x & 7) * per + (blockIdx.x >> 3) : total;
  }
  if (t < 0 || t >= total) return;
  int tm, tn;
  band_tile(t, tiles_m, tiles_n, tm, tn);
  if (op.tri && tm * BM > tn * BN + BN - 1) return;  // wholly below the diagonal: see the mirror
  direct_tile<MODE, TA, TB, TC, TX, LA, LB, TM, TN, NB, 0>(op, tm, tn);
}

// Products of uneven shapes: one workgroup per tile of the concatenated tile lists, dealt to the XCDs in
// short runs. Tiles of a stopped system return at once.
template <int MODE, typename TA, typename TB, typename TC, typename TX, int LA, int LB, int TM,
          int TN, int NB, int OCC>
__global__ __launch_bounds__(WK * 64, OCC) void gemm_direct_grouped(GroupedArgs g) {
  constexpr int BM = TM * 16, BN = TN * 16;
  const int total = g.tile_start[g.nops];
  const int t = dealt_tile(blockIdx.x, total);
  if (t >= total) return;
  int lo = 0, hi = g.nops - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (g.tile_start[mid] <= t) lo = mid; else hi = mid - 1;
  }
  const int* dn = g.done[lo];
  if (dn && *dn) return;
  const GemmOp& op = g.ops[lo];  // by reference: a local copy would sit in scratch memory
  const int tiles_m = (op.M + BM - 1) / BM, tiles_n = (op.N + BN - 1) / BN;
  int tm, tn;
  band_tile(t - g.tile_start[lo], tiles_m, tiles_n, tm, tn);
  if (op.tri && tm * BM > tn * BN + BN - 1) return;
  direct_tile<MODE, TA, TB, TC, TX, LA, LB, TM, TN, NB, 1>(op, tm, tn);
}

// The tile shapes (TM, TN, ring steps NB, workgroups per CU OCC), macro tiles DIRECT_TILE0 ..
template <int MODE, typename TA, typename TB, typename TC, typename TX, int LA, int LB>
gemm_fn pick_direct(int tile) {
  switch (tile - DIRECT_TILE0) {
    case 0: return gemm_direct_kernel<MODE, TA, TB, TC, TX, LA, LB, 1, 2, 4, 1>;
    case 1: return gemm_direct_kernel<MODE, TA, TB, TC, TX, LA, LB, 2, 2, 2, 1>;
    case 2: return gemm_direct_kernel<MODE, TA, TB, TC, TX, LA, LB, 3, 3, 2, 1>;
    case 3: return gemm_direct_kernel<MODE, TA, TB, TC, TX, LA, LB, 3, 4, 2, 1>;
    case 4: return gemm_direct_kernel<MODE, TA, TB, TC, TX, LA, LB, 4, 4, 2, 2>;
    case 5: return gemm_direct_kernel<MODE, TA, TB, TC, TX, LA, LB, 4, 6, 2, 1>;
    default: return nullptr;
  }
}
template <int MODE, typename TA, typename TB, typename TC, typename TX, int LA, int LB>
grouped_fn pick_direct_grouped(int tile) {
  switch (tile - DIRECT_TILE0) {
    case 0: return gemm_direct_grouped<MODE, TA, TB, TC, TX, LA, LB, 1, 2, 4, 1>;
    case 1: return gemm_direct_grouped<MODE, TA, TB, TC, TX, LA, LB, 2, 2, 2, 1>;
    case 2: return gemm_direct_grouped<MODE, TA, TB, TC, TX, LA, LB, 3, 3, 2, 1>;
    case 3: return gemm_direct_grouped<MODE, TA, TB, TC, TX, LA, LB, 3, 4, 2, 1>;
    case 4: return gemm_direct_grouped<MODE, TA, TB, TC, TX, LA, LB, 4, 4, 2, 2>;
    case 5: return gemm_direct_grouped<MODE, TA, TB, TC, TX, LA, LB, 4, 6, 2, 1>;
    default: return nullptr;
  }
}

}  // namespace gemm_detail
}  // namespace omm
