// Complex GEMM tile of the substitutions and of the factorization's sweep on
// the matrix cores: BM rows x BN columns per block of 4 waves.
//
// Row operand.  BM = 64: each wave owns 16 rows and all columns, so the row
// operand needs no LDS: a lane loads its consecutive k of one row straight in
// the MFMA operand layout.  BM = 32: two waves share 16 rows and take half of
// the columns each.
// Column operand.  Loaded once per block, laid out for the MFMA by the thread
// that loaded it and passed through LDS.  Two buffers, one barrier per K
// step; the global loads of a step are issued before the MFMAs of the step
// before it.
// Rows and columns past the operands are clamped to the last valid one (their
// results are never stored); past the K range the column operand is zero and
// the row operand clamped, so no out-of-range value is read.
//
// complex64: on the bf16 matrix cores, at FP32 accuracy (the three-way split of
// Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence
// Datatype For Higher-Precision Computations", ARITH 2019).  A float x is split
// into three bf16 numbers, x = h + m + l: h is x rounded to bf16, m the rounded
// rest, l what is left (24 = 3 x 8 significant bits).  The split is exact for
// 2^-110 <= |x| < 2^128 (1 - 2^-9); below, l ends on bf16's smallest
// subnormal (an error of 2^-134), above, h rounds to infinity.  A real product
// is then formed from the six bf16 products
//   h h' + h m' + m h' + h l' + l h' + m m',
// accumulated in FP32 by the matrix cores, smallest first; the dropped ones
// (m l', l m', l l') are below 2^-24 of |x||x'| (with them the errors below
// are the same).  Root mean square error of a length-K product against FP64,
// normal data, K = 32 / 64 / 256 / 1024, in 1e-7:
//   v_mfma_f32_16x16x4f32     1.02 / 1.45 / 2.86 / 5.72
//   sums running through      0.38 / 0.93 / 2.28 / 4.88
//   a sum per K step (STEP)   0.38 / 0.47 / 0.69 / 1.18
// Running sums are rounded by every one of a step's six instructions, a step's
// own sum only once at the size of the whole.  STEP costs the substitutions 2 to
// 4% (96^3, 64 columns 882 -> 906 us a pruned layer solve) without any effect
// on their error, which the factors' decides, so they let the sums run; the
// factorization takes STEP at the same time (160^3 754 and 755 ms): at 200^3
// (layered) the layer solves' error against complex128 has geometric mean
// 0.97e-5 and largest value 1.2e-4, with running sums 1.03e-5 and 2.2e-4, with
// the FP32 tile of three real products before 1.13e-5 and 1.8e-4.  The largest
// values belong to four nearly singular layers and move by a factor 2 with any
// change of rounding.  Why the split: on gfx950 the FP32 matrix instructions
// run at 134 TFLOP/s (measured loop) and the bf16 ones at 2100, so six products
// per real one still leave 350.  What bounds the tile then is the latency of
// its operand loads, not the matrix cores.  Against the FP32 tile it replaced
// (three real products, both operands in LDS): one interior layer of 100^3 with
// 64 columns 1.75 -> 1.57 ms, a whole refined solve of 64 sources on 96^3 419
// -> 362 ms.
//
// complex128: v_mfma_f64_16x16x4f64 on the real and imaginary parts, four
// real products per complex one, in 144 to 165 registers at 64 columns where
// the tile with both operands in LDS took 376 (one wave per SIMD).  Pruned
// layer solves at 97^3: 21 columns 1240 -> 1045 us, 64 columns 2358 -> 1940
// (with the finer K chunks that the launch lists then take).
#pragma once

#include "kernels_common.h"

namespace helm {
namespace kern {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d4 __attribute__((ext_vector_type(4)));

// K step (complex elements)
template <typename T> constexpr int tile_k() { return sizeof(T) == 4 ? 32 : 16; }

// W floats split into their three bf16 planes (vectors of W elements).  The
// rest of a rounding, x - h, is one v_dot2_f32_bf16 on the rounded pair with
// (-1, 0) or (0, -1), exact as the rest is representable (checked on the
// device bit for bit against the subtraction), instead of an unpacking and a
// subtraction: the conversions are about as many cycles as the MFMAs of a
// 32-column tile.  The selectors go through registers: as an inline constant
// the low half is read as a float's.
template <int W> struct Split3 {
  typedef __bf16 V __attribute__((ext_vector_type(W)));
  V p[3];
};
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
struct SplitSel {
  bf2 s0, s1;   // (-1, 0) and (0, -1)
  __device__ __forceinline__ SplitSel() {
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
    asm("" : "+v"(lo), "+v"(hi));
    s0 = __builtin_bit_cast(bf2, lo);
    s1 = __builtin_bit_cast(bf2, hi);
  }
};
template <int W>
__device__ __forceinline__ Split3<W> split3(const float (&x)[W], const SplitSel& sel) {
  Split3<W> s;
#pragma unroll
  for (int i = 0; i < W; i += 2) {
    float a = x[i], b = x[i + 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const bf2 h = {(__bf16)a, (__bf16)b};
      s.p[q][i] = h[0];
      s.p[q][i + 1] = h[1];
      if (q < 2) {
        a = __builtin_amdgcn_fdot2_f32_bf16(h, sel.s0, a, false);
        b = __builtin_amdgcn_fdot2_f32_bf16(h, sel.s1, b, false);
      }
    }
  }
  return s;
}

// A complex value at a byte offset from a block-uniform base.
template <typename C> __device__ __forceinline__ C ld_at(const char* base, unsigned off) {
  return ld(reinterpret_cast<const C*>(base + off));
}
// The K order of a step.  Lane group kg = l / 16 of the row operand holds KP
// values of k; which ones is free as long as the column operand agrees.  Value
// j of group kg is k = 8 (j / 2) + 2 kg + j % 2 in complex64 and 4 j + kg in
// complex128: the four groups' 16-byte loads of one instruction then cover 64
// contiguous bytes of each row, where consecutive k per group would touch four
// times the cache lines per instruction (97^3 complex128: 21 columns 1016 ->
// 967 us, 64 columns 1870 -> 1781; the 100^3 sweep 126 -> 118 ms).
template <typename T> __device__ __forceinline__ constexpr int tile_kk(int kg, int j) {
  return sizeof(T) == 4 ? 8 * (j / 2) + 2 * kg + j % 2 : 4 * j + kg;
}
// A lane's values of a row with contiguous k (base and offset at the step's
// k = 0 of the row), aligned to one complex value: two complex64 per load.
__device__ __forceinline__ void ld_run(const char* base, unsigned off, int kg, float2 (&x)[8]) {
  typedef float V __attribute__((ext_vector_type(4), aligned(8)));
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const V v = *(const HELM_AS1 V*)(const HELM_AS1 char*)(base + (off + 16u * kg) + 32 * i);
    x[i] = make_float2(v.x, v.y);
    x[i + 1] = make_float2(v.z, v.w);
  }
}
__device__ __forceinline__ void ld_run(const char* base, unsigned off, int kg, double2 (&x)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = ld_at<double2>(base + 64 * i, off + 16u * kg);
}

template <typename T, int BM, int BN> struct TileShape {
  static constexpr int K = tile_k<T>(), KP = K / 4;     // K step; k per lane
  static constexpr int WR = BM / 16, WC = 4 / WR;       // waves along rows, columns
  static constexpr int NB = BN / 16 / WC;               // 16-column blocks per wave
  static constexpr int KPT = K * BN / 256;              // k per thread of the column operand
  static_assert((BM == 64 || BM == 32) && NB >= 1, "4 waves of 16 rows");
};

// LDS of the column operand: per buffer
//  complex64: [plane: re h m l, im h m l][8 k][column] of 8 bf16, so that
//   stores and reads of 16 lanes are 256 contiguous bytes;
//  complex128: [re, im][k][column], rows padded so that the four k rows of a
//   read start on different quarters of the banks.
template <typename T, int BN> struct TileSmem;
template <int BN> struct TileSmem<float, BN> {
  bf8 q[2][6][4][BN];
};
template <int BN> struct TileSmem<double, BN> {
  double q[2][2][16][BN + 8];
};

// Accumulators of one wave: 16 rows x NB 16-column blocks.  STEP (complex64):
// every K step is summed from zero on the matrix cores and then added to the
// rest; else the sums run through (complex64 keeps Pi Qi apart until finish()).
template <typename T, int BM, int BN, bool STEP = false> struct TileAcc;
template <int BM, int BN> struct TileAcc<float, BM, BN, false> {
  static constexpr int NB = TileShape<float, BM, BN>::NB;
  f4 re[NB], im[NB], ii[NB];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] = im[b] = ii[b] = f4{0, 0, 0, 0};
  }
  __device__ __forceinline__ void finish() {
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] -= ii[b];
  }
};
template <int BM, int BN> struct TileAcc<float, BM, BN, true> {
  static constexpr int NB = TileShape<float, BM, BN>::NB;
  f4 re[NB], im[NB];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] = im[b] = f4{0, 0, 0, 0};
  }
  __device__ __forceinline__ void finish() {}
};
template <int BM, int BN, bool STEP> struct TileAcc<double, BM, BN, STEP> {
  static constexpr int NB = TileShape<double, BM, BN>::NB;
  d4 re[NB], im[NB];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int b = 0; b < NB; ++b) re[b] = im[b] = d4{0, 0, 0, 0};
  }
  __device__ __forceinline__ void finish() {}
};

// Output rows and columns (tile offsets) of this lane's accumulators: element
// v of an MFMA result vector is row 4 (l / 16) + v in FP32 and 4 v + l / 16 in
// FP64, column l % 16 (both checked on the device).
template <typename T, int BM, int BN> struct TileOut {
  using G = TileShape<T, BM, BN>;
  static constexpr int NR = 4, NC = G::NB;
  int r[NR], c[NC];
  __device__ __forceinline__ TileOut() {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      r[v] = (wave / G::WC) * 16 + (sizeof(T) == 4 ? 4 * (lane >> 4) + v : 4 * v + (lane >> 4));
#pragma unroll
    for (int b = 0; b < NC; ++b) c[b] = ((wave % G::WC) * NC + b) * 16 + (lane & 15);
  }
};
template <typename T, int BM, int BN, bool STEP>
__device__ __forceinline__ C_t<T> acc_at(const TileAcc<T, BM, BN, STEP>& acc, int i, int j) {
  C_t<T> z;
  z.x = acc.re[j][i];
  z.y = acc.im[j][i];
  return z;
}

// Row operand: element (r, k) at base[r ld + k] when CONTIG (a lane's k are
// contiguous), else at base[k ld + r]; r < rows.
// Column operand: element (k, c) at base[row(k) ld + c], c < cols, with
// row(k) = k, or kmap[k] when QMODE is kMap; with kGather the children's
// updates landing on row k are added, U[i][inv[i][k] ldu + c] where inv[i] is
// given and its entry is not negative.
enum QMode { kDirect, kMap, kGather };
template <typename T> struct TileP {
  const C_t<T>* base;
  long long ld;
  int rows;
};
template <typename T> struct TileQ {
  const C_t<T>* base;
  long long ld;
  int cols;
  const int* kmap;
  const C_t<T>* U[2];
  const int* inv[2];
};

// One K step of MFMAs of a wave on the lane's row values p (lane l: row
// l % 16, k in the step's order) and the block's staged columns.
template <int BM, int BN, bool STEP>
__device__ __forceinline__ void tile_mfma(const TileSmem<float, BN>& sm, int buf,
                                          TileAcc<float, BM, BN, STEP>& acc, const Split3<8>& ar,
                                          const Split3<8>& ai, int wc, int lane, int nbv) {
  constexpr int NB = TileShape<float, BM, BN>::NB;
  const int kg = lane >> 4;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (b >= nbv) break;
    bf8 br[3], bi[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      br[s] = sm.q[buf][s][kg][(wc * NB + b) * 16 + (lane & 15)];
      bi[s] = sm.q[buf][3 + s][kg][(wc * NB + b) * 16 + (lane & 15)];
    }
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pc[6] = {0, 2, 1, 0, 1, 0};
    if constexpr (STEP) {
      // two chains at a time
      f4 u = {0, 0, 0, 0}, v = u;
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        u = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai.p[pa[s]], bi[pc[s]], u, 0, 0, 0);
        v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai.p[pa[s]], br[pc[s]], v, 0, 0, 0);
      }
      acc.re[b] -= u;
      acc.im[b] += v;
      u = v = f4{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        u = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar.p[pa[s]], br[pc[s]], u, 0, 0, 0);
        v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar.p[pa[s]], bi[pc[s]], v, 0, 0, 0);
      }
      acc.re[b] += u;
      acc.im[b] += v;
      // the sums are formed here: moved past the branch they keep every
      // block's chains alive, which spills
      asm("" : "+v"(acc.re[b]), "+v"(acc.im[b]));
    } else {
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        acc.re[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar.p[pa[s]], br[pc[s]], acc.re[b], 0, 0, 0);
        acc.im[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar.p[pa[s]], bi[pc[s]], acc.im[b], 0, 0, 0);
        acc.ii[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai.p[pa[s]], bi[pc[s]], acc.ii[b], 0, 0, 0);
        acc.im[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai.p[pa[s]], br[pc[s]], acc.im[b], 0, 0, 0);
      }
    }
  }
}
template <int BM, int BN, bool STEP>
__device__ __forceinline__ void tile_mfma(const TileSmem<double, BN>& sm, int buf,
                                          TileAcc<double, BM, BN, STEP>& acc,
                                          const double2 (&p)[4], int wc, int lane, int nbv) {
  constexpr int NB = TileShape<double, BM, BN>::NB;
  const int kg = lane >> 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (b >= nbv) break;
      const int c = (wc * NB + b) * 16 + (lane & 15);
      const double qr = sm.q[buf][0][4 * j + kg][c], qi = sm.q[buf][1][4 * j + kg][c];
      acc.re[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[j].x, qr, acc.re[b], 0, 0, 0);
      acc.im[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[j].x, qi, acc.im[b], 0, 0, 0);
      acc.re[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-p[j].y, qi, acc.re[b], 0, 0, 0);
      acc.im[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[j].y, qr, acc.im[b], 0, 0, 0);
    }
  }
}

// The tile's product over k in [kbeg, kend).  The loads of a step are issued
// one step ahead.  The main loop knows that the next step is whole, so its
// loads are one straight sequence: with a branch between a whole and a clamped
// load the compiler merges their registers by copies right after the loads,
// each waiting for its load, and nothing is ahead any more (a pruned layer
// solve of 160^3, 32 columns: 1528 us with the branch, 1467 without).
template <typename T, int BM, int BN, bool CONTIG, QMode QM, bool STEP>
__device__ __forceinline__ void tile_gemm(TileSmem<T, BN>& sm, TileAcc<T, BM, BN, STEP>& acc,
                                          const TileP<T>& P, const TileQ<T>& Q, int r0, int c0,
                                          int kbeg, int kend) {
  using C = C_t<T>;
  using G = TileShape<T, BM, BN>;
  constexpr int K = G::K, KP = G::KP, KPT = G::KPT;
  constexpr unsigned E = sizeof(C);
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wr = wave / G::WC, wc = wave % G::WC;
  const int kg = lane >> 4;
  acc.zero();
  // a wave whose rows all lie past the operand only stages columns
  const bool live = r0 + wr * 16 < P.rows;
  const int nbv = live ? min(G::NB, (Q.cols - c0 - wc * G::NB * 16 + 15) / 16) : 0;
  const int row = min(wr * 16 + (lane & 15), P.rows - 1 - r0);
  const char* pb = reinterpret_cast<const char*>(CONTIG ? P.base + (long long)r0 * P.ld
                                                        : P.base + r0);
  const unsigned pld = (unsigned)P.ld * E;
  const unsigned prow = (unsigned)row * (CONTIG ? pld : E);
  const int qc = min(t % BN, Q.cols - 1 - c0);
  // this thread's values of k within a step: positions qk.. of the order in
  // complex64 (8 per group), rows qk.. in complex128
  const int qk = (t / BN) * KPT;
  auto kof = [&](int i) {
    return sizeof(T) == 4 ? tile_kk<T>(qk / 8, qk % 8 + i) : qk + i;
  };
  const char* qb = reinterpret_cast<const char*>(Q.base + c0);
  const unsigned qld = (unsigned)Q.ld * E;
  const unsigned qoff = (unsigned)kof(0) * qld + (unsigned)qc * E;
  const SplitSel sel;

  constexpr bool MAP = QM == kMap, GAT = QM == kGather;
  C p[KP], q[KPT], u0[GAT ? KPT : 1], u1[GAT ? KPT : 1];
  int ki[KPT], kj[GAT ? KPT : 1];
  // rows of the column operand (kMap) or of the children's updates (kGather),
  // loaded one step before the values they address
  auto load_index = [&](int k0) {
    if constexpr (MAP) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) ki[i] = ld(Q.kmap + min(k0 + kof(i), kend - 1));
    }
    if constexpr (GAT) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        const int kk = min(k0 + kof(i), kend - 1);
        ki[i] = Q.inv[0] ? ld(Q.inv[0] + kk) : -1;
        kj[i] = Q.inv[1] ? ld(Q.inv[1] + kk) : -1;
      }
    }
  };
  auto load_updates = [&] {
    if constexpr (GAT) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        u0[i] = ld_or_zero(ki[i] >= 0, Q.U[0] + (long long)ki[i] * Q.ld + c0 + qc);
        u1[i] = ld_or_zero(kj[i] >= 0, Q.U[1] + (long long)kj[i] * Q.ld + c0 + qc);
      }
    }
  };
  auto load_mapped = [&] {
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      q[i] = ld(reinterpret_cast<const C*>(qb) + (long long)ki[i] * Q.ld + qc);
  };
  auto load_whole = [&](int k0) {   // k0 + K <= kend
    const char* b = pb + (long long)k0 * (CONTIG ? (long long)E : P.ld * (long long)E);
    if constexpr (CONTIG) {
      ld_run(b, prow, kg, p);
    } else {
#pragma unroll
      for (int i = 0; i < KP; ++i)
        p[i] = ld_at<C>(b + (long long)tile_kk<T>(0, i) * P.ld * E,
                        prow + (unsigned)tile_kk<T>(kg, 0) * pld);
    }
    if constexpr (MAP) {
      load_mapped();
    } else {
      const char* c = qb + (long long)k0 * Q.ld * E;
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        q[i] = ld_at<C>(c + (long long)(sizeof(T) == 4 ? tile_kk<T>(0, i) : i) * Q.ld * E, qoff);
    }
    load_updates();
  };
  auto load_part = [&](int k0) {    // k0 < kend: clamped to the last k
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      const long long kk = min(k0 + tile_kk<T>(kg, i), kend - 1);
      p[i] = ld(reinterpret_cast<const C*>(pb + prow) + kk * (CONTIG ? 1LL : P.ld));
    }
    if constexpr (MAP) {
      load_mapped();
    } else {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        q[i] = ld(reinterpret_cast<const C*>(qb) + (long long)min(k0 + kof(i), kend - 1) * Q.ld + qc);
    }
    load_updates();
  };
  // the loaded columns to LDS and the rows to the operand form; then the next
  // loads (ahead), the barrier and the MFMAs
  auto step = [&](int buf, int kleft, auto&& ahead) {
    if constexpr (GAT) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) q[i] = cadd(q[i], cadd(u0[i], u1[i]));
    }
    if (kleft < K) {
#pragma unroll
      for (int i = 0; i < KPT; ++i)
        if (kof(i) >= kleft) q[i] = czero<C>();
    }
    if constexpr (sizeof(T) == 4) {
      float x[KPT], y[KPT];
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        x[i] = q[i].x;
        y[i] = q[i].y;
      }
      const Split3<KPT> sx = split3<KPT>(x, sel), sy = split3<KPT>(y, sel);
      typedef typename Split3<KPT>::V V;
      char* dst = reinterpret_cast<char*>(&sm.q[buf][0][qk / 8][t % BN]) + (qk % 8) * 2;
      constexpr int PL = sizeof(sm.q[0][0]);
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        *reinterpret_cast<V*>(dst + u * PL) = sx.p[u];
        *reinterpret_cast<V*>(dst + (3 + u) * PL) = sy.p[u];
      }
      float u[8], v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        u[i] = p[i].x;
        v[i] = p[i].y;
      }
      const Split3<8> ar = split3<8>(u, sel), ai = split3<8>(v, sel);
      ahead();
      __syncthreads();
      tile_mfma(sm, buf, acc, ar, ai, wc, lane, nbv);
    } else {
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        sm.q[buf][0][qk + i][t % BN] = q[i].x;
        sm.q[buf][1][qk + i][t % BN] = q[i].y;
      }
      double2 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = p[i];
      ahead();
      __syncthreads();
      tile_mfma(sm, buf, acc, a, wc, lane, nbv);
    }
  };
  if (kbeg >= kend) return;   // an empty product
  load_index(kbeg);
  if (kbeg + K <= kend) load_whole(kbeg); else load_part(kbeg);
  load_index(kbeg + K);
  int k0 = kbeg, buf = 0;
  for (; k0 + 2 * K <= kend; k0 += K, buf ^= 1)
    step(buf, K, [&] {
      load_whole(k0 + K);
      load_index(k0 + 2 * K);
    });
  // the last whole step and a partial one
  for (; k0 < kend; k0 += K, buf ^= 1)
    step(buf, kend - k0, [&] {
      if (k0 + K < kend) load_part(k0 + K);
    });
  acc.finish();
}

}  // namespace kern
}  // namespace helm
