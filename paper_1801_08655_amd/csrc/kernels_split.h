// Complex64 GEMM tile on the bf16 matrix cores, at (better than) FP32
// accuracy.
//
// A float x is split exactly into three bf16 numbers, x = h + m + l: h is x
// rounded to bf16, m the rounded rest, l what is left (24 = 3 x 8 significant
// bits).  A real product is then formed from the six bf16 products
//   h h' + h m' + m h' + h l' + l h' + m m',
// accumulated in FP32 by the matrix cores, smallest first; the dropped ones
// (m l', l m', l l') are below 2^-24 of |x||x'|.  Measured against FP64 on
// normal data, the error of a length-K product is 0.37 (K = 32), 0.79 (256)
// and 0.85 (1024) of the v_mfma_f32_16x16x4f32 chain's: an MFMA of K = 32
// rounds once where the FP32 instruction rounds 32 times.
//
// Why: on gfx950 the FP32 matrix instructions run at 134 TFLOP/s (measured
// loop) and the bf16 ones at 2100, so six products per real one still leave
// 350.  What bounds the tile then is the latency of its operand loads, not the
// matrix cores.  Against the FP32 tile it replaced (three real products, both
// operands in LDS): one interior layer of 100^3 with 64 columns 1.75 -> 1.57
// ms (21 columns 0.98 -> 0.91), a whole refined solve of 64 sources on 96^3
// 419 -> 362 ms, of 32 on 160^3 1049 -> 999 ms; the local solve's error
// against complex128 2.15e-6 -> 2.05e-6 (25^3: 8.8e-7 -> 7.7e-7), smaller at
// every width.  The complex product takes four real ones (three accumulators: Pr Qr,
// Pi Qi, Pr Qi + Pi Qr), whose error is bounded per component.
//
// Tile: BM rows x BN columns, K steps of 32, 4 waves.  BM = 64: each wave
// owns 16 rows and all columns, so the row operand needs no LDS: a lane
// loads its 8 consecutive k of one row straight in the MFMA operand layout
// (lane l: row l % 16, k = 8 (l / 16) + 0..7) and splits them in registers.
// BM = 32: two waves share 16 rows and take half of the columns each.  The
// column operand is split once per block by the thread that loaded it and
// passed through LDS, 16 bytes per (plane, 8 k, column): stores and reads of
// 16 lanes are 256 contiguous bytes.  Two LDS buffers, one barrier per step;
// the global loads of a step are issued before the MFMAs of the step before
// it.  Rows and columns past the operands are clamped to the last valid one
// (their results are never stored); past the K range the column operand is
// zero and the row operand clamped, so no out-of-range value is read.
#pragma once

#include "kernels_common.h"

namespace helm {
namespace kern {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int SK = 32;   // K step (complex elements)

// W floats split into their three bf16 planes (vectors of W elements).
template <int W> struct Split3 {
  typedef __bf16 V __attribute__((ext_vector_type(W)));
  V p[3];
};
template <int W> __device__ __forceinline__ Split3<W> split3(const float (&x)[W]) {
  Split3<W> s;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const __bf16 h = (__bf16)x[i];
    const float r = x[i] - (float)h;
    const __bf16 m = (__bf16)r;
    s.p[0][i] = h;
    s.p[1][i] = m;
    s.p[2][i] = (__bf16)(r - (float)m);
  }
  return s;
}

// A float2 at a byte offset from a block-uniform base.
__device__ __forceinline__ float2 ld_at(const char* base, unsigned off) {
  typedef float V __attribute__((ext_vector_type(2)));
  const V v = *(const HELM_AS1 V*)(const HELM_AS1 char*)(base + off);
  return make_float2(v.x, v.y);
}
// Two float2 (16 bytes, 8-byte aligned).
__device__ __forceinline__ void ld_at2(const char* base, unsigned off, float2& a, float2& b) {
  typedef float V __attribute__((ext_vector_type(4), aligned(8)));
  const V v = *(const HELM_AS1 V*)(const HELM_AS1 char*)(base + off);
  a = make_float2(v.x, v.y);
  b = make_float2(v.z, v.w);
}

template <int BM, int BN> struct SplitShape {
  static constexpr int WR = BM / 16, WC = 4 / WR;   // waves along rows, columns
  static constexpr int NB = BN / 16 / WC;           // 16-column blocks per wave
  static constexpr int KPT = BN / 8;                // k per thread of the column operand
  static_assert((BM == 64 || BM == 32) && NB >= 1, "4 waves of 16 rows");
};

// LDS of the column operand: [buffer][plane: re h m l, im h m l][8 k][column]
template <int BN> struct SplitSmem {
  bf8 q[2][6][SK / 8][BN];
};

// Accumulators of one wave: 16 rows x NB 16-column blocks.
template <int BM, int BN> struct SplitAcc {
  static constexpr int NB = SplitShape<BM, BN>::NB;
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

// Output rows and columns (tile offsets) of this lane's accumulators.
template <int BM, int BN> struct SplitOut {
  using G = SplitShape<BM, BN>;
  static constexpr int NR = 4, NC = G::NB;
  int r[NR], c[NC];
  __device__ __forceinline__ SplitOut() {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = (wave / G::WC) * 16 + 4 * (lane >> 4) + v;
#pragma unroll
    for (int b = 0; b < NC; ++b) c[b] = ((wave % G::WC) * NC + b) * 16 + (lane & 15);
  }
};
template <int BM, int BN>
__device__ __forceinline__ float2 acc_at(const SplitAcc<BM, BN>& acc, int i, int j) {
  return make_float2(acc.re[j][i], acc.im[j][i]);
}

// Row operand: element (r, k) at base[r ldr + k ldk], r < rows.  CONTIG: ldk
// is 1 (a lane's 8 k are 64 contiguous bytes), else ldr is 1.
// Column operand: element (k, c) at base[row(k) ldk + c], c < cols, with
// row(k) = k, or kmap[k] when a map is given.
struct SplitP {
  const float2* base;
  long long ld;    // stride of k (or of r when CONTIG)
  int rows;
};
struct SplitQ {
  const float2* base;
  long long ld;
  int cols;
  const int* kmap;
};

template <int BM, int BN, bool CONTIG, bool MAP>
__device__ __forceinline__ void split_tile(SplitSmem<BN>& sm, SplitAcc<BM, BN>& acc,
                                           const SplitP& P, const SplitQ& Q, int r0, int c0,
                                           int kbeg, int kend) {
  using G = SplitShape<BM, BN>;
  constexpr int KPT = G::KPT;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wr = wave / G::WC, wc = wave % G::WC;
  const int kg = lane >> 4;
  acc.zero();
  if (kbeg >= kend) return;
  // a wave whose rows all lie past the operand only stages columns
  const bool live = r0 + wr * 16 < P.rows;
  const int nbv = min(G::NB, (Q.cols - c0 - wc * G::NB * 16 + 15) / 16);
  const int row = min(wr * 16 + (lane & 15), P.rows - 1 - r0);
  const char* pb = reinterpret_cast<const char*>(CONTIG ? P.base + (long long)r0 * P.ld
                                                        : P.base + r0);
  const unsigned ld8 = (unsigned)P.ld * 8u;
  const unsigned prow = CONTIG ? (unsigned)row * ld8 : (unsigned)row * 8u;
  const int qc = min(t % BN, Q.cols - 1 - c0);
  const int qk = (t / BN) * KPT;                  // this thread's k within a step
  const char* qb = reinterpret_cast<const char*>(Q.base + c0);
  const unsigned qld8 = (unsigned)Q.ld * 8u;

  float2 p[8], q[KPT];
  int ki[KPT];
  auto load_index = [&](int k0) {   // rows of the column operand (MAP), clamped
    if (MAP) {
#pragma unroll
      for (int i = 0; i < KPT; ++i) ki[i] = ld(Q.kmap + min(k0 + qk + i, kend - 1));
    }
  };
  auto load = [&](int k0) {
    const int left = kend - k0;
    if (live) {
      const char* b = pb + (CONTIG ? (long long)k0 * 8 : (long long)k0 * P.ld * 8);
      if (left >= SK) {
        if (CONTIG) {
#pragma unroll
          for (int i = 0; i < 8; i += 2)
            ld_at2(b, prow + (unsigned)(kg * 8 + i) * 8u, p[i], p[i + 1]);
        } else {
#pragma unroll
          for (int i = 0; i < 8; ++i)
            p[i] = ld_at(b + (long long)i * P.ld * 8, prow + (unsigned)(kg * 8) * ld8);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const unsigned kk = (unsigned)min(kg * 8 + i, left - 1);
          p[i] = ld_at(b, prow + (CONTIG ? kk * 8u : kk * ld8));
        }
      }
    }
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      if (MAP) {
        q[i] = ld(reinterpret_cast<const float2*>(qb) + (long long)ki[i] * Q.ld + qc);
      } else {
        const unsigned kk = (unsigned)min(qk + i, left - 1);
        q[i] = ld_at(qb + (long long)k0 * Q.ld * 8, kk * qld8 + (unsigned)qc * 8u);
      }
    }
  };
  load_index(kbeg);
  load(kbeg);
  load_index(kbeg + SK);
  int buf = 0;
  for (int k0 = kbeg; k0 < kend; k0 += SK, buf ^= 1) {
    // column operand: split and to LDS
    {
      float x[KPT], y[KPT];
#pragma unroll
      for (int i = 0; i < KPT; ++i) {
        const bool ok = k0 + qk + i < kend;
        x[i] = ok ? q[i].x : 0.0f;
        y[i] = ok ? q[i].y : 0.0f;
      }
      const Split3<KPT> sx = split3<KPT>(x), sy = split3<KPT>(y);
      typedef typename Split3<KPT>::V V;
      char* dst = reinterpret_cast<char*>(&sm.q[buf][0][qk / 8][t % BN]) + (qk % 8) * 2;
      constexpr int PL = sizeof(sm.q[0][0]);
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        *reinterpret_cast<V*>(dst + s * PL) = sx.p[s];
        *reinterpret_cast<V*>(dst + (3 + s) * PL) = sy.p[s];
      }
    }
    // row operand: split in registers
    Split3<8> ar, ai;
    if (live) {
      float x[8], y[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[i] = p[i].x;
        y[i] = p[i].y;
      }
      ar = split3<8>(x);
      ai = split3<8>(y);
    }
    if (k0 + SK < kend) {
      load(k0 + SK);
      load_index(k0 + 2 * SK);
    }
    __syncthreads();
    if (live) {
#pragma unroll
      for (int b = 0; b < G::NB; ++b) {
        if (b >= nbv) break;
        bf8 br[3], bi[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          br[s] = sm.q[buf][s][kg][(wc * G::NB + b) * 16 + (lane & 15)];
          bi[s] = sm.q[buf][3 + s][kg][(wc * G::NB + b) * 16 + (lane & 15)];
        }
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pc[6] = {0, 2, 1, 0, 1, 0};
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
  acc.finish();
}

}  // namespace kern
}  // namespace helm
