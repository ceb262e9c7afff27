// Multi-RHS substitutions over a layer's front tree (online stage: every
// local solve (H^l)^-1 of Algorithms 2-10).
//
// With the stored blocks [F11^-1; -F21 F11^-1] of every front:
//   forward (leaves -> root): X(S) += children's updates (extend-add, in
//     place; leaves have none), Z(S) <- F11^-1 X(S),
//     update_B <- children's updates - F21 F11^-1 X(S)
//   backward (root -> leaves): X(S) <- Z(S) + (-F21 F11^-1)^T X(B)
// Both passes are dense complex GEMMs with the RHS columns as N.  X (the
// solve vector) and Z are stored in nested-dissection order with the columns
// fastest; update_B lives in a per-depth-parity buffer.
#include <hip/hip_ext.h>

#include "kernels.h"
#include "kernels_common.h"
#include "kernels_tile.h"

namespace helm {
namespace kern {

namespace {

template <typename T>
__device__ __forceinline__ C_t<T>* ub_ptr(const LayerDev& L, int parity) {
  return reinterpret_cast<C_t<T>*>(L.Ub[parity]);
}

// Sum of the children's updates landing on front row `row` (extend-add in
// pull form through the front-row -> child-boundary maps).
template <typename T> struct ChildSum {
  const C_t<T>* Uc;
  long long cub[2];
  const int* inv[2];
  __device__ __forceinline__ ChildSum(const SolveFront& f, const LayerDev& L) {
    Uc = reinterpret_cast<const C_t<T>*>(L.Ub[f.ub_parity ^ 1]);
#pragma unroll
    for (int slot = 0; slot < 2; ++slot) {
      cub[slot] = f.cub[slot];
      inv[slot] = f.inv[slot] >= 0 ? L.inv + f.inv[slot] : nullptr;
    }
  }
};

// forward, step 1 (fronts with children): X(S) += children's updates on the
// pivot rows, in place.  The boundary rows are summed in the GEMM epilogue.
template <typename T, int NT>
__global__ void __launch_bounds__(NT)
k_fwd_gather(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
             const LayerDev* __restrict__ layers, int k) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int r0 = tm.y * RT;
  C* X = reinterpret_cast<C*>(L.X);
  const ChildSum<T> cs(f, L);
  const int rows = (f.s - r0) < RT ? (f.s - r0) : RT;
  const int total = rows * k;
  // EPT elements (row, column) per thread and pass: child rows first, then
  // every value, then the stores (one latency per group of loads, not one
  // per element)
  constexpr int EPT = 4;
  for (int e0 = 0; e0 < total; e0 += NT * EPT) {
    int q[2][EPT], rr[EPT], cc[EPT];
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      const int e = e0 + (int)threadIdx.x + j * NT;
      const bool ok = e < total;
      rr[j] = ok ? r0 + e / k : -1;
      cc[j] = ok ? e % k : 0;
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
        q[sl][j] = (ok && cs.inv[sl]) ? ld(cs.inv[sl] + rr[j]) : -1;
    }
    C v[EPT];
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      C u[2];
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
        u[sl] = ld_or_zero(q[sl][j] >= 0, cs.Uc + (cs.cub[sl] + q[sl][j]) * k + cc[j]);
      const C x = ld_or_zero(rr[j] >= 0, X + (long long)(f.off + rr[j]) * k + cc[j]);
      v[j] = cadd(x, cadd(cadd(czero<C>(), u[0]), u[1]));
    }
#pragma unroll
    for (int j = 0; j < EPT; ++j)
      if (rr[j] >= 0) st(X + (long long)(f.off + rr[j]) * k + cc[j], v[j]);
  }
}

// Partial products of a split front: rows [m0, ...) < n of chunk `chunk`.
template <typename T, class O, class Acc>
__device__ __forceinline__ void store_partial(const Acc& acc, C_t<T>* S, long long row0, int m0,
                                              int n0, int n, int k) {
  const O o;
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gm = m0 + o.r[i], gc = n0 + o.c[j];
      if (gm < n && gc < k) st(S + (row0 + gm) * k + gc, acc_at(acc, i, j));
    }
}

// Forward GEMM epilogue of an unsplit front: pivot rows to Z, boundary rows
// to the update buffer with the children's updates added.  The child rows of
// all of this lane's outputs are loaded first, then the child values, then
// the results are stored, so that the latencies of each group of loads
// overlap instead of following one another output by output.
template <typename T, class O, class Acc>
__device__ __forceinline__ void fwd_epilogue(const Acc& acc, const SolveFront& f,
                                             const ChildSum<T>& cs, C_t<T>* Z, C_t<T>* Uo,
                                             int m0, int n0, int k) {
  using C = C_t<T>;
  const O o;
  const int n = f.s + f.b;
  int q[2][O::NR];
#pragma unroll
  for (int i = 0; i < O::NR; ++i) {
    const int gm = m0 + o.r[i];
    const bool bnd = gm >= f.s && gm < n;
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) q[sl][i] = (bnd && cs.inv[sl]) ? ld(cs.inv[sl] + gm) : -1;
  }
  C add[O::NR][O::NC];
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) add[i][j] = czero<C>();
  if (cs.inv[0] || cs.inv[1]) {   // uniform: leaves have no children
#pragma unroll
    for (int i = 0; i < O::NR; ++i)
#pragma unroll
      for (int j = 0; j < O::NC; ++j) {
        const int gc = n0 + o.c[j];
        C u[2];
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
          u[sl] = ld_or_zero(q[sl][i] >= 0 && gc < k, cs.Uc + (cs.cub[sl] + q[sl][i]) * k + gc);
        add[i][j] = cadd(cadd(add[i][j], u[0]), u[1]);
      }
  }
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gm = m0 + o.r[i], gc = n0 + o.c[j];
      if (gm >= n || gc >= k) continue;
      const C z = acc_at(acc, i, j);
      if (gm < f.s) st(Z + (long long)(f.off + gm) * k + gc, z);
      else st(Uo + (f.ub + gm - f.s) * k + gc, cadd(z, add[i][j]));
    }
}

// Occupancy asked of the compiler (waves per SIMD) for a tile of BN columns:
// 4 for the complex64 tiles of 16 and 32 columns (128 registers), 3 for the
// 64-column one (168); complex128 2.
template <typename T> constexpr int tile_waves(int bn) {
  return sizeof(T) == 4 ? (bn == 64 ? 3 : 4) : 2;
}

// forward, step 2: [X(S); Ub] = [F11^-1 w_S; Ub - F21 F11^-1 w_S], the K
// (pivot) dimension optionally split into chunks (partials to scratch).
template <typename T, int BN, bool GATHER>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(tile_waves<T>(BN) - (GATHER && sizeof(T) == 4 && BN > 16), 8)))
k_fwd_gemm(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
           const LayerDev* __restrict__ layers, int k, void* scratch) {
  using C = C_t<T>;
  constexpr int BM = FWD_BM;
  using O = TileOut<T, BM, BN>;
  __shared__ TileSmem<T, BN> sm;
  const int ntn = (k + BN - 1) / BN;
  const int mt = blockIdx.x / ntn, nt = blockIdx.x % ntn;
  const int2 tm = tmap[mt];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b;
  const int chunk = tm.y % f.nch;
  const int m0 = (tm.y / f.nch) * BM, n0 = nt * BN;
  const int kb = chunk * f.kc;
  const int ke = min(f.s, kb + f.kc);
  // P = FT (col-major, rows m), Q = X(S) (rows = pivots, columns = RHS)
  const C* FT = reinterpret_cast<const C*>(L.fac) + f.fac;
  const C* X = reinterpret_cast<const C*>(L.X) + (long long)f.off * k;
  TileAcc<T, BM, BN> acc;
  const ChildSum<T> cs(f, L);
  TileQ<T> Q{X, k, k};
  if (GATHER)
    for (int sl = 0; sl < 2; ++sl) {
      Q.U[sl] = cs.Uc + cs.cub[sl] * k;
      Q.inv[sl] = cs.inv[sl];
    }
  tile_gemm<T, BM, BN, false, GATHER ? kGather : kDirect>(sm, acc, TileP<T>{FT, n, n}, Q, m0, n0,
                                                          kb, ke);
  if (f.nch > 1)
    store_partial<T, O>(acc, reinterpret_cast<C*>(scratch), f.scr + (long long)chunk * n, m0, n0,
                        n, k);
  else
    fwd_epilogue<T, O>(acc, f, cs, reinterpret_cast<C*>(L.Wt), ub_ptr<T>(L, f.ub_parity), m0,
                       n0, k);
}

// elements per thread and pass of the split-K reductions, and chunks whose
// partial products are loaded together (one latency for the group)
constexpr int RED_EPT = 4, RED_CH = 4;

// z[j] += the partial products of element gm[j], gc[j] (gm < 0: none), in
// order of the chunks; `rows` partial rows per chunk from row0.
template <typename T>
__device__ __forceinline__ void add_partials(C_t<T> (&z)[RED_EPT], const int (&gm)[RED_EPT],
                                             const int (&gc)[RED_EPT], const C_t<T>* S,
                                             long long row0, int rows, int nch, int k) {
  using C = C_t<T>;
  for (int c0 = 0; c0 < nch; c0 += RED_CH) {
    C v[RED_CH][RED_EPT];
#pragma unroll
    for (int i = 0; i < RED_CH; ++i)
#pragma unroll
      for (int j = 0; j < RED_EPT; ++j) {
        const bool ok = gm[j] >= 0 && c0 + i < nch;
        v[i][j] = ld_or_zero(ok, S + (ok ? (row0 + (long long)(c0 + i) * rows + gm[j]) * k + gc[j]
                                         : 0));
      }
#pragma unroll
    for (int i = 0; i < RED_CH; ++i)
#pragma unroll
      for (int j = 0; j < RED_EPT; ++j) z[j] = cadd(z[j], v[i][j]);
  }
}

// forward, step 3 (split fronts only): sum the chunk partials in order
template <typename T, int NT>
__global__ void __launch_bounds__(NT)
k_fwd_reduce(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
             const LayerDev* __restrict__ layers, int k, const void* scratch) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b;
  const int r0 = tm.y * RT;
  const int rows = min(RT, n - r0);
  const C* S = reinterpret_cast<const C*>(scratch);
  C* Z = reinterpret_cast<C*>(L.Wt);
  C* Uo = ub_ptr<T>(L, f.ub_parity);
  const ChildSum<T> cs(f, L);
  // RED_EPT elements per thread at a time: all their loads, then the stores
  for (int e0 = 0; e0 < rows * k; e0 += NT * RED_EPT) {
    int gm[RED_EPT], gc[RED_EPT], q[2][RED_EPT];
    C z[RED_EPT], u[2][RED_EPT];
#pragma unroll
    for (int j = 0; j < RED_EPT; ++j) {
      const int e = e0 + (int)threadIdx.x + j * NT;
      gm[j] = e < rows * k ? r0 + e / k : -1;
      gc[j] = e % k;
      z[j] = czero<C>();
      // (a boundary row takes its children's updates)
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
        q[sl][j] = (gm[j] >= f.s && cs.inv[sl]) ? ld(cs.inv[sl] + gm[j]) : -1;
    }
#pragma unroll
    for (int j = 0; j < RED_EPT; ++j)
#pragma unroll
      for (int sl = 0; sl < 2; ++sl)
        u[sl][j] = ld_or_zero(q[sl][j] >= 0, cs.Uc + (cs.cub[sl] + q[sl][j]) * k + gc[j]);
    add_partials<T>(z, gm, gc, S, f.scr, n, f.nch, k);
#pragma unroll
    for (int j = 0; j < RED_EPT; ++j) {
      if (gm[j] < 0) continue;
      if (gm[j] < f.s) st(Z + (long long)(f.off + gm[j]) * k + gc[j], z[j]);
      else st(Uo + (f.ub + gm[j] - f.s) * k + gc[j], cadd(z[j], cadd(u[0][j], u[1][j])));
    }
  }
}

// backward: X(S) = Z(S) + (-F21 F11^-1)^T X(B); X(B) is read in place
// through the front's boundary index list, the K (boundary) dimension
// optionally split.  Fronts without boundary (roots) just copy Z(S).
template <typename T, int BM, int BN>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(tile_waves<T>(BN), 8)))
k_bwd_gemm(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
           const LayerDev* __restrict__ layers, int k, void* scratch) {
  using C = C_t<T>;
  using O = TileOut<T, BM, BN>;
  __shared__ TileSmem<T, BN> sm;
  const int ntn = (k + BN - 1) / BN;
  const int mt = blockIdx.x / ntn, nt = blockIdx.x % ntn;
  const int2 tm = tmap[mt];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b;
  const int chunk = tm.y % f.nch;
  const int m0 = (tm.y / f.nch) * BM, n0 = nt * BN;
  const int kb = chunk * f.kc;
  const int ke = min(f.b, kb + f.kc);
  // P(m, q) = FT[(s + q) + m n]  (transposed lower block, contiguous in q),
  // Q(q, c) = X[B[q] k + c]
  const C* FT = reinterpret_cast<const C*>(L.fac) + f.fac + f.s;
  C* X = reinterpret_cast<C*>(L.X);
  TileAcc<T, BM, BN> acc;
  tile_gemm<T, BM, BN, true, kMap>(sm, acc, TileP<T>{FT, n, f.s},
                                   TileQ<T>{X, k, k, L.bidx + f.bidx}, m0, n0, kb, ke);
  if (f.nch > 1) {
    store_partial<T, O>(acc, reinterpret_cast<C*>(scratch), f.scr + (long long)chunk * f.s, m0,
                        n0, f.s, k);
    return;
  }
  // X(S) = Z(S) + product: every Z value of the lane is loaded before the
  // first store (X and Z are distinct buffers, but the compiler cannot tell)
  const O o;
  const C* Z = reinterpret_cast<const C*>(L.Wt);
  C zv[O::NR][O::NC];
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gm = m0 + o.r[i], gc = n0 + o.c[j];
      zv[i][j] = ld_or_zero(gm < f.s && gc < k && !f.zero_z,
                            Z + (long long)(f.off + gm) * k + gc);
    }
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gm = m0 + o.r[i], gc = n0 + o.c[j];
      if (gm < f.s && gc < k)
        st(X + (long long)(f.off + gm) * k + gc, cadd(zv[i][j], acc_at(acc, i, j)));
    }
}

template <typename T, int NT>
__global__ void __launch_bounds__(NT)
k_bwd_reduce(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
             const LayerDev* __restrict__ layers, int k, const void* scratch) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int r0 = tm.y * RT;
  const int rows = min(RT, f.s - r0);
  const C* S = reinterpret_cast<const C*>(scratch);
  C* X = reinterpret_cast<C*>(L.X);
  const C* Z = reinterpret_cast<const C*>(L.Wt);
  for (int e0 = 0; e0 < rows * k; e0 += NT * RED_EPT) {
    int gm[RED_EPT], gc[RED_EPT];
    C z[RED_EPT];
#pragma unroll
    for (int j = 0; j < RED_EPT; ++j) {
      const int e = e0 + (int)threadIdx.x + j * NT;
      gm[j] = e < rows * k ? r0 + e / k : -1;
      gc[j] = e % k;
      const bool ok = gm[j] >= 0 && !f.zero_z;
      z[j] = ld_or_zero(ok, Z + (ok ? (long long)(f.off + gm[j]) * k + gc[j] : 0));
    }
    add_partials<T>(z, gm, gc, S, f.scr, f.s, f.nch, k);
#pragma unroll
    for (int j = 0; j < RED_EPT; ++j)
      if (gm[j] >= 0) st(X + (long long)(f.off + gm[j]) * k + gc[j], z[j]);
  }
}

// ---------------------------------------------------------------------------
// Vector path for batches of KC <= 4 columns (a template argument): the GEMMs
// above would pad the columns to a 16-wide MFMA tile, so the substitutions are
// done with plain FMAs while streaming the factor blocks once.  Large fronts
// are bound by HBM bandwidth, the others by the latency of the chain of
// dependent loads in one launch, so a depth is one launch per pass: the
// children's updates of the pivot rows are added while the right-hand side
// is staged in LDS (no gather launch), and a depth with few tiles takes
// narrower ones instead of a split K with a reduction launch.  Against
// gather, GEMV and reduction launches, one pruned layer solve of one column:
// 25^3 complex128 167 -> 103 us, 60^3 complex64 336 -> 219, 100^3 complex64
// 476 -> 356 (factor blocks at 3 to 4 TB/s per launch) and complex128 627 ->
// 561 (4 to 5 TB/s).
// ---------------------------------------------------------------------------

// forward: RTILE rows of one front per block (64, or 32 or 16 where 64-row
// tiles are too few).  The 256 / RTILE threads of a row take the pivot columns
// round robin; U columns are loaded ahead of the U being multiplied, and the
// first ones before the right-hand side is staged.
template <typename T, int KC, int RTILE>
__global__ void __launch_bounds__(256)
k_fwd_gemv(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
           const LayerDev* __restrict__ layers) {
  using C = C_t<T>;
  constexpr int NKP = 256 / RTILE, U = RTILE < 64 && sizeof(T) == 4 ? 16 : 8;
  constexpr int QC = KC == 1 ? 1024 : (KC == 2 ? 512 : 256);   // pivots staged at a time
  constexpr int EPT = QC * KC / 256;
  static_assert(QC % (U * NKP) == 0, "whole batches per stage");
  __shared__ C w[QC * KC];
  __shared__ C red[3][RTILE][KC];
  const int2 tm = tmap[blockIdx.x];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b, t = threadIdx.x;
  const int row = t % RTILE, kp = t / RTILE;
  const int m = tm.y * RTILE + row;
  const C* col = reinterpret_cast<const C*>(L.fac) + f.fac + min(m, n - 1);
  const C* X = reinterpret_cast<const C*>(L.X) + (long long)f.off * KC;
  const ChildSum<T> cs(f, L);
  // the row's children's updates, in flight under everything that follows
  C add[2][KC];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
    const bool own = kp == 0 && m < n && m >= f.s && cs.inv[sl];
    const int q = own ? ld(cs.inv[sl] + m) : -1;
#pragma unroll
    for (int c = 0; c < KC; ++c)
      add[sl][c] = ld_or_zero(q >= 0, cs.Uc + (cs.cub[sl] + q) * KC + c);
  }
  C acc[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) acc[c] = czero<C>();
  for (int qb = 0; qb < f.s; qb += QC) {
    const int nq = min(QC, f.s - qb);
    C p[U], pn[U];
    auto load = [&](C (&x)[U], int batch) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = min(qb + (batch * U + u) * NKP + kp, f.s - 1);
        x[u] = ld(col + (long long)q * n);
      }
    };
    load(p, 0);
    if (qb) __syncthreads();
    // w = X(S) + children's updates, zero past the last pivot
    {
      int iq[2][EPT];
      C v[EPT], u0[EPT], u1[EPT];
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const int e = t + 256 * i, q = e / KC;
        const bool ok = q < nq;
#pragma unroll
        for (int sl = 0; sl < 2; ++sl)
          iq[sl][i] = (ok && cs.inv[sl]) ? ld(cs.inv[sl] + qb + q) : -1;
        v[i] = ld_or_zero(ok, X + (long long)qb * KC + e);
      }
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const int c = (t + 256 * i) % KC;
        u0[i] = ld_or_zero(iq[0][i] >= 0, cs.Uc + (cs.cub[0] + iq[0][i]) * KC + c);
        u1[i] = ld_or_zero(iq[1][i] >= 0, cs.Uc + (cs.cub[1] + iq[1][i]) * KC + c);
      }
#pragma unroll
      for (int i = 0; i < EPT; ++i) w[t + 256 * i] = cadd(v[i], cadd(u0[i], u1[i]));
    }
    __syncthreads();
    // two batches in turn, the loads of one (past the end: the last column
    // again) issued before the products of the other
    const int nbatch = (nq + U * NKP - 1) / (U * NKP);
    auto use = [&](const C (&x)[U], int b) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const C* wq = &w[((b * U + u) * NKP + kp) * KC];
#pragma unroll
        for (int c = 0; c < KC; ++c) cfma(acc[c], x[u], wq[c]);
      }
    };
    int b = 0;
    for (; b + 2 <= nbatch; b += 2) {
      load(pn, b + 1);
      use(p, b);
      load(p, b + 2);
      use(pn, b + 1);
    }
    if (b < nbatch) use(p, b);
  }
  // the row's partial sums: the lanes of a wave, then the 4 waves, in order
#pragma unroll
  for (int c = 0; c < KC; ++c)
#pragma unroll
    for (int o = RTILE; o < 64; o <<= 1) {
      acc[c].x += __shfl_xor(acc[c].x, o, 64);
      acc[c].y += __shfl_xor(acc[c].y, o, 64);
    }
  const int wave = t >> 6;
  if (wave > 0 && (t & 63) < RTILE) {
#pragma unroll
    for (int c = 0; c < KC; ++c) red[wave - 1][row][c] = acc[c];
  }
  __syncthreads();
  if (kp != 0 || m >= n) return;
  C* Z = reinterpret_cast<C*>(L.Wt);
  C* Uo = ub_ptr<T>(L, f.ub_parity);
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const C z = cadd(cadd(acc[c], red[0][row][c]), cadd(red[1][row][c], red[2][row][c]));
    if (m < f.s) st(Z + (long long)(f.off + m) * KC + c, z);
    else st(Uo + (f.ub + m - f.s) * KC + c, cadd(z, cadd(add[0][c], add[1][c])));
  }
}

// forward, depths whose fronts all have at most 64 NS pivots (the deep ones,
// thousands of small fronts): one wave per 64-row tile, lane = row.  Lane q
// holds the gathered right-hand side of pivots q, q + 64, ..., broadcast by
// lane reads, so nothing waits at a barrier: the gather's two dependent loads
// overlap the first U factor columns.
template <typename T, int KC, int NS>
__global__ void __launch_bounds__(256)
k_fwd_gemv_wave(const SolveFront* __restrict__ list, const int2* __restrict__ tmap, int total,
                const LayerDev* __restrict__ layers) {
  using C = C_t<T>;
  constexpr int U = 8;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = blockIdx.x * 4 + wave, lane = threadIdx.x & 63;
  if (tile >= total) return;
  const int2 tm = tmap[tile];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b, m = tm.y * 64 + lane;
  const C* col = reinterpret_cast<const C*>(L.fac) + f.fac + min(m, n - 1);
  const C* X = reinterpret_cast<const C*>(L.X) + (long long)f.off * KC;
  const ChildSum<T> cs(f, L);
  C p[U], pn[U];
  auto load = [&](C (&x)[U], int q0) {
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = ld(col + (long long)min(q0 + u, f.s - 1) * n);
  };
  load(p, 0);
  // every index, then every value: the tile's boundary rows and the pivots
  int iq[2][NS], im[2];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int q = lane + 64 * i;
      iq[sl][i] = (q < f.s && cs.inv[sl]) ? ld(cs.inv[sl] + q) : -1;
    }
    im[sl] = (m >= f.s && m < n && cs.inv[sl]) ? ld(cs.inv[sl] + m) : -1;
  }
  C w[NS][KC], add[KC], acc[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const C a0 = ld_or_zero(im[0] >= 0, cs.Uc + (cs.cub[0] + im[0]) * KC + c);
    const C a1 = ld_or_zero(im[1] >= 0, cs.Uc + (cs.cub[1] + im[1]) * KC + c);
    add[c] = cadd(a0, a1);
    acc[c] = czero<C>();
  }
#pragma unroll
  for (int i = 0; i < NS; ++i)
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const int q = lane + 64 * i;
      const C x = ld_or_zero(q < f.s, X + (long long)q * KC + c);
      const C u0 = ld_or_zero(iq[0][i] >= 0, cs.Uc + (cs.cub[0] + iq[0][i]) * KC + c);
      const C u1 = ld_or_zero(iq[1][i] >= 0, cs.Uc + (cs.cub[1] + iq[1][i]) * KC + c);
      w[i][c] = cadd(x, cadd(u0, u1));
    }
  // pivots in groups of U, two in turn (past the last pivot the right-hand
  // side is zero and the loads repeat the last column)
  auto use = [&](const C (&x)[U], const C (&wi)[KC], int q0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        C v;
        v.x = lane_read(wi[c].x, q0 + u);
        v.y = lane_read(wi[c].y, q0 + u);
        cfma(acc[c], x[u], v);
      }
  };
#pragma unroll
  for (int i = 0; i < NS; ++i)
    for (int q0 = 0; q0 < 64 && 64 * i + q0 < f.s; q0 += 2 * U) {
      load(pn, 64 * i + q0 + U);
      use(p, w[i], q0);
      load(p, 64 * i + q0 + 2 * U);
      use(pn, w[i], q0 + U);
    }
  if (m >= n) return;
  C* Z = reinterpret_cast<C*>(L.Wt);
  C* Uo = ub_ptr<T>(L, f.ub_parity);
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    if (m < f.s) st(Z + (long long)(f.off + m) * KC + c, acc[c]);
    else st(Uo + (f.ub + m - f.s) * KC + c, cadd(acc[c], add[c]));
  }
}

template <typename T> __device__ __forceinline__ T shfl_xor_t(T v, int mask) {
  return __shfl_xor(v, mask, 64);
}

// backward: 8 RPG rows of one front per block; the 256 threads form 8 groups
// of 32 lanes and group g takes the rows m0 + g, m0 + g + 8, ... (RPG of
// them) together: its lanes walk the boundary index q (contiguous in the
// stored block), load X(B[q]) once for all those rows and the factor entry
// of every row, so that several independent factor loads are in flight per
// lane (fewer rows per group where the depth has few tiles, with more of the
// boundary in flight instead).
template <typename T, int KC, int RPG>
__global__ void __launch_bounds__(256)
k_bwd_gemv(const SolveFront* __restrict__ list, const int2* __restrict__ tmap,
           const LayerDev* __restrict__ layers) {
  using C = C_t<T>;
  constexpr int GW = 32, NG = 256 / GW;
  const int2 tm = tmap[blockIdx.x];
  const SolveFront f = list[tm.x];
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b;
  const int m0 = tm.y * NG * RPG;
  const int g = threadIdx.x / GW, gl = threadIdx.x % GW;
  const C* FT = reinterpret_cast<const C*>(L.fac) + f.fac;
  C* X = reinterpret_cast<C*>(L.X);
  const C* Z = reinterpret_cast<const C*>(L.Wt);
  const int* B = L.bidx + f.bidx;
  bool row_ok[RPG];
  const C* col[RPG];
#pragma unroll
  for (int r = 0; r < RPG; ++r) {
    const int m = m0 + g + NG * r;
    row_ok[r] = m < f.s;
    col[r] = FT + f.s + (long long)(row_ok[r] ? m : 0) * n;
  }
  // the row and column this lane will write, and its forward result
  int rsel = 0;
#pragma unroll
  for (int h = RPG / 2, off = GW / 2; h >= 1; h >>= 1, off >>= 1)
    if (gl & off) rsel += h;
  const int lo = gl & (GW / RPG - 1);
  const int m = m0 + g + NG * rsel;
  const bool mine = m < f.s && lo < KC;
  const long long idx = (long long)(f.off + m) * KC + lo;
  const C z0 = ld_or_zero(mine && !f.zero_z, Z + idx);
  C acc[RPG][KC];
#pragma unroll
  for (int r = 0; r < RPG; ++r)
#pragma unroll
    for (int c = 0; c < KC; ++c) acc[r][c] = czero<C>();
#pragma unroll(RPG >= 4 ? 2 : (RPG == 2 ? 4 : 8))
  for (int q = gl; q < f.b; q += GW) {
    const C* xb = X + (long long)ld(B + q) * KC;
    C fa[RPG], xv[KC];
#pragma unroll
    for (int r = 0; r < RPG; ++r) fa[r] = ld_or_zero(row_ok[r], col[r] + q);
#pragma unroll
    for (int c = 0; c < KC; ++c) xv[c] = ld(xb + c);
#pragma unroll
    for (int r = 0; r < RPG; ++r)
#pragma unroll
      for (int c = 0; c < KC; ++c) cfma(acc[r][c], fa[r], xv[c]);
  }
  // reduce-scatter over the group: each halving step trades half of the
  // lane's row sums with the partner lane (offset GW/2, GW/4, ...), so
  // that after log2(RPG) steps the lane holds one row's partial sum (the
  // row given by its high bits); a butterfly over the GW/RPG lanes that
  // share the row completes it (RPG = 8: 18 exchanges per column instead
  // of 80 for a butterfly per row)
  static_assert((RPG & (RPG - 1)) == 0 && RPG <= GW && KC <= GW / RPG, "group shape");
#pragma unroll
  for (int h = RPG / 2, off = GW / 2; h >= 1; h >>= 1, off >>= 1) {
    const bool up = (gl & off) != 0;
#pragma unroll
    for (int i = 0; i < h; ++i)
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const C send = up ? acc[i][c] : acc[i + h][c];
        const C keep = up ? acc[i + h][c] : acc[i][c];
        acc[i][c].x = keep.x + shfl_xor_t(send.x, off);
        acc[i][c].y = keep.y + shfl_xor_t(send.y, off);
      }
  }
#pragma unroll
  for (int c = 0; c < KC; ++c)
#pragma unroll
    for (int off = GW / (2 * RPG); off > 0; off >>= 1) {
      acc[0][c].x += shfl_xor_t(acc[0][c].x, off);
      acc[0][c].y += shfl_xor_t(acc[0][c].y, off);
    }
  if (!mine) return;
  C z = acc[0][0];
#pragma unroll
  for (int c = 1; c < KC; ++c)
    if (lo == c) z = acc[0][c];
  st(X + idx, cadd(z0, z));
}

}  // namespace

// Launch with the start and stop events t0, t1 recorded by the launch itself
// when given.
#define HELM_SOLVE_LAUNCH(KERNEL, GRID, ...)                                               \
  do {                                                                                     \
    if (t0)                                                                                \
      hipExtLaunchKernelGGL(KERNEL, dim3(GRID), dim3(256), 0, st, t0, t1, 0, __VA_ARGS__); \
    else                                                                                   \
      hipLaunchKernelGGL(KERNEL, dim3(GRID), dim3(256), 0, st, __VA_ARGS__);               \
  } while (0)

template <typename T>
void launch_fwd_gemv(const SolveFront* list, const int2* tmap, int total, const LayerDev* layers,
                     int k, int rtile, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  if (total <= 0) return;
  const int waves = (total + 3) / 4;   // rtile 1, 2: a wave per tile, 64 or 128 pivots
#define HELM_FWDV(KC_)                                                                    \
  switch (rtile) {                                                                        \
    case 1:                                                                               \
      HELM_SOLVE_LAUNCH((k_fwd_gemv_wave<T, KC_, 1>), waves, list, tmap, total, layers);  \
      break;                                                                              \
    case 2:                                                                               \
      HELM_SOLVE_LAUNCH((k_fwd_gemv_wave<T, KC_, 2>), waves, list, tmap, total, layers);  \
      break;                                                                              \
    case 16: HELM_SOLVE_LAUNCH((k_fwd_gemv<T, KC_, 16>), total, list, tmap, layers); break; \
    case 32: HELM_SOLVE_LAUNCH((k_fwd_gemv<T, KC_, 32>), total, list, tmap, layers); break; \
    default: HELM_SOLVE_LAUNCH((k_fwd_gemv<T, KC_, 64>), total, list, tmap, layers); break; \
  }
  switch (k) {
    case 1: HELM_FWDV(1); break;
    case 2: HELM_FWDV(2); break;
    case 3: HELM_FWDV(3); break;
    default: HELM_FWDV(4); break;
  }
#undef HELM_FWDV
}
template <typename T>
void launch_bwd_gemv(const SolveFront* list, const int2* tmap, int total, const LayerDev* layers,
                     int k, int rpg, hipStream_t st, hipEvent_t t0, hipEvent_t t1) {
  if (total <= 0) return;
#define HELM_BWDV(KC_)                                                                     \
  switch (rpg) {                                                                           \
    case 1: HELM_SOLVE_LAUNCH((k_bwd_gemv<T, KC_, 1>), total, list, tmap, layers); break;  \
    case 2: HELM_SOLVE_LAUNCH((k_bwd_gemv<T, KC_, 2>), total, list, tmap, layers); break;  \
    case 4: HELM_SOLVE_LAUNCH((k_bwd_gemv<T, KC_, 4>), total, list, tmap, layers); break;  \
    default: HELM_SOLVE_LAUNCH((k_bwd_gemv<T, KC_, 8>), total, list, tmap, layers); break; \
  }
  switch (k) {
    case 1: HELM_BWDV(1); break;
    case 2: HELM_BWDV(2); break;
    case 3: HELM_BWDV(3); break;
    default: HELM_BWDV(4); break;
  }
#undef HELM_BWDV
}

template <typename T>
void launch_fwd_gather(const SolveFront* list, const int2* tmap, int total,
                       const LayerDev* layers, int k, hipStream_t st) {
  if (total <= 0) return;
  // a tile is RT rows x k columns: one wave per tile for few columns
  if (k <= 4)
    hipLaunchKernelGGL((k_fwd_gather<T, 64>), dim3(total), dim3(64), 0, st, list, tmap, layers, k);
  else
    hipLaunchKernelGGL((k_fwd_gather<T, 256>), dim3(total), dim3(256), 0, st, list, tmap, layers,
                       k);
}
template <typename T>
void launch_fwd_gemm(const SolveFront* list, const int2* tmap, int total, const LayerDev* layers,
                     int k, void* scratch, int bn, bool gather, hipStream_t st, hipEvent_t t0,
                     hipEvent_t t1) {
  if (total <= 0) return;
  const int grid = total * ((k + bn - 1) / bn);
#define HELM_FWD(BN_)                                                                          \
  if (gather)                                                                                  \
    HELM_SOLVE_LAUNCH((k_fwd_gemm<T, BN_, true>), grid, list, tmap, layers, k, scratch);       \
  else                                                                                         \
    HELM_SOLVE_LAUNCH((k_fwd_gemm<T, BN_, false>), grid, list, tmap, layers, k, scratch)
  if (bn == 16) { HELM_FWD(16); } else if (bn == 32) { HELM_FWD(32); } else { HELM_FWD(64); }
#undef HELM_FWD
}
template <typename T>
void launch_fwd_reduce(const SolveFront* list, const int2* tmap, int total,
                       const LayerDev* layers, int k, const void* scratch, hipStream_t st) {
  if (total <= 0) return;
  if (k <= 4)
    hipLaunchKernelGGL((k_fwd_reduce<T, 64>), dim3(total), dim3(64), 0, st, list, tmap, layers, k,
                       scratch);
  else
    hipLaunchKernelGGL((k_fwd_reduce<T, 256>), dim3(total), dim3(256), 0, st, list, tmap, layers,
                       k, scratch);
}
template <typename T>
void launch_bwd_gemm(const SolveFront* list, const int2* tmap, int total, const LayerDev* layers,
                     int k, void* scratch, int bm, int bn, hipStream_t st, hipEvent_t t0,
                     hipEvent_t t1) {
  if (total <= 0) return;
  // a 32 x 16 tile has fewer MFMA blocks than waves: use 32 columns there
  if (bm == 32 && bn == 16) bn = 32;
  const int grid = total * ((k + bn - 1) / bn);
#define HELM_BWD(BM_, BN_) \
  HELM_SOLVE_LAUNCH((k_bwd_gemm<T, BM_, BN_>), grid, list, tmap, layers, k, scratch)
  if (bm == 32) {
    if (bn == 32) HELM_BWD(32, 32); else HELM_BWD(32, 64);
  } else {
    if (bn == 16) HELM_BWD(64, 16); else if (bn == 32) HELM_BWD(64, 32); else HELM_BWD(64, 64);
  }
#undef HELM_BWD
}
template <typename T>
void launch_bwd_reduce(const SolveFront* list, const int2* tmap, int total,
                       const LayerDev* layers, int k, const void* scratch, hipStream_t st) {
  if (total <= 0) return;
  if (k <= 4)
    hipLaunchKernelGGL((k_bwd_reduce<T, 64>), dim3(total), dim3(64), 0, st, list, tmap, layers, k,
                       scratch);
  else
    hipLaunchKernelGGL((k_bwd_reduce<T, 256>), dim3(total), dim3(256), 0, st, list, tmap, layers,
                       k, scratch);
}

#define HELM_INST_SOLVE(T)                                                                     \
  template void launch_fwd_gather<T>(const SolveFront*, const int2*, int, const LayerDev*,     \
                                     int, hipStream_t);                                        \
  template void launch_fwd_gemm<T>(const SolveFront*, const int2*, int, const LayerDev*, int,  \
                                   void*, int, bool, hipStream_t, hipEvent_t, hipEvent_t);     \
  template void launch_fwd_reduce<T>(const SolveFront*, const int2*, int, const LayerDev*,     \
                                     int, const void*, hipStream_t);                           \
  template void launch_bwd_gemm<T>(const SolveFront*, const int2*, int, const LayerDev*, int,  \
                                   void*, int, int, hipStream_t, hipEvent_t, hipEvent_t);      \
  template void launch_bwd_reduce<T>(const SolveFront*, const int2*, int, const LayerDev*,     \
                                     int, const void*, hipStream_t);                           \
  template void launch_fwd_gemv<T>(const SolveFront*, const int2*, int, const LayerDev*, int,  \
                                   int, hipStream_t, hipEvent_t, hipEvent_t);                  \
  template void launch_bwd_gemv<T>(const SolveFront*, const int2*, int, const LayerDev*, int,  \
                                   int, hipStream_t, hipEvent_t, hipEvent_t);
HELM_INST_SOLVE(float)
HELM_INST_SOLVE(double)

}  // namespace kern
}  // namespace helm
