// Multifrontal factorization kernels (offline stage, Algorithm 1).
//
// Every front holds an (s+b) x (s+b) column-major frontal matrix
//   F = [F11 F12; F21 F22]   (s pivots, b boundary variables).
// Instead of an LU with separate triangular solves, the s pivots are
// eliminated by a blocked Gauss-Jordan sweep with partial pivoting restricted
// to the rows of F11.  After the sweep the front holds
//   [F11^-1, F11^-1 F12; -F21 F11^-1, F22 - F21 F11^-1 F12],
// i.e. the inverse of the pivot block, the multipliers and the Schur
// complement passed to the parent.  Each block step of nb pivots is a small
// panel factorization (pivot choice), a row swap, and one rank-nb update of
// the whole front -- a dense complex GEMM that runs on the matrix cores.
// With the complex-symmetric operator (H = H^T) the stored left block
// [F11^-1; -F21 F11^-1] is all the substitutions need: the backward step uses
// the transpose of -F21 F11^-1 in place of F11^-1 F12.
#include "kernels.h"
#include "kernels_common.h"
#include "kernels_tile.h"

namespace helm {
namespace kern {

namespace {

template <typename T>
__device__ __forceinline__ C_t<T>* front_ptr(void* ws0, void* ws1, const FrontDev& f) {
  C_t<T>* base = reinterpret_cast<C_t<T>*>(f.ws_parity ? ws1 : ws0);
  return base + f.ws;
}

// The Schur complement of a complex-symmetric front is symmetric whatever
// rows the pivoting of F11 exchanged, so of the boundary x boundary block only
// the 64 x 64 tiles on and below the diagonal are assembled and updated: a
// tile of rows i0.. and columns j0.. is left out when this holds, and whoever
// reads the block takes the lower of the two mirror entries.  28% of the
// sweep's tiles at 100^3: complex64 sweep 80 -> 56 ms, complex128 175 -> 124.
__device__ __forceinline__ bool mirrored(const FrontDev& f, int i0, int j0) {
  return i0 >= f.s && j0 >= i0 + GT;
}

// --------------------------------------------------------------------------
// front assembly: frontal matrix = extend-add of the children's Schur
// complements (pull form: every entry is written once) ...
// The front-row -> child-boundary maps increase, so a tile above the diagonal
// reads the children's mirror entries: its columns' lanes walk their
// contiguous rows, and the tile is turned in LDS.
// --------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_extend_add(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
             int n_ids, const int2* __restrict__ tmap,
             const LayerDev* __restrict__ layers, void* ws0, void* ws1) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const int a = tm.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int nt = (n + GT - 1) / GT;
  const int tile = tm.y;
  const int i0 = (tile % nt) * GT, j0 = (tile / nt) * GT;
  if (mirrored(f, i0, j0)) return;   // uniform per block
  __shared__ int inv_r[2][GT], inv_c[2][GT];
  __shared__ C turn[GT][GT + 1];
  const LayerDev& L = layers[f.layer];
  const int t = threadIdx.x;
  if (t < 2 * GT) {
    int slot = t / GT, q = t % GT;
    int vr = -1, vc = -1;
    if (f.inv[slot] >= 0) {
      if (i0 + q < n) vr = L.inv[f.inv[slot] + i0 + q];
      if (j0 + q < n) vc = L.inv[f.inv[slot] + j0 + q];
    }
    inv_r[slot][q] = vr;
    inv_c[slot][q] = vc;
  }
  __syncthreads();
  C* F = front_ptr<T>(ws0, ws1, f);
  const C* S[2] = {nullptr, nullptr};
  int ldc[2] = {0, 0}, sc[2] = {0, 0};
  for (int slot = 0; slot < 2; ++slot) {
    if (f.child[slot] >= 0) {
      const FrontDev c = fronts[f.child[slot]];
      S[slot] = front_ptr<T>(ws0, ws1, c);
      ldc[slot] = c.s + c.b;
      sc[slot] = c.s;
    }
  }
  // the lane's 16 entries are all gathered before the first store; lanes
  // walk the tile's rows, above the diagonal its columns
  const bool upper = j0 > i0;
  constexpr int NJ = GT / (256 / GT);
  const int p = t % GT;
  C v[NJ];
#pragma unroll
  for (int u = 0; u < NJ; ++u) {
    const int q = t / GT + u * (256 / GT);
    const int ii = upper ? q : p, jj = upper ? p : q;
    const int gi = i0 + ii, gj = j0 + jj;
    C acc = czero<C>();
#pragma unroll
    for (int slot = 0; slot < 2; ++slot) {
      const int ri = inv_r[slot][ii], cj = inv_c[slot][jj];
      const bool hit = gi < n && gj < n && S[slot] && ri >= 0 && cj >= 0;
      const int lo = min(ri, cj), hi = max(ri, cj);
      acc = cadd(acc, ld_or_zero(hit, S[slot] + (hit ? (long long)(sc[slot] + hi) +
                                                         (long long)(sc[slot] + lo) * ldc[slot]
                                                     : 0)));
    }
    v[u] = acc;
  }
  if (upper) {   // uniform per block
#pragma unroll
    for (int u = 0; u < NJ; ++u) turn[t / GT + u * (256 / GT)][p] = v[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NJ; ++u) v[u] = turn[p][t / GT + u * (256 / GT)];
  }
  const int gi = i0 + p;
#pragma unroll
  for (int u = 0; u < NJ; ++u) {
    const int gj = j0 + t / GT + u * (256 / GT);
    if (gi < n && gj < n) st(F + (long long)gi + (long long)gj * n, v[u]);
  }
}

// ... plus the entries of H^l whose first-eliminated variable is a pivot of
// this front.  Discrete operator of Eq. discrete_local_Helmholtz in the
// complex-symmetric form: off-diagonal h^-2 beta_a(half) / (other two betas),
// diagonal minus their sum plus omega^2 m / (beta_x beta_y beta_z).
__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zdiv(double2 a, double2 b) { return cdiv(a, b); }

template <typename T>
__global__ void __launch_bounds__(256)
k_orig_entries(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
               int n_ids, const int2* __restrict__ tmap,
               const LayerDev* __restrict__ layers, void* ws0, void* ws1,
               GridDev g, int skip_front, FactorStatus* status) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const int a = tm.x;
  const FrontDev f = fronts[ids[a]];
  const int r = tm.y * 256 + threadIdx.x;
  // a front left unassembled on request (exercises the zero-pivot status)
  const bool valid = r < f.s && ids[a] != skip_front;
  const LayerDev& L = layers[f.layer];
  const int n = f.s + f.b;
  C* F = front_ptr<T>(ws0, ws1, f);
  const int nx = g.nx, ny = g.ny;
  int x = 0, y = 0, z = 0;
  double2 cpl[6];
  double2 dg = make_double2(0.0, 0.0);
  const double ih2 = 1.0 / (g.h * g.h);
  if (valid) {
    const int nat = L.nd2nat[f.off + r];
    x = nat % nx; y = (nat / nx) % ny; z = nat / (nx * ny);
    const double2 bx = g.bx[x], by = g.by[y], bz = L.bz[z];
    const double2 bxy = zmul(bx, by), bxz = zmul(bx, bz), byz = zmul(by, bz);
    // six couplings: -x, +x, -y, +y, -z, +z
    cpl[0] = zdiv(g.bxh[x], byz);
    cpl[1] = zdiv(g.bxh[x + 1], byz);
    cpl[2] = zdiv(g.byh[y], bxz);
    cpl[3] = zdiv(g.byh[y + 1], bxz);
    cpl[4] = zdiv(L.bzh[z], bxy);
    cpl[5] = zdiv(L.bzh[z + 1], bxy);
    int zg = L.lo + z;
    zg = zg < L.s ? L.s : (zg > L.e ? L.e : zg);   // model copied into the local PML
    const double mm = g.m[(long long)x + (long long)nx * ((long long)y + (long long)ny * zg)];
    dg = zdiv(make_double2(g.omega * g.omega * mm, 0.0), zmul(bxy, bz));
    for (int q = 0; q < 6; ++q) { dg.x -= cpl[q].x * ih2; dg.y -= cpl[q].y * ih2; }
  }
  {
    // largest |diagonal entry|^2 of the operator: a wave-wide maximum, then
    // one atomic per wave (bit patterns of non-negative doubles order like
    // the numbers)
    double d2 = dg.x * dg.x + dg.y * dg.y;
    for (int off = 32; off > 0; off >>= 1) d2 = fmax(d2, __shfl_xor(d2, off));
    if ((threadIdx.x & 63) == 0 && d2 > 0.0)
      atomicMax(&status->dmax, (unsigned long long)__double_as_longlong(d2));
  }
  if (!valid) return;
  {
    C& d = F[(long long)r + (long long)r * n];
    d = cadd(d, from_d2<C>(dg));
  }
  const int dx[6] = {-1, 1, 0, 0, 0, 0}, dy[6] = {0, 0, -1, 1, 0, 0},
            dz[6] = {0, 0, 0, 0, -1, 1};
  const int* B = L.bidx + f.bidx;
  for (int q = 0; q < 6; ++q) {
    int xx = x + dx[q], yy = y + dy[q], zz = z + dz[q];
    if (xx < 0 || xx >= nx || yy < 0 || yy >= ny || zz < 0 || zz >= L.t) continue;
    int ndn = L.nat2nd[xx + nx * (yy + ny * zz)];
    if (ndn < f.off) continue;  // assembled in a descendant front
    C v = from_d2<C>(make_double2(cpl[q].x * ih2, cpl[q].y * ih2));
    if (ndn < f.off + f.s) {
      int col = ndn - f.off;
      C& e = F[(long long)r + (long long)col * n];
      e = cadd(e, v);
    } else {
      // boundary variable: binary search in the sorted boundary list
      int lo = 0, hi = f.b - 1;
      while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (B[mid] < ndn) lo = mid + 1; else hi = mid;
      }
      if (f.b == 0 || B[lo] != ndn) continue;   // cannot happen for a valid plan
      int col = f.s + lo;
      C& e1 = F[(long long)r + (long long)col * n];
      e1 = cadd(e1, v);
      C& e2 = F[(long long)col + (long long)r * n];
      e2 = cadd(e2, v);
    }
  }
}

// --------------------------------------------------------------------------
// panel: LU with partial pivoting of rows [k, s) x columns [k, k+nbf) on a
// copy, to choose the nbf pivot rows; then D = (pivoted diagonal block)^-1.
// One workgroup of NT threads per front.  Three kernels: the panel in
// registers (k_panel_regs, every leaf front's), the current column block in
// registers and the rest in the global panel buffer (k_panel_rb), all of it in
// that buffer (k_panel, panels taller than the others take); only D, the pivots
// and the permutation leave a kernel.
// --------------------------------------------------------------------------
constexpr int NBMAX = 64;
constexpr int PB = 8;   // column block of the panel LU

// The largest v of a wave and the smallest index among the lanes that hold it
// (both uniform; v must not be NaN in the winning lane): the maximum through
// DPP moves, ties by a ballot.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = (int)(b & 0xffffffffll), hi = (int)(b >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
  return fmax(v, __longlong_as_double(((long long)h2 << 32) | (unsigned)l2));
}
__device__ __forceinline__ void wave_argmax(double& v, int& idx) {
  double m = dpp_max<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: lane 15 of each row
  m = dpp_max<0x112, 0xf>(m);
  m = dpp_max<0x114, 0xf>(m);
  m = dpp_max<0x118, 0xf>(m);
  m = dpp_max<0x142, 0xa>(m);          // row_bcast 15, 31: lane 63
  m = dpp_max<0x143, 0xc>(m);
  const long long b = __double_as_longlong(m);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), 63);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
  m = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  unsigned long long who = __ballot(v == m);
  int best = 0x7fffffff;
  while (who) {   // one lane but for ties
    const int l = __ffsll((long long)who) - 1;
    best = min(best, __builtin_amdgcn_readlane(idx, l));
    who &= who - 1;
  }
  v = m;
  idx = best;
}

// D = U^-1 L^-1 of the leading nbf x nbf block of the factored panel P
// (R rows, column-major): X = L^-1 by eliminating below each unit pivot, then
// D = U^-1 X from the last row up.  Wave w of the first four holds rows 16 w ..
// 16 w + 15 in registers, lane = column; each step passes one row of X through
// LDS (one barrier) and updates the rows it touches.
// With X in LDS and its entries dealt to the threads one by one (an integer
// division each), this was half of a tall panel's time.
template <typename T, int NT>
__device__ __forceinline__ void panel_inverse(const C_t<T>* P, int R, int nbf, int nb,
                                              C_t<T>* D) {
  using C = C_t<T>;
  static_assert(NT >= 256, "four waves hold the rows");
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  __shared__ C LU[NBMAX][NBMAX + 2];   // LU[c][r]: a column's rows are contiguous
  __shared__ C row[2][NBMAX];
  {
    // the factors, every load before the first store
    constexpr int PER = (NBMAX * NBMAX + NT - 1) / NT;
    C v[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = t + NT * i, r = e % NBMAX, c = e / NBMAX;
      const bool ok = r < nbf && c < nbf;
      v[i] = ld_or_zero(ok, P + (ok ? r + (long long)c * R : 0));
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = t + NT * i, r = e % NBMAX, c = e / NBMAX;
      if (NT * PER == NBMAX * NBMAX || e < NBMAX * NBMAX) LU[c][r] = v[i];
    }
  }
  const bool mine = w < 4;
  const int r0 = 16 * w;
  C x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = cmake<C>(r0 + i == lane ? 1.0 : 0.0, 0.0);
  __syncthreads();
  // X[i][:] -= L[i][q] X[q][:] for i > q
  for (int qg = 0; 16 * qg < nbf; ++qg) {
#pragma unroll
    for (int qi = 0; qi < 16; ++qi) {
      const int q = 16 * qg + qi;
      if (q + 1 >= nbf) break;
      if (w == qg) row[qi & 1][lane] = x[qi];
      __syncthreads();
      if (mine && w >= qg) {
        const C xq = row[qi & 1][lane];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (w > qg || i > qi) cfms(x[i], LU[q][r0 + i], xq);
      }
    }
  }
  // rows from the last one up: D[q] = X[q] / U[q][q], X[i] -= U[i][q] D[q]
  __syncthreads();
  for (int qg = (nbf - 1) / 16; qg >= 0; --qg) {
#pragma unroll
    for (int qi = 15; qi >= 0; --qi) {
      const int q = 16 * qg + qi;
      if (q >= nbf) continue;
      if (w == qg) {
        C u = LU[q][q];
        if (cabs2(u) == 0.0) u = cmake<C>(1.0, 0.0);
        x[qi] = cmul(x[qi], cdiv(cmake<C>(1.0, 0.0), u));
        row[qi & 1][lane] = x[qi];
      }
      __syncthreads();
      if (mine && w <= qg) {
        const C xq = row[qi & 1][lane];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (w < qg || i < qi) cfms(x[i], LU[q][r0 + i], xq);
      }
    }
  }
  if (mine && lane < nbf) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (r0 + i < nbf) st(D + (r0 + i) + (long long)lane * nb, x[i]);
  }
}

template <typename T, int NT>
__global__ void __launch_bounds__(NT)
k_panel(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
        int k, int nb, void* ws0, void* ws1, void* panel_base,
        const long long* __restrict__ panel_off, void* D_base, int* ipiv_base,
        int* perm_base, const long long* __restrict__ perm_off, FactorStatus* status) {
  using C = C_t<T>;
  constexpr int NW = NT / 64;
  const int a = blockIdx.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int R = f.s - k;
  if (R <= 0) return;
  const int nbf = R < nb ? R : nb;
  const int t = threadIdx.x;
  const C* F = front_ptr<T>(ws0, ws1, f);
  C* P = reinterpret_cast<C*>(panel_base) + panel_off[a];
  C* D = reinterpret_cast<C*>(D_base) + panel_off[a];
  int* ipiv = ipiv_base + perm_off[a];
  int* perm = perm_base + perm_off[a];
  if (k == 0)
    for (int i = t; i < f.s; i += NT) perm[i] = i;
  for (long long e = t; e < (long long)R * nbf; e += NT) {
    int r = e % R, c = e / R;
    P[r + (long long)c * R] = ld(F + (long long)(k + r) + (long long)(k + c) * n);
  }
  __shared__ double red_v[NW];
  __shared__ int red_i[NW];
  __shared__ int piv_row;
  // smallest and largest |pivot|^2 of this panel (thread 0)
  double pv_min = INFINITY, pv_max = 0.0;
  __syncthreads();
  // Blocked right-looking LU of the panel: columns in blocks of PB; inside
  // a block every column is pivoted, scaled and applied to the block's
  // remaining columns; then the block rows of the trailing columns are
  // solved with the block's unit lower triangle and the trailing columns
  // get one rank-PB update (one pass over them per block instead of one per
  // column).
  __shared__ C U12[PB][NBMAX];
  for (int c0 = 0; c0 < nbf; c0 += PB) {
    const int c1 = (c0 + PB < nbf) ? c0 + PB : nbf;
    for (int c = c0; c < c1; ++c) {
      // arg max |P[r][c]|, r >= c (ties: smallest row, so the choice is
      // reproducible)
      double best = -1.0;
      int bi = R;
      for (int r = c + t; r < R; r += NT) {
        double v = cabs2(P[r + (long long)c * R]);
        if (v > best) { best = v; bi = r; }
      }
      wave_argmax(best, bi);
      if ((t & 63) == 0) { red_v[t >> 6] = best; red_i[t >> 6] = bi; }
      __syncthreads();
      if (t == 0) {
        double bv = red_v[0];
        int bidx = red_i[0];
        for (int w = 1; w < NW; ++w)
          if (red_v[w] > bv || (red_v[w] == bv && red_i[w] < bidx)) {
            bv = red_v[w];
            bidx = red_i[w];
          }
        if (!(bv > 0.0) || !isfinite(bv)) {
          atomicExch(&status->flag, 1);   // zero or non-finite pivot
          bidx = c;
        } else {
          pv_min = fmin(pv_min, bv);
          pv_max = fmax(pv_max, bv);
        }
        piv_row = bidx;
        ipiv[c] = bidx;
        if (bidx != c) {
          int tmp = perm[k + c];
          perm[k + c] = perm[k + bidx];
          perm[k + bidx] = tmp;
        }
      }
      __syncthreads();
      const int p = piv_row;
      if (p != c)
        for (int cc = t; cc < nbf; cc += NT) {
          C x = P[c + (long long)cc * R];
          P[c + (long long)cc * R] = P[p + (long long)cc * R];
          P[p + (long long)cc * R] = x;
        }
      __syncthreads();
      C piv = P[c + (long long)c * R];
      if (cabs2(piv) == 0.0) piv = cmake<C>(1.0, 0.0);
      const C one = cmake<C>(1.0, 0.0);
      const C ipv = cdiv(one, piv);
      for (int r = c + 1 + t; r < R; r += NT)
        P[r + (long long)c * R] = cmul(P[r + (long long)c * R], ipv);
      __syncthreads();
      // rank-1 update of the block's remaining columns
      const int rows = R - c - 1, cols = c1 - c - 1;
      for (long long e = t; e < (long long)rows * cols; e += NT) {
        int r = c + 1 + (int)(e % rows), cc = c + 1 + (int)(e / rows);
        C& x = P[r + (long long)cc * R];
        cfms(x, P[r + (long long)c * R], P[c + (long long)cc * R]);
      }
      __syncthreads();
    }
    if (c1 >= nbf) break;
    const int W = nbf - c1, bw = c1 - c0;
    // block rows of the trailing columns: U12 = L11^-1 A12 (unit lower)
    for (int cc = t; cc < W; cc += NT) {
      const long long col = (long long)(c1 + cc) * R;
      for (int i = 0; i < bw; ++i) {
        C x = P[c0 + i + col];
        for (int j = 0; j < i; ++j) cfms(x, P[c0 + i + (long long)(c0 + j) * R], U12[j][cc]);
        U12[i][cc] = x;
        P[c0 + i + col] = x;
      }
    }
    __syncthreads();
    // rank-bw update of the trailing columns below the block
    for (int r = c1 + t; r < R; r += NT) {
      C l[PB];
#pragma unroll
      for (int j = 0; j < PB; ++j)
        l[j] = j < bw ? P[r + (long long)(c0 + j) * R] : czero<C>();
      for (int cc = 0; cc < W; ++cc) {
        C& x = P[r + (long long)(c1 + cc) * R];
        C y = x;
#pragma unroll
        for (int j = 0; j < PB; ++j)
          if (j < bw) cfms(y, l[j], U12[j][cc]);
        x = y;
      }
    }
    __syncthreads();
  }
  if (t == 0 && pv_max > 0.0) {
    atomicMin(&status->pmin, (unsigned long long)__double_as_longlong(pv_min));
    atomicMax(&status->pmax, (unsigned long long)__double_as_longlong(pv_max));
  }
  panel_inverse<T, NT>(P, R, nbf, nb, D);
}

// Panels of at most 64 RW rows: the panel in registers, a row per lane (its
// 64 columns in CH parts over as many waves, so that complex128 fits).
// Gauss-Jordan elimination with partial pivoting turns the panel into the
// inverse of its pivoted diagonal block in place: at column c the chosen row
// is scaled by the pivot's inverse and removed from every other row, and
// column c's slot, no longer needed, takes column c of the inverse (the
// eliminated unit column carried along).  The slots of the part that holds
// column c move down by one in the same step, so that the current column is
// always slot 0 and no register is chosen at run time.  Rows never leave their
// lanes; each tracks the index its row would have if rows were exchanged as in
// the LU, which gives the pivot choice of the LU with partial pivoting
// (largest |entry| among the rows not yet chosen, ties to the smallest index),
// the same exchange record ipiv and the same permutation.  With one wave of
// rows the pivot row comes by lane reads, with several through LDS (two
// barriers per column; one, or none, otherwise).  Bound: the chain of column
// steps (5 us each at 512 rows).  Panels of a 100^3 factorization 65 -> 43 ms
// in complex64 (512 rows 577 -> 318 us a launch; 768 rows were the taller
// kernel's 690) and 93 -> 65 ms in complex128 (whose 64-row panels took an LDS
// copy of 130 KB, one block per compute unit); 200^3 complex64 448 -> 350 ms.
template <typename T, int RW, int CH>
__global__ void __launch_bounds__(64 * RW * CH)
k_panel_regs(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
             int k, int nb, void* ws0, void* ws1, void* D_base, int* ipiv_base,
             int* perm_base, const long long* __restrict__ perm_off,
             const long long* __restrict__ panel_off, FactorStatus* status) {
  using C = C_t<T>;
  constexpr int NC = NBMAX / CH;
  const int a = blockIdx.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int R = f.s - k;
  if (R <= 0) return;
  const int nbf = R < nb ? R : nb;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int part = wave / RW, rw = wave % RW;
  const int t = rw * 64 + lane;   // this thread's panel row
  const bool row = t < R;
  const C* F = front_ptr<T>(ws0, ws1, f);
  C* D = reinterpret_cast<C*>(D_base) + panel_off[a];
  int* ipiv = ipiv_base + perm_off[a];
  int* perm = perm_base + perm_off[a];
  __shared__ double red_v[2][RW];
  __shared__ int red_i[2][RW];
  __shared__ C gcol[2][CH > 1 ? 64 * RW : 1];          // column c of every row
  __shared__ C prow[RW > 1 ? CH : 1][RW > 1 ? NC : 1];  // the pivot row
  __shared__ C piv_s;
  C x[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int c = part * NC + j;
    const bool ok = row && c < nbf;
    x[j] = ld_or_zero(ok, F + (ok ? (long long)(k + t) + (long long)(k + c) * n : 0));
  }
  // the permutation entry of this thread's row, read before any is written
  const int pold = k == 0 ? t : (row ? ld(perm + k + t) : 0);
  if (RW * CH > 1) __syncthreads();
  int pos = t;           // the row's index were rows exchanged as in the LU
  bool chosen = false;   // the row is the pivot row of an earlier column
  double pv_min = INFINITY, pv_max = 0.0;
  for (int c = 0; c < nbf; ++c) {
    const bool owner = CH == 1 || c / NC == part;
    const int buf = c & 1;
    const bool cand = row && !chosen;
    C g = x[0];
    double bv = -1.0;
    int P = R;
    if (owner) {
      bv = cand ? cabs2(g) : -1.0;
      P = cand ? pos : R;
      wave_argmax(bv, P);
      if (RW * CH > 1 && lane == 0) {
        red_v[buf][rw] = bv;
        red_i[buf][rw] = P;
      }
      if (CH > 1) gcol[buf][t] = g;
    }
    if (RW * CH > 1) {
      __syncthreads();
      bv = red_v[buf][0];
      P = red_i[buf][0];
#pragma unroll
      for (int w = 1; w < RW; ++w)
        if (red_v[buf][w] > bv || (red_v[buf][w] == bv && red_i[buf][w] < P)) {
          bv = red_v[buf][w];
          P = red_i[buf][w];
        }
      if (CH > 1) g = gcol[buf][t];
    }
    // a zero or non-finite maximum: flagged, the row at index c taken
    const bool bad = !(bv > 0.0) || !isfinite(bv);
    if (bad) {
      P = c;
      if (threadIdx.x == 0) atomicExch(&status->flag, 1);
    } else {
      pv_min = fmin(pv_min, bv);
      pv_max = fmax(pv_max, bv);
    }
    if (threadIdx.x == 0) ipiv[c] = P;
    const bool win = cand && pos == P;
    C piv;
    int pl = 0;
    if (RW == 1) {
      pl = __builtin_amdgcn_readfirstlane(__ffsll((long long)__ballot(win)) - 1);
      piv.x = lane_read(g.x, pl);
      piv.y = lane_read(g.y, pl);
    } else {
      if (win) {
#pragma unroll
        for (int j = 0; j < NC; ++j) prow[part][j] = x[j];
        if (owner) piv_s = g;
      }
      __syncthreads();
      piv = piv_s;
    }
    // exchange of indices c and P: the row at c moves to P, the pivot row to c
    if (pos == c) pos = P;
    if (win) {
      pos = c;
      chosen = true;
    }
    if (cabs2(piv) == 0.0) piv = cmake<C>(1.0, 0.0);
    const C ipv = cdiv(cmake<C>(1.0, 0.0), piv);
    // row -= gw w with w the pivot row: gw = g / piv, and for the pivot row
    // itself (read as zero) -1 / piv; column c of the inverse is -gw
    const C gw = win ? cneg(ipv) : cmul(g, ipv);
    auto reduced = [&](int j) {
      C w;
      if (RW == 1) {
        w.x = lane_read(x[j].x, pl);
        w.y = lane_read(x[j].y, pl);
      } else {
        w = prow[part][j];
      }
      C y = win ? czero<C>() : x[j];
      cfms(y, gw, w);
      return y;
    };
    if (owner) {
#pragma unroll
      for (int j = 1; j < NC; ++j) x[j - 1] = reduced(j);
      x[NC - 1] = cneg(gw);
    } else {
#pragma unroll
      for (int j = 0; j < NC; ++j) x[j] = reduced(j);
    }
  }
  if (threadIdx.x == 0 && pv_max > 0.0) {
    atomicMin(&status->pmin, (unsigned long long)__double_as_longlong(pv_min));
    atomicMax(&status->pmax, (unsigned long long)__double_as_longlong(pv_max));
  }
  if (row && part == 0) perm[k + pos] = pold;
  if (row && pos < nbf) {
    const int turned = min(max(nbf - part * NC, 0), NC);   // steps its slots moved
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int c = part * NC + (j + turned) % NC;
      if (c < nbf) st(D + pos + (long long)c * nb, x[j]);
    }
  }
}

// Tall panels (more rows than k_panel_regs takes): the same blocked LU with
// partial pivoting, with the current column block of every row held in
// registers.  Thread t owns the rows t, t + NT, ... (RPT of them); a column
// step (pivot search, row exchange, scaling, rank-1 update of the block)
// works on registers and LDS only, so the panel copy in global memory is
// passed over once per block (the trailing update) instead of once per
// column.  Pivots, swaps and arithmetic are those of k_panel.
template <typename T, int NT, int RPT, int BW>
__global__ void __launch_bounds__(NT)
k_panel_rb(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
           int k, int nb, void* ws0, void* ws1, void* panel_base,
           const long long* __restrict__ panel_off, void* D_base, int* ipiv_base,
           int* perm_base, const long long* __restrict__ perm_off, FactorStatus* status) {
  using C = C_t<T>;
  constexpr int NW = NT / 64;
  const int a = blockIdx.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int R = f.s - k;
  if (R <= 0) return;
  const int nbf = R < nb ? R : nb;
  const int t = threadIdx.x;
  const C* F = front_ptr<T>(ws0, ws1, f);
  C* P = reinterpret_cast<C*>(panel_base) + panel_off[a];
  C* D = reinterpret_cast<C*>(D_base) + panel_off[a];
  int* ipiv = ipiv_base + perm_off[a];
  int* perm = perm_base + perm_off[a];
  if (k == 0)
    for (int i = t; i < f.s; i += NT) perm[i] = i;
  // the panel's columns past the first block to the global copy (each
  // thread its own rows, a group of columns' loads before their stores);
  // the first block goes straight to registers
  constexpr int CG = sizeof(T) == 4 ? BW : BW / 2;   // columns per load group
  for (int cg = BW; cg < nbf; cg += CG) {
    C v[RPT][CG];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = t + i * NT;
#pragma unroll
      for (int j = 0; j < CG; ++j)
        v[i][j] = ld_or_zero(r < R && cg + j < nbf,
                             F + (long long)(k + (r < R ? r : 0)) + (long long)(k + cg + j) * n);
    }
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = t + i * NT;
#pragma unroll
      for (int j = 0; j < CG; ++j)
        if (r < R && cg + j < nbf) P[r + (long long)(cg + j) * R] = v[i][j];
    }
  }
  __shared__ double red_v[NW];
  __shared__ int red_i[NW];
  __shared__ C xch[BW];      // row c's block values, for the pivot row's owner
  __shared__ C prow[BW];     // the pivot row's block values
  __shared__ int bsw[BW];    // the block's pivot rows (swap c0 + j <-> bsw[j])
  __shared__ int src[2 * BW], dst[2 * BW];   // the block's composed row moves
  __shared__ int nmove;
  __shared__ C mv[NBMAX][2 * BW];            // staged values of the moves
  __shared__ C L11[BW][BW];  // the block rows' factors (unit lower part used)
  __shared__ C U12[BW][NBMAX];
  double pv_min = INFINITY, pv_max = 0.0;
  C x[RPT][BW];
  for (int c0 = 0; c0 < nbf; c0 += BW) {
    const int c1 = (c0 + BW < nbf) ? c0 + BW : nbf;
    const int bw = c1 - c0;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = t + i * NT;
#pragma unroll
      for (int j = 0; j < BW; ++j) {
        const bool ok = r < R && j < bw;
        x[i][j] = c0 == 0 ? ld_or_zero(ok, F + (long long)(k + (ok ? r : 0)) + (long long)(k + j) * n)
                          : (ok ? P[r + (long long)(c0 + j) * R] : czero<C>());
      }
    }
    if (c0 == 0) __syncthreads();   // the copy is complete before any row swap
#pragma unroll
    for (int jc = 0; jc < BW; ++jc) {
      if (jc >= bw) break;
      const int c = c0 + jc;
      // arg max |P[r][c]|, r >= c (ties: smallest row): wave maxima to LDS,
      // then every thread reduces them (no second barrier)
      double best = -1.0;
      int bi = R;
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r = t + i * NT;
        if (r >= c && r < R) {
          const double v = cabs2(x[i][jc]);
          if (v > best) { best = v; bi = r; }
        }
      }
      wave_argmax(best, bi);
      if ((t & 63) == 0) { red_v[t >> 6] = best; red_i[t >> 6] = bi; }
      __syncthreads();
      double bv = red_v[0];
      int p = red_i[0];
#pragma unroll
      for (int w = 1; w < NW; ++w)
        if (red_v[w] > bv || (red_v[w] == bv && red_i[w] < p)) {
          bv = red_v[w];
          p = red_i[w];
        }
      if (!(bv > 0.0) || !isfinite(bv)) {
        if (t == 0) atomicExch(&status->flag, 1);   // zero or non-finite pivot
        p = c;
      } else if (t == 0) {
        pv_min = fmin(pv_min, bv);
        pv_max = fmax(pv_max, bv);
      }
      if (t == 0) {
        ipiv[c] = p;
        bsw[jc] = p;
      }
      // rows c and p trade places: the pivot row's block values go to prow
      // (every thread reads them), row c's to xch (for row p's owner)
      const int tc = c % NT, ic = c / NT, tp = p % NT, ip = p / NT;
      if (t == tp)
#pragma unroll
        for (int i = 0; i < RPT; ++i)
          if (i == ip)
#pragma unroll
            for (int j = 0; j < BW; ++j) prow[j] = x[i][j];
      if (t == tc && p != c)
#pragma unroll
        for (int i = 0; i < RPT; ++i)
          if (i == ic)
#pragma unroll
            for (int j = 0; j < BW; ++j) xch[j] = x[i][j];
      __syncthreads();
      if (p != c) {
        if (t == tc)
#pragma unroll
          for (int i = 0; i < RPT; ++i)
            if (i == ic)
#pragma unroll
              for (int j = 0; j < BW; ++j) x[i][j] = prow[j];
        if (t == tp)
#pragma unroll
          for (int i = 0; i < RPT; ++i)
            if (i == ip)
#pragma unroll
              for (int j = 0; j < BW; ++j) x[i][j] = xch[j];
      }
      C piv = prow[jc];
      if (cabs2(piv) == 0.0) piv = cmake<C>(1.0, 0.0);
      const C ipv = cdiv(cmake<C>(1.0, 0.0), piv);
      // scale the column below the pivot, rank-1 update of the block's
      // remaining columns
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r = t + i * NT;
        if (r > c && r < R) {
          const C l = cmul(x[i][jc], ipv);
          x[i][jc] = l;
#pragma unroll
          for (int j = 0; j < BW; ++j)
            if (j > jc && j < bw) cfms(x[i][j], l, prow[j]);
        }
      }
    }
    // the block's row swaps, composed into moves dst <- src (at most 2 BW
    // rows), applied at once to the columns outside the block and to the
    // row permutation: every value is loaded before any is stored
    if (t == 0) {
      // dst[q]: a touched row, src[q]: the row whose content ends there
      int m = 0;
      for (int j = 0; j < bw; ++j) {
        const int ra = c0 + j, rb = bsw[j];
        int qa = -1, qb = -1;
        for (int q = 0; q < m; ++q) {
          if (dst[q] == ra) qa = q;
          if (dst[q] == rb) qb = q;
        }
        if (qa < 0) { qa = m; dst[m] = ra; src[m] = ra; ++m; }
        if (qb < 0) { qb = m; dst[m] = rb; src[m] = rb; ++m; }
        const int y = src[qa];
        src[qa] = src[qb];
        src[qb] = y;
      }
      int nm = 0;
      for (int q = 0; q < m; ++q)
        if (src[q] != dst[q]) { dst[nm] = dst[q]; src[nm] = src[q]; ++nm; }
      nmove = nm;
    }
    __syncthreads();
    const int nm = nmove;
    if (nm > 0) {
      // through LDS: every moved value is read before any is written (all
      // of a thread's loads issued before its first LDS store)
      constexpr int MV = (NBMAX * 2 * BW + NT - 1) / NT;
      C mvv[MV];
#pragma unroll
      for (int i = 0; i < MV; ++i) {
        const int e = t + NT * i, cc = e / nm, q = e % nm;
        const bool ok = e < nbf * nm && (cc < c0 || cc >= c1);
        mvv[i] = ld_or_zero(ok, P + (ok ? src[q] + (long long)cc * R : 0));
      }
#pragma unroll
      for (int i = 0; i < MV; ++i) {
        const int e = t + NT * i, cc = e / nm, q = e % nm;
        if (e < nbf * nm && (cc < c0 || cc >= c1)) mv[cc][q] = mvv[i];
      }
      int pv = 0;
      if (t < nm) pv = perm[k + src[t]];
      __syncthreads();
      for (int e = t; e < nbf * nm; e += NT) {
        const int cc = e / nm, q = e % nm;
        if (cc < c0 || cc >= c1) P[dst[q] + (long long)cc * R] = mv[cc][q];
      }
      if (t < nm) perm[k + dst[t]] = pv;
    }
    // the block's columns back to the global copy; the block rows' factors
    // to LDS for the trailing solve
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int r = t + i * NT;
      if (r < R)
#pragma unroll
        for (int j = 0; j < BW; ++j)
          if (j < bw) P[r + (long long)(c0 + j) * R] = x[i][j];
      if (r >= c0 && r < c1)
#pragma unroll
        for (int j = 0; j < BW; ++j) L11[r - c0][j] = x[i][j];
    }
    __syncthreads();
    if (c1 >= nbf) break;
    const int W = nbf - c1;
    // block rows of the trailing columns: U12 = L11^-1 A12 (unit lower),
    // the column's block rows loaded together first
    for (int cc = t; cc < W; cc += NT) {
      const long long col = (long long)(c1 + cc) * R;
      C u[BW];
#pragma unroll
      for (int i = 0; i < BW; ++i) u[i] = i < bw ? P[c0 + i + col] : czero<C>();
#pragma unroll
      for (int i = 0; i < BW; ++i) {
        if (i >= bw) break;
        C y = u[i];
#pragma unroll
        for (int j = 0; j < BW; ++j)
          if (j < i) cfms(y, L11[i][j], u[j]);
        u[i] = y;
        U12[i][cc] = y;
        P[c0 + i + col] = y;
      }
    }
    __syncthreads();
    // rank-bw update of the trailing columns below the block (own rows):
    // a group of TG columns of all the thread's rows loaded before any of
    // their stores, so that RPT x TG loads are in flight per thread
    constexpr int TG = CG < (NT >= 1024 ? 16 : 32) / RPT ? CG : (NT >= 1024 ? 16 : 32) / RPT;
    for (int cg = 0; cg < W; cg += TG) {
      C y[RPT][TG];
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r = t + i * NT;
        const bool ok = r >= c1 && r < R;
#pragma unroll
        for (int q = 0; q < TG; ++q) {
          const bool in = ok && cg + q < W;
          y[i][q] = ld_or_zero(in, P + (in ? r + (long long)(c1 + cg + q) * R : 0));
        }
      }
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r = t + i * NT;
        if (r < c1 || r >= R) continue;
#pragma unroll
        for (int q = 0; q < TG; ++q) {
          if (cg + q >= W) break;
#pragma unroll
          for (int j = 0; j < BW; ++j)
            if (j < bw) cfms(y[i][q], x[i][j], U12[j][cg + q]);
          P[r + (long long)(c1 + cg + q) * R] = y[i][q];
        }
      }
    }
    __syncthreads();
  }
  if (t == 0 && pv_max > 0.0) {
    atomicMin(&status->pmin, (unsigned long long)__double_as_longlong(pv_min));
    atomicMax(&status->pmax, (unsigned long long)__double_as_longlong(pv_max));
  }
  panel_inverse<T, NT>(P, R, nbf, nb, D);
}

// --------------------------------------------------------------------------
// apply the nbf row swaps to every column, then rows J <- D * rows J for the
// columns outside J.  One workgroup per 64-column tile.
// The swaps are composed first (one wave, in registers): row k + jj of J
// ends up holding old row srcJ[jj], and each row outside J that a swap
// touches (at most nbf of them) holds old row srcO[i].  Every new value is
// then one independent load, so the column tile is read once, in parallel,
// instead of through nbf dependent swaps per column.
// complex128 takes the product on the matrix-core tile (whole operands in LDS
// were 133 KB, one block per CU): 71^3 8.6 -> 5.9 ms.  complex64 keeps FP32
// products: the tile's split took 100^3 from 14.7 to 9.9 ms, but the layer
// solves' error against complex128 grew by 9% on smooth media (geometric mean
// 1.95e-6 -> 2.12e-6).
// --------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_swap_JO(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
          int n_active, const int2* __restrict__ tmap, int k, int nb,
          void* ws0, void* ws1, const void* D_base, const int* __restrict__ ipiv_base,
          const long long* __restrict__ panel_off, const long long* __restrict__ perm_off) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const int a = tm.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int nbf = (f.s - k) < nb ? (f.s - k) : nb;
  const int c0 = tm.y * GT;
  C* F = front_ptr<T>(ws0, ws1, f);
  const int* ipiv = ipiv_base + perm_off[a];
  const C* D = reinterpret_cast<const C*>(D_base) + panel_off[a];
  const int t = threadIdx.x;
  __shared__ int srcJ[NBMAX], rowO[NBMAX], srcO[NBMAX];
  __shared__ int nO;
  if (t < 64) {
    // lane i holds srcJ[i] and outside entry i (row ro, source so)
    int vJ = k + t, ro = -1, so = 0, cnt = 0;
    const int piv = ld(ipiv + (t < nbf ? t : 0));
    for (int jj = 0; jj < nbf; ++jj) {
      const int r2 = k + __builtin_amdgcn_readlane(piv, jj);
      const int cur = __builtin_amdgcn_readlane(vJ, jj);
      if (r2 < k + nbf) {
        const int other = __builtin_amdgcn_readlane(vJ, r2 - k);
        if (t == jj) vJ = other;
        if (t == r2 - k) vJ = cur;
      } else {
        const unsigned long long hit = __ballot(ro == r2);
        if (hit) {
          const int i = __ffsll((long long)hit) - 1;
          const int other = __builtin_amdgcn_readlane(so, i);
          if (t == jj) vJ = other;
          if (t == i) so = cur;
        } else {
          if (t == jj) vJ = r2;
          if (t == cnt) { ro = r2; so = cur; }
          ++cnt;
        }
      }
    }
    if (t < nbf) srcJ[t] = vJ;
    if (t < cnt) { rowO[t] = ro; srcO[t] = so; }
    if (t == 0) nO = cnt;
  }
  __syncthreads();
  const int no = nO;
  // every read of the tile before any write
  constexpr int WPT = NBMAX * GT / 256;
  C w[WPT];
#pragma unroll
  for (int i = 0; i < WPT; ++i) {
    const int e = t + 256 * i, r = e / GT, gc = c0 + e % GT;
    const bool ok = r < no && gc < n;
    w[i] = ld_or_zero(ok, F + (ok ? (long long)srcO[r] + (long long)gc * n : 0));
  }
  if constexpr (sizeof(T) == 8) {
    // the rows are swapped in place and read back as the tile's row operand
    C vj[WPT];
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int e = t + 256 * i, r = e % NBMAX, gc = c0 + e / NBMAX;
      const bool ok = r < nbf && gc < n;
      vj[i] = ld_or_zero(ok, F + (ok ? (long long)srcJ[r] + (long long)gc * n : 0));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int e = t + 256 * i, r = e / GT, gc = c0 + e % GT;
      if (r < no && gc < n) st(F + (long long)rowO[r] + (long long)gc * n, w[i]);
      const int rj = e % NBMAX, gj = c0 + e / NBMAX;
      if (rj < nbf && gj < n) st(F + (long long)(k + rj) + (long long)gj * n, vj[i]);
    }
    __syncthreads();
    // P rows = columns gc of F: V^T(gc, q) = F[(k + q) + gc n], swapped above
    // Q columns = rows r of J: D^T(q, r) = D[r + q nb]
    __shared__ TileSmem<T, 64> sm;
    TileAcc<T, 64, 64, true> acc;
    tile_gemm<T, 64, 64, true, kDirect>(sm, acc, TileP<T>{F + k, n, n}, TileQ<T>{D, nb, nbf},
                                        c0, 0, 0, nbf);
    __syncthreads();   // in place: every read before any write
    using O = TileOut<T, 64, 64>;
    const O o;
#pragma unroll
    for (int i = 0; i < O::NR; ++i)
#pragma unroll
      for (int j = 0; j < O::NC; ++j) {
        const int gc = c0 + o.r[i], r = o.c[j];
        if (r >= nbf || gc >= n || (gc >= k && gc < k + nbf)) continue;
        st(F + (long long)(k + r) + (long long)gc * n, acc_at(acc, i, j));
      }
  } else {
    __shared__ C V[NBMAX][GT + 1];
    __shared__ C DsT[NBMAX][NBMAX + 1];  // DsT[q][r] = D(r, q)
    // the rows J of the tile and D: every load issued before the first store
    C vj[WPT], dw[WPT];
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int e = t + 256 * i, r = e % NBMAX, c = e / NBMAX, gc = c0 + c;
      const bool ok = r < nbf && gc < n;
      vj[i] = ld_or_zero(ok, F + (ok ? (long long)srcJ[r] + (long long)gc * n : 0));
      const bool dok = r < nbf && c < nbf;
      dw[i] = ld_or_zero(dok, D + (dok ? r + c * nb : 0));
    }
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int e = t + 256 * i, r = e % NBMAX, c = e / NBMAX;
      V[r][c] = vj[i];
      DsT[c][r] = dw[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WPT; ++i) {
      const int e = t + 256 * i, r = e / GT, gc = c0 + e % GT;
      if (r < no && gc < n) st(F + (long long)rowO[r] + (long long)gc * n, w[i]);
    }
    // rows J of the tile: thread (rg, cg) owns rows rg + 16 i and columns
    // cg + 16 j (i, j < 4), so each LDS value read feeds four products
    const int rg = t & 15, cg = t >> 4;
    C acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = czero<C>();
    for (int q = 0; q < nbf; ++q) {
      C dv[4], vv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) dv[i] = DsT[q][rg + 16 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) vv[j] = V[q][cg + 16 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) cfma(acc[i][j], dv[i], vv[j]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = rg + 16 * i, c = cg + 16 * j, gc = c0 + c;
        if (r >= nbf || gc >= n) continue;
        const bool inJ = gc >= k && gc < k + nbf;
        st(F + (long long)(k + r) + (long long)gc * n, inJ ? V[r][c] : acc[i][j]);
      }
  }
}

// --------------------------------------------------------------------------
// rank-nb update of every entry outside the pivot rows / columns J:
//   F(O, O) -= F(O, J) F(J, O)     (J rows already hold D * F(J, O))
// Computed as C^T = B^T A^T so that the MFMA column index walks the
// contiguous (row) dimension of the column-major front.  Entries of rows
// already eliminated (< k) in boundary columns (>= s) are skipped: they
// would accumulate F11^-1 F12, which neither the factor store (the
// symmetric operator's backward step uses the transpose of -F21 F11^-1) nor
// the parent's extend-add (the Schur block) ever reads.  Tiles that lie
// wholly in J or in that block, and the mirrored ones of the Schur block,
// return at once.
// Bound: the trailing entries streamed from and to HBM once per pivot block
// (complex64 at 200^3: 3.6 TB in 1.13 s, 3.2 TB/s) and the latency of a two-step
// product between them.  complex64 runs on the split bf16 tile: against the FP32
// tile, the mirrored tiles still among them, 1916 -> 1604 ms of a 200^3
// factorization and 93 -> 80 ms of a 100^3 one (complex128 at 100^3: 186 ->
// 175); now 1129, 56 and 121.  Loading the tile's entries before the product
// needs 200 registers (2 waves per SIMD): 1809 ms against 1639; kept at 3 waves
// it spills: 3688.
// --------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 2, 8)))
k_sweep_gemm(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
             int n_active, const int2* __restrict__ tmap, int k, int nb,
             void* ws0, void* ws1) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const int a = tm.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int nbf = (f.s - k) < nb ? (f.s - k) : nb;
  const int nt = (n + GT - 1) / GT;
  const int tile = tm.y;
  const int i0 = (tile % nt) * GT;   // rows of F
  const int j0 = (tile / nt) * GT;   // columns of F
  const bool rowsJ = i0 >= k && i0 + GT <= k + nbf, colsJ = j0 >= k && j0 + GT <= k + nbf;
  if (rowsJ || colsJ || (i0 + GT <= k && j0 >= f.s) || mirrored(f, i0, j0))
    return;   // uniform per block
  C* F = front_ptr<T>(ws0, ws1, f);
  // P rows = C columns j: B^T(j, q) = F[(k + q) + j n]
  // Q columns = C rows i: A^T(q, i) = F[i + (k + q) n]
  __shared__ TileSmem<T, 64> sm;
  TileAcc<T, 64, 64, true> acc;
  tile_gemm<T, 64, 64, true, kDirect>(sm, acc, TileP<T>{F + k, n, n},
                                      TileQ<T>{F + (long long)k * n, n, n}, j0, i0, 0, nbf);
  // F(i, j) -= product: every entry of the lane is loaded before the first
  // store (one latency for the group instead of a load-store chain per entry)
  using O = TileOut<T, 64, 64>;
  const O o;
  auto outside = [&](int gi, int gj) {
    return gi < n && gj < n && (gi < k || gi >= k + nbf) && (gj < k || gj >= k + nbf) &&
           !(gi < k && gj >= f.s);
  };
  C cv[O::NR][O::NC];
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gi = i0 + o.c[j], gj = j0 + o.r[i];
      cv[i][j] = ld_or_zero(outside(gi, gj), F + (long long)gi + (long long)gj * n);
    }
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gi = i0 + o.c[j], gj = j0 + o.r[i];
      if (outside(gi, gj))
        st(F + (long long)gi + (long long)gj * n, csub(cv[i][j], acc_at(acc, i, j)));
    }
}

// --------------------------------------------------------------------------
// columns J: rows outside J <- -F(O, J) D, rows J <- D.  One workgroup per
// 64-row tile, as one product of the matrix-core tile (K = the pivot block).
// Bound by the latency of its loads: with both operands held whole in LDS
// (133 KB in complex128) one block ran per CU.  Factorization of 100^3
// complex64 10.6 -> 6.0 ms, 71^3 complex128 6.9 -> 4.2; the error of the
// complex64 layer solves against complex128 is the same to 0.5%.
// --------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_update_OJ(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
            int n_active, const int2* __restrict__ tmap, int k, int nb,
            void* ws0, void* ws1, const void* D_base,
            const long long* __restrict__ panel_off) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const int a = tm.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int nbf = (f.s - k) < nb ? (f.s - k) : nb;
  const int r0 = tm.y * GT;
  C* F = front_ptr<T>(ws0, ws1, f);
  const C* D = reinterpret_cast<const C*>(D_base) + panel_off[a];
  // P rows = columns c of the panel: D^T(c, q) = D[q + c nb]
  // Q columns = rows i of F: F(i, q) = F[i + (k + q) n]
  __shared__ TileSmem<T, 64> sm;
  TileAcc<T, 64, 64, true> acc;
  tile_gemm<T, 64, 64, true, kDirect>(sm, acc, TileP<T>{D, nb, nbf},
                                      TileQ<T>{F + (long long)k * n, n, n}, 0, r0, 0, nbf);
  __syncthreads();   // the tile is updated in place: every read before any write
  using O = TileOut<T, 64, 64>;
  const O o;
#pragma unroll
  for (int i = 0; i < O::NR; ++i)
#pragma unroll
    for (int j = 0; j < O::NC; ++j) {
      const int gr = r0 + o.c[j], c = o.r[i];
      if (gr >= n || c >= nbf) continue;
      const bool inJ = gr >= k && gr < k + nbf;
      st(F + (long long)gr + (long long)(k + c) * n,
         inJ ? ld(D + (gr - k) + c * nb) : cneg(acc_at(acc, i, j)));
    }
}

// --------------------------------------------------------------------------
// copy the first s columns to the factor store, undoing the row pivoting of
// F11 (which permuted the columns of the swept inverse): true column perm[i]
// <- swept column i.
// --------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_store_factor(const FrontDev* __restrict__ fronts, const int* __restrict__ ids,
               int n_ids, const int2* __restrict__ tmap,
               const LayerDev* __restrict__ layers, void* ws0, void* ws1,
               const int* __restrict__ perm_base, const long long* __restrict__ perm_off) {
  using C = C_t<T>;
  const int2 tm = tmap[blockIdx.x];
  const int a = tm.x;
  const FrontDev f = fronts[ids[a]];
  const int n = f.s + f.b;
  const int nrt = (n + GT - 1) / GT;
  const int tile = tm.y;
  const int i0 = (tile % nrt) * GT, j0 = (tile / nrt) * GT;
  const C* F = front_ptr<T>(ws0, ws1, f);
  C* FT = reinterpret_cast<C*>(layers[f.layer].fac) + f.fac;
  const int* perm = perm_base + perm_off[a];
  const int t = threadIdx.x;
  const int i = t % GT;
  for (int jj = t / GT; jj < GT; jj += 256 / GT) {
    int gi = i0 + i, gj = j0 + jj;
    if (gi >= n || gj >= f.s) continue;
    FT[(long long)gi + (long long)perm[gj] * n] = F[(long long)gi + (long long)gj * n];
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T>
void launch_extend_add(const FrontDev* fronts, const int* ids, int n_ids,
                       const int2* tmap, int total, const LayerDev* layers,
                       void* ws0, void* ws1, hipStream_t st) {
  if (total <= 0) return;
  hipLaunchKernelGGL(k_extend_add<T>, dim3(total), dim3(256), 0, st, fronts, ids,
                     n_ids, tmap, layers, ws0, ws1);
}
template <typename T>
void launch_orig_entries(const FrontDev* fronts, const int* ids, int n_ids,
                         const int2* tmap, int total, const LayerDev* layers,
                         void* ws0, void* ws1, const GridDev& g, int skip_front,
                         FactorStatus* status, hipStream_t st) {
  if (total <= 0) return;
  hipLaunchKernelGGL(k_orig_entries<T>, dim3(total), dim3(256), 0, st, fronts, ids,
                     n_ids, tmap, layers, ws0, ws1, g, skip_front, status);
}
template <typename T>
void launch_panel(const FrontDev* fronts, const int* ids, int n_active, int max_rows,
                  int k, int nb, void* ws0, void* ws1, void* panel,
                  const long long* panel_off, void* D, int* ipiv, int* perm,
                  const long long* perm_off, FactorStatus* status, hipStream_t st) {
  if (n_active <= 0) return;
  // threads and panel home from the tallest panel of the launch
#define HELM_PANEL(NT)                                                              \
  hipLaunchKernelGGL((k_panel<T, NT>), dim3(n_active), dim3(NT), 0, st,            \
                     fronts, ids, k, nb, ws0, ws1, panel, panel_off, D, ipiv, perm, \
                     perm_off, status)
#define HELM_PANEL_RB(NT, RPT, BW)                                                  \
  hipLaunchKernelGGL((k_panel_rb<T, NT, RPT, BW>), dim3(n_active), dim3(NT), 0, st, \
                     fronts, ids, k, nb, ws0, ws1, panel, panel_off, D, ipiv, perm, \
                     perm_off, status)
  // up to 768 rows (complex128: 256) the panel in registers; above, the column
  // block in registers, 4 rows per thread at most (complex128 at 512 threads:
  // at 1024 a lane's register share of 128 would spill), else the global copy
  // alone
  constexpr bool C64 = sizeof(T) == 4;
#define HELM_PANEL_REGS(RW, CH)                                                        \
  hipLaunchKernelGGL((k_panel_regs<T, RW, CH>), dim3(n_active), dim3(64 * RW * CH), 0, \
                     st, fronts, ids, k, nb, ws0, ws1, D, ipiv, perm, perm_off,        \
                     panel_off, status)
  if constexpr (C64) {
    // (few small fronts: four waves share a panel's columns, 25^3 2.7 -> 2.4 ms;
    // thousands: a wave each, without a barrier, 100^3 51 -> 47 ms)
    if (max_rows <= 64 && n_active < 256) HELM_PANEL_REGS(1, 4);
    else if (max_rows <= 64) HELM_PANEL_REGS(1, 1);
    else if (max_rows <= 128) HELM_PANEL_REGS(2, 1);
    else if (max_rows <= 192) HELM_PANEL_REGS(3, 1);
    else if (max_rows <= 256) HELM_PANEL_REGS(4, 1);
    else if (max_rows <= 384) HELM_PANEL_REGS(6, 1);
    else if (max_rows <= 512) HELM_PANEL_REGS(8, 1);
    else if (max_rows <= 768) HELM_PANEL_REGS(12, 1);
    else if (max_rows <= 1024) HELM_PANEL_RB(256, 4, PB);
    else if (max_rows <= 2048) HELM_PANEL_RB(1024, 2, PB);
    else if (max_rows <= 4096) HELM_PANEL_RB(1024, 4, PB);
    else if (max_rows <= 6144) HELM_PANEL_RB(1024, 6, PB / 2);
    else HELM_PANEL(1024);
  } else {
    if (max_rows <= 64) HELM_PANEL_REGS(1, 4);
    else if (max_rows <= 128) HELM_PANEL_REGS(2, 4);
    else if (max_rows <= 192) HELM_PANEL_REGS(3, 4);
    else if (max_rows <= 256) HELM_PANEL_REGS(4, 4);
    else if (max_rows <= 1024) HELM_PANEL_RB(256, 4, PB);
    else if (max_rows <= 2048) HELM_PANEL_RB(512, 4, PB);
    else HELM_PANEL(1024);
  }
#undef HELM_PANEL_REGS
#undef HELM_PANEL_RB
#undef HELM_PANEL
}
template <typename T>
void launch_swap_JO(const FrontDev* fronts, const int* ids, int n_active,
                    const int2* tmap, int total, int k, int nb, void* ws0,
                    void* ws1, const void* D, const int* ipiv,
                    const long long* panel_off, const long long* perm_off,
                    hipStream_t st) {
  if (total <= 0) return;
  hipLaunchKernelGGL(k_swap_JO<T>, dim3(total), dim3(256), 0, st, fronts, ids,
                     n_active, tmap, k, nb, ws0, ws1, D, ipiv, panel_off, perm_off);
}
template <typename T>
void launch_sweep_gemm(const FrontDev* fronts, const int* ids, int n_active,
                       const int2* tmap, int total, int k, int nb, void* ws0,
                       void* ws1, hipStream_t st) {
  if (total <= 0) return;
  hipLaunchKernelGGL(k_sweep_gemm<T>, dim3(total), dim3(256), 0, st, fronts, ids, n_active,
                     tmap, k, nb, ws0, ws1);
}
template <typename T>
void launch_update_OJ(const FrontDev* fronts, const int* ids, int n_active,
                      const int2* tmap, int total, int k, int nb, void* ws0,
                      void* ws1, const void* D, const long long* panel_off,
                      hipStream_t st) {
  if (total <= 0) return;
  hipLaunchKernelGGL(k_update_OJ<T>, dim3(total), dim3(256), 0, st, fronts, ids,
                     n_active, tmap, k, nb, ws0, ws1, D, panel_off);
}
template <typename T>
void launch_store_factor(const FrontDev* fronts, const int* ids, int n_ids,
                         const int2* tmap, int total, const LayerDev* layers,
                         void* ws0, void* ws1, const int* perm,
                         const long long* perm_off, hipStream_t st) {
  if (total <= 0) return;
  hipLaunchKernelGGL(k_store_factor<T>, dim3(total), dim3(256), 0, st, fronts, ids,
                     n_ids, tmap, layers, ws0, ws1, perm, perm_off);
}

#define HELM_INST_FACTOR(T)                                                        \
  template void launch_extend_add<T>(const FrontDev*, const int*, int, const int2*, \
                                     int, const LayerDev*, void*, void*,           \
                                     hipStream_t);                                 \
  template void launch_orig_entries<T>(const FrontDev*, const int*, int,          \
                                       const int2*, int, const LayerDev*, void*,    \
                                       void*, const GridDev&, int, FactorStatus*,   \
                                       hipStream_t);                                \
  template void launch_panel<T>(const FrontDev*, const int*, int, int, int, int, void*, \
                                void*, void*, const long long*, void*, int*, int*, \
                                const long long*, FactorStatus*, hipStream_t);     \
  template void launch_swap_JO<T>(const FrontDev*, const int*, int, const int2*,    \
                                  int, int, int, void*, void*, const void*,        \
                                  const int*, const long long*, const long long*,  \
                                  hipStream_t);                                    \
  template void launch_sweep_gemm<T>(const FrontDev*, const int*, int, const int2*, \
                                     int, int, int, void*, void*, hipStream_t);       \
  template void launch_update_OJ<T>(const FrontDev*, const int*, int, const int2*,  \
                                    int, int, int, void*, void*, const void*,      \
                                    const long long*, hipStream_t);                \
  template void launch_store_factor<T>(const FrontDev*, const int*, int,          \
                                       const int2*, int, const LayerDev*, void*,    \
                                       void*, const int*, const long long*,        \
                                       hipStream_t);
HELM_INST_FACTOR(float)
HELM_INST_FACTOR(double)

}  // namespace kern
}  // namespace helm
