// Volume, interface-trace and Krylov kernels of the online stage.
//
//  * source partition f^l = f chi_l (Algorithm 2) and the volume
//    reconstruction (the last step of Algorithm 2) between the global grid (RHS-major, FP64)
//    and a layer's solve vector (ND order, columns fastest, working precision);
//  * interface sources: the plane deltas of Section "Formulation" scaled to
//    this discretisation (coefficient B = 1/(h^2 beta_x beta_y), the matrix
//    coupling across an interior interface):
//      top of layer l:    -B a on plane s_l,  +B b on plane s_l - 1,
//      bottom of layer l: -B b on plane e_l,  +B a on plane e_l + 1,
//    and the trace read-outs of two planes (Algorithms 3-10);
//  * FP64 column-batched BLAS-1 for GMRES on the interface system;
//  * the FP64 residual f - H u of the global 7-point operator.
// Interface pair vectors use the layout [plane a|b][y][x][column], FP64.
#include "kernels.h"
#include "kernels_common.h"

namespace helm {
namespace kern {

namespace {

// Volume <-> layer copies of the bulk planes [s, e] for a few columns: one
// element per thread, consecutive threads on consecutive nodes.
template <typename T>
__global__ void k_scatter_flat(LayerDev L, const double2* __restrict__ f, int nx, int ny,
                               long long N, int k) {
  using C = C_t<T>;
  const long long plane = (long long)nx * ny;
  const long long nb = plane * (L.e - L.s + 1);
  C* X = reinterpret_cast<C*>(L.X);
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nb * k;
       e += (long long)gridDim.x * blockDim.x) {
    const long long sp = e % nb;
    const int c = (int)(e / nb);
    X[(long long)L.nat2nd[sp + plane * (L.s - L.lo)] * k + c] =
        from_d2<C>(f[(long long)c * N + sp + plane * L.s]);
  }
}
template <typename T>
__global__ void k_gather_flat(LayerDev L, double2* __restrict__ u, int nx, int ny,
                              long long N, int k) {
  using C = C_t<T>;
  const long long plane = (long long)nx * ny;
  const long long nb = plane * (L.e - L.s + 1);
  const C* X = reinterpret_cast<const C*>(L.X);
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nb * k;
       e += (long long)gridDim.x * blockDim.x) {
    const long long sp = e % nb;
    const int c = (int)(e / nb);
    u[(long long)c * N + sp + plane * L.s] =
        to_d2(X[(long long)L.nat2nd[sp + plane * (L.s - L.lo)] * k + c]);
  }
}

// The same copies for many columns, as tiles of 64 nodes x
// 64 columns staged in LDS: f and u hold each column contiguously over the
// nodes, X holds each node's k values contiguously, so both sides are read
// or written along their contiguous direction.  Grid: (node tiles, column
// tiles); wave w of the block handles tile rows w, w + 4, ...
constexpr int VT = 64;
constexpr int RESID_COLS = 8;   // columns per block row of k_residual

template <typename T>
__global__ void __launch_bounds__(256)
k_scatter_source(LayerDev L, const double2* __restrict__ f, int nx, int ny, long long N, int k) {
  using C = C_t<T>;
  __shared__ C tile[VT][VT + 1];   // [node][column]
  const long long plane = (long long)nx * ny;
  const long long nb = plane * (L.e - L.s + 1);
  const long long n0 = (long long)blockIdx.x * VT;
  const int c0 = blockIdx.y * VT, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  C* X = reinterpret_cast<C*>(L.X);
  {
    const long long sp = n0 + lane;
#pragma unroll
    for (int j = 0; j < VT / 4; ++j) {
      const int c = w + 4 * j;
      const bool ok = sp < nb && c0 + c < k;
      tile[lane][c] = from_d2<C>(ld_or_zero(ok, f + (ok ? (long long)(c0 + c) * N + sp + plane * L.s : 0)));
    }
  }
  __syncthreads();
  long long dst[VT / 4];
#pragma unroll
  for (int j = 0; j < VT / 4; ++j) {
    const long long sp = n0 + w + 4 * j;
    dst[j] = sp < nb ? (long long)ld(L.nat2nd + sp + plane * (L.s - L.lo)) * k : -1;
  }
  if (c0 + lane < k)
#pragma unroll
    for (int j = 0; j < VT / 4; ++j)
      if (dst[j] >= 0) st(X + dst[j] + c0 + lane, tile[w + 4 * j][lane]);
}

template <typename T>
__global__ void __launch_bounds__(256)
k_gather_volume(LayerDev L, double2* __restrict__ u, int nx, int ny, long long N, int k) {
  using C = C_t<T>;
  __shared__ C tile[VT][VT + 1];   // [node][column]
  const long long plane = (long long)nx * ny;
  const long long nb = plane * (L.e - L.s + 1);
  const long long n0 = (long long)blockIdx.x * VT;
  const int c0 = blockIdx.y * VT, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const C* X = reinterpret_cast<const C*>(L.X);
  long long src[VT / 4];
#pragma unroll
  for (int j = 0; j < VT / 4; ++j) {
    const long long sp = n0 + w + 4 * j;
    src[j] = sp < nb ? (long long)ld(L.nat2nd + sp + plane * (L.s - L.lo)) * k : -1;
  }
#pragma unroll
  for (int j = 0; j < VT / 4; ++j) {
    const bool ok = src[j] >= 0 && c0 + lane < k;
    tile[w + 4 * j][lane] = ld_or_zero(ok, X + (ok ? src[j] + c0 + lane : 0));
  }
  __syncthreads();
  const long long sp = n0 + lane;
  if (sp < nb)
#pragma unroll
    for (int j = 0; j < VT / 4; ++j) {
      const int c = w + 4 * j;
      if (c0 + c < k) u[(long long)(c0 + c) * N + sp + plane * L.s] = to_d2(tile[lane][c]);
    }
}

// Whether complex64 substitutions take a column of largest magnitude a as it
// is.  A float of 2^-110 and more splits exactly into three bf16 numbers, and
// the substitutions move values by the size of H^-1 (2^-10 at 36^3 on the unit
// cube), so both ends keep well away from the format's.
constexpr double kScaleLow = 0x1p-60, kScaleHigh = 0x1p60;

__device__ __forceinline__ bool out_of_range(double2 v) {
  const double a = fmax(fabs(v.x), fabs(v.y));
  return (a > 0.0 && a < kScaleLow) || a > kScaleHigh;
}
__global__ void __launch_bounds__(256)
k_range_check(const double2* __restrict__ x, long long n, int* odd) {
  bool out = false;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += gridDim.x * 256LL)
    out = out || out_of_range(x[e]);
  if (out) *odd = 1;
}

// whole extended layer, natural order <-> ND order (inspection entry point);
// SCALED: columns times, and divided by, scale[column]
template <typename T, bool SCALED>
__global__ void k_local_to_X(LayerDev L, const double2* __restrict__ r, int k,
                             const double* __restrict__ scale, int* odd) {
  using C = C_t<T>;
  C* X = reinterpret_cast<C*>(L.X);
  const long long total = (long long)L.n_loc * k;
  bool out = false;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long sp = e % L.n_loc;
    const int c = (int)(e / L.n_loc);
    double2 v = r[e];
    if (SCALED) v = make_double2(v.x * scale[c], v.y * scale[c]);
    else if (sizeof(T) == 4) out = out || out_of_range(v);
    X[(long long)L.nat2nd[sp] * k + c] = from_d2<C>(v);
  }
  if (!SCALED && sizeof(T) == 4 && out) *odd = 1;
}
template <typename T, bool SCALED>
__global__ void k_X_to_local(LayerDev L, double2* __restrict__ w, int k,
                             const double* __restrict__ scale) {
  using C = C_t<T>;
  const C* X = reinterpret_cast<const C*>(L.X);
  const long long total = (long long)L.n_loc * k;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long sp = e % L.n_loc;
    const int c = (int)(e / L.n_loc);
    double2 v = to_d2(X[(long long)L.nat2nd[sp] * k + c]);
    if (SCALED) v = make_double2(v.x / scale[c], v.y / scale[c]);
    w[e] = v;
  }
}
// largest |Re|, |Im| of each column, a part per block: part[c gridDim.x + block]
__global__ void __launch_bounds__(256)
k_column_max(const double2* __restrict__ x, long long N, double* __restrict__ part) {
  const double2* col = x + (long long)blockIdx.y * N;
  double m = 0.0;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < N; i += gridDim.x * 256LL)
    m = fmax(m, fmax(fabs(col[i].x), fabs(col[i].y)));
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  __shared__ double wm[4];
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    part[(long long)blockIdx.y * gridDim.x + blockIdx.x] =
        fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
}
__global__ void __launch_bounds__(64)
k_column_scale(const double* __restrict__ part, int parts, double* __restrict__ scale,
               int* scaled) {
  double m = (int)threadIdx.x < parts ? part[(long long)blockIdx.x * parts + threadIdx.x] : 0.0;
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  if (threadIdx.x) return;
  const bool keep = !(m > 0.0) || isinf(m) || (m >= kScaleLow && m <= kScaleHigh);
  // (an inverse power of two stays a normal number)
  scale[blockIdx.x] = keep ? 1.0 : ldexp(1.0, -max(ilogb(m), -1000));
  if (!keep) *scaled = 1;
}

// Interface source of a pair (a, b) = c0 in0 + c1 in1 + c2 in2 (null entries
// skipped) at element e of the pair's planes, on plane a (which = 0) or b:
//   top:    a -> s (coefficient -B), b -> s - 1 (+B)
//   bottom: b -> e (-B),             a -> e + 1 (+B)
template <typename T>
__device__ __forceinline__ C_t<T> jump_value(const JumpTerms& t, double2 B, int bottom, int which,
                                             long long e, long long total) {
  double2 a = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (!t.in[i]) continue;
    const double2 v = t.in[i][e + which * total];
    a.x += t.c[i] * v.x;
    a.y += t.c[i] * v.y;
  }
  const double s = (bottom != which) ? 1.0 : -1.0;
  return from_d2<C_t<T>>(make_double2(s * (B.x * a.x - B.y * a.y), s * (B.x * a.y + B.y * a.x)));
}

// add an interface source to X
template <typename T>
__global__ void k_jump(LayerDev L, JumpTerms t, const double2* __restrict__ B, int bottom,
                       int nx, int ny, int k) {
  using C = C_t<T>;
  C* X = reinterpret_cast<C*>(L.X);
  const long long plane = (long long)nx * ny;
  const long long total = plane * k;
  const int za = bottom ? L.e + 1 : L.s;
  const int zb = bottom ? L.e : L.s - 1;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long sp = e / k;
    const int c = (int)(e % k);
    const double2 cf = B[sp];
    const long long ia = L.nat2nd[sp + plane * (za - L.lo)];
    const long long ib = L.nat2nd[sp + plane * (zb - L.lo)];
    C& xa = X[ia * k + c];
    xa = cadd(xa, jump_value<T>(t, cf, bottom, 0, e, total));
    C& xb = X[ib * k + c];
    xb = cadd(xb, jump_value<T>(t, cf, bottom, 1, e, total));
  }
}

// X = the interface sources of the layer's two sides, zero elsewhere: a sweep
// solve's whole right-hand side in one pass in ND order (a fill and up to
// three additions to X before; at 96^3 and 64 columns 13 + 11 to 22 us).
template <typename T>
__global__ void __launch_bounds__(256)
k_sources(LayerDev L, JumpTerms top, JumpTerms bot, const double2* __restrict__ B, int nx, int ny,
          int k) {
  using C = C_t<T>;
  C* X = reinterpret_cast<C*>(L.X);
  const int plane = nx * ny;
  const long long total = (long long)plane * k, n = (long long)L.n_loc * k;
  const bool has_top = top.in[0], has_bot = bot.in[0];
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
    const long long node = i / k;
    const int c = (int)(i % k);
    const int nat = ld(L.nd2nat + node);
    const int z = nat / plane + L.lo, sp = nat % plane;
    C v = czero<C>();
    const bool t = has_top && (z == L.s || z == L.s - 1);
    const bool b = has_bot && (z == L.e || z == L.e + 1);
    if (t || b) {
      const double2 cf = B[sp];
      const long long e = (long long)sp * k + c;
      if (t) v = cadd(v, jump_value<T>(top, cf, 0, z == L.s ? 0 : 1, e, total));
      if (b) v = cadd(v, jump_value<T>(bot, cf, 1, z == L.e ? 1 : 0, e, total));
    }
    st(X + i, v);
  }
}

// read-outs of a layer's traces, one per block row
template <typename T>
__global__ void __launch_bounds__(256) k_readout(LayerDev L, ReadOuts ro, int nx, int ny, int k) {
  using C = C_t<T>;
  const C* X = reinterpret_cast<const C*>(L.X);
  const ReadOut& r = ro.r[blockIdx.y];
  const long long plane = (long long)nx * ny;
  const long long total = plane * k;
  // R_top = (w(s - 1), w(s)),  R_bot = (w(e), w(e + 1))
  const int z0 = r.bottom ? L.e : L.s - 1;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < 2 * total;
       e += (long long)gridDim.x * 256) {
    const int p = e >= total;
    if (!((r.terms.planes >> p) & 1)) continue;
    const long long q = p ? e - total : e;
    const long long sp = q / k;
    const int c = (int)(q % k);
    double2 v = make_double2(0.0, 0.0);
    if (r.sx != 0.0) {
      const long long idx = L.nat2nd[sp + plane * (z0 + p - L.lo)];
      double2 x = to_d2(X[idx * k + c]);
      v.x = r.sx * x.x;
      v.y = r.sx * x.y;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (!r.terms.in[i]) continue;
      const double cf = p ? r.terms.cb[i] : r.terms.ca[i];
      if (cf == 0.0) continue;
      const double2 y = r.terms.in[i][e];
      v.x += cf * y.x;
      v.y += cf * y.y;
    }
    r.out[e] = v;
  }
}

// ----------------------------------------------------------------------------
// FP64 column-batched vector kernels; vectors are V x k with k fastest.
// ----------------------------------------------------------------------------
constexpr int DOT_BLOCKS = 256;

// partial[c][blk] = sum_v conj(x[v, c]) y[v, c] over this block's rows: COLS
// columns (the power of two that holds a narrow batch, at most 32) by
// 256 / COLS rows at a time.  Bound by memory once every lane has a column:
// with 32 columns at every width one column used one lane in 32.  Kernel times:
// 100^3, 1 column 37.6 -> 4.2 us; 97^3, 21 columns 42.6 -> 26.8 (two loads in
// flight); 25^3, 1 column, no gain (3 us, a launch's own time).
template <int COLS>
__global__ void __launch_bounds__(256)
k_dot_partial(const double2* __restrict__ x, const double2* __restrict__ y,
              long long V, int k, double2* __restrict__ partial) {
  constexpr int ROWS = 256 / COLS;
  const int tx = threadIdx.x % COLS, ty = threadIdx.x / COLS;
  const int c = blockIdx.y * COLS + tx;
  double re = 0, im = 0;
  if (c < k) {
#pragma unroll 2
    for (long long v = blockIdx.x * ROWS + ty; v < V; v += (long long)gridDim.x * ROWS) {
      const double2 a = x[v * k + c], b = y[v * k + c];
      re += a.x * b.x + a.y * b.y;
      im += a.x * b.y - a.y * b.x;
    }
  }
  // the rows of a wave by a butterfly, then the four waves in order
  for (int o = COLS; o < 64; o <<= 1) {
    re += __shfl_xor(re, o);
    im += __shfl_xor(im, o);
  }
  __shared__ double sre[4][COLS], sim[4][COLS];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) < COLS) {
    sre[wave][tx] = re;
    sim[wave][tx] = im;
  }
  __syncthreads();
  if (threadIdx.x < COLS && c < k) {
    for (int q = 1; q < 4; ++q) {
      re += sre[q][tx];
      im += sim[q][tx];
    }
    partial[(long long)c * gridDim.x + blockIdx.x] = make_double2(re, im);
  }
}

// out[c] = sum over blocks (fixed order, reproducible): a wave per column,
// the blocks' sums dealt to its lanes, then a butterfly (a thread per column
// walked them one load after another: 25 us against 3).
__global__ void __launch_bounds__(64)
k_dot_final(const double2* __restrict__ partial, int nblk, double2* __restrict__ out) {
  const int c = blockIdx.x, lane = threadIdx.x;
  double re = 0, im = 0;
  for (int b = lane; b < nblk; b += 64) {
    const double2 v = partial[(long long)c * nblk + b];
    re += v.x;
    im += v.y;
  }
  for (int o = 32; o > 0; o >>= 1) {
    re += __shfl_xor(re, o);
    im += __shfl_xor(im, o);
  }
  if (lane == 0) out[c] = make_double2(re, im);
}

// y[v, c] += sign * alpha[c] * x[v, c]     (alpha per column, complex)
__global__ void k_axpy_cols(double2* __restrict__ y, const double2* __restrict__ x,
                            const double2* __restrict__ alpha, double sign,
                            long long V, int k) {
  const long long total = V * k;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int c = (int)(e % k);
    const double2 a = alpha[c], b = x[e];
    double2 o = y[e];
    o.x += sign * (a.x * b.x - a.y * b.y);
    o.y += sign * (a.x * b.y + a.y * b.x);
    y[e] = o;
  }
}

// y[v, c] = x[v, c] * s[c]  (s real, per column); y may be x (each element
// is read and written by one thread), so y and x are not restrict
__global__ void k_scale_cols(double2* y, const double2* x, const double* __restrict__ s,
                             long long V, int k) {
  const long long total = V * k;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const double a = s[e % k];
    const double2 b = x[e];
    y[e] = make_double2(a * b.x, a * b.y);
  }
}

// volumes: column c's N elements contiguous, one grid row per column
__global__ void k_scale_volumes(double2* y, const double2* x, const double* __restrict__ s,
                                long long N) {
  const double a = s[blockIdx.y];
  const long long base = blockIdx.y * N;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < N;
       e += (long long)gridDim.x * blockDim.x) {
    const double2 b = x[base + e];
    y[base + e] = make_double2(a * b.x, a * b.y);
  }
}

// the columns map.col[0..m) of an interleaved batch of k into a batch of w
__global__ void k_gather_cols(double2* __restrict__ out, const double2* __restrict__ in,
                              long long V, int k, int w, int m, ColMap map) {
  const long long total = V * w;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const long long e = i / w;
    const int j = (int)(i % w);
    out[i] = j < m ? in[e * k + map.col[j]] : make_double2(0.0, 0.0);
  }
}

// back: column c of the batch of k from slot slot.col[c] of the batch of w
__global__ void k_scatter_cols(double2* __restrict__ out, const double2* __restrict__ in,
                               long long V, int k, int w, ColMap slot) {
  const long long total = V * k;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const long long e = i / k;
    const int s = slot.col[i % k];
    out[i] = s >= 0 ? in[e * w + s] : make_double2(0.0, 0.0);
  }
}

// y = x + z (elementwise); y may be x or z
__global__ void k_add(double2* y, const double2* x, const double2* z, long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    y[e] = make_double2(x[e].x + z[e].x, x[e].y + z[e].y);
  }
}

// y[v, c] = x[v, c] + alpha[c] y[v, c]   (alpha per column, complex)
__global__ void k_xpay_cols(double2* __restrict__ y, const double2* __restrict__ x,
                            const double2* __restrict__ alpha, long long V, int k) {
  const long long total = V * k;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const double2 a = alpha[e % k], b = y[e], c = x[e];
    y[e] = make_double2(c.x + a.x * b.x - a.y * b.y, c.y + a.x * b.y + a.y * b.x);
  }
}

// y = z - y in place: each element is read and written by one thread, so y
// is the only pointer that aliases nothing else
__global__ void k_rsub(double2* y, const double2* __restrict__ z, long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    const double2 a = y[e], b = z[e];
    y[e] = make_double2(b.x - a.x, b.y - a.y);
  }
}

// FP64 residual r = f - H u on the global grid (volumes RHS-major); f may be
// null (then r = H u).  Same operator as the local assembly.
__global__ void __launch_bounds__(256)
k_residual(GridDev g, const double2* __restrict__ f, const double2* __restrict__ u,
           double2* __restrict__ r, int k) {
  // one node per thread and RESID_COLS columns per block row: the node's
  // stencil coefficients are formed once for all of its columns
  const long long N = (long long)g.nx * g.ny * g.nz;
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= N) return;
  const double ih2 = 1.0 / (g.h * g.h);
  const int x = (int)(idx % g.nx);
  const int y = (int)((idx / g.nx) % g.ny);
  const int z = (int)(idx / ((long long)g.nx * g.ny));
  const double2 bx = g.bx[x], by = g.by[y], bz = g.bz[z];
  auto mul = [](double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
  };
  const double2 bxy = mul(bx, by), bxz = mul(bx, bz), byz = mul(by, bz);
  double2 cp[6];
  cp[0] = cdiv(g.bxh[x], byz);
  cp[1] = cdiv(g.bxh[x + 1], byz);
  cp[2] = cdiv(g.byh[y], bxz);
  cp[3] = cdiv(g.byh[y + 1], bxz);
  cp[4] = cdiv(g.bzh[z], bxy);
  cp[5] = cdiv(g.bzh[z + 1], bxy);
  const double2 dg = cdiv(make_double2(g.omega * g.omega * g.m[idx], 0.0), mul(bxy, bz));
  const long long st[6] = {-1, 1, -(long long)g.nx, (long long)g.nx,
                           -(long long)g.nx * g.ny, (long long)g.nx * g.ny};
  const bool ok[6] = {x > 0, x < g.nx - 1, y > 0, y < g.ny - 1, z > 0, z < g.nz - 1};
  const int cend = min(k, (int)(blockIdx.y + 1) * RESID_COLS);
  for (int c = blockIdx.y * RESID_COLS; c < cend; ++c) {
    const double2* uc = u + (long long)c * N;
    const double2 u0 = uc[idx];
    double2 acc = mul(dg, u0);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      double2 nb = ok[q] ? uc[idx + st[q]] : make_double2(0.0, 0.0);
      double2 d = make_double2((nb.x - u0.x) * ih2, (nb.y - u0.y) * ih2);
      double2 t = mul(cp[q], d);
      acc.x += t.x;
      acc.y += t.y;
    }
    const long long e = (long long)c * N + idx;
    double2 out;
    if (f) out = make_double2(f[e].x - acc.x, f[e].y - acc.y);
    else out = acc;
    r[e] = out;
  }
}


// point sources: f[c * N + node[c]] = amp[c] / h^3 (f zeroed before)
__global__ void k_point_sources(double2* __restrict__ f, const long long* __restrict__ node,
                                const double2* __restrict__ amp, double inv_h3,
                                long long N, int k) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= k) return;
  f[(long long)c * N + node[c]] = make_double2(amp[c].x * inv_h3, amp[c].y * inv_h3);
}

// u[c] += d[c]  over volumes (refinement update)
__global__ void k_accumulate(double2* __restrict__ u, const double2* __restrict__ d,
                             long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    u[e] = make_double2(u[e].x + d[e].x, u[e].y + d[e].y);
  }
}

// per-column squared norms of RHS-major volumes: out[c] = sum |x|^2
__global__ void __launch_bounds__(256)
k_volume_norm2(const double2* __restrict__ x, long long N, int k,
               double* __restrict__ partial) {
  const int c = blockIdx.y;
  double s = 0;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < N; e += (long long)gridDim.x * 256) {
    const double2 v = x[(long long)c * N + e];
    s += v.x * v.x + v.y * v.y;
  }
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[(long long)c * gridDim.x + blockIdx.x] = red[0];
}
__global__ void __launch_bounds__(64)
k_norm_final(const double* __restrict__ partial, int nblk, double* __restrict__ out) {
  const int c = blockIdx.x, lane = threadIdx.x;
  double s = 0;
  for (int b = lane; b < nblk; b += 64) s += partial[(long long)c * nblk + b];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) out[c] = s;
}

inline int grid_for(long long n, int block = 256) {
  long long g = (n + block - 1) / block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

// ---------------------------------------------------------------------------
template <typename T>
void launch_scatter_source(const LayerDev& L, const double2* f, int nx, int ny,
                           long long N, int k, hipStream_t st) {
  const long long nb = (long long)nx * ny * (L.e - L.s + 1);
  if (nb <= 0 || k <= 0) return;
  if (k <= 8) {   // a 64-column tile would leave most lanes idle
    hipLaunchKernelGGL(k_scatter_flat<T>, dim3(grid_for(nb * k)), dim3(256), 0, st, L, f, nx, ny, N, k);
    return;
  }
  const dim3 grid((unsigned)((nb + VT - 1) / VT), (unsigned)((k + VT - 1) / VT));
  hipLaunchKernelGGL(k_scatter_source<T>, grid, dim3(256), 0, st, L, f, nx, ny, N, k);
}
template <typename T>
void launch_gather_volume(const LayerDev& L, double2* u, int nx, int ny,
                          long long N, int k, hipStream_t st) {
  const long long nb = (long long)nx * ny * (L.e - L.s + 1);
  if (nb <= 0 || k <= 0) return;
  if (k <= 8) {   // a 64-column tile would leave most lanes idle
    hipLaunchKernelGGL(k_gather_flat<T>, dim3(grid_for(nb * k)), dim3(256), 0, st, L, u, nx, ny, N, k);
    return;
  }
  const dim3 grid((unsigned)((nb + VT - 1) / VT), (unsigned)((k + VT - 1) / VT));
  hipLaunchKernelGGL(k_gather_volume<T>, grid, dim3(256), 0, st, L, u, nx, ny, N, k);
}
template <typename T>
void launch_local_to_X(const LayerDev& L, const double2* r, int k, const double* scale,
                       int* odd, hipStream_t st) {
  const dim3 grid(grid_for((long long)L.n_loc * k));
  if (scale)
    hipLaunchKernelGGL((k_local_to_X<T, true>), grid, dim3(256), 0, st, L, r, k, scale, odd);
  else
    hipLaunchKernelGGL((k_local_to_X<T, false>), grid, dim3(256), 0, st, L, r, k, scale, odd);
}
template <typename T>
void launch_X_to_local(const LayerDev& L, double2* w, int k, const double* scale,
                       hipStream_t st) {
  const dim3 grid(grid_for((long long)L.n_loc * k));
  if (scale)
    hipLaunchKernelGGL((k_X_to_local<T, true>), grid, dim3(256), 0, st, L, w, k, scale);
  else
    hipLaunchKernelGGL((k_X_to_local<T, false>), grid, dim3(256), 0, st, L, w, k, scale);
}
template <typename T>
void launch_jump(const LayerDev& L, const JumpTerms& t, const double2* B, int bottom, int nx,
                 int ny, int k, hipStream_t st) {
  long long n = (long long)nx * ny * k;
  hipLaunchKernelGGL(k_jump<T>, dim3(grid_for(n)), dim3(256), 0, st, L, t, B, bottom, nx,
                     ny, k);
}
template <typename T>
void launch_sources(const LayerDev& L, const JumpTerms& top, const JumpTerms& bot,
                    const double2* B, int nx, int ny, int k, hipStream_t st) {
  hipLaunchKernelGGL(k_sources<T>, dim3(grid_for((long long)L.n_loc * k)), dim3(256), 0, st, L,
                     top, bot, B, nx, ny, k);
}
template <typename T>
void launch_readout(const LayerDev& L, const ReadOuts& ro, int nx, int ny, int k,
                    hipStream_t st) {
  const long long n = 2LL * nx * ny * k;
  hipLaunchKernelGGL(k_readout<T>, dim3(grid_for(n), ro.n), dim3(256), 0, st, L, ro, nx, ny, k);
}

void launch_dot(const double2* x, const double2* y, long long V, int k,
                double2* partial, double2* out, hipStream_t st) {
#define HELM_DOT(COLS)                                                                      \
  hipLaunchKernelGGL(k_dot_partial<COLS>, dim3(DOT_BLOCKS, (k + COLS - 1) / COLS), dim3(256), 0, \
                     st, x, y, V, k, partial)
  if (k == 1) HELM_DOT(1);
  else if (k == 2) HELM_DOT(2);
  else if (k <= 4) HELM_DOT(4);
  else if (k <= 8) HELM_DOT(8);
  else if (k <= 16) HELM_DOT(16);
  else HELM_DOT(32);
#undef HELM_DOT
  hipLaunchKernelGGL(k_dot_final, dim3(k), dim3(64), 0, st, partial, DOT_BLOCKS, out);
}
void launch_axpy_cols(double2* y, const double2* x, const double2* alpha,
                      double sign, long long V, int k, hipStream_t st) {
  hipLaunchKernelGGL(k_axpy_cols, dim3(grid_for(V * k)), dim3(256), 0, st, y, x, alpha,
                     sign, V, k);
}
void launch_gather_cols(double2* out, const double2* in, long long V, int k, int w, int m,
                        const ColMap& map, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_cols, dim3(grid_for(V * w)), dim3(256), 0, st, out, in, V, k, w,
                     m, map);
}
void launch_scatter_cols(double2* out, const double2* in, long long V, int k, int w,
                         const ColMap& slot, hipStream_t st) {
  hipLaunchKernelGGL(k_scatter_cols, dim3(grid_for(V * k)), dim3(256), 0, st, out, in, V, k, w,
                     slot);
}
void launch_scale_cols(double2* y, const double2* x, const double* s, long long V,
                       int k, hipStream_t st) {
  hipLaunchKernelGGL(k_scale_cols, dim3(grid_for(V * k)), dim3(256), 0, st, y, x, s, V,
                     k);
}
void launch_scale_volumes(double2* y, const double2* x, const double* s, long long N, int k,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_scale_volumes, dim3(grid_for(N), k), dim3(256), 0, st, y, x, s, N);
}
void launch_range_check(const double2* x, long long n, int* odd, hipStream_t st) {
  hipLaunchKernelGGL(k_range_check, dim3(grid_for(n)), dim3(256), 0, st, x, n, odd);
}
void launch_column_scale(const double2* x, long long N, int k, double* scale, int* scaled,
                         hipStream_t st) {
  const int parts = (int)std::min<long long>(64, 1 + N / 1024);
  double* part = scale + k;
  hipLaunchKernelGGL(k_column_max, dim3(parts, k), dim3(256), 0, st, x, N, part);
  hipLaunchKernelGGL(k_column_scale, dim3(k), dim3(64), 0, st, part, parts, scale, scaled);
}
void launch_add(double2* y, const double2* x, const double2* z, long long n,
                hipStream_t st) {
  hipLaunchKernelGGL(k_add, dim3(grid_for(n)), dim3(256), 0, st, y, x, z, n);
}
void launch_xpay_cols(double2* y, const double2* x, const double2* alpha, long long V, int k,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_xpay_cols, dim3(grid_for(V * k)), dim3(256), 0, st, y, x, alpha, V, k);
}
void launch_rsub(double2* y, const double2* z, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_rsub, dim3(grid_for(n)), dim3(256), 0, st, y, z, n);
}
void launch_residual(const GridDev& g, const double2* f, const double2* u,
                     double2* r, int k, hipStream_t st) {
  const long long N = (long long)g.nx * g.ny * g.nz;
  if (N <= 0 || k <= 0) return;
  const dim3 grid((unsigned)((N + 255) / 256), (unsigned)((k + RESID_COLS - 1) / RESID_COLS));
  hipLaunchKernelGGL(k_residual, grid, dim3(256), 0, st, g, f, u, r, k);
}
void launch_point_sources(double2* f, const long long* node, const double2* amp,
                          double inv_h3, long long N, int k, hipStream_t st) {
  hipLaunchKernelGGL(k_point_sources, dim3((k + 63) / 64), dim3(64), 0, st, f, node,
                     amp, inv_h3, N, k);
}
void launch_accumulate(double2* u, const double2* d, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_accumulate, dim3(grid_for(n)), dim3(256), 0, st, u, d, n);
}
void launch_volume_norm2(const double2* x, long long N, int k, double* partial,
                         double* out, hipStream_t st) {
  const int nblk = 128;
  hipLaunchKernelGGL(k_volume_norm2, dim3(nblk, k), dim3(256), 0, st, x, N, k, partial);
  hipLaunchKernelGGL(k_norm_final, dim3(k), dim3(64), 0, st, partial, nblk, out);
}

#define HELM_INST_VOL(T)                                                             \
  template void launch_scatter_source<T>(const LayerDev&, const double2*, int, int,  \
                                         long long, int, hipStream_t);               \
  template void launch_gather_volume<T>(const LayerDev&, double2*, int, int,         \
                                        long long, int, hipStream_t);                \
  template void launch_local_to_X<T>(const LayerDev&, const double2*, int,           \
                                     const double*, int*, hipStream_t);              \
  template void launch_X_to_local<T>(const LayerDev&, double2*, int, const double*,  \
                                     hipStream_t);                                   \
  template void launch_jump<T>(const LayerDev&, const JumpTerms&, const double2*, int, \
                               int, int, int, hipStream_t);                          \
  template void launch_sources<T>(const LayerDev&, const JumpTerms&, const JumpTerms&, \
                                  const double2*, int, int, int, hipStream_t);       \
  template void launch_readout<T>(const LayerDev&, const ReadOuts&, int, int, int,   \
                                  hipStream_t);
HELM_INST_VOL(float)
HELM_INST_VOL(double)

}  // namespace kern
}  // namespace helm
