// Allocation-free variant of the local solve entry point (helm_layer_solve_dev):
// the same substitution kernels, with every buffer they need beyond the
// caller's input and output taken from one file-scope device array instead of
// the handle's hipMalloc'ed workspace.
//
// The array holds, from its start, each at a 256-byte boundary:
//   - the layer table the kernels index (one LayerDev per layer; only the
//     solved layer's entry is written),
//   - X (the solve vector, n_loc x k), Z (the forward results, n_loc x k),
//   - the two depth-parity update buffers (ub_rows[0] x k, ub_rows[1] x k),
//   - the split-K partial products (scratch_rows x k), or these in the caller's
//     output,
// in the precision of the factors, k being the columns of one pass.  Every byte
// that the kernels read is written earlier in the same call (X by the copy-in,
// Z and the update buffers by the forward pass, the partials by the GEMM
// chunks), so nothing has to start at zero and the previous call's contents
// never matter.
#include <algorithm>
#include <mutex>

#include "api_common.h"
#include "kernels.h"

namespace helm {

namespace {

// One copy per GPU, held until the process ends.  In host code `scratch`
// names a host-side stand-in: its device address comes from
// hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[HELM_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_mu;
void* g_scratch[kMaxDevices] = {};

__global__ void k_put_layer(LayerDev* dst, LayerDev v) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *dst = v;
}

size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

// Device address of the current device's copy of the array, looked up on the
// first call for that device (the factorization calls it with the handle's
// device current, so the solve entry point finds it cached).
void* noalloc_scratch(int device) {
  std::lock_guard<std::mutex> lock(g_mu);
  HELM_REQUIRE(device >= 0 && device < kMaxDevices, HELM_EINVAL,
               "device ordinal out of range for the static scratch table");
  if (!g_scratch[device]) {
    int cur = -1;
    HELM_HIP(hipGetDevice(&cur));
    HELM_REQUIRE(cur == device, HELM_EINVAL, "static scratch looked up on another device");
    void* p = nullptr;
    HELM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    HELM_REQUIRE(p != nullptr, HELM_EHIP, "no device address for the static scratch");
    g_scratch[device] = p;
  }
  return g_scratch[device];
}

namespace {

template <typename T>
void solve_noalloc(Handle& H, int l, int k, const double2* r, double2* w, unsigned char* base) {
  const LayerPlan& P = H.G.layers[l];
  const LayerSet& S = *H.single_sets[l];
  const size_t e = H.elem, cap = HELM_NOALLOC_SCRATCH_BYTES;
  const size_t table = round256((size_t)H.G.L * sizeof(LayerDev));
  const size_t u0 = std::max<long long>(P.ub_rows[0], 1), u1 = std::max<long long>(P.ub_rows[1], 1);
  auto bytes = [&](size_t rows, size_t cols) { return round256(rows * cols * e); };
  auto need = [&](size_t cols, long long split_rows) {
    return table + 2 * bytes((size_t)P.n_loc, cols) + bytes(u0, cols) + bytes(u1, cols) +
           bytes((size_t)std::max<long long>(split_rows, 1), cols);
  };
  const size_t asked = need((size_t)k, S.limit_rows);
  HELM_REQUIRE(asked <= cap, HELM_ENOMEM,
               "local solve needs " + std::to_string(asked) +
                   " bytes of workspace, more than the static scratch of " + std::to_string(cap) +
                   " bytes (use fewer columns or helm_layer_solve_dev)");
  // The launches' own partials can take more than the limit counts.  Then they
  // go into the caller's result, which is written last (complex128, 68 x 68 x
  // 30, 16 columns: 897 us, in two passes of 8 columns 1570); where they
  // cannot (it is also the right-hand side), the columns go in passes of equal
  // width.  Up to 4 columns (the vector kernels) have no partials, so a pass
  // always fits.
  const long long n = (long long)P.n_loc * k;
  const bool apart = r + n <= w || w + n <= r;
  int cols = k;
  while (cols > 4 && need((size_t)cols, S.scratch_rows) > cap) --cols;
  const bool in_w = cols < k && apart && (size_t)S.scratch_rows * e <= P.n_loc * sizeof(double2);
  if (in_w) cols = k;
  const int passes = (k + cols - 1) / cols;
  cols = (k + passes - 1) / passes;
  LayerDev* tab = reinterpret_cast<LayerDev*>(base);
  LayerDev v = H.layers_h[l];
  unsigned char* p = base + table;
  v.X = p;
  p += bytes((size_t)P.n_loc, cols);
  v.Wt = p;
  p += bytes((size_t)P.n_loc, cols);
  v.Ub[0] = p;
  p += bytes(u0, cols);
  v.Ub[1] = p;
  p += bytes(u1, cols);
  void* splitk = in_w ? static_cast<void*>(w) : p;
  hipLaunchKernelGGL(k_put_layer, dim3(1), dim3(64), 0, H.st, tab + l, v);
  H.local_solve<T>(v, r, w, k, cols,
                   [&](int n) { H.run_layers_t<T>(S, n, tab, splitk, nullptr, false); });
}

}  // namespace

}  // namespace helm

using namespace helm;

extern "C" int helm_layer_solve_noalloc_dev(helm_handle* h, int l, int k, const double* r_dev,
                                            double* w_dev) {
  return guard([&] {
    HELM_REQUIRE(h && r_dev && w_dev && k >= 1, HELM_EINVAL, "bad argument");
    Handle& H = h->impl;
    HELM_REQUIRE(l >= 0 && l < H.G.L, HELM_EINVAL, "layer index out of range");
    HELM_REQUIRE((int)H.single_sets.size() == H.G.L && H.single_sets[l], HELM_EINVAL,
                 "handle has no factorized layer plans");
    HELM_HIP(hipSetDevice(H.device));
    unsigned char* base = static_cast<unsigned char*>(noalloc_scratch(H.device));
    const double2* r = reinterpret_cast<const double2*>(r_dev);
    double2* w = reinterpret_cast<double2*>(w_dev);
    if (H.prec == HELM_FP64) solve_noalloc<double>(H, l, k, r, w, base);
    else solve_noalloc<float>(H, l, k, r, w, base);
    return HELM_OK;
  });
}
