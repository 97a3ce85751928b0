// Non-orthogonal bases (Sec. II.A): the inverse factor Z of the overlap O
// (Z^T O Z = I) by the cubically convergent recursion the paper gives,
//   X_n = Z_n^T O Z_n,   Z_{n+1} = Z_n (1.875 I - 1.25 X_n + 0.375 X_n^2),
// started from Z_0 = c I with c^2 = 1 / (Gershgorin bound of O), and the
// congruences Z A Z that take H0, H1 to the orthogonalised representation and
// the density matrices back (D = Z D_perp Z^T).  With Z_0 a multiple of I every
// iterate is a polynomial in O, so Z is the symmetric (Lowdin) factor O^{-1/2}
// and Z^T = Z.  All products run on the direct MFMA kernels (FP64 or FP32):
// single products C = A B with symmetric operands, stored either on the upper
// tiles and mirrored (symmetric C) or on every tile (general C).
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <string>
#include <vector>

#include "layer_common.h"

namespace dmpt {

namespace {

// Z = c I on the N x N block, zero elsewhere (padded rows x ld storage).
template <typename M>
__global__ void __launch_bounds__(kBlk) k_scaled_identity(M* z, double c, int64_t n, int64_t total,
                                                         int64_t ld) {
  for (int64_t q = (int64_t)blockIdx.x * kBlk + threadIdx.x; q < total;
       q += (int64_t)gridDim.x * kBlk) {
    const int64_t i = q / ld, j = q - i * ld;
    z[q] = (M)((i == j && i < n) ? c : 0.0);
  }
}

// The first iterate's products with Z_0 = c I: X = (c O) c on the N x N block, zero
// elsewhere, the lower triangle of O standing for both.  One term of every dot
// product is not zero, so this is what the product kernels give, bit for bit (adding
// 0 makes a zero term's sign theirs), at the cost of a pass over memory: at N = 4096
// in FP64 0.05 ms in place of 2.0 + 1.3 ms.  A workgroup reads a 32 x 32 tile of the
// lower triangle by rows and writes it and, through the LDS, its mirror by rows.  The
// upper triangle enters with a factor of zero, as it did in the dot products: what is
// not finite there is NaN in X.
constexpr int kMirTile = 32;
template <typename M>
__global__ void __launch_bounds__(kBlk) k_first_x(const M* o, double c, M* x, int64_t n,
                                                 int64_t ld) {
  __shared__ M sh[kMirTile][kMirTile + 1];
  const int ti = blockIdx.y, tj = blockIdx.x;
  if (tj > ti) return;
  const M cm = (M)c;
  const int col = threadIdx.x % kMirTile, row0 = threadIdx.x / kMirTile;
  const int64_t i0 = (int64_t)ti * kMirTile, j0 = (int64_t)tj * kMirTile;
  for (int row = row0; row < kMirTile; row += kBlk / kMirTile) {
    const int64_t i = i0 + row, j = j0 + col;
    M v = (M)0;
    if (i < n && j < n) {
      const M y = cm * o[i * ld + j] + (M)0;
      v = y * cm + (M)0;
    }
    sh[row][col] = v;
    if (j <= i) x[i * ld + j] = v;
  }
  __syncthreads();
  for (int row = row0; row < kMirTile; row += kBlk / kMirTile) {
    const int64_t i = j0 + row, j = i0 + col;
    if (j > i) x[i * ld + j] = sh[col][row] + (j < n ? (M)0 * o[i * ld + j] : (M)0);
  }
}

// Q = a0 I + a1 X + a2 T on the N x N block (T = X^2), zero elsewhere; q may be t.
// FIRST: c Q, the update Z_0 Q of the first iterate.
template <typename M, bool FIRST>
__global__ void __launch_bounds__(kBlk) k_poly2(const M* x, const M* t, M* q, int64_t n,
                                               int64_t total, int64_t ld, double c) {
  const double a0 = 1.875, a1 = -1.25, a2 = 0.375;
  for (int64_t p = (int64_t)blockIdx.x * kBlk + threadIdx.x; p < total;
       p += (int64_t)gridDim.x * kBlk) {
    const int64_t i = p / ld, j = p - i * ld;
    double v = 0.0;
    if (i < n && j < n) v = (i == j ? a0 : 0.0) + a1 * (double)x[p] + a2 * (double)t[p];
    M w = (M)v;
    if constexpr (FIRST) w = (M)c * w + (M)0;
    q[p] = w;
  }
}

// ||X - I||_F^2 partials over the N x N block (FP64, fixed grid).
template <typename M>
__global__ void __launch_bounds__(kBlk) k_dev_identity(const M* x, int64_t n, int64_t ld,
                                                      double* part) {
  double v = 0.0;
  const int64_t total = n * n;
  for (int64_t p = (int64_t)blockIdx.x * kBlk + threadIdx.x; p < total;
       p += (int64_t)gridDim.x * kBlk) {
    const int64_t i = p / n, j = p - i * n;
    const double d = (double)x[i * ld + j] - (i == j ? 1.0 : 0.0);
    v += d * d;
  }
  v = block_sum(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v;
}

__global__ void __launch_bounds__(kBlk) k_sum_partials(const double* part, int nb, double* out) {
  const double v = serial_sum(part, nb);
  if (threadIdx.x == 0) *out = v;
}

dmpt_status ofail(dmpt_status s, const std::string& m) {
  set_last_error(m.c_str());
  return s;
}

// Workspace of the single products: padded matrices and the two item lists, in one
// allocation (mapping and unmapping device memory costs about 0.1 ms per call and
// 1 ms per GB).
struct ProductWork {
  dmpt_precision prec;
  int64_t n = 0, np = 0, ld = 0;
  size_t eb = 0;
  char* base = nullptr;
  TileItem* items_sym = nullptr;
  TileItem* items_all = nullptr;
  int n_sym = 0, n_all = 0;
  DirectTile tile_sym{}, tile_all{};
  double* part = nullptr;
  double* dscal = nullptr;

  // An FP64 matrix that the product kernels can read where it lies: no padding to
  // add, rows on their 16-byte loads.
  bool in_place(const double* m) const {
    return prec == DMPT_FP64 && np == n && ((uintptr_t)m & 15) == 0;
  }
  // the lists, scalars and `mats` matrices (mat[0 .. mats))
  hipError_t init(dmpt_precision pr, int64_t nn, int mats, void** mat, hipStream_t s) {
    prec = pr;
    n = nn;
    const int tile = product_tile(prec);
    np = (n + tile - 1) / tile * tile;
    ld = np;
    eb = prec == DMPT_FP64 ? 8 : 4;
    tile_sym = direct_tile(prec, n, 1, 0, true);
    tile_all = direct_tile(prec, n, 1, 0, false);
    const int Ts = (int)((n + tile_sym.edge - 1) / tile_sym.edge);
    const int Ta = (int)((n + tile_all.edge - 1) / tile_all.edge);
    n_sym = Ts * (Ts + 1) / 2;
    n_all = Ta * Ta;
    std::vector<TileItem> items(n_sym + n_all);
    product_items(Ts, 1, items.data());
    product_items(Ta, 2, items.data() + n_sym);
    const size_t item_bytes = items.size() * sizeof(TileItem);
    const size_t mbytes = (size_t)np * ld * eb;             // a multiple of 64 KB
    const size_t small = (3 * 512 + 16) * sizeof(double);
    hipError_t e = hipMalloc((void**)&base, mats * mbytes + small + item_bytes);
    if (e != hipSuccess) {
      base = nullptr;
      return e;
    }
    for (int i = 0; i < mats; ++i) mat[i] = base + i * mbytes;
    part = (double*)(base + mats * mbytes);
    dscal = part + 3 * 512;
    items_sym = (TileItem*)(dscal + 16);
    items_all = items_sym + n_sym;
    e = hipMemcpy(items_sym, items.data(), item_bytes, hipMemcpyHostToDevice);
    // padding that a product reads but none writes; without padding every element
    // is written before it is read
    if (e == hipSuccess && np != n) e = hipMemsetAsync(base, 0, mats * mbytes, s);
    return e;
  }
  // C = A B (A, B symmetric); symmetric C on mirrored upper tiles, else every tile
  hipError_t product(const void* A, const void* B, void* C, bool symmetric, hipStream_t s) {
    ProductArgs a;
    memset(&a, 0, sizeof(a));
    a.s_hi = A;
    a.s1_hi[0] = B;
    a.x = C;
    a.items = symmetric ? items_sym : items_all;
    a.n_items = symmetric ? n_sym : n_all;
    a.ld = ld;
    a.kdim = np;
    a.kext = direct_kext(n);
    a.tile = symmetric ? tile_sym : tile_all;
    a.mode = symmetric ? 1 : 2;
    return launch_products(prec, a, s);
  }
  ~ProductWork() {
    if (base) (void)hipFree(base);
  }
};

bool direct_precision(int32_t p) { return p == DMPT_FP64 || p == DMPT_FP32; }

}  // namespace

}  // namespace dmpt

using namespace dmpt;

extern "C" {

dmpt_status dmpt_inverse_factor(int32_t precision, const double* O, int64_t N, double* Z,
                                int32_t max_iter, double tol, int32_t* iters, double* err,
                                void* stream) {
  if (!O || !Z || N < 1 || N > (1 << 17) || max_iter < 1 || !(tol > 0.0))
    return ofail(DMPT_EINVAL, "bad arguments");
  if (!direct_precision(precision))
    return ofail(DMPT_ENOTSUP, "the inverse factor runs in DMPT_FP64 or DMPT_FP32");
  hipStream_t s = (hipStream_t)stream;
  const dmpt_precision prec = (dmpt_precision)precision;
  ProductWork w;
  void* m[5] = {};
  hipError_t e = w.init(prec, N, 5, m, s);
  if (e != hipSuccess)
    return ofail(e == hipErrorOutOfMemory ? DMPT_ENOMEM : DMPT_EHIP, "workspace allocation failed");
  void *z = m[0], *y = m[1], *x = m[2], *t = m[3], *q = t;
  const void* om = m[4];
  const int64_t total = w.np * w.ld;
  double eps[2] = {0.0, 0.0};
  e = launch_gershgorin(O, N, w.part, nullptr, w.dscal, s);
  if (e == hipSuccess) e = hipMemcpyAsync(eps, w.dscal, sizeof(eps), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return ofail(DMPT_EHIP, hipGetErrorString(e));
  if (!(eps[1] > 0.0) || !isfinite(eps[1]))
    return ofail(DMPT_ENONFINITE, "overlap matrix without a positive spectral bound");
  if (w.in_place(O))
    om = O;
  else
    e = launch_from_f64(prec, O, N, w.np, w.ld, 0, 0, m[4], nullptr, nullptr, s);
  if (e != hipSuccess) return ofail(DMPT_EHIP, hipGetErrorString(e));
  const double c = 1.0 / sqrt(eps[1]);
  int it = 0;
  double r = INFINITY;
  for (;; ++it) {
    // X = Z O Z (Y = Z O, general; X = Y Z, symmetric).  Y is formed in full although
    // Z and O commute: with its lower half mirrored the recursion loses the
    // stability that its rounding errors need (on a matrix of condition 100 the
    // residual grew sevenfold with every step past convergence).
    if (it == 0) {
      const dim3 grid((unsigned)(w.np / kMirTile), (unsigned)(w.np / kMirTile));
      if (prec == DMPT_FP64)
        hipLaunchKernelGGL(k_first_x<double>, grid, dim3(kBlk), 0, s, (const double*)om, c,
                           (double*)x, N, w.ld);
      else
        hipLaunchKernelGGL(k_first_x<float>, grid, dim3(kBlk), 0, s, (const float*)om, c,
                           (float*)x, N, w.ld);
    } else {
      e = w.product(z, om, y, false, s);
      if (e == hipSuccess) e = w.product(y, z, x, true, s);
    }
    if (e != hipSuccess) break;
    if (prec == DMPT_FP64)
      hipLaunchKernelGGL(k_dev_identity<double>, dim3(512), dim3(kBlk), 0, s, (const double*)x, N,
                         w.ld, w.part);
    else
      hipLaunchKernelGGL(k_dev_identity<float>, dim3(512), dim3(kBlk), 0, s, (const float*)x, N,
                         w.ld, w.part);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kBlk), 0, s, w.part, 512, w.dscal);
    double r2 = 0.0;
    e = hipMemcpyAsync(&r2, w.dscal, sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) break;
    r = sqrt(r2);
    if (!isfinite(r)) {
      e = hipSuccess;
      break;
    }
    if (r < tol || it >= max_iter) break;
    // Z <- Z (a0 I + a1 X + a2 X^2)
    e = w.product(x, x, t, true, s);
    if (e != hipSuccess) break;
    if (it == 0) {
      if (prec == DMPT_FP64)
        hipLaunchKernelGGL((k_poly2<double, true>), dim3(2048), dim3(kBlk), 0, s, (const double*)x,
                           (const double*)t, (double*)z, N, total, w.ld, c);
      else
        hipLaunchKernelGGL((k_poly2<float, true>), dim3(2048), dim3(kBlk), 0, s, (const float*)x,
                           (const float*)t, (float*)z, N, total, w.ld, c);
      continue;
    }
    if (prec == DMPT_FP64)
      hipLaunchKernelGGL((k_poly2<double, false>), dim3(2048), dim3(kBlk), 0, s, (const double*)x,
                         (const double*)t, (double*)q, N, total, w.ld, c);
    else
      hipLaunchKernelGGL((k_poly2<float, false>), dim3(2048), dim3(kBlk), 0, s, (const float*)x,
                         (const float*)t, (float*)q, N, total, w.ld, c);
    e = w.product(z, q, y, true, s);
    if (e != hipSuccess) break;
    std::swap(z, y);
  }
  if (e != hipSuccess) return ofail(DMPT_EHIP, hipGetErrorString(e));
  if (it == 0) {                               // Z_0 = c I
    if (prec == DMPT_FP64)
      hipLaunchKernelGGL(k_scaled_identity<double>, dim3(2048), dim3(kBlk), 0, s, (double*)z, c, N,
                         total, w.ld);
    else
      hipLaunchKernelGGL(k_scaled_identity<float>, dim3(2048), dim3(kBlk), 0, s, (float*)z, c, N,
                         total, w.ld);
  }
  e = launch_copy_plain(prec, z, w.ld, Z, N, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return ofail(DMPT_EHIP, hipGetErrorString(e));
  if (iters) *iters = it;
  if (err) *err = r;
  if (!isfinite(r)) return ofail(DMPT_ENONFINITE, "inverse factor iteration diverged");
  if (!(r < tol)) return ofail(DMPT_ENOCONV, "inverse factor: tolerance not reached");
  return DMPT_OK;
}

dmpt_status dmpt_congruence(int32_t precision, int64_t N, const double* Z, const double* A,
                            double* out, void* stream) {
  if (!Z || !A || !out || N < 1 || N > (1 << 17)) return ofail(DMPT_EINVAL, "bad arguments");
  if (!direct_precision(precision))
    return ofail(DMPT_ENOTSUP, "congruences run in DMPT_FP64 or DMPT_FP32");
  hipStream_t s = (hipStream_t)stream;
  const dmpt_precision prec = (dmpt_precision)precision;
  ProductWork w;
  void* m[3] = {};
  // Y and, where the operands cannot be read or the result not be written in place
  // (Y Z is written while Z is read), copies of Z and of A, which the result replaces
  w.prec = prec;
  w.n = N;
  w.np = (N + product_tile(prec) - 1) / product_tile(prec) * product_tile(prec);
  const double* end = Z + (size_t)N * N;
  const bool direct = w.in_place(Z) && w.in_place(A) &&
                      (out + (size_t)N * N <= Z || out >= end);
  hipError_t e = w.init(prec, N, direct ? 1 : 3, m, s);
  if (e != hipSuccess)
    return ofail(e == hipErrorOutOfMemory ? DMPT_ENOMEM : DMPT_EHIP, "workspace allocation failed");
  if (direct) {
    e = w.product(Z, A, m[0], false, s);                           // Y = Z A
    if (e == hipSuccess) e = w.product(m[0], Z, out, true, s);     // Z A Z
  } else {
    e = launch_from_f64(prec, Z, N, w.np, w.ld, 0, 0, m[1], nullptr, nullptr, s);
    if (e == hipSuccess) e = launch_from_f64(prec, A, N, w.np, w.ld, 0, 0, m[2], nullptr, nullptr, s);
    if (e == hipSuccess) e = w.product(m[1], m[2], m[0], false, s);
    if (e == hipSuccess) e = w.product(m[0], m[1], m[2], true, s);
    if (e == hipSuccess) e = launch_copy_plain(prec, m[2], w.ld, out, N, s);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  return e == hipSuccess ? DMPT_OK : ofail(DMPT_EHIP, hipGetErrorString(e));
}

}  // extern "C"
