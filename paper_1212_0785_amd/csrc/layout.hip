// Conversion between the canonical array-of-structures layout (complex128,
// site-major, the form fields are imported and exported in) and the
// structure-of-arrays device layouts of device.h, plus precision
// conversion for the mixed-precision solver.  Sec. 3's tensor structure
// (Outer x Spin x Color x Reality) is kept: the outer (site) level becomes
// the fastest-varying index so that each spin/colour/reality component of
// a field is one contiguous array.
#include "device.h"
#include "internal.h"

namespace hmc {


// Gauge and spinor conversions go through LDS: a block takes kTile
// consecutive lexicographic sites, whose canonical entries are one contiguous
// range and which hold kTile / 2 consecutive checkerboard sites of each parity,
// so both sides are read or written in whole cache lines.  With one work-item
// per site the canonical side was touched in 16-byte pieces, 576 (links) or
// 192 bytes (spinors) apart: 183 / 246 us to import / export the links of
// 20^2x22x44 (2 x 223 MB), against 90 / 67 us through the tile (spinors 54 ->
// 28 us).
constexpr int kTile = 64;
constexpr int kLinkRow = 37;    // 36 entries per site, padded against bank conflicts
constexpr int kSpinorRow = 13;  // 12

// Position within its pair of sites (2q, 2q + 1) of the site of parity par.
__device__ __forceinline__ int site_of_pair(const Lat& g, int pair, int par) {
  return par ^ parity_of_lex(g, 2 * pair);
}

// Links that are not SU(3) to within `tol` in any real component: rows 0 and 1
// not orthonormal (|row|^2 - 1, <row0, row1>), or the stored third row not
// conj(row0 x row1) (which then makes det U = 1).  The compact link forms
// rebuild entries from exactly these relations.
__device__ __forceinline__ bool not_su3(const mat3<double>& u, double tol) {
  mat3<double> r = u;
  third_row(r);
  bool bad = false;
#pragma unroll
  for (int k = 6; k < 9; ++k)
    bad |= !(fabs(u.m[k].re - r.m[k].re) <= tol) || !(fabs(u.m[k].im - r.m[k].im) <= tol);
  const double n0 = norm2(u.m[0]) + norm2(u.m[1]) + norm2(u.m[2]);
  const double n1 = norm2(u.m[3]) + norm2(u.m[4]) + norm2(u.m[5]);
  cx<double> o = cmadd_conj(cx<double>{0, 0}, u.m[0], u.m[3]);
  o = cmadd_conj(o, u.m[1], u.m[4]);
  o = cmadd_conj(o, u.m[2], u.m[5]);
  bad |= !(fabs(n0 - 1.0) <= tol) || !(fabs(n1 - 1.0) <= tol) || !(fabs(o.re) <= tol) || !(fabs(o.im) <= tol);
  return bad;
}

// Also counts the block's links that are not SU(3) (one of the tile's 256 per
// work-item) into bad[blockIdx.x], which spares the import a second sweep of
// the links (46 us of the 230 at 20^2x22x44).
__global__ void __launch_bounds__(kBlock) k_pack_gauge(Lat g, const double2* canon, double2* U, double tol,
                                                       double* bad) {
  static_assert(kTile * 4 == kBlock, "one link per work-item");
  __shared__ double2 tile[kTile * kLinkRow];
  const int i0 = blockIdx.x * kTile, n = min(kTile, 2 * g.Vh - i0);
  for (int j = threadIdx.x; j < n * 36; j += kBlock) tile[j / 36 * kLinkRow + j % 36] = canon[(size_t)i0 * 36 + j];
  __syncthreads();
  const int r = threadIdx.x & (kTile - 1), par = r / (kTile / 2), q = r % (kTile / 2);
  if (2 * q < n) {
    const int pair = i0 / 2 + q;
    const double2* src = tile + (2 * q + site_of_pair(g, pair, par)) * kLinkRow;
    for (int c = threadIdx.x / kTile; c < 36; c += kBlock / kTile) {
      const int mu = c / 9, k = c - 9 * mu;
      U[((size_t)(mu * 2 + par) * 9 + k) * g.stride + pair] = src[c];
    }
  }
  double v[1] = {0.0};
  if ((int)threadIdx.x < 4 * n) {
    const double2* src = tile + (threadIdx.x >> 2) * kLinkRow + 9 * (threadIdx.x & 3);
    mat3<double> u;
#pragma unroll
    for (int k = 0; k < 9; ++k) u.m[k] = {src[k].x, src[k].y};
    v[0] = not_su3(u, tol) ? 1.0 : 0.0;
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) bad[blockIdx.x] = v[0];
}

__global__ void __launch_bounds__(kBlock) k_unpack_gauge(Lat g, const double2* U, double2* canon) {
  __shared__ double2 tile[kTile * kLinkRow];
  const int i0 = blockIdx.x * kTile, n = min(kTile, 2 * g.Vh - i0);
  const int r = threadIdx.x & (kTile - 1), par = r / (kTile / 2), q = r % (kTile / 2);
  if (2 * q < n) {
    const int pair = i0 / 2 + q;
    double2* dst = tile + (2 * q + site_of_pair(g, pair, par)) * kLinkRow;
#pragma unroll
    for (int m = 0; m < 9; ++m) {
      const int c = threadIdx.x / kTile + m * (kBlock / kTile), mu = c / 9, k = c - 9 * mu;
      dst[c] = U[((size_t)(mu * 2 + par) * 9 + k) * g.stride + pair];
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < n * 36; j += kBlock) canon[(size_t)i0 * 36 + j] = tile[j / 36 * kLinkRow + j % 36];
}

// canonical full spinor -> half spinor of parity par0, or (par0 < 0) both.
__global__ void __launch_bounds__(kBlock) k_pack_spinor(Lat g, const double2* canon, double2* half, int par0) {
  __shared__ double2 tile[kTile * kSpinorRow];
  const int i0 = blockIdx.x * kTile, n = min(kTile, 2 * g.Vh - i0);
  for (int j = threadIdx.x; j < n * 12; j += kBlock) {
    const int l = j / 12;
    if (par0 < 0 || parity_of_lex(g, i0 + l) == par0)
      tile[l * kSpinorRow + j % 12] = canon[(size_t)i0 * 12 + j];
  }
  __syncthreads();
  const int r = threadIdx.x & (kTile - 1), par = r / (kTile / 2), q = r % (kTile / 2);
  if (2 * q >= n || (par0 >= 0 && par != par0)) return;
  const int pair = i0 / 2 + q;
  const double2* src = tile + (2 * q + site_of_pair(g, pair, par)) * kSpinorRow;
  double2* dst = half + (par0 < 0 ? (size_t)par * 12 * g.stride : 0);
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    const int c = threadIdx.x / kTile + m * (kBlock / kTile);
    dst[(size_t)c * g.stride + pair] = src[c];
  }
}

// half spinor(s) -> canonical full spinor, zeros on the other parity's sites.
__global__ void __launch_bounds__(kBlock) k_unpack_spinor(Lat g, const double2* half, double2* canon, int par0) {
  __shared__ double2 tile[kTile * kSpinorRow];
  const int i0 = blockIdx.x * kTile, n = min(kTile, 2 * g.Vh - i0);
  const int r = threadIdx.x & (kTile - 1), par = r / (kTile / 2), q = r % (kTile / 2);
  if (2 * q < n) {
    const int pair = i0 / 2 + q;
    double2* dst = tile + (2 * q + site_of_pair(g, pair, par)) * kSpinorRow;
    const double2* src = half + (par0 < 0 ? (size_t)par * 12 * g.stride : 0);
    const bool zero = par0 >= 0 && par != par0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const int c = threadIdx.x / kTile + m * (kBlock / kTile);
      dst[c] = zero ? make_double2(0.0, 0.0) : src[(size_t)c * g.stride + pair];
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < n * 12; j += kBlock) canon[(size_t)i0 * 12 + j] = tile[j / 12 * kSpinorRow + j % 12];
}

__global__ void k_pack_momenta(Lat g, const double2* canon, double* P) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= 2 * g.Vh) return;
  int par = parity_of_lex(g, i), s = i >> 1;
  for (int mu = 0; mu < 4; ++mu) {
    const double2* m = canon + ((size_t)i * 4 + mu) * 9;
    double c[8] = {m[0].x, m[4].x, m[1].x, m[1].y, m[2].x, m[2].y, m[5].x, m[5].y};
    store_compact(P, g.stride, mu, par, s, c);
  }
}

__global__ void k_unpack_momenta(Lat g, const double* P, double2* canon) {
  int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= 2 * g.Vh) return;
  int par = parity_of_lex(g, i), s = i >> 1;
  for (int mu = 0; mu < 4; ++mu) {
    double c[8];
    load_compact(P, g.stride, mu, par, s, c);
    mat3<double> h = herm_from_compact(c);
    double2* m = canon + ((size_t)i * 4 + mu) * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) m[k] = make_double2(h.m[k].re, h.m[k].im);
  }
}

template <class LK>
__global__ void k_convert_gauge(Lat g, const void* U64, void* Ulow) {
  int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= g.Vh) return;
  int mu = blockIdx.y >> 1, par = blockIdx.y & 1;
  mat3<double> u = LkF64::load(U64, g.stride, mu, par, s);
  LK::store(Ulow, g.stride, mu, par, s, u);
}

// Per-block counts of the links that are not SU(3) to within `tol`.
__global__ void __launch_bounds__(kBlock) k_su3_check(Lat g, const void* U, double tol, double* part) {
  double v[1] = {0.0};
  for (int j = blockIdx.x * kBlock + threadIdx.x; j < 2 * g.Vh; j += gridDim.x * kBlock) {
    const int par = j >= g.Vh, s = j - par * g.Vh;
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) v[0] += not_su3(LkF64::load(U, g.stride, mu, par, s), tol) ? 1.0 : 0.0;
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

template <class SI, class SO>
__global__ void k_convert_spinor(Lat g, const void* in, void* out, const void* const* tin, void* const* tout,
                                 const int* gate) {
  if (gate && *gate == 0) return;  // gated: a device-driven reliable update that was not requested
  int s = blockIdx.x * kBlock + threadIdx.x;
  if (s >= g.Vh) return;
  const void* src = tin ? tin[blockIdx.y] : in;
  void* dst = tout ? tout[blockIdx.y] : out;
  cx<typename SI::R> a[12];
  cx<typename SO::R> b[12];
  SI::load(src, g.stride, s, a);
#pragma unroll
  for (int k = 0; k < 12; ++k) b[k] = {(typename SO::R)a[k].re, (typename SO::R)a[k].im};
  SO::store(dst, g.stride, s, b);
}

int pack_gauge_blocks(int Vh) { return ceil_div(2LL * Vh, kTile); }

hipError_t launch_pack_gauge(const LatArg& g, const void* canon, void* U, double tol, double* bad, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_gauge, dim3(pack_gauge_blocks(g.Vh)), dim3(kBlock), 0, st, to_lat(g),
                     (const double2*)canon, (double2*)U, tol, bad);
  return hipGetLastError();
}
hipError_t launch_unpack_gauge(const LatArg& g, const void* U, void* canon, hipStream_t st) {
  hipLaunchKernelGGL(k_unpack_gauge, dim3(ceil_div(2LL * g.Vh, kTile)), dim3(kBlock), 0, st, to_lat(g),
                     (const double2*)U, (double2*)canon);
  return hipGetLastError();
}
hipError_t launch_pack_spinor(const LatArg& g, const void* canon, void* half, int par, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_spinor, dim3(ceil_div(2LL * g.Vh, kTile)), dim3(kBlock), 0, st, to_lat(g),
                     (const double2*)canon, (double2*)half, par);
  return hipGetLastError();
}
hipError_t launch_unpack_spinor(const LatArg& g, const void* half, void* canon, int par, hipStream_t st) {
  hipLaunchKernelGGL(k_unpack_spinor, dim3(ceil_div(2LL * g.Vh, kTile)), dim3(kBlock), 0, st, to_lat(g),
                     (const double2*)half, (double2*)canon, par);
  return hipGetLastError();
}
hipError_t launch_pack_momenta(const LatArg& g, const void* canon, double* P, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_momenta, dim3(ceil_div(2LL * g.Vh, kBlock)), dim3(kBlock), 0, st, to_lat(g),
                     (const double2*)canon, P);
  return hipGetLastError();
}
hipError_t launch_unpack_momenta(const LatArg& g, const double* P, void* canon, hipStream_t st) {
  hipLaunchKernelGGL(k_unpack_momenta, dim3(ceil_div(2LL * g.Vh, kBlock)), dim3(kBlock), 0, st, to_lat(g), P,
                     (double2*)canon);
  return hipGetLastError();
}

hipError_t launch_su3_check(const LatArg& g, const void* U, double tol, double* part, int nb, hipStream_t st) {
  hipLaunchKernelGGL(k_su3_check, dim3(nb), dim3(kBlock), 0, st, to_lat(g), U, tol, part);
  return hipGetLastError();
}

hipError_t launch_convert_gauge(const LatArg& g, const void* U64, void* Ulow, hmc_prec prec, hipStream_t st) {
  dim3 grid(site_blocks(g.Vh), 8), block(kBlock);
  switch (prec) {
    case HMC_F32: hipLaunchKernelGGL(k_convert_gauge<LkF32>, grid, block, 0, st, to_lat(g), U64, Ulow); break;
    case HMC_F16: hipLaunchKernelGGL(k_convert_gauge<LkF16>, grid, block, 0, st, to_lat(g), U64, Ulow); break;
    case HMC_BF16: hipLaunchKernelGGL(k_convert_gauge<LkBF16>, grid, block, 0, st, to_lat(g), U64, Ulow); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class SI>
static hipError_t conv_out(const LatArg& g, const void* in, void* out, hmc_prec pout, int nbatch,
                           const void* const* tin, void* const* tout, hipStream_t st, const int* gate) {
  dim3 grid(site_blocks(g.Vh), nbatch), block(kBlock);
  switch (pout) {
    case HMC_F64: hipLaunchKernelGGL((k_convert_spinor<SI, SpF64>), grid, block, 0, st, to_lat(g), in, out, tin, tout, gate); break;
    case HMC_F32: hipLaunchKernelGGL((k_convert_spinor<SI, SpF32>), grid, block, 0, st, to_lat(g), in, out, tin, tout, gate); break;
    case HMC_F16: hipLaunchKernelGGL((k_convert_spinor<SI, SpF16>), grid, block, 0, st, to_lat(g), in, out, tin, tout, gate); break;
    case HMC_BF16: hipLaunchKernelGGL((k_convert_spinor<SI, SpBF16>), grid, block, 0, st, to_lat(g), in, out, tin, tout, gate); break;
  }
  return hipGetLastError();
}

hipError_t launch_convert_spinor(const LatArg& g, const void* in, hmc_prec pin, void* out, hmc_prec pout,
                                 int nbatch, const void* const* tab_in, void* const* tab_out, hipStream_t st,
                                 const int* gate) {
  switch (pin) {
    case HMC_F64: return conv_out<SpF64>(g, in, out, pout, nbatch, tab_in, tab_out, st, gate);
    case HMC_F32: return conv_out<SpF32>(g, in, out, pout, nbatch, tab_in, tab_out, st, gate);
    case HMC_F16: return conv_out<SpF16>(g, in, out, pout, nbatch, tab_in, tab_out, st, gate);
    case HMC_BF16: return conv_out<SpBF16>(g, in, out, pout, nbatch, tab_in, tab_out, st, gate);
  }
  return hipErrorInvalidValue;
}

}  // namespace hmc
