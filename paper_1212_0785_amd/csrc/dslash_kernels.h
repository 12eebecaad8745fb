// Kernels and launchers of the Wilson hopping term, instantiated once per
// storage precision (dslash_f64.hip, dslash_f32.hip, dslash_f16.hip,
// dslash_bf16.hip; dslash.hip dispatches).
//
// Wilson hopping term on one checkerboard (the dominant kernel of the
// fermion-matrix inversion that the paper's introduction singles out as
// the bulk of the floating-point work):
//   (D psi)(x) = sum_mu [(1 - gamma_mu) U_mu(x) psi(x+mu)
//                      + (1 + gamma_mu) U_mu(x-mu)^dag psi(x-mu)]
// with -1 on hops across the time boundary; the dagger swaps the
// projectors.  One work-item per output site (Sec. 3's site-per-thread
// mapping); the 4x4 spin structure is applied through the rank-2
// projections (1 +- gamma_mu), so each hop multiplies only two colour
// vectors by the link.
//
// The kernel is HBM-bound (about 0.86 flop per byte in FP64).  Fields are
// stored component-major so every load instruction of a wave covers one
// contiguous 1 KiB (FP64) span; neighbour spinors are re-read through L2,
// and the XCD-aware block order keeps the +-y/+-z neighbours of a block on
// the XCD that owns it.
#pragma once

#include <hip/hip_ext.h>

#include <climits>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace hmc {

#ifndef HMC_DSLASH_WAVES
#define HMC_DSLASH_WAVES
#endif
#ifndef HMC_HOP_CHAIN
#define HMC_HOP_CHAIN 1
#endif

// Makes `idx` depend on every accumulator without changing either.  The
// loads of a hop use indices chained to the accumulators left by the
// previous hop, so the compiler cannot issue all sixteen hops' loads up
// front (that needs ~600 registers and spills); a wave keeps one hop
// (HMC_HOP_CHAIN = 1) or one direction (= 2) of loads in flight and
// occupancy supplies the memory parallelism.
template <typename R>
__device__ __forceinline__ int chain(int idx, cx<R>* acc) {
#if HMC_HOP_CHAIN
#pragma unroll
  for (int k = 0; k < 12; ++k) asm volatile("" : "+v"(acc[k].re), "+v"(acc[k].im));
  asm volatile("" : "+v"(idx));
#endif
  return idx;
}

// Half spinor (1 + SIG gamma_MU) psi of site s.
template <class SP, int MU, int SIG>
__device__ __forceinline__ void load_projected(const void* in, int stride, int s, cx<typename SP::R>* h) {
  if constexpr (SP::kScaled) {
    SP::template load_projected<MU, SIG>(in, stride, s, h);
  } else {
    cx<typename SP::R> psi[12];
    SP::load(in, stride, s, psi);
    spin_project<MU, SIG>(psi, h);
  }
}

template <class SP, class LK, int MU, bool DAG>
__device__ __forceinline__ void hop_dir(const Lat& g, const Site& st, int out_par, int s, const void* U,
                                        const void* in, cx<typename SP::R>* acc) {
  using R = typename SP::R;
  constexpr int SF = DAG ? +1 : -1;  // forward hop carries (1 + SF gamma_mu)
  constexpr int SB = -SF;
  bool wf, wb;
  const int lf = neighbour_lex<MU, +1>(g, st, &wf);
  const int lb = neighbour_lex<MU, -1>(g, st, &wb);
  {
    cx<R> h[6], uh[6];
    const int sn = chain(lf >> 1, acc), sl = chain(s, acc);
    load_projected<SP, MU, SF>(in, g.stride, sn, h);
    if (MU == 3) {  // antiperiodic time boundary
      const R sg = wf ? R(-1) : R(1);
#pragma unroll
      for (int k = 0; k < 6; ++k) h[k] = sg * h[k];
    }
    const mat3<R> u = LK::load_u(U, g.stride, MU, out_par, sl);
    mv(u, h, uh);
    mv(u, h + 3, uh + 3);
    spin_accum<MU, SF>(acc, uh);
  }
  {
    cx<R> h[6], uh[6];
    const int sn = HMC_HOP_CHAIN == 1 ? chain(lb >> 1, acc) : lb >> 1;
    load_projected<SP, MU, SB>(in, g.stride, sn, h);
    if (MU == 3) {
      const R sg = wb ? R(-1) : R(1);
#pragma unroll
      for (int k = 0; k < 6; ++k) h[k] = sg * h[k];
    }
    const mat3<R> u = LK::load_u(U, g.stride, MU, out_par ^ 1, sn);
    mdv(u, h, uh);
    mdv(u, h + 3, uh + 3);
    spin_accum<MU, SB>(acc, uh);
  }
}

// Block 0 computes the solver step length from the partial sums of the
// previous kernels (see DslashArgs::alpha_out); the other blocks skip it.
template <int W = kBlock / 64>
__device__ __forceinline__ void alpha_prologue(const DslashArgs& e, int label) {
  if (!e.alpha_out || blockIdx.x != 0) return;
  const double* part[2] = {e.alpha_pp[label & 1], e.alpha_den};
  const int n[2] = {e.alpha_n_pp, e.alpha_n_den};
  double s[2];
  sum_partials_n<W, 2>(part, n, s);
  if (threadIdx.x == 0) *(HMC_GLOBAL double*)e.alpha_out = s[0] / s[1];
}

// The block's |out|^2 (thread 0's v) into its partial-sum slot or slots.
__device__ __forceinline__ void put_partial(const DslashArgs& e, int label, int b, double v) {
  if (threadIdx.x != 0) return;
  if (e.partial) ((HMC_GLOBAL double*)e.partial)[b] = v;
  if (e.partial_pp[0])
    ((HMC_GLOBAL double*)(e.partial || (label & 1) ? e.partial_pp[0] : e.partial_pp[1]))[b] = v;
}

// BATCH: blockIdx.y selects an entry of `table` (same-volume requests share
// one launch); otherwise the single entry `one` is read from the kernel
// arguments.
template <class SP, class LK, bool DAG, int EPI, bool BATCH>
__global__ void __launch_bounds__(kBlock) HMC_DSLASH_WAVES k_dslash(Lat g, int out_par,
                                                                    const DslashArgs* __restrict__ table,
                                                                    DslashArgs one, int j) {
  using R = typename SP::R;
  const DslashArgs* ep;
  if constexpr (BATCH)
    ep = table + blockIdx.y;
  else
    ep = &one;
  const DslashArgs& e = *ep;
  const int label = e.iter0 + j + (e.label_base ? *(const HMC_GLOBAL int*)e.label_base : 0);
  if (e.stop_at && label >= *(const HMC_GLOBAL int*)e.stop_at) return;
  alpha_prologue(e, label);
  int b;
  const int s = dslash_site(g, &b);
  double nrm[1] = {0.0};
  if (s < g.Vh) {
    const Site st = cb_site(g, out_par, s);
    cx<R> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
    hop_dir<SP, LK, 0, DAG>(g, st, out_par, s, e.U, e.in, acc);
    hop_dir<SP, LK, 1, DAG>(g, st, out_par, s, e.U, e.in, acc);
    hop_dir<SP, LK, 2, DAG>(g, st, out_par, s, e.U, e.in, acc);
    hop_dir<SP, LK, 3, DAG>(g, st, out_par, s, e.U, e.in, acc);
    if (EPI != EPI_PLAIN) {
      const R a = (R)e.a, bb = (R)e.b;
      if (e.y) {
        cx<R> y[12];
        SP::load(e.y, g.stride, s, y);
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {fma(bb, acc[k].re, a * y[k].re), fma(bb, acc[k].im, a * y[k].im)};
      } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = bb * acc[k];
      }
    }
    if (EPI == EPI_CG) {  // acc = q = A p;  r <- r - alpha q
      const R al = (R)(*(const HMC_GLOBAL double*)e.alpha_in);
      cx<R> r[12];
      SP::load(e.r, g.stride, s, r);
#pragma unroll
      for (int k = 0; k < 12; ++k) acc[k] = {fma(-al, acc[k].re, r[k].re), fma(-al, acc[k].im, r[k].im)};
    }
    if (EPI == EPI_AXPY_NORM || EPI == EPI_CG)
#pragma unroll
      for (int k = 0; k < 12; ++k) nrm[0] += (double)acc[k].re * acc[k].re + (double)acc[k].im * acc[k].im;
    SP::template store<LK::kStream>(e.out, g.stride, s, acc);
  }
  if (EPI == EPI_AXPY_NORM || EPI == EPI_CG) {
    block_sum<1>(nrm);
    put_partial(e, label, b, nrm[0]);
  }
}

// Direction split: a block of NW = 2 or 4 wavefronts covers 64 sites; wavefront
// w computes the hops along two directions, 2w and 2w + 1, or along direction w,
// and parks its partial sum in LDS; after a barrier each work-item combines the
// partials of 12 / NW of the 12 components of one site (coalesced stores).  NW
// times the wavefronts of the one-site-per-work-item kernel at the same registers
// per work-item, and 1 / NW of its serial hop chain.
template <class SP, class LK, bool DAG, int EPI, bool BATCH, int NW>
__global__ void __launch_bounds__(64 * NW) k_dslash_split(Lat g, int out_par, const DslashArgs* __restrict__ table,
                                                      DslashArgs one, int j) {
  using R = typename SP::R;
  constexpr int kSites = 64, NC = 12 / NW;
  __shared__ cx<R> part[NW][12][kSites];
  const DslashArgs* ep;
  if constexpr (BATCH)
    ep = table + blockIdx.y;
  else
    ep = &one;
  const DslashArgs& e = *ep;
  const int label = e.iter0 + j + (e.label_base ? *(const HMC_GLOBAL int*)e.label_base : 0);
  if (e.stop_at && label >= *(const HMC_GLOBAL int*)e.stop_at) return;
  alpha_prologue<NW>(e, label);
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int w = threadIdx.x >> 6;  // wave index (uniform per wave)
  const int ls = threadIdx.x & (kSites - 1);
  const int s = b * kSites + ls;
  {
    cx<R> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
    if (s < g.Vh) {
      const Site st = cb_site(g, out_par, s);
      if constexpr (NW == 4) {
        switch (w) {
          case 0: hop_dir<SP, LK, 0, DAG>(g, st, out_par, s, e.U, e.in, acc); break;
          case 1: hop_dir<SP, LK, 1, DAG>(g, st, out_par, s, e.U, e.in, acc); break;
          case 2: hop_dir<SP, LK, 2, DAG>(g, st, out_par, s, e.U, e.in, acc); break;
          default: hop_dir<SP, LK, 3, DAG>(g, st, out_par, s, e.U, e.in, acc); break;
        }
      } else if (w == 0) {
        hop_dir<SP, LK, 0, DAG>(g, st, out_par, s, e.U, e.in, acc);
        hop_dir<SP, LK, 1, DAG>(g, st, out_par, s, e.U, e.in, acc);
      } else {
        hop_dir<SP, LK, 2, DAG>(g, st, out_par, s, e.U, e.in, acc);
        hop_dir<SP, LK, 3, DAG>(g, st, out_par, s, e.U, e.in, acc);
      }
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) part[w][k][ls] = acc[k];
  }
  __syncthreads();
  // work-item (ls, w) now owns components NC w .. NC w + NC - 1 of site s
  double nrm[1] = {0.0};
  cx<R> o[NC];
  const bool active = s < g.Vh;
  if (active) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      o[c] = part[0][NC * w + c][ls];
#pragma unroll
      for (int q = 1; q < NW; ++q) o[c] = o[c] + part[q][NC * w + c][ls];
    }
    if (EPI != EPI_PLAIN) {
      const R a = (R)e.a, bb = (R)e.b;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (e.y) {
          const cx<R> y = SP::load_one(e.y, g.stride, s, NC * w + c);
          o[c] = {fma(bb, o[c].re, a * y.re), fma(bb, o[c].im, a * y.im)};
        } else {
          o[c] = bb * o[c];
        }
      }
    }
    if (EPI == EPI_CG) {
      const R al = (R)(*(const HMC_GLOBAL double*)e.alpha_in);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const cx<R> rv = SP::load_one(e.r, g.stride, s, NC * w + c);
        o[c] = {fma(-al, o[c].re, rv.re), fma(-al, o[c].im, rv.im)};
      }
    }
    if (EPI == EPI_AXPY_NORM || EPI == EPI_CG)
#pragma unroll
      for (int c = 0; c < NC; ++c) nrm[0] += (double)o[c].re * o[c].re + (double)o[c].im * o[c].im;
  }
  if constexpr (SP::kScaled) {
    // the per-site scale needs the largest |re|, |im| over all 12 components
    __shared__ float smax[NW][kSites];
    float m = 0.f;
    if (active)
#pragma unroll
      for (int c = 0; c < NC; ++c) m = fmaxf(m, fmaxf(fabsf((float)o[c].re), fabsf((float)o[c].im)));
    smax[w][ls] = m;
    __syncthreads();
    m = smax[0][ls];
#pragma unroll
    for (int q = 1; q < NW; ++q) m = fmaxf(m, smax[q][ls]);
    m = SP::live_scale(m);
    const float inv = m > 0.f ? 1.f / m : 0.f;
    if (active) {
      if (w == 0) SP::template store_scale<LK::kStream>(e.out, g.stride, s, m);
#pragma unroll
      for (int c = 0; c < NC; ++c) SP::template store_one_scaled<LK::kStream>(e.out, g.stride, s, NC * w + c, o[c], inv);
    }
  } else {
    if (active)
#pragma unroll
      for (int c = 0; c < NC; ++c) SP::template store_one<LK::kStream>(e.out, g.stride, s, NC * w + c, o[c]);
  }
  if (EPI == EPI_AXPY_NORM || EPI == EPI_CG) {
    block_sum<1, NW>(nrm);
    put_partial(e, label, b, nrm[0]);
  }
}

// Index of the neighbour of hop w (direction w / 2, forward if w is even);
// *wrap is set where the hop crosses the boundary.
__device__ __forceinline__ int hop_neighbour(const Lat& g, const Site& st, int w, bool* wrap) {
  switch (w) {
    case 0: return neighbour_lex<0, +1>(g, st, wrap) >> 1;
    case 1: return neighbour_lex<0, -1>(g, st, wrap) >> 1;
    case 2: return neighbour_lex<1, +1>(g, st, wrap) >> 1;
    case 3: return neighbour_lex<1, -1>(g, st, wrap) >> 1;
    case 4: return neighbour_lex<2, +1>(g, st, wrap) >> 1;
    case 5: return neighbour_lex<2, -1>(g, st, wrap) >> 1;
    case 6: return neighbour_lex<3, +1>(g, st, wrap) >> 1;
    default: return neighbour_lex<3, -1>(g, st, wrap) >> 1;
  }
}

// The projected spinor of hop w.
template <bool DAG, typename R>
__device__ __forceinline__ void hop_project(int w, const cx<R>* psi, cx<R>* h) {
  constexpr int SF = DAG ? +1 : -1, SB = -SF;
  switch (w) {
    case 0: spin_project<0, SF>(psi, h); break;
    case 1: spin_project<0, SB>(psi, h); break;
    case 2: spin_project<1, SF>(psi, h); break;
    case 3: spin_project<1, SB>(psi, h); break;
    case 4: spin_project<2, SF>(psi, h); break;
    case 5: spin_project<2, SB>(psi, h); break;
    case 6: spin_project<3, SF>(psi, h); break;
    default: spin_project<3, SB>(psi, h); break;
  }
}

// Hop w's half spinor uh = U h (forward) or U^dag h (backward), h the projected
// neighbour with the time boundary's sign.  The spinor's registers are free
// before the rest of the link is rebuilt.
template <class LK, bool DAG, typename R>
__device__ __forceinline__ void hop_half(const Lat& g, const void* U, int w, int lpar, int lsite, bool wrap,
                                         const cx<R>* psi, mat3<R>& u, cx<R>* uh) {
  cx<R> h[6];
  hop_project<DAG>(w, psi, h);
  if (w >= 6 && wrap)
#pragma unroll
    for (int k = 0; k < 6; ++k) h[k] = -h[k];
  LK::finish_u(U, g.stride, w >> 1, lpar, lsite, u);
  if (w & 1) {
    mdv(u, h, uh);
    mdv(u, h + 3, uh + 3);
  } else {
    mv(u, h, uh);
    mv(u, h + 3, uh + 3);
  }
}

// Adds hop (MU, SIG)'s share of spin component SPIN, colour c, to acc.
template <int MU, int SIG, int SPIN, typename R>
__device__ __forceinline__ cx<R> hop_share(cx<R> acc, const cx<R> (*h)[64], int c, int ls) {
  if (SPIN == 0) return acc + h[c][ls];
  if (SPIN == 1) return acc + h[3 + c][ls];
  const bool first = MU == 0 || MU == 1 ? SPIN == 3 : SPIN == 2;  // from h0, else from h1
  const cx<R> v = h[first ? c : 3 + c][ls];
  if (MU == 0) return acc + (SIG > 0 ? mul_mi(v) : mul_i(v));
  if (MU == 1) return (SPIN == 2) == (SIG > 0) ? acc + v : acc - v;
  if (MU == 2) return acc + ((SPIN == 2) == (SIG > 0) ? mul_mi(v) : mul_i(v));
  return SIG > 0 ? acc + v : acc - v;
}

// Component (SPIN, c) of D psi from the eight parked half spinors: one after the
// other, as the one-site kernel adds them, or (PAIRS) direction by direction, as
// the direction split does.
template <bool DAG, bool PAIRS, int SPIN, typename R>
__device__ __forceinline__ cx<R> hops_combine(const cx<R> (*half)[6][64], int c, int ls) {
  constexpr int SF = DAG ? +1 : -1, SB = -SF;
  const cx<R> zero = {R(0), R(0)};
  cx<R> t, p;
  t = hop_share<0, SF, SPIN>(zero, half[0], c, ls);
  t = hop_share<0, SB, SPIN>(t, half[1], c, ls);
  p = hop_share<1, SF, SPIN>(PAIRS ? zero : t, half[2], c, ls);
  p = hop_share<1, SB, SPIN>(p, half[3], c, ls);
  t = PAIRS ? t + p : p;
  p = hop_share<2, SF, SPIN>(PAIRS ? zero : t, half[4], c, ls);
  p = hop_share<2, SB, SPIN>(p, half[5], c, ls);
  t = PAIRS ? t + p : p;
  p = hop_share<3, SF, SPIN>(PAIRS ? zero : t, half[6], c, ls);
  p = hop_share<3, SB, SPIN>(p, half[7], c, ls);
  return PAIRS ? t + p : p;
}

// The sum's own rounding counts in FP32 storage, which takes the pairs (error of
// Mhat at 18x10x14x26 4.94e-8 one after the other, 4.83e-8 in pairs; 20^3x40 35.9
// and 36.1 us).  The narrower storages round far more than it does (FP16 2.6e-4),
// and FP64 errs less in sequence (9.36e-17 against 9.47e-17).
template <class SP, bool DAG, typename R>
__device__ __forceinline__ cx<R> hops_component(const cx<R> (*half)[6][64], int spin, int c, int ls) {
  constexpr bool kPairs = std::is_same_v<SP, SpF32>;
  switch (spin) {
    case 0: return hops_combine<DAG, kPairs, 0>(half, c, ls);
    case 1: return hops_combine<DAG, kPairs, 1>(half, c, ls);
    case 2: return hops_combine<DAG, kPairs, 2>(half, c, ls);
    default: return hops_combine<DAG, kPairs, 3>(half, c, ls);
  }
}

// Four-way direction split, one wavefront per hop: a block of eight
// wavefronts covers 64 sites; wavefront 2 mu (2 mu + 1) loads the forward
// (backward) neighbour along mu, and parks the six components of the
// projected, link-multiplied spinor in LDS (six, not the twelve of a full
// partial sum: 48 KB in FP64).  After one barrier the wavefronts rebuild and
// add the eight hops, two or one of the twelve components per work-item.
//
// What bounds a hop on a small lattice is the latency of its loads (the
// one-site kernel waits for eight rounds of them, one after the other); here
// every load of a site is in flight at once, 98 VGPRs per work-item in FP64.
// Mhat (two hops), against the same split with one wavefront per direction
// and two rounds of loads: FP64 8^4 9.9 -> 8.9 us (one-site 16.8), 12^3x24
// 14.9 -> 13.3 (21.6), 16^3x32 32.2 -> 29.9 (34.6; two-way 31.1); FP32
// 16^3x32 19.6 -> 17.5, FP16 14.9 -> 14.1, BF16 13.7 -> 12.7; FP64 24^3x48
// with streaming 161 -> 158.
constexpr int kHopThreads = 8 * 64;
constexpr int kAlphaAhead = 2;  // partial sums per work-item requested ahead (1024 in all, a 2^16-site launch's)

// Arguments of one launch.  The host writes a kernel's arguments on the
// caller's thread: 2.9 us a launch with at most 112 bytes of them and no use of
// the grid's extent (which adds 256 bytes), 3.7 us with more, and the launches
// are what a solve on a small lattice waits for (8^4, FP32: 650 of them).  So a
// single entry travels without what the kernel can derive (number of sites and
// blocks, the stop's neighbour in the solver state) or its epilogue does not
// read; every addend enters with the factor 1, and EPI_CG works in place.
template <int EPI>
struct HopEpilogue {  // EPI_PLAIN
  const double *alpha_pp[2], *alpha_den;
  double* alpha_out;
  int alpha_n_pp, alpha_n_den;
  HopEpilogue(const DslashArgs& d)
      : alpha_pp{d.alpha_pp[0], d.alpha_pp[1]}, alpha_den(d.alpha_den), alpha_out(d.alpha_out),
        alpha_n_pp(d.alpha_n_pp), alpha_n_den(d.alpha_n_den) {}
  __device__ void expand(DslashArgs& d) const {
    d.alpha_pp[0] = alpha_pp[0], d.alpha_pp[1] = alpha_pp[1], d.alpha_den = alpha_den, d.alpha_out = alpha_out;
    d.alpha_n_pp = alpha_n_pp, d.alpha_n_den = alpha_n_den;
  }
};
template <>
struct HopEpilogue<EPI_AXPY> {
  const void* y;
  double b;
  HopEpilogue(const DslashArgs& d) : y(d.y), b(d.b) {}
  __device__ void expand(DslashArgs& d) const { d.y = y, d.a = 1.0, d.b = b; }
};
template <>
struct HopEpilogue<EPI_AXPY_NORM> {
  const void* y;
  double b;
  double *partial, *partial_pp[2];
  HopEpilogue(const DslashArgs& d)
      : y(d.y), b(d.b), partial(d.partial), partial_pp{d.partial_pp[0], d.partial_pp[1]} {}
  __device__ void expand(DslashArgs& d) const {
    d.y = y, d.a = 1.0, d.b = b, d.partial = partial, d.partial_pp[0] = partial_pp[0], d.partial_pp[1] = partial_pp[1];
  }
};
template <>
struct HopEpilogue<EPI_CG> {
  const void* y;
  double b;
  double* partial_pp[2];
  const double* alpha_in;
  HopEpilogue(const DslashArgs& d)
      : y(d.y), b(d.b), partial_pp{d.partial_pp[0], d.partial_pp[1]}, alpha_in(d.alpha_in) {}
  __device__ void expand(DslashArgs& d) const {
    d.y = y, d.a = 1.0, d.b = b, d.partial = nullptr, d.partial_pp[0] = partial_pp[0], d.partial_pp[1] = partial_pp[1];
    d.r = d.out, d.alpha_in = alpha_in;
  }
};

template <int EPI>
struct HopOne {
  int L[4];
  unsigned mul[3];
  unsigned packed;  // the three division shifts and the output parity, a byte each
  const void *U, *in;
  void* out;
  const int* stop_at;
  int base;   // the label base is this far behind *stop_at (0: none)
  int label;  // without the base
  HopEpilogue<EPI> x;

  HopOne(const Lat& g, int out_par, const DslashArgs& d, int j)
      : L{g.L[0], g.L[1], g.L[2], g.L[3]}, mul{g.mul[0], g.mul[1], g.mul[2]},
        packed(g.shift[0] | g.shift[1] << 8 | g.shift[2] << 16 | (unsigned)out_par << 24), U(d.U), in(d.in), out(d.out),
        stop_at(d.stop_at), base(d.label_base ? (int)(d.label_base - d.stop_at) : 0), label(d.iter0 + j), x(d) {}
  // What the launch relies on.
  static bool holds(const Lat& g, const DslashArgs& d) {
    const long long V = (long long)g.L[0] * g.L[1] * g.L[2] * g.L[3];
    return g.stride == g.Vh && 2LL * g.Vh == V && (!d.y || d.a == 1.0) && (!d.label_base || d.stop_at) &&
           (EPI != EPI_CG || (d.r == d.out && !d.partial));
  }
};
static_assert(sizeof(HopOne<EPI_PLAIN>) <= 112 && sizeof(HopOne<EPI_AXPY_NORM>) <= 112 && sizeof(HopOne<EPI_CG>) <= 112,
              "launch arguments");
struct HopBatch {  // blockIdx.y selects an entry of `table`
  Lat g;
  int out_par;
  const DslashArgs* table;
  int j;
  HopBatch(const Lat& lat, int par, const DslashArgs* t, int jj) : g(lat), out_par(par), table(t), j(jj) {}
};

template <class SP, class LK, bool DAG, int EPI, bool BATCH>
__global__ void __launch_bounds__(kHopThreads) k_dslash_hops(std::conditional_t<BATCH, HopBatch, HopOne<EPI>> h) {
  using R = typename SP::R;
  constexpr int kSites = 64;
  __shared__ cx<R> half[8][6][kSites];
  Lat g;
  DslashArgs one;
  const DslashArgs* ep = &one;
  int out_par, label;
  if constexpr (BATCH) {
    g = h.g;
    ep = h.table + blockIdx.y;
    out_par = h.out_par;
    label = ep->iter0 + h.j;
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) g.L[k] = h.L[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) g.mul[k] = h.mul[k], g.shift[k] = h.packed >> (8 * k) & 255;
    g.Vh = g.stride = (h.L[0] >> 1) * h.L[1] * h.L[2] * h.L[3];
    out_par = h.packed >> 24;
    label = h.label;
    one.U = h.U, one.in = h.in, one.out = h.out, one.stop_at = h.stop_at;
    one.label_base = h.base ? h.stop_at + h.base : nullptr;
    h.x.expand(one);
  }
  const DslashArgs& e = *ep;
  // Everything the hop reads is requested before anything is waited for: the
  // solver control, the step length, block 0's partial sums, the epilogue's
  // inputs, the spinor and the link.  A launch past the stop then reads them in
  // vain, so launches of which many are past it look at the control first: the
  // low-precision iterations queued up to the next reliable update, and the
  // gated launches of the update itself (which have no label base).
  if (e.label_base) label += *(const HMC_GLOBAL int*)e.label_base;
  int stop = INT_MAX;
  if (sizeof(R) == 4 || !e.label_base) {
    if (e.stop_at && label >= *(const HMC_GLOBAL int*)e.stop_at) return;
    asm volatile("" ::: "memory");  // (or the compiler waits for the control on both paths)
  } else if (e.stop_at) {
    stop = *(const HMC_GLOBAL int*)e.stop_at;
  }
  const double alpha = EPI == EPI_CG ? *(const HMC_GLOBAL double*)e.alpha_in : 0.0;
  const bool sums = EPI == EPI_PLAIN && e.alpha_out && blockIdx.x == 0;
  double ta[kAlphaAhead], tb[kAlphaAhead];
  if (sums) {
    const double* pp = label & 1 ? e.alpha_pp[1] : e.alpha_pp[0];
#pragma unroll
    for (int u = 0; u < kAlphaAhead; ++u) {
      const int i = threadIdx.x + u * kHopThreads;
      ta[u] = i < e.alpha_n_pp ? pp[i] : 0.0;
      tb[u] = i < e.alpha_n_den ? e.alpha_den[i] : 0.0;
    }
  }
  const int b = xcd_remap(blockIdx.x, (g.Vh + kSites - 1) / kSites);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ls = threadIdx.x & (kSites - 1);
  const int s = b * kSites + ls;
  const bool active = s < g.Vh;
  // wavefront w combines spin w % 4, colours 0 and 1 (w < 4) or 2 (w >= 4)
  const int spin = w & 3, c0 = w < 4 ? 0 : 2, nc = w < 4 ? 2 : 1;
  const int lmu = w >> 1, lpar = out_par ^ (w & 1);
  int lsite = s;
  bool wrap = false;
  cx<R> yv[2], rv[2], psi[12];
  mat3<R> u;
  if (active) {
    if (EPI != EPI_PLAIN && e.y)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (q < nc) yv[q] = SP::load_one(e.y, g.stride, s, 3 * spin + c0 + q);
    if (EPI == EPI_CG)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (q < nc) rv[q] = SP::load_one(e.r, g.stride, s, 3 * spin + c0 + q);
    const Site st = cb_site(g, out_par, s);
    const int sn = hop_neighbour(g, st, w, &wrap);
    if (w & 1) lsite = sn;  // a backward hop's link belongs to the neighbour
    SP::load(e.in, g.stride, sn, psi);
    LK::raw_u(e.U, g.stride, lmu, lpar, lsite, u);
  }
  asm volatile("" ::: "memory");  // the loads above stay above
  if (label >= stop) return;
  if (active) {
    cx<R> uh[6];
    hop_half<LK, DAG>(g, e.U, w, lpar, lsite, wrap, psi, u, uh);
#pragma unroll
    for (int k = 0; k < 6; ++k) half[w][k][ls] = uh[k];
  }
  __syncthreads();
  double nrm[1] = {0.0};
  cx<R> o[2];
  if (active) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q >= nc) break;
      const int c = c0 + q;
      o[q] = hops_component<SP, DAG>(half, spin, c, ls);
      if (EPI != EPI_PLAIN) {
        const R a = (R)e.a, bb = (R)e.b;
        if (e.y)
          o[q] = {fma(bb, o[q].re, a * yv[q].re), fma(bb, o[q].im, a * yv[q].im)};
        else
          o[q] = bb * o[q];
      }
      if (EPI == EPI_CG) {
        const R al = (R)alpha;
        o[q] = {fma(-al, o[q].re, rv[q].re), fma(-al, o[q].im, rv[q].im)};
      }
      if (EPI == EPI_AXPY_NORM || EPI == EPI_CG)
        nrm[0] += (double)o[q].re * o[q].re + (double)o[q].im * o[q].im;
    }
  }
  if constexpr (SP::kScaled) {
    __shared__ float smax[8][kSites];
    float m = 0.f;
    if (active)
      for (int q = 0; q < 2; ++q)
        if (q < nc) m = fmaxf(m, fmaxf(fabsf((float)o[q].re), fabsf((float)o[q].im)));
    smax[w][ls] = m;
    __syncthreads();
    m = smax[0][ls];
#pragma unroll
    for (int q = 1; q < 8; ++q) m = fmaxf(m, smax[q][ls]);
    m = SP::live_scale(m);
    const float inv = m > 0.f ? 1.f / m : 0.f;
    if (active) {
      if (w == 7) SP::template store_scale<LK::kStream>(e.out, g.stride, s, m);
      for (int q = 0; q < 2; ++q)
        if (q < nc) SP::template store_one_scaled<LK::kStream>(e.out, g.stride, s, 3 * spin + c0 + q, o[q], inv);
    }
  } else {
    if (active)
      for (int q = 0; q < 2; ++q)
        if (q < nc) SP::template store_one<LK::kStream>(e.out, g.stride, s, 3 * spin + c0 + q, o[q]);
  }
  if (EPI == EPI_AXPY_NORM || EPI == EPI_CG) {
    block_sum<1, 8>(nrm);
    put_partial(e, label, b, nrm[0]);
  }
  if (sums) {  // the step length for the next hop, after this one's stores
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < kAlphaAhead; ++q) v[0] += ta[q], v[1] += tb[q];
    const double* pp = label & 1 ? e.alpha_pp[1] : e.alpha_pp[0];
    for (int i = threadIdx.x + kAlphaAhead * kHopThreads; i < e.alpha_n_pp; i += kHopThreads) v[0] += pp[i];
    for (int i = threadIdx.x + kAlphaAhead * kHopThreads; i < e.alpha_n_den; i += kHopThreads) v[1] += e.alpha_den[i];
    block_sum<2, 8>(v);
    if (threadIdx.x == 0) *(HMC_GLOBAL double*)e.alpha_out = v[0] / v[1];
  }
}

// Mhat on a lattice of at most kSmallSites half-lattice sites in one launch of
// one block: sixteen wavefronts, one hop of 64 sites each as above, take the
// odd sites and then, from LDS, the even ones (the odd field stays in the
// arithmetic's precision).  The second hop's links and the addend are
// requested before the first one's barriers (with its own loads they spill).  At this size a hop is one round of loads and its
// launch costs more than it does: 4^4, FP64, 10.2 us in two launches, 7.1 in
// one.  Twice the sites would need two steps per hop (4^3x8 12.9 us against
// 10.0 in two launches).
constexpr int kSmallThreads = 16 * 64;
static_assert(kSmallSites == 2 * 64, "two groups of 64 sites per block");

template <class SP, class LK, bool DAG>
__global__ void __launch_bounds__(kSmallThreads) k_mhat_small(Lat g, const void* U, const void* in, void* out,
                                                              double b) {
  using R = typename SP::R;
  __shared__ cx<R> half[2][8][6][64];
  __shared__ cx<R> odd[12][kSmallSites];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = wave & 7, pair = wave >> 3;
  const int spin = w & 3, c0 = w < 4 ? 0 : 2, nc = w < 4 ? 2 : 1;
  const int s = 64 * pair + lane, back = w & 1;
  const bool active = s < g.Vh;
  bool wrap_o = false, wrap_e = false;
  int sn_o = 0, sn_e = 0;
  cx<R> psi[12], uh[6], y[2], o[2];
  mat3<R> u;
  if (active) {
    sn_o = hop_neighbour(g, cb_site(g, 1, s), w, &wrap_o);
    sn_e = hop_neighbour(g, cb_site(g, 0, s), w, &wrap_e);
    SP::load(in, g.stride, sn_o, psi);
    LK::raw_u(U, g.stride, w >> 1, 1 ^ back, back ? sn_o : s, u);
    hop_half<LK, DAG>(g, U, w, 1 ^ back, back ? sn_o : s, wrap_o, psi, u, uh);
#pragma unroll
    for (int k = 0; k < 6; ++k) half[pair][w][k][lane] = uh[k];
    LK::raw_u(U, g.stride, w >> 1, back, back ? sn_e : s, u);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (q < nc) y[q] = SP::load_one(in, g.stride, s, 3 * spin + c0 + q);
  }
  __syncthreads();
  if (active)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (q < nc) odd[3 * spin + c0 + q][s] = hops_component<SP, DAG>(half[pair], spin, c0 + q, lane);
  __syncthreads();
  if (active) {
#pragma unroll
    for (int k = 0; k < 12; ++k) psi[k] = odd[k][sn_e];
    hop_half<LK, DAG>(g, U, w, back, back ? sn_e : s, wrap_e, psi, u, uh);
#pragma unroll
    for (int k = 0; k < 6; ++k) half[pair][w][k][lane] = uh[k];
  }
  __syncthreads();
  if (active)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q >= nc) break;
      const R bb = (R)b;
      o[q] = hops_component<SP, DAG>(half[pair], spin, c0 + q, lane);
      o[q] = {fma(bb, o[q].re, y[q].re), fma(bb, o[q].im, y[q].im)};
      if constexpr (!SP::kScaled) SP::template store_one<false>(out, g.stride, s, 3 * spin + c0 + q, o[q]);
    }
  if constexpr (SP::kScaled) {  // the site's scale: its largest component
    __shared__ float smax[16][64];
    float m = 0.f;
    if (active)
      for (int q = 0; q < 2; ++q)
        if (q < nc) m = fmaxf(m, fmaxf(fabsf((float)o[q].re), fabsf((float)o[q].im)));
    smax[wave][lane] = m;
    __syncthreads();
    m = smax[8 * pair][lane];
#pragma unroll
    for (int q = 1; q < 8; ++q) m = fmaxf(m, smax[8 * pair + q][lane]);
    m = SP::live_scale(m);
    const float inv = m > 0.f ? 1.f / m : 0.f;
    if (active) {
      if (w == 7) SP::template store_scale<false>(out, g.stride, s, m);
      for (int q = 0; q < 2; ++q)
        if (q < nc) SP::template store_one_scaled<false>(out, g.stride, s, 3 * spin + c0 + q, o[q], inv);
    }
  }
}

// out = in + b D_eo D_oe in (dagger: of D^dag) on at most kSmallSites sites.
template <class SP, class LK>
hipError_t launch_mhat_small_links(hmc_prec prec, int dagger, const LatArg& g, const void* U, const void* in, void* out,
                                   double b, bool su3, hipStream_t st) {
  if (g.Vh > kSmallSites) return hipErrorInvalidValue;
  const int form = link_form_for(su3, dslash_link_form(g, prec));
  const int lb = form == LINK_ROWCOL ? LkRowCol<LK>::kBytes : form == LINK_ROWS2 ? LkRows2<LK>::kBytes : LK::kBytes;
  // the links of the two hops, the input as spinor and as addend, the output
  const KernelEvents ev = timing_kernel_events(TK_DSLASH, (16.0 * LK::kBytes + 3 * SP::kBytes) * g.Vh,
                                               (16.0 * lb + 3 * SP::kBytes) * g.Vh);
  const Lat lat = to_lat(g);
#define HMC_SMALL(LKF)                                                                                              \
  do {                                                                                                              \
    if (dagger)                                                                                                     \
      hipExtLaunchKernelGGL((k_mhat_small<SP, LKF, true>), dim3(1), dim3(kSmallThreads), 0, st, ev.start, ev.stop,  \
                            0, lat, U, in, out, b);                                                                 \
    else                                                                                                            \
      hipExtLaunchKernelGGL((k_mhat_small<SP, LKF, false>), dim3(1), dim3(kSmallThreads), 0, st, ev.start, ev.stop, \
                            0, lat, U, in, out, b);                                                                 \
  } while (0)
  if (form == LINK_ROWCOL)
    HMC_SMALL(LkRowCol<LK>);
  else if (form == LINK_ROWS2)
    HMC_SMALL(LkRows2<LK>);
  else
    HMC_SMALL(LK);
#undef HMC_SMALL
  return hipGetLastError();
}

// Batched launches of the hop-per-wavefront shape split by direction instead from
// kBatchSites on: what they wait for there is their bytes, which four wavefronts
// of two hops each request with half the LDS traffic and barriers a wavefront.
// Requests in the service, hop / direction per wavefront, ms: FP32 12^3x24 one
// 2.78 / 2.80, four 5.66 / 5.43; 14^3x28 3.36 / 3.40, 8.27 / 7.85; 16^3x32 3.99 /
// 3.96, 11.8 / 11.1, sixteen 57.8 / 51.9; 24^3x48 14.7 / 13.8, 63.3 / 56.6; FP64
// 12^3x24 2.41 / 2.57, 6.47 / 6.15; 14^3x28 3.56 / 3.39, 10.6 / 9.9; 16^3x32
// sixteen 89.0 / 76.6.
template <class SP, class LK>
static hipError_t launch_typed(hmc_prec prec, int dagger, int epi, const LatArg& ga, int out_par,
                               const DslashArgs* table, int nbatch, const DslashArgs& one, hipStream_t st, int j,
                               KernelEvents ev) {
  Lat g = to_lat(ga);
  const int shape = one.shape ? one.shape : dslash_run_shape(ga, prec);
  const int order = shape == 1 ? dslash_tiled_order(ga, prec) : 0;
  if (order) {
    g.tiled = 1;
    g.plane = ga.L[0] * ga.L[1] / 2;
    g.slice = g.plane * ga.L[2];
    g.tile_r = g.plane % 64 == 0 ? g.plane / 64 : 0;
    g.tile_t = ga.L[3] / 8;
    g.tile_y = order == 1 ? g.tile_r : order;  // 0: chunks of the t-slices
  }
  const dim3 grid(dslash_shape_blocks(ga.Vh, shape), nbatch);
  const bool four = table && shape == 4 && ga.Vh >= kBatchSites;
  const dim3 block(four ? 256 : shape == 4 ? kHopThreads : shape == 2 ? 128 : kBlock);
  // The tiled order may reserve LDS it does not use: 54,000 bytes per block
  // leave room for two blocks per CU (2 wavefronts per SIMD), so an XCD's
  // wavefronts in flight span a few (z, t) rows instead of dozens and the
  // neighbours they share are still in its L2 (measured at 48^3x96 with
  // whole z-planes: FP64 1.36 ms without the cap, 1.24 ms with it, 1.27-1.31
  // ms for the linear order; with y-blocks the FP32 and FP16 kernels run
  // faster without it).
  const size_t lds_cap = g.tiled && dslash_tiled_occupancy(ga, prec) == 2 ? 54000 : 0;
#define HMC_LAUNCH(KERNEL) \
  hipExtLaunchKernelGGL(KERNEL, grid, block, lds_cap, st, ev.start, ev.stop, 0, g, out_par, table, one, j)
#define HMC_HOPS(D, E, B)                                                                                         \
  do {                                                                                                            \
    if constexpr (B) {                                                                                            \
      hipExtLaunchKernelGGL((k_dslash_hops<SP, LK, D, E, B>), grid, block, 0, st, ev.start, ev.stop, 0,           \
                            HopBatch(g, out_par, table, j));                                                      \
    } else {                                                                                                      \
      if (!HopOne<E>::holds(g, one)) return hipErrorInvalidValue;                                                 \
      hipExtLaunchKernelGGL((k_dslash_hops<SP, LK, D, E, B>), grid, block, 0, st, ev.start, ev.stop, 0,           \
                            HopOne<E>(g, out_par, one, j));                                                       \
    }                                                                                                             \
  } while (0)
#define HMC_DS_B(D, E, B)                                       \
  do {                                                          \
    if (B && four) /* (four wavefronts: in batches only) */     \
      HMC_LAUNCH((k_dslash_split<SP, LK, D, E, B, B ? 4 : 2>)); \
    else if (shape == 4)                                        \
      HMC_HOPS(D, E, B);                                        \
    else if (shape == 2)                                        \
      HMC_LAUNCH((k_dslash_split<SP, LK, D, E, B, 2>));         \
    else                                                        \
      HMC_LAUNCH((k_dslash<SP, LK, D, E, B>));                  \
  } while (0)
#define HMC_DS(D, E)            \
  do {                          \
    if (table)                  \
      HMC_DS_B(D, E, true);     \
    else                        \
      HMC_DS_B(D, E, false);    \
  } while (0)
  if (epi == EPI_CG) {  // last hop of a CG iteration: dagger, one solve
    if (table || !dagger) return hipErrorInvalidValue;
    HMC_DS_B(true, EPI_CG, false);
    return hipGetLastError();
  }
  if (dagger) {
    if (epi == EPI_PLAIN) HMC_DS(true, EPI_PLAIN);
    else if (epi == EPI_AXPY) HMC_DS(true, EPI_AXPY);
    else HMC_DS(true, EPI_AXPY_NORM);
  } else {
    if (epi == EPI_PLAIN) HMC_DS(false, EPI_PLAIN);
    else if (epi == EPI_AXPY) HMC_DS(false, EPI_AXPY);
    else HMC_DS(false, EPI_AXPY_NORM);
  }
#undef HMC_DS
#undef HMC_DS_B
#undef HMC_HOPS
#undef HMC_LAUNCH
  return hipGetLastError();
}

// Link form (SU(3) fields: the tuned compact form and streaming choice,
// else all entries), then shape and epilogue.
template <class SP, class LK>
hipError_t launch_links(hmc_prec prec, int dagger, int epi, const LatArg& g, int out_par, const DslashArgs* table,
                        int nbatch, const DslashArgs& one, hipStream_t st, int j) {
  const int form = link_form_for(one.su3, dslash_link_form(g, prec));
  const bool stream = form != LINK_FULL && dslash_link_stream(g, prec);
  const int link_bytes = form == LINK_ROWCOL ? LkRowCol<LK>::kBytes : form == LINK_ROWS2 ? LkRows2<LK>::kBytes
                                                                                          : LK::kBytes;
  // bytes per site: 8 links + 1 input + 1 output spinor (+1 for y, +1 more
  // for the residual read by the CG epilogue); algorithmic with whole links,
  // moved with the stored reals of the link form
  const double spinor_bytes = 2 * SP::kBytes + (epi ? SP::kBytes : 0) + (epi == EPI_CG ? SP::kBytes : 0);
  const double alg = (8.0 * LK::kBytes + spinor_bytes) * g.Vh * nbatch;
  const double moved = (8.0 * link_bytes + spinor_bytes) * g.Vh * nbatch;
  const KernelEvents ev = timing_kernel_events(TK_DSLASH, alg, moved);
  if (form == LINK_ROWCOL) {
    if (stream)
      return launch_typed<SP, LkRowCol<LK, true>>(prec, dagger, epi, g, out_par, table, nbatch, one, st, j, ev);
    return launch_typed<SP, LkRowCol<LK>>(prec, dagger, epi, g, out_par, table, nbatch, one, st, j, ev);
  }
  if (form == LINK_ROWS2) {
    if (stream)
      return launch_typed<SP, LkRows2<LK, true>>(prec, dagger, epi, g, out_par, table, nbatch, one, st, j, ev);
    return launch_typed<SP, LkRows2<LK>>(prec, dagger, epi, g, out_par, table, nbatch, one, st, j, ev);
  }
  return launch_typed<SP, LK>(prec, dagger, epi, g, out_par, table, nbatch, one, st, j, ev);
}

}  // namespace hmc
