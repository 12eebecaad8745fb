// Global sums (the QDP++ sum / innerProduct / sumMulti functions named in
// the paper's QDP-JIT feature list, Sec. 1) and the fused vector updates
// of the Krylov solvers.
//
// Every reduction is deterministic and independent of other work in the
// same launch: a work-item accumulates its sites in a fixed grid-stride
// order, a wave64 butterfly and a fixed wave order give one partial per
// block, and consumers sum the partials in index order.  The solver
// kernels re-sum the partials they need in every block (the same bits in
// every block), which removes the separate finalisation launches from the
// iteration.
#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace hmc {


// ------------------------------------------------------------- sums

// Longest run of inner iterations between two device-driven reliable updates.
constexpr int kMaxInner = 48;

// The kernels taking `gate` do nothing while *gate == 0 (gate may be null).
__device__ __forceinline__ bool gate_closed(const int* gate) { return gate && *gate == 0; }

template <class SP>
__global__ void __launch_bounds__(kBlock) k_norm2_partials(Lat g, const void* x, double* part, const int* gate) {
  if (gate_closed(gate)) return;
  double v[1] = {0.0};
  for (int s = blockIdx.x * kBlock + threadIdx.x; s < g.Vh; s += gridDim.x * kBlock) {
    cx<typename SP::R> a[12];
    SP::load(x, g.stride, s, a);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[0] += (double)a[k].re * a[k].re + (double)a[k].im * a[k].im;
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

__global__ void __launch_bounds__(kBlock) k_inner_partials(Lat g, const double2* a, const double2* b, double* part) {
  double v[2] = {0.0, 0.0};
  const size_t n = (size_t)12 * g.stride;
  for (size_t j = (size_t)blockIdx.x * kBlock + threadIdx.x; j < n; j += (size_t)gridDim.x * kBlock) {
    if ((int)(j % g.stride) >= g.Vh) continue;
    double2 x = a[j], y = b[j];
    v[0] += x.x * y.x + x.y * y.y;  // Re conj(x) y
    v[1] += x.x * y.y - x.y * y.x;  // Im conj(x) y
  }
  block_sum<2>(v);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = v[0];
    part[gridDim.x + blockIdx.x] = v[1];
  }
}

__global__ void __launch_bounds__(kBlock) k_finalize(const double* part, int n, int nvals, double* out, double scale,
                                                     int accumulate, const int* gate) {
  if (gate_closed(gate)) return;
  for (int v = 0; v < nvals; ++v) {
    double s = sum_partials(part + (size_t)v * n, n);
    if (threadIdx.x == 0) out[v] = (accumulate ? out[v] : 0.0) + scale * s;
  }
}

// sumMulti: per-wavefront histograms of |x|^2 over the subsets, in LDS.  A
// wavefront takes the subset ids among its 64 sites one after the other (most
// often one or two: time slices and blocks are contiguous in the site order),
// adds that subset's values up in a butterfly and one lane adds the sum to the
// wavefront's bin, so every bin is summed in a fixed order: no atomics.  One
// work-item adding the block's 256 values in turn took 41 us at 20^2x22x44
// (44 slices; 74 MB), this 15 us.
constexpr int kMaxSub = 1024;

__global__ void __launch_bounds__(kBlock) k_sum_multi_partials(Lat g, const void* x, const int* subset, int nsub,
                                                               double* part) {
  constexpr int W = kBlock / 64;
  extern __shared__ double bins[];  // [W][nsub]
  for (int k = threadIdx.x; k < W * nsub; k += kBlock) bins[k] = 0.0;
  __syncthreads();
  const int half = blockIdx.y, lane = threadIdx.x & 63;
  double* mine = bins + (threadIdx.x >> 6) * nsub;
  const char* xh = (const char*)x + (size_t)half * 12 * g.stride * sizeof(v2d);
  const int* sh = subset + (size_t)half * g.Vh;
  // (the bound is rounded up to whole wavefronts: every lane takes part in the butterflies)
  for (int s = blockIdx.x * kBlock + threadIdx.x; s - lane < g.Vh; s += gridDim.x * kBlock) {
    double v = 0.0;
    int sub = -1;
    if (s < g.Vh) {
      cx<double> a[12];
      SpF64::load(xh, g.stride, s, a);
#pragma unroll
      for (int k = 0; k < 12; ++k) v += a[k].re * a[k].re + a[k].im * a[k].im;
      sub = sh[s];
    }
    // ids outside [0, nsub) are ignored
    unsigned long long left = __ballot(sub >= 0 && sub < nsub);
    while (left) {
      const int id = __shfl(sub, __ffsll((long long)left) - 1, 64);
      const bool in = sub == id;
      const double t = wave_sum(in ? v : 0.0);
      if (lane == 0) mine[id] += t;
      left &= ~__ballot(in);
    }
  }
  __syncthreads();
  // one row of block sums per subset, so that the final sum reads them in order
  const int nrows = gridDim.x * gridDim.y, row = half * gridDim.x + blockIdx.x;
  for (int k = threadIdx.x; k < nsub; k += kBlock) {
    double t = bins[k];
#pragma unroll
    for (int w = 1; w < W; ++w) t += bins[w * nsub + k];
    part[(size_t)k * nrows + row] = t;
  }
}

// One block per subset (one lane per subset, adding up to 2048 block sums in
// turn, took 361 us for 44 subsets; this 4 us).
__global__ void __launch_bounds__(kBlock) k_sum_multi_final(const double* part, int nrows, double* out) {
  const double s = sum_partials(part + (size_t)blockIdx.x * nrows, nrows);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// ------------------------------------------------------- element-wise

// STREAM triad a = b + s c over n2 double2 elements, four per work-item
// (all loads before the stores), optionally with non-temporal hints: the
// attainable streaming rate of this chip for the access pattern of the
// field kernels (16-byte lanes, contiguous waves).
template <bool NT>
__global__ void __launch_bounds__(kBlock) k_triad(void* a, const void* b, const void* c, double sc, size_t n2) {
  constexpr int U = 4;
  const size_t step = (size_t)gridDim.x * kBlock;
  for (size_t j0 = (size_t)blockIdx.x * kBlock + threadIdx.x; j0 < n2; j0 += step * U) {
    v2d x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t j = j0 + u * step;
      if (j < n2) {
        x[u] = gld_link<v2d, NT>((const char*)b + j * 16, 0);
        y[u] = gld_link<v2d, NT>((const char*)c + j * 16, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t j = j0 + u * step;
      if (j < n2) gput<NT>((char*)a + j * 16, 0, v2d{fma(sc, y[u].x, x[u].x), fma(sc, y[u].y, x[u].y)});
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_xmy_norm(Lat g, const double2* b, const double2* q, double2* r,
                                                    double* part, const int* gate) {
  if (gate_closed(gate)) return;
  double v[1] = {0.0};
  for (int s = blockIdx.x * kBlock + threadIdx.x; s < g.Vh; s += gridDim.x * kBlock) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      size_t j = (size_t)k * g.stride + s;
      double2 d = make_double2(b[j].x - q[j].x, b[j].y - q[j].y);
      r[j] = d;
      v[0] += d.x * d.x + d.y * d.y;
    }
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

__global__ void k_zero(uint4* p, size_t n16, unsigned char* tail, size_t ntail) {
  for (size_t j = (size_t)blockIdx.x * kBlock + threadIdx.x; j < n16; j += (size_t)gridDim.x * kBlock)
    p[j] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

__global__ void k_copy(uint4* d, const uint4* s, size_t n16, unsigned char* dt, const unsigned char* st,
                       size_t ntail, const int* gate) {
  if (gate && *gate == 0) return;
  for (size_t j = (size_t)blockIdx.x * kBlock + threadIdx.x; j < n16; j += (size_t)gridDim.x * kBlock) d[j] = s[j];
  if (blockIdx.x == 0 && threadIdx.x < ntail) dt[threadIdx.x] = st[threadIdx.x];
}

// ------------------------------------------------------------ solvers

// x = 0, r = p = b, partials of |b|^2 (FP64 vectors).
__global__ void __launch_bounds__(kBlock) k_cg_init(Lat g, const double2* b, double2* x, double2* r, double2* p,
                                                    double* part) {
  double v[1] = {0.0};
  for (int s = blockIdx.x * kBlock + threadIdx.x; s < g.Vh; s += gridDim.x * kBlock) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      size_t j = (size_t)k * g.stride + s;
      double2 a = b[j];
      x[j] = make_double2(0.0, 0.0);
      r[j] = a;
      p[j] = a;
      v[0] += a.x * a.x + a.y * a.y;
    }
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

// The arguments of this block's solve: entry blockIdx.y of a batch table,
// or the single entry passed by value.  Chosen at compile time, so the
// by-value entry is read in place from the kernel arguments (a run-time
// choice copies the struct to per-lane scratch memory).
// Arguments of the two launches below: single entries in at most 112 bytes and
// the block count inside, for which a launch costs the host 2.9 us instead of
// 3.7 (as the Dslash's).
struct CgOne {
  int Vh, label;  // (label without the base)
  void *x, *p, *r;
  const void* qs;  // q (update) or s (p-update)
  double* pp;
  int pp1;    // pp[1] - pp[0]
  int flags;  // blocks per XCD, mixed, cgls
  double *pq, *pr;
  int n_pp, n_pq, n_pr, max_iters;
  SolverState* state;
  double delta2;
  void* x64;

  CgOne(int Vh_, int blocks, const CgArgs& a, const void* qs_, int j)
      : Vh(Vh_), label(a.iter0 + j), x(a.x), p(a.p), r(a.r), qs(qs_), pp(a.pp[0]), pp1((int)(a.pp[1] - a.pp[0])),
        flags((blocks >> 3) << 2 | (a.mixed ? 2 : 0) | (a.cgls ? 1 : 0)), pq(a.pq), pr(a.pr), n_pp(a.n_pp),
        n_pq(a.n_pq), n_pr(a.n_pr), max_iters(a.max_iters), state(a.state), delta2(a.delta2), x64(a.x64) {}
  // What the launch relies on: both partial buffers are cut from one.
  static bool holds(const CgArgs& a) {
    const long long d = a.pp[1] - a.pp[0];
    return d == (int)d;
  }
};
static_assert(sizeof(CgOne) <= 112, "launch arguments");
struct CgBatch {  // blockIdx.y selects an entry of `table`
  int Vh, blocks;
  const CgArgs* table;
  int j;
};
template <bool BATCH>
using CgParam = std::conditional_t<BATCH, CgBatch, CgOne>;

// The entry's arguments, its label without the base and the blocks per XCD.
__device__ __forceinline__ CgArgs cg_args(const CgOne& h, int* label, int* nbx) {
  CgArgs a;
  a.x = h.x, a.p = h.p, a.r = h.r, a.q = a.s = h.qs;
  a.pp[0] = h.pp, a.pp[1] = h.pp + h.pp1, a.pq = h.pq, a.pr = h.pr;
  a.n_pp = h.n_pp, a.n_pq = h.n_pq, a.n_pr = h.n_pr, a.max_iters = h.max_iters;
  a.state = h.state, a.delta2 = h.delta2, a.x64 = h.x64;
  a.cgls = h.flags & 1, a.mixed = h.flags >> 1 & 1;
  *label = h.label;
  *nbx = h.flags >> 2;
  return a;
}
__device__ __forceinline__ const CgArgs& cg_args(const CgBatch& h, int* label, int* nbx) {
  const CgArgs& a = h.table[blockIdx.y];
  *label = a.iter0 + h.j;
  *nbx = h.blocks >> 3;
  return a;
}

// One solver iteration with label k = iter0 + j; cur = k & 1, nxt = cur ^ 1.
//   update (CGLS): alpha = sum(pp[cur]) / sum(pq) (block 0: into the solver
//            state);  r -= alpha q;  per-block |r|^2 -> pr
//   pupdate: beta = sum(pp[nxt]) / sum(pp[cur]);  x += alpha p;  p = src +
//            beta p with src = r (CG) or s (CGLS); convergence measure
//            |r|^2 = sum(pp[nxt]) (CG) or sum(pr) (CGLS).
// (CG: pp holds |r|^2, pq = <p, A p> = |Mhat p|^2.  CGLS: pp holds
// |s|^2 = |Mhat^dag r|^2, pq = |q|^2 = |Mhat p|^2.)
// CG launches no update: its third Dslash computes alpha (block 0, into the
// solver state) and the fourth does r -= alpha q in its epilogue.  x is left
// to the p-update in both, which reads p anyway: with x in the CGLS update p
// was read twice (24^3x48, FP64: update 67 -> 34 us, p-update 39 -> 54).
//
// NP = 4 work-items share a site in both kernels: work-item (part, s) updates the
// components 3 part .. 3 part + 2 of site s.  For a storage with a per-site
// scale, which needs all twelve components, the four are the wavefronts of one
// block, which exchange their largest components through LDS.  Batches from
// kBatchSites on have work-items enough with one per site (NP = 1), and a quarter
// of the blocks then repeats the sums over the partials (requests in the service,
// four parts / one, ms: sixteen of 16^3x32 FP64 75.5 / 76.0, FP32 52.1 / 50.0,
// FP16 46.6 / 43.6, BF16 45.4 / 42.4; one FP32 3.95 / 3.93; but one of 8^3x16 FP64
// 1.70 / 1.79).  XCD x (hardware blocks b with b % 8 == x; their number is a
// multiple of 8) takes the sites [x Vh / 8, (x + 1) Vh / 8), the range the
// Dslash's XCD-aware block order gives the same XCD, so the vectors stay in the
// L2 of the XCD that reads them next.  The first element's loads depend on no sum
// and are issued before anything is waited for, but where many launches are past
// their stop.
struct VecRange {
  int lo, nsx, nwork, first, step;
};
// Element i of a range is part i / nsx of site lo + i % nsx (NP = 1: site
// lo + i); SHARED: wavefront w of a block has part w of 64 sites, so i runs over
// groups of 64 sites times four parts, and all four wavefronts of a block make
// the same steps.
template <int NP, bool SHARED>
__device__ __forceinline__ VecRange vec_range(int Vh, int nbx) {
  VecRange v;
  const int xcd = blockIdx.x & 7;
  v.lo = (int)((long long)Vh * xcd / 8);
  v.nsx = (int)((long long)Vh * (xcd + 1) / 8) - v.lo;
  v.nwork = SHARED ? (v.nsx + 63) / 64 * kBlock : v.nsx * NP;
  v.first = (blockIdx.x >> 3) * kBlock + threadIdx.x;
  v.step = nbx * kBlock;
  return v;
}
// Part and site of element i (site -1: beyond the range).
template <int NP, bool SHARED>
__device__ __forceinline__ int vec_site(const VecRange& v, int i, int* part) {
  if (SHARED) {
    *part = (i >> 6) & 3;
    const int s = (i >> 8) * 64 + (i & 63);
    return s < v.nsx ? v.lo + s : -1;
  }
  *part = NP == 1 ? 0 : i / v.nsx;
  return v.lo + i - *part * v.nsx;
}
// Part `part` of the NP equal parts of site s of a vector.
template <class SP, int NP>
__device__ __forceinline__ void load_components(const void* v, int stride, int s, int part, cx<typename SP::R>* out) {
  if constexpr (NP == 1) {
    SP::load(v, stride, s, out);
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c) out[c] = SP::load_one(v, stride, s, 3 * part + c);
  }
}
// (SP::kScaled and NP = 4: every work-item of the block calls it, with s < 0 where it has nothing to store)
template <class SP, int NP>
__device__ __forceinline__ void store_components(void* v, int stride, int s, int part, const cx<typename SP::R>* in) {
  if constexpr (NP == 1) {
    SP::store(v, stride, s, in);
  } else if constexpr (SP::kScaled) {
    __shared__ float smax[4][64];
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) m = fmaxf(m, fmaxf(fabsf(in[c].re), fabsf(in[c].im)));
    const int lane = threadIdx.x & 63;
    __syncthreads();  // the previous step's maxima have been read
    smax[part][lane] = m;
    __syncthreads();
    m = SP::live_scale(fmaxf(fmaxf(smax[0][lane], smax[1][lane]), fmaxf(smax[2][lane], smax[3][lane])));
    const float inv = m > 0.f ? 1.f / m : 0.f;
    if (s < 0) return;
    if (part == 0) SP::store_scale(v, stride, s, m);
#pragma unroll
    for (int c = 0; c < 3; ++c) SP::store_one_scaled(v, stride, s, 3 * part + c, in[c], inv);
  } else {
    SP::store_part(v, stride, s, part, in);
  }
}

template <class SP, bool BATCH, int NP>
__global__ void __launch_bounds__(kBlock) k_cg_update(CgParam<BATCH> h) {
  using R = typename SP::R;
  constexpr int NC = 12 / NP;
  constexpr bool kShared = SP::kScaled && NP == 4;
  int label, nbx;
  const CgArgs& a = cg_args(h, &label, &nbx);
  const int Vh = h.Vh;
  const VecRange w = vec_range<NP, kShared>(Vh, nbx);
  cx<R> q[NC] = {}, r[NC] = {};  // (zero where a work-item has no site)
  auto load = [&](int i) {
    int part;
    const int s = vec_site<NP, kShared>(w, i, &part);
    if (kShared && s < 0) return;
    load_components<SP, NP>(a.q, Vh, s, part, q);
    load_components<SP, NP>(a.r, Vh, s, part, r);
  };
  const int k = label + a.state->base;
  if (NP == 1 || a.mixed) {  // many launches of a mixed chunk or a batch are past its stop: they leave before they load
    if (k >= a.state->stop_at) return;
    asm volatile("" ::: "memory");
  }
  if (w.first < w.nwork) load(w.first);
  const int stop = a.state->stop_at;
  asm volatile("" ::: "memory");  // the loads above stay above
  if (k >= stop) return;
  const double* part[2] = {k & 1 ? a.pp[1] : a.pp[0], a.pq};
  const int n[2] = {a.n_pp, a.n_pq};
  double sums[2];
  sum_partials_n<kBlock / 64, 2>(part, n, sums);
  const double alpha = sums[0] / sums[1];
  if (blockIdx.x == 0 && threadIdx.x == 0) a.state->alpha = alpha;
  const R al = (R)alpha;
  double v[1] = {0.0};
  for (int i = w.first; i < w.nwork; i += w.step) {
    if (i != w.first) load(i);
    int part;
    const int s = vec_site<NP, kShared>(w, i, &part);
    if (!kShared || s >= 0)
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        r[m].re = fma(-al, q[m].re, r[m].re);
        r[m].im = fma(-al, q[m].im, r[m].im);
        v[0] += (double)r[m].re * r[m].re + (double)r[m].im * r[m].im;
      }
    store_components<SP, NP>(a.r, Vh, s, part, r);
  }
  block_sum<1>(v);
  if (threadIdx.x == 0) a.pr[blockIdx.x] = v[0];
}

// Block 0 records the iteration and, when |r|^2 <= thr (or, in mixed
// precision, when the inner residual fell by delta since the last FP64
// update), sets stop_at = k + 1; blocks of this launch compare k only, so
// none of them can observe a change that concerns it.
// Every input of an element is loaded before any output is stored (x, p and r
// are distinct arrays), so a work-item makes one round trip to memory.
template <class SP, class SX, bool BATCH, int NP>
__global__ void __launch_bounds__(kBlock) k_cg_pupdate(CgParam<BATCH> h) {
  int label, nbx;
  const CgArgs& a = cg_args(h, &label, &nbx);
  const int Vh = h.Vh;
  SolverState* stt = a.state;
  using R = typename SP::R;
  using XR = typename SX::R;
  constexpr int NC = 12 / NP;  // components per work-item
  constexpr bool kShared = SP::kScaled && NP == 4;
  const void* src = a.cgls ? a.s : a.r;
  const VecRange w = vec_range<NP, kShared>(Vh, nbx);
  const int nwork = w.nwork, i0 = w.first;
  cx<R> p[NC] = {}, q[NC] = {};  // (zero where a work-item has no site)
  cx<XR> x[NC];
  auto load = [&](int i) {
    int part;
    const int s = vec_site<NP, kShared>(w, i, &part);
    if (kShared && s < 0) return;
    load_components<SP, NP>(a.p, Vh, s, part, p);
    load_components<SX, NP>(a.x, Vh, s, part, x);
    load_components<SP, NP>(src, Vh, s, part, q);
  };
  // the state as the launch found it, read once (block 0 writes iters, last,
  // rr, the other parity's sum_pp, stop_at beyond this label, and maxrr only to
  // a value that leaves the decision below as it is)
  const int k = label + stt->base;
  if (NP == 1 || a.mixed) {  // many launches of a mixed chunk or a batch are past its stop: they leave before they load
    if (k >= stt->stop_at) return;
    asm volatile("" ::: "memory");
  }
  if (i0 < nwork) load(i0);
  const int stop = stt->stop_at, ru_label = stt->ru_label, ru_iter = stt->ru_iter;
  const int iters = stt->iters;
  const double thr = stt->thr, maxrr = stt->maxrr, alpha = stt->alpha, sum0 = stt->sum_pp[0], sum1 = stt->sum_pp[1];
  asm volatile("" ::: "memory");  // the loads above stay above
  if (k >= stop) return;
  const int cur = k & 1, nxt = cur ^ 1;
  const double *pp_cur = cur ? a.pp[1] : a.pp[0], *pp_nxt = cur ? a.pp[0] : a.pp[1];
  // the sums of this step in one block reduction (same order, hence the same
  // bits, in every block).  sum(pp[cur]) is the previous iteration's
  // sum(pp[nxt]), which its block 0 left in the state: it is summed again only
  // by the first iteration after a start or restart.  (The state keeps both
  // parities, so no block reads what this launch writes.)
  __shared__ double bc[3];
  __shared__ int fold_sh;
  {
    // each work-item adds its partials in index order; the loads of up to
    // eight of them are issued together
    constexpr int U = 8;
    double v[3] = {0.0, 0.0, 0.0};
    const bool restarted = k == ru_label;
    for (int base = threadIdx.x; base < a.n_pp; base += U * kBlock) {
      double t0[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = base + u * kBlock;
        t0[u] = i < a.n_pp ? pp_nxt[i] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) v[0] += t0[u];
      if (restarted)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = base + u * kBlock;
          v[1] += i < a.n_pp ? pp_cur[i] : 0.0;
        }
    }
    if (a.cgls)
      for (int base = threadIdx.x; base < a.n_pr; base += U * kBlock) {
        double t2[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = base + u * kBlock;
          t2[u] = i < a.n_pr ? a.pr[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) v[2] += t2[u];
      }
    block_sum<3>(v);
    if (threadIdx.x == 0) {
      bc[0] = v[0], bc[1] = restarted ? v[1] : (cur ? sum1 : sum0), bc[2] = v[2];
      // mixed precision with device-driven updates: does this iteration ask
      // for one?  (Block 0 may already have raised maxrr to max(maxrr, rr):
      // every block gets the same answer.)
      const double r2 = a.cgls ? v[2] : v[0];
      // (ru_iter and ru_label change only between chunks, so every block
      // counts the same iterations.)
      const int done_after = ru_iter + (k + 1 - ru_label);
      fold_sh = a.x64 && (r2 <= thr || r2 < a.delta2 * fmax(maxrr, r2) || !(r2 == r2) ||
                          k + 1 - ru_label >= kMaxInner || (a.max_iters > 0 && done_after >= a.max_iters));
    }
    __syncthreads();
  }
  const double nw = bc[0], old = bc[1];
  const double rr = a.cgls ? bc[2] : nw;
  const bool conv = rr <= thr;
  // the iteration that asks for an update folds the inner solution into
  // the FP64 one (x64 += xl, xl = 0) for the update that follows
  const bool fold = fold_sh != 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    stt->iters = iters + 1;
    stt->last = k;
    stt->rr = rr;
    stt->sum_pp[nxt] = nw;
    if (a.mixed) {
      double mx = fmax(maxrr, rr);
      stt->maxrr = mx;
      // updates also come every kMaxInner iterations, so a low-precision
      // recursion that stagnates cannot run away (the host-driven updates
      // of the solve service: since the restart at ru_label), and, device
      // driven, at the iteration limit
      if (a.x64 ? fold : (conv || rr < a.delta2 * mx || !(rr == rr) || k + 1 - ru_label >= kMaxInner)) {
        stt->reason = 2;
        stt->stop_at = k + 1;
        stt->ru_gate = INT_MAX;  // a device-driven solve updates next
      }
    } else if (conv || !(rr == rr)) {
      stt->reason = conv ? 1 : 3;
      stt->stop_at = k + 1;
    }
  }
  const bool p_done = conv && !a.mixed;  // converged: the search direction is not needed
  const R beta = (R)(nw / old);
  for (int i = i0; i < nwork; i += w.step) {
    int part;
    const int s = vec_site<NP, kShared>(w, i, &part);
    const bool on = !kShared || s >= 0;
    if (i != i0) load(i);
    if (on) {
      // x += alpha p with the p of this iteration
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        x[m].re = fma((XR)alpha, (XR)p[m].re, x[m].re);
        x[m].im = fma((XR)alpha, (XR)p[m].im, x[m].im);
      }
      if (fold) {
#pragma unroll
        for (int m = 0; m < NC; ++m) {
          double2* h = (double2*)a.x64 + (size_t)(NC * part + m) * Vh + s;
          const double2 v = *h;
          *h = make_double2(v.x + (double)x[m].re, v.y + (double)x[m].im);
          x[m] = {(XR)0, (XR)0};
        }
      }
      store_components<SX, NP>(a.x, Vh, s, part, x);
    }
    if (p_done) continue;
    if (on)
#pragma unroll
      for (int m = 0; m < NC; ++m) {
        p[m].re = fma(beta, p[m].re, q[m].re);
        p[m].im = fma(beta, p[m].im, q[m].im);
      }
    store_components<SP, NP>(a.p, Vh, s, part, p);
  }
}

// Start or resume a solve: stop_at = INT_MAX, reason = 0, no reliable
// update pending, maxrr from a device slot (null -> 0), threshold thr; a
// start also clears the counts and the label base.
__global__ void k_state_reset(SolverState* st, const double* maxrr, int nbatch, int reset_iters, double thr,
                              int label) {
  int k = blockIdx.x * kBlock + threadIdx.x;
  if (k >= nbatch) return;
  st[k].stop_at = INT_MAX;
  st[k].reason = 0;
  st[k].ru_gate = 0;
  st[k].thr = thr;
  if (reset_iters) {
    st[k].iters = 0;
    st[k].last = -1;
    st[k].rr = 0.0;
    st[k].base = 0;
    st[k].done = 0;
    st[k].nru = 0;
    st[k].ru_iter = 0;
    st[k].ru_label = 0;
    st[k].rr64 = 0.0;
  }
  st[k].maxrr = maxrr ? maxrr[k] : 0.0;
  if (label >= 0) st[k].ru_label = label;
}

__global__ void k_advance_base(SolverState* st, int n) {
  if (threadIdx.x == 0) st->base += n;
}

__global__ void k_ru_request(SolverState* st) {
  if (threadIdx.x != 0) return;
  st->ru_gate = INT_MAX;
  st->stop_at = min(st->stop_at, st->base);
}

// The end of a device-driven reliable update (see launch_ru_finish).  One
// block; every thread reads the gate before thread 0 clears it (the sum
// synchronises the block in between).
__global__ void __launch_bounds__(kBlock) k_ru_finish(SolverState* st, const double* part64, int n, double* slot,
                                                     int advance, int max_ru, int max_iters) {
  if (st->ru_gate == 0) {
    if (threadIdx.x == 0) st->restart = 0, st->base += advance;
    return;
  }
  const double rr64 = sum_partials(part64, n);
  if (threadIdx.x != 0) return;
  *slot = rr64;
  // The reliable update keeps the search direction p, which is conjugate
  // for the recursive residual it replaces.  Where the two differ by more
  // than a factor 2 in |r|^2, or a whole cycle of inner iterations did not
  // lower the FP64 residual, the low-precision recursion has lost track
  // (BF16 storage with a small delta does this) and keeping p makes the
  // iteration diverge: p restarts from the new residual instead.
  st->restart = rr64 > 2.0 * st->rr || (st->nru > 0 && rr64 >= st->rr64);
  st->nru += 1;
  st->base += advance;
  st->ru_iter = st->iters;
  st->ru_label = st->base;
  st->rr64 = rr64;
  if (rr64 <= st->thr) {
    st->done = 1;
  } else if (!isfinite(rr64)) {
    st->done = 3;
  } else if (st->nru >= max_ru || st->iters >= max_iters) {
    st->done = 4;
  } else {  // resume: the iterations of the next chunk run
    st->stop_at = INT_MAX;
    st->reason = 0;
    st->maxrr = rr64;
  }
  st->ru_gate = 0;
}

// Device-driven reliable update after q = A x (see launch_ru_residual).  The
// |r|^2 of the stored low-precision r is summed from its stored values, as
// the norm of a freshly converted vector is.
template <class SP>
__global__ void __launch_bounds__(kBlock) k_ru_residual(Lat g, const double2* rhs, const double2* q, double2* r64,
                                                        void* rlow, double* part64, double* pp0, double* pp1,
                                                        const int* gate) {
  if (*gate == 0) return;
  using R = typename SP::R;
  double v[2] = {0.0, 0.0};
  for (int s = blockIdx.x * kBlock + threadIdx.x; s < g.Vh; s += gridDim.x * kBlock) {
    cx<R> a[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const size_t j = (size_t)k * g.stride + s;
      const double2 d = make_double2(rhs[j].x - q[j].x, rhs[j].y - q[j].y);
      r64[j] = d;
      v[0] += d.x * d.x + d.y * d.y;
      a[k] = {(R)d.x, (R)d.y};
    }
    SP::store(rlow, g.stride, s, a);
    if (pp0) {
      SP::load(rlow, g.stride, s, a);
#pragma unroll
      for (int k = 0; k < 12; ++k) v[1] += (double)a[k].re * a[k].re + (double)a[k].im * a[k].im;
    }
  }
  block_sum<2>(v);
  if (threadIdx.x == 0) {
    part64[blockIdx.x] = v[0];
    if (pp0) pp0[blockIdx.x] = v[1], pp1[blockIdx.x] = v[1];
  }
}

// x64 += x32; x32 = 0 (mixed precision accumulator hand-over).
__global__ void k_add_low_to_f64(Lat g, double2* x64, float2* x32, const int* gate) {
  if (gate_closed(gate)) return;
  const size_t n = (size_t)12 * g.stride;
  for (size_t j = (size_t)blockIdx.x * kBlock + threadIdx.x; j < n; j += (size_t)gridDim.x * kBlock) {
    float2 l = x32[j];
    double2 h = x64[j];
    x64[j] = make_double2(h.x + (double)l.x, h.y + (double)l.y);
    x32[j] = make_float2(0.f, 0.f);
  }
}

// ------------------------------------------------------------ launchers

// One wavefront that does nothing: the floor of a launch timed through a
// kernel-stamped event pair.
__global__ void k_empty() {}

hipError_t launch_empty_timed(hipStream_t st) {
  const KernelEvents ev = timing_kernel_events(TK_OTHER, 0.0);
  hipExtLaunchKernelGGL(k_empty, dim3(1), dim3(64), 0, st, ev.start, ev.stop, 0);
  return hipGetLastError();
}

hipError_t launch_triad(void* a, const void* b, const void* c, double sc, size_t n2, bool nt, hipStream_t st) {
  TimedScope ts(TK_OTHER, st, 48.0 * n2);
  const int nb = (int)std::min<size_t>((n2 + 4 * kBlock - 1) / (4 * kBlock), 65536);
  if (nt)
    hipLaunchKernelGGL(k_triad<true>, dim3(nb), dim3(kBlock), 0, st, a, b, c, sc, n2);
  else
    hipLaunchKernelGGL(k_triad<false>, dim3(nb), dim3(kBlock), 0, st, a, b, c, sc, n2);
  return hipGetLastError();
}

hipError_t launch_norm2_partials(const LatArg& g, hmc_prec prec, const void* x, double* part, int nb,
                                 hipStream_t st, const int* gate) {
  const double kb[4] = {SpF64::kBytes, SpF32::kBytes, SpF16::kBytes, SpBF16::kBytes};
  TimedScope ts(TK_REDUCE, st, kb[prec] * g.Vh);
  switch (prec) {
    case HMC_F64: hipLaunchKernelGGL(k_norm2_partials<SpF64>, dim3(nb), dim3(kBlock), 0, st, to_lat(g), x, part, gate); break;
    case HMC_F32: hipLaunchKernelGGL(k_norm2_partials<SpF32>, dim3(nb), dim3(kBlock), 0, st, to_lat(g), x, part, gate); break;
    case HMC_F16: hipLaunchKernelGGL(k_norm2_partials<SpF16>, dim3(nb), dim3(kBlock), 0, st, to_lat(g), x, part, gate); break;
    case HMC_BF16: hipLaunchKernelGGL(k_norm2_partials<SpBF16>, dim3(nb), dim3(kBlock), 0, st, to_lat(g), x, part, gate); break;
  }
  return hipGetLastError();
}

hipError_t launch_inner_partials(const LatArg& g, const void* a, const void* b, double* part, int nb,
                                 hipStream_t st) {
  TimedScope ts(TK_REDUCE, st, 2.0 * SpF64::kBytes * g.Vh);
  hipLaunchKernelGGL(k_inner_partials, dim3(nb), dim3(kBlock), 0, st, to_lat(g), (const double2*)a,
                     (const double2*)b, part);
  return hipGetLastError();
}

hipError_t launch_finalize(const double* part, int n, int nvals, double* out, double scale, int accumulate,
                           hipStream_t st, const int* gate) {
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(kBlock), 0, st, part, n, nvals, out, scale, accumulate, gate);
  return hipGetLastError();
}

hipError_t launch_sum_multi(const LatArg& g, const void* x, int nhalves, const int* subset, int nsub, double* part,
                            int nb, double* out, hipStream_t st) {
  if (nsub > kMaxSub || nsub < 1) return hipErrorInvalidValue;
  const size_t lds = (size_t)(kBlock / 64) * nsub * sizeof(double);
  hipLaunchKernelGGL(k_sum_multi_partials, dim3(nb, nhalves), dim3(kBlock), lds, st, to_lat(g), x, subset, nsub, part);
  hipLaunchKernelGGL(k_sum_multi_final, dim3(nsub), dim3(kBlock), 0, st, part, nb * nhalves, out);
  return hipGetLastError();
}

// out = sum_k c_k y_k over n <= 4 F64 half spinors (complex coefficients).
struct LinComb {
  const double2* y[4];
  double2 c[4];
  int n;
};

__global__ void __launch_bounds__(kBlock) k_lincomb(Lat g, LinComb a, double2* out) {
  const size_t total = (size_t)12 * g.stride;
  for (size_t j = (size_t)blockIdx.x * kBlock + threadIdx.x; j < total; j += (size_t)gridDim.x * kBlock) {
    double re = 0.0, im = 0.0;
    for (int k = 0; k < a.n; ++k) {
      const double2 v = a.y[k][j];
      re += a.c[k].x * v.x - a.c[k].y * v.y;
      im += a.c[k].x * v.y + a.c[k].y * v.x;
    }
    out[j] = make_double2(re, im);
  }
}

hipError_t launch_lincomb(const LatArg& g, const void* const* y, const double* c, int n, void* out, hipStream_t st) {
  if (n < 1 || n > 4) return hipErrorInvalidValue;
  LinComb a{};
  for (int k = 0; k < n; ++k) {
    a.y[k] = (const double2*)y[k];
    a.c[k] = make_double2(c[2 * k], c[2 * k + 1]);
  }
  a.n = n;
  hipLaunchKernelGGL(k_lincomb, dim3(blas_blocks(g.Vh)), dim3(kBlock), 0, st, to_lat(g), a, (double2*)out);
  return hipGetLastError();
}

hipError_t launch_xmy_norm(const LatArg& g, const void* b, const void* q, void* r, double* part, int nb,
                           hipStream_t st, const int* gate) {
  hipLaunchKernelGGL(k_xmy_norm, dim3(nb), dim3(kBlock), 0, st, to_lat(g), (const double2*)b, (const double2*)q,
                     (double2*)r, part, gate);
  return hipGetLastError();
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
  size_t n16 = bytes / 16, nt = bytes % 16;
  int nb = (int)std::min<size_t>(std::max<size_t>((n16 + kBlock - 1) / kBlock, 1), 4096);
  hipLaunchKernelGGL(k_zero, dim3(nb), dim3(kBlock), 0, st, (uint4*)p, n16, (unsigned char*)p + n16 * 16, nt);
  return hipGetLastError();
}

hipError_t launch_copy_gated(void* dst, const void* src, size_t bytes, const int* gate, hipStream_t st) {
  size_t n16 = bytes / 16, nt = bytes % 16;
  int nb = (int)std::min<size_t>(std::max<size_t>((n16 + kBlock - 1) / kBlock, 1), 4096);
  hipLaunchKernelGGL(k_copy, dim3(nb), dim3(kBlock), 0, st, (uint4*)dst, (const uint4*)src, n16,
                     (unsigned char*)dst + n16 * 16, (const unsigned char*)src + n16 * 16, nt, gate);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
  return launch_copy_gated(dst, src, bytes, nullptr, st);
}

hipError_t launch_cg_init(const LatArg& g, hmc_prec prec, const void* b, void* x, void* r, void* p, double* part,
                          int nb, hipStream_t st) {
  if (prec != HMC_F64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cg_init, dim3(nb), dim3(kBlock), 0, st, to_lat(g), (const double2*)b, (double2*)x,
                     (double2*)r, (double2*)p, part);
  return hipGetLastError();
}

// Bytes of a solver-vector update per site: x read and written in its own
// storage, `nsp` reads or writes of vectors of the iteration's storage.
static double cg_vec_bytes(hmc_prec prec, bool with_x, int nsp) {
  const double sp = prec == HMC_F64 ? SpF64::kBytes : prec == HMC_F32 ? SpF32::kBytes
                    : prec == HMC_F16 ? SpF16::kBytes : SpBF16::kBytes;
  const double sx = prec == HMC_F64 ? SpF64::kBytes : SpF32::kBytes;
  return (with_x ? 2 * sx : 0.0) + nsp * sp;
}

int cg_vec_parts(int Vh, bool batch) { return batch && Vh >= kBatchSites ? 1 : 4; }
// One share per XCD of a grid that gives every work-item an element up to 2048
// blocks (512 to 4096 measure the same).
int cg_vec_blocks(int Vh, bool batch) {
  return std::min(8 * ceil_div((long long)cg_vec_parts(Vh, batch) * Vh, 8 * kBlock), 2048);
}

hipError_t launch_cg_update(const LatArg& g, hmc_prec prec, const CgArgs& a, const CgArgs* table, int nbatch, int j,
                            hipStream_t st) {
  // r -= alpha q: q read, r read + written
  TimedScope ts(TK_CG_BLAS, st, cg_vec_bytes(prec, false, 3) * g.Vh * nbatch);
  if (g.stride != g.Vh || (!table && !CgOne::holds(a))) return hipErrorInvalidValue;
  const dim3 grid(cg_vec_blocks(g.Vh, table != nullptr), nbatch), block(kBlock);
  const CgBatch batch{g.Vh, (int)grid.x, table, j};
  auto go = [&](auto sp) {
    using SP = decltype(sp);
    if (!table)
      hipLaunchKernelGGL((k_cg_update<SP, false, 4>), grid, block, 0, st, CgOne(g.Vh, grid.x, a, a.q, j));
    else if (cg_vec_parts(g.Vh, true) == 1)
      hipLaunchKernelGGL((k_cg_update<SP, true, 1>), grid, block, 0, st, batch);
    else
      hipLaunchKernelGGL((k_cg_update<SP, true, 4>), grid, block, 0, st, batch);
  };
  switch (prec) {
    case HMC_F64: go(SpF64{}); break;
    case HMC_F32: go(SpF32{}); break;
    case HMC_F16: go(SpF16{}); break;
    case HMC_BF16: go(SpBF16{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_cg_pupdate(const LatArg& g, hmc_prec prec, const CgArgs& a, const CgArgs* table, int nbatch, int j,
                             hipStream_t st) {
  // x += alpha p, p = r + beta p: x and p read + written, r read
  TimedScope ts(TK_CG_BLAS, st, cg_vec_bytes(prec, true, 3) * g.Vh * nbatch);
  if (g.stride != g.Vh || (!table && !CgOne::holds(a))) return hipErrorInvalidValue;
  const dim3 grid(cg_vec_blocks(g.Vh, table != nullptr), nbatch), block(kBlock);
  const CgBatch batch{g.Vh, (int)grid.x, table, j};
  auto go = [&](auto sp, auto sx) {
    using SP = decltype(sp);
    using SX = decltype(sx);
    if (!table)
      hipLaunchKernelGGL((k_cg_pupdate<SP, SX, false, 4>), grid, block, 0, st, CgOne(g.Vh, grid.x, a, a.s, j));
    else if (cg_vec_parts(g.Vh, true) == 1)
      hipLaunchKernelGGL((k_cg_pupdate<SP, SX, true, 1>), grid, block, 0, st, batch);
    else
      hipLaunchKernelGGL((k_cg_pupdate<SP, SX, true, 4>), grid, block, 0, st, batch);
  };
  switch (prec) {
    case HMC_F64: go(SpF64{}, SpF64{}); break;
    case HMC_F32: go(SpF32{}, SpF32{}); break;
    case HMC_F16: go(SpF16{}, SpF32{}); break;
    case HMC_BF16: go(SpBF16{}, SpF32{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_state_reset(SolverState* st_dev, const double* maxrr, int nbatch, int reset_iters, double thr,
                              hipStream_t st, int label) {
  hipLaunchKernelGGL(k_state_reset, dim3(ceil_div(nbatch, kBlock)), dim3(kBlock), 0, st, st_dev, maxrr, nbatch,
                     reset_iters, thr, label);
  return hipGetLastError();
}

hipError_t launch_advance_base(SolverState* st_dev, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_advance_base, dim3(1), dim3(64), 0, st, st_dev, n);
  return hipGetLastError();
}

hipError_t launch_ru_request(SolverState* st_dev, hipStream_t st) {
  hipLaunchKernelGGL(k_ru_request, dim3(1), dim3(64), 0, st, st_dev);
  return hipGetLastError();
}

hipError_t launch_ru_finish(SolverState* st_dev, const double* part64, int n, double* rr64_slot, int advance,
                            int max_ru, int max_iters, hipStream_t st) {
  hipLaunchKernelGGL(k_ru_finish, dim3(1), dim3(kBlock), 0, st, st_dev, part64, n, rr64_slot, advance, max_ru,
                     max_iters);
  return hipGetLastError();
}

hipError_t launch_ru_residual(const LatArg& g, hmc_prec prec, const void* rhs, const void* q, void* r64, void* rlow,
                              double* part64, double* pp0, double* pp1, int nb, const int* gate, hipStream_t st) {
  const dim3 grid(nb), block(kBlock);
  const Lat lat = to_lat(g);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, lat, (const double2*)rhs, (const double2*)q, (double2*)r64, rlow,
                       part64, pp0, pp1, gate);
  };
  switch (prec) {
    case HMC_F64: return hipErrorInvalidValue;  // FP64 solves need no update
    case HMC_F32: go(k_ru_residual<SpF32>); break;
    case HMC_F16: go(k_ru_residual<SpF16>); break;
    case HMC_BF16: go(k_ru_residual<SpBF16>); break;
  }
  return hipGetLastError();
}

hipError_t launch_add_low_to_f64(const LatArg& g, void* x64, void* xlow, hipStream_t st, const int* gate) {
  hipLaunchKernelGGL(k_add_low_to_f64, dim3(blas_blocks(g.Vh)), dim3(kBlock), 0, st, to_lat(g), (double2*)x64,
                     (float2*)xlow, gate);
  return hipGetLastError();
}

}  // namespace hmc
