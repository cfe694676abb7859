// Layout conversion and vector (BLAS-1) kernels of the solver.
//
// Layout conversion: the ABI's canonical site-major complex128 arrays
// [V][nc] are transposed, through LDS, into the internal even/odd
// structure-of-arrays [parity][nc][V/2], so both the global reads and the
// global writes are unit-stride across a wavefront.
//
// Vector kernels work on flat arrays of n complex numbers (grid-stride,
// unit-stride).  Reductions write block partials; the one-block finalize
// kernel sums them in a fixed order (deterministic, see block_partials).
#include <algorithm>

#include "lgt_internal.h"

namespace lgt {

// A packed field is 6 to 36 planes of one complex number per site, and a wave
// reads the same sites of every plane at once.  On lattices past the caches
// whose planes are a large power of two apart (8 MB at 32^3x64 in FP32) those
// reads crowd onto a part of the memory channels: a plain sum over 24 float2
// planes runs at 5.35 TB/s with planes 2^21 elements apart and at 6.2 TB/s
// with them a little off that distance; the two-row hops at 32^3x64 take 125
// (FP32) and 264 us (FP64) dense, 120 and 248 us padded, the smeared force
// there 218.7 and 209.6 ms.  In the caches the same holds for L2 channels, and
// dense fields of 16^4 come out in one of two ways from process to process
// (mixed FP32 force 5.27 or 5.51 ms; padded 5.16 to 5.26; rational force 5.25
// and 5.10 ms).  Planes of more than 16384 sites that are a multiple of 16384
// are therefore 2112 = 33 * 64 sites further apart (64, 1088 and 4160 measured
// within 1 %).  Padded against dense on further lattices of that kind: solves
// in FP64, FP32 and BF16 and 1 to 12 shifts 1 % faster at 16^3x24 (49152
// sites), 1.5 to 2 % at 16^3x32, 1 to 2 % at 16^3x48, 2 to 4 % at 32^4; staple
// force 3 % from 16^3x32 on; slower only one pass of its own, the Schur
// operator (83 -> 86 us) and the plaquette sum (121 -> 124), at 16^3x32.  Others stay dense: at 24^3x48 (81 * 2^12 sites) the padding
// gave the FP64 hop 4 % and cost the smearing 0.6 %, and 8x16^3 (16384 sites)
// lost by it (FP64 solve 4.90 -> 4.99 ms, rational force 3.34 -> 3.42).  A lattice
// that only fits the 32-bit field offsets without the padding (for 1..16
// batched fields, or the gauge field of the 32-site hop blocks) stays dense
// too, so that no call is lost to it.
constexpr int kPadMinVh = 16384;
constexpr int kPadAlign = 16384;
constexpr int kPadSites = 2112;
int plane_stride(int vh) {
  if (vh <= kPadMinVh || vh % kPadAlign != 0) return vh;
  const int vs = vh + kPadSites;
  const size_t lim = (size_t)1 << 32, e = sizeof(double2);
  for (size_t n = 1; n <= 16; ++n)
    if (12 * n * vh * e < lim && 12 * n * vs * e >= lim) return vh;
  if ((size_t)72 * vh * e < lim && (size_t)72 * vs * e >= lim) return vh;
  return vs;
}

constexpr int kPackSites = 64;  // lexicographic sites per pack block (32 per parity)

template <int NC, bool W32>
__global__ __launch_bounds__(256) void k_pack(Geom g, const double2* __restrict__ canon,
                                              double2* __restrict__ out64, float2* __restrict__ out32,
                                              int* nonfinite) {
  __shared__ double2 tile[NC][kPackSites];
  __shared__ int par[kPackSites];
  const int V = 2 * g.vh;
  const int s0 = blockIdx.x * kPackSites;
  const int nsite = min(kPackSites, V - s0);
  bool bad = false;
  for (int e = threadIdx.x; e < nsite * NC; e += 256) {
    double2 v = canon[(size_t)s0 * NC + e];
    bad |= !(isfinite(v.x) && isfinite(v.y));
    tile[e % NC][e / NC] = v;
  }
  if (threadIdx.x < nsite) {
    int c[4];
    lex_coords(g, s0 + threadIdx.x, c);
    par[threadIdx.x] = parity_of(c);
  }
  if (bad && nonfinite) atomicOr(nonfinite, 1);
  __syncthreads();
  const int half = kPackSites / 2;
  const int cb0 = s0 / 2;
  for (int e = threadIdx.x; e < 2 * NC * half; e += 256) {
    const int p = e / (NC * half);
    const int k = (e / half) % NC;
    const int j = e % half;
    if (2 * j >= nsite) continue;
    // of the two sites s0+2j, s0+2j+1 (same cb index) pick the one of parity p
    const int site = (par[2 * j] == p) ? 2 * j : 2 * j + 1;
    const double2 v = tile[k][site];
    const size_t o = ((size_t)p * NC + k) * g.vs + cb0 + j;
    out64[o] = v;
    if (W32) out32[o] = make_float2((float)v.x, (float)v.y);
  }
}

template <int NC>
__global__ __launch_bounds__(256) void k_unpack(Geom g, const double2* __restrict__ packed,
                                                double2* __restrict__ canon) {
  __shared__ double2 tile[NC][kPackSites];
  __shared__ int par[kPackSites];
  const int V = 2 * g.vh;
  const int s0 = blockIdx.x * kPackSites;
  const int nsite = min(kPackSites, V - s0);
  if (threadIdx.x < nsite) {
    int c[4];
    lex_coords(g, s0 + threadIdx.x, c);
    par[threadIdx.x] = parity_of(c);
  }
  __syncthreads();
  const int half = kPackSites / 2;
  const int cb0 = s0 / 2;
  for (int e = threadIdx.x; e < 2 * NC * half; e += 256) {
    const int p = e / (NC * half);
    const int k = (e / half) % NC;
    const int j = e % half;
    if (2 * j >= nsite) continue;
    const int site = (par[2 * j] == p) ? 2 * j : 2 * j + 1;
    tile[k][site] = packed[((size_t)p * NC + k) * g.vs + cb0 + j];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nsite * NC; e += 256) canon[(size_t)s0 * NC + e] = tile[e % NC][e / NC];
}

hipError_t launch_pack(const Geom& g, int nc, const double2* canon, double2* out64, float2* out32,
                       int* nonfinite, hipStream_t s) {
  const int V = 2 * g.vh;
  const int nb = (V + kPackSites - 1) / kPackSites;
  if (nc == 12) {
    if (out32) hipLaunchKernelGGL((k_pack<12, true>), dim3(nb), dim3(256), 0, s, g, canon, out64, out32, nonfinite);
    else hipLaunchKernelGGL((k_pack<12, false>), dim3(nb), dim3(256), 0, s, g, canon, out64, out32, nonfinite);
  } else if (nc == 36) {
    if (out32) hipLaunchKernelGGL((k_pack<36, true>), dim3(nb), dim3(256), 0, s, g, canon, out64, out32, nonfinite);
    else hipLaunchKernelGGL((k_pack<36, false>), dim3(nb), dim3(256), 0, s, g, canon, out64, out32, nonfinite);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// HMC momentum refresh (Sec. III B): Pi = i sum_a c_a T_a, T_a = lambda_a / 2
// (Gell-Mann), from eight normals c_a per link, canonical [V][4][3][3].
// Written out per element (traceless anti-Hermitian by construction).
__global__ __launch_bounds__(256) void k_momenta(size_t nlinks, const double* __restrict__ c,
                                                 double2* __restrict__ P) {
  const size_t l = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (l >= nlinks) return;
  const double* a = c + 8 * l;
  const double h = 0.5, r3 = 0.57735026918962576451;  // 1/sqrt(3)
  double2* q = P + 9 * l;
  q[0] = make_double2(0.0, h * (a[2] + r3 * a[7]));
  q[1] = make_double2(h * a[1], h * a[0]);
  q[2] = make_double2(h * a[4], h * a[3]);
  q[3] = make_double2(-h * a[1], h * a[0]);
  q[4] = make_double2(0.0, h * (-a[2] + r3 * a[7]));
  q[5] = make_double2(h * a[6], h * a[5]);
  q[6] = make_double2(-h * a[4], h * a[3]);
  q[7] = make_double2(-h * a[6], h * a[5]);
  q[8] = make_double2(0.0, -2.0 * h * r3 * a[7]);
}
hipError_t launch_momenta(const Geom& g, const double* normals, double2* P, hipStream_t s) {
  const size_t n = (size_t)2 * g.vh * 4;
  hipLaunchKernelGGL(k_momenta, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, normals, P);
  return hipGetLastError();
}

hipError_t launch_unpack(const Geom& g, int nc, const double2* packed, double2* canon, hipStream_t s) {
  const int V = 2 * g.vh;
  const int nb = (V + kPackSites - 1) / kPackSites;
  if (nc == 12) hipLaunchKernelGGL((k_unpack<12>), dim3(nb), dim3(256), 0, s, g, packed, canon);
  else if (nc == 36) hipLaunchKernelGGL((k_unpack<36>), dim3(nb), dim3(256), 0, s, g, packed, canon);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Vector kernels
// ---------------------------------------------------------------------------
static inline int vec_blocks(int n) {
  int nb = (n + 255) / 256;
  return nb < 1024 ? (nb < 1 ? 1 : nb) : 1024;
}

template <typename R>
__global__ __launch_bounds__(256) void k_cg_init(int n, const R2<R>* __restrict__ b, R2<R>* __restrict__ r,
                                                 R2<R>* __restrict__ p, R2<R>* __restrict__ x, double* partials) {
  double acc = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const R2<R> v = b[i];
    r[i] = v;
    p[i] = v;
    R2<R> z;
    z.x = R(0);
    z.y = R(0);
    x[i] = z;
    acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
  }
  double v[1] = {acc};
  block_partials<256, 1>(v, partials, blockIdx.x);
}

template <typename R>
hipError_t launch_cg_init(int n, const R2<R>* b, R2<R>* r, R2<R>* p, R2<R>* x, SolverState* st,
                          Reduce red, double tol, int max_iter, hipStream_t s) {
  const int nb = vec_blocks(n);
  hipLaunchKernelGGL((k_cg_init<R>), dim3(nb), dim3(256), 0, s, n, b, r, p, x, red.partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_finalize(kFinCgInit, nb, red, st, 0, tol, max_iter, s);
}

// One block: sum the partials of the previous launch and act on the totals.
template <int NV>
__global__ __launch_bounds__(256) void k_finalize(int mode, int nblk, const double* __restrict__ partials,
                                                  SolverState* st, double* result, double tol, int max_iter,
                                                  Mailbox* mb) {
  double tot[NV];
  sum_partials<256, NV>(partials, nblk, tot);
  if (threadIdx.x != 0) return;
  if (mode == kFinResult1 || mode == kFinResult2) {
#pragma unroll
    for (int k = 0; k < NV; ++k) result[k] = tot[k];
  } else if (mode == kFinCgInit) {
    const double rr = tot[0];
    st->rr = rr;
    st->rr0 = rr;
    st->rr_max = rr;
    st->rr_stop = tol * tol * rr;
    st->iter = 0;
    st->max_iter = max_iter;
    st->alpha = 0.0;
    st->beta = 0.0;
    st->pap = 0.0;
    st->delta2 = 0.0;
    st->done = !isfinite(rr) ? kDoneBreakdown : (rr == 0.0 ? kDoneConverged : kDoneRunning);
  }
}

hipError_t launch_finalize(int mode, int nblk, Reduce red, SolverState* st, int slot, double tol, int max_iter,
                           hipStream_t s) {
  if (nblk > red.capacity) return hipErrorInvalidValue;
  if (mode == kFinResult2)
    hipLaunchKernelGGL(k_finalize<2>, dim3(1), dim3(256), 0, s, mode, nblk, red.partials, st, red.result + slot,
                       tol, max_iter, red.mbox);
  else
    hipLaunchKernelGGL(k_finalize<1>, dim3(1), dim3(256), 0, s, mode, nblk, red.partials, st, red.result + slot,
                       tol, max_iter, red.mbox);
  return hipGetLastError();
}

// Elements of the direction update: as many components as one 16-byte vector
// of T holds, with the same components of the R2<R> fields x and r (two
// vectors of them for BF16-stored p, whose planes hold a colour's four spins;
// see Planes).  e: element, n / W of them; vs: plane stride.
template <typename R, typename T> struct StepElem;
template <> struct StepElem<double, double2> {
  static constexpr int W = 1;
  static __device__ __forceinline__ void ld_p(const double2* p, int e, C<double>* v) { v[0] = lgt::ld<double>(p + e); }
  static __device__ __forceinline__ void st_p(double2* p, int e, const C<double>* v) { lgt::st<double>(p + e, v[0]); }
  static __device__ __forceinline__ void ld_x(const double2* x, int e, int, C<double>* v) { v[0] = lgt::ld<double>(x + e); }
  static __device__ __forceinline__ void st_x(double2* x, int e, int, const C<double>* v) { lgt::st<double>(x + e, v[0]); }
};
template <> struct StepElem<float, float2> {
  static constexpr int W = 2;
  static __device__ __forceinline__ void ld_p(const float2* p, int e, C<float>* v) {
    halves(reinterpret_cast<const v4f32*>(p)[e], v[0], v[1]);
  }
  static __device__ __forceinline__ void st_p(float2* p, int e, const C<float>* v) {
    reinterpret_cast<v4f32*>(p)[e] = v4f32{v[0].re, v[0].im, v[1].re, v[1].im};
  }
  static __device__ __forceinline__ void ld_x(const float2* x, int e, int, C<float>* v) { ld_p(x, e, v); }
  static __device__ __forceinline__ void st_x(float2* x, int e, int, const C<float>* v) { st_p(x, e, v); }
};
template <> struct StepElem<float, Bf16c> {
  static constexpr int W = 4;
  static __device__ __forceinline__ void ld_p(const Bf16c* p, int e, C<float>* v) { Planes<float, Bf16c>::ld(p, 0, 0, e, v); }
  static __device__ __forceinline__ void st_p(Bf16c* p, int e, const C<float>* v) { Planes<float, Bf16c>::st(p, 0, 0, e, v); }
  static __device__ __forceinline__ void ld_x(const float2* x, int e, int vs, C<float>* v) {
    const int own = e / vs;
    Planes<float, float2>::ld(x, vs, own, e - own * vs, v);
  }
  static __device__ __forceinline__ void st_x(float2* x, int e, int vs, const C<float>* v) {
    const int own = e / vs;
    Planes<float, float2>::st(x, vs, own, e - own * vs, v);
  }
};

constexpr int kStepThreads = 512;

template <typename R, typename T>
__global__ __launch_bounds__(kStepThreads) void k_cg_step(int n, int vs, int nblk, const double* __restrict__ partials,
                                                          const R2<R>* __restrict__ r, T* __restrict__ p,
                                                          SolverState* st, Mailbox* mb, R2<R>* __restrict__ x) {
  // what the third hop recorded: done itself is block 0's to set below, while
  // other blocks may only be starting
  const int done0 = st->done_prev;
  if (done0 != kDoneRunning) {  // the iteration was skipped
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      if (done0 == kDoneUpdate) st->done = kDoneUpdateHeld;
      // the same action as the stop itself, in case the host has not seen it
      post_progress(mb, st->iter, action_word(st->epoch, done0 == kDoneUpdateHeld ? kDoneUpdate : done0));
    }
    return;
  }
  // every block forms the same rr (same partials, same order) and so takes
  // the same decision; the inputs are the copies the third hop made, which
  // block 0's writes below do not touch
  __shared__ double s_rr;
  double tot[1];
  sum_partials<kStepThreads, 1>(partials, nblk, tot);
  if (threadIdx.x == 0) s_rr = tot[0];
  __syncthreads();
  const double rr = s_rr;
  const double beta = rr / st->rr_prev;
  const int iter = st->iter_prev + 1;
  const double rr_max = fmax(st->rr_max, rr);  // block 0 may have stored this same value already
  int code = kDoneRunning;
  if (!isfinite(rr)) code = kDoneBreakdown;
  else if (rr <= st->rr_stop) code = st->delta2 > 0.0 ? kDoneUpdate : kDoneConverged;
  else if (rr <= st->delta2 * rr_max) code = kDoneUpdate;
  else if (iter >= st->max_iter) code = kDoneMaxIter;
  {
    // x += alpha p (this iteration's step, taken whatever the decision), then
    // p = r + beta p unless the recursion stops
    using E = StepElem<R, T>;
    const R b = R(beta), a = R(st->alpha);
    const bool upd = code == kDoneRunning;
    const int stride = gridDim.x * kStepThreads, ne = n / E::W;
    for (int i = blockIdx.x * kStepThreads + threadIdx.x; i < ne; i += stride) {
      C<R> rv[E::W], pv[E::W], xv[E::W];
      E::ld_p(p, i, pv);
      E::ld_x(x, i, vs, xv);
      if (upd) E::ld_x(r, i, vs, rv);
#pragma unroll
      for (int q = 0; q < E::W; ++q) {
        xv[q] += a * pv[q];
        if (upd) pv[q] = C<R>{rv[q].re + b * pv[q].re, rv[q].im + b * pv[q].im};
      }
      E::st_x(x, i, vs, xv);
      if (upd) E::st_p(p, i, pv);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->beta = beta;
    st->rr = rr;
    st->iter = iter;
    st->rr_max = rr_max;
    if (code != kDoneRunning) st->done = code;
    post_progress(mb, iter, code != kDoneRunning ? action_word(st->epoch, code) : 0u);
  }
}

template <typename R, typename T>
hipError_t launch_cg_step(int vs, const R2<R>* r, T* p, SolverState* st, Reduce red, int nblk, hipStream_t s,
                          R2<R>* x) {
  const int n = 12 * vs;
  if (nblk > red.capacity) return hipErrorInvalidValue;
  // Bound by HBM and the memory-side cache; but each block also sums the nblk
  // partials, one for 64 sites: at 32^3x64 128 KB a block, so blocks beyond
  // one a CU cost more than they hide.  256 blocks of 512 threads (8 waves a
  // CU) against 1024 or 2048 of 256 threads that took two or four elements a
  // trip: FP32 at 32^3x64 104.6 -> 74.5 us, BF16 at 24^3x48 25.3 -> 20.9,
  // FP64 at 24^3x48 52.2 -> 48.9 and at 32^3x64 182.9 -> 163.5.
  const int nb = std::max(1, std::min((n / StepElem<R, T>::W + kStepThreads - 1) / kStepThreads, 256));
  hipLaunchKernelGGL((k_cg_step<R, T>), dim3(nb), dim3(kStepThreads), 0, s, n, vs, nblk, red.partials, r, p, st, red.mbox, x);
  return hipGetLastError();
}
template hipError_t launch_cg_step<double, double2>(int, const double2*, double2*, SolverState*, Reduce, int,
                                                    hipStream_t, double2*);
template hipError_t launch_cg_step<float, float2>(int, const float2*, float2*, SolverState*, Reduce, int,
                                                  hipStream_t, float2*);
template hipError_t launch_cg_step<float, Bf16c>(int, const float2*, Bf16c*, SolverState*, Reduce, int,
                                                 hipStream_t, float2*);

__global__ __launch_bounds__(256) void k_norm_dot(int n, const double2* __restrict__ a,
                                                  const double2* __restrict__ b, double* partials) {
  double nn = 0.0, dd = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double2 av = a[i];
    nn += av.x * av.x + av.y * av.y;
    if (b) {
      const double2 bv = b[i];
      dd += av.x * bv.x + av.y * bv.y;
    }
  }
  double v[2] = {nn, dd};
  block_partials<256, 2>(v, partials, blockIdx.x);
}

hipError_t launch_norm_dot(int n, const double2* a, const double2* b, Reduce red, int slot, hipStream_t s) {
  const int nb = vec_blocks(n);
  hipLaunchKernelGGL(k_norm_dot, dim3(nb), dim3(256), 0, s, n, a, b, red.partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_finalize(kFinResult2, nb, red, nullptr, slot, 0.0, 0, s);
}

__global__ __launch_bounds__(256) void k_axpy64(int n, double a, const double2* __restrict__ x,
                                                double2* __restrict__ y) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double2 xv = x[i];
    double2 yv = y[i];
    yv.x += a * xv.x;
    yv.y += a * xv.y;
    y[i] = yv;
  }
}
hipError_t launch_axpy64(int n, double a, const double2* x, double2* y, hipStream_t s) {
  hipLaunchKernelGGL(k_axpy64, dim3((n + 255) / 256), dim3(256), 0, s, n, a, x, y);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_copy64(int n, const double2* __restrict__ x, double2* __restrict__ y) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) y[i] = x[i];
}
hipError_t launch_copy64(int n, const double2* x, double2* y, hipStream_t s) {
  hipLaunchKernelGGL(k_copy64, dim3((n + 255) / 256), dim3(256), 0, s, n, x, y);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_zero64(int n, double2* __restrict__ y) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) y[i] = make_double2(0.0, 0.0);
}
hipError_t launch_zero64(int n, double2* y, hipStream_t s) {
  hipLaunchKernelGGL(k_zero64, dim3((n + 255) / 256), dim3(256), 0, s, n, y);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_zero32(int n, float2* __restrict__ y) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) y[i] = make_float2(0.f, 0.f);
}
hipError_t launch_zero32(int n, float2* y, hipStream_t s) {
  hipLaunchKernelGGL(k_zero32, dim3((n + 255) / 256), dim3(256), 0, s, n, y);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_convert_64_32(int n, const double2* __restrict__ x, float2* __restrict__ y) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double2 v = x[i];
    y[i] = make_float2((float)v.x, (float)v.y);
  }
}
hipError_t launch_convert_64_32(int n, const double2* x, float2* y, hipStream_t s) {
  hipLaunchKernelGGL(k_convert_64_32, dim3((n + 255) / 256), dim3(256), 0, s, n, x, y);
  return hipGetLastError();
}

// Two-row copy of a packed link field ([2][4][9][vs] -> six complex planes a
// link in FP64, three planes of two in FP32, see load_two_rows) and
// the check that the links are SU(3): flag is set when a stored third row
// differs from the conjugate cross product of the first two by more than tol
// (per component, |re| + |im|), or is not finite.
// FP64 links whose stored third row is within this of the rebuilt one (a few
// dozen rounding units) are taken as SU(3) by the FP64 solver's hops.
constexpr double kTwoRowTol64 = 1e-14;

template <typename R>
__global__ __launch_bounds__(256) void k_compress_links(int vh, int vs, const R2<R>* __restrict__ U, R2<R>* __restrict__ Uc,
                                                        int* flag, R tol) {
  const int t = blockIdx.x * 256 + threadIdx.x;  // link (parity, mu) slowest, site fastest
  if (t >= 8 * vh) return;
  const int pm = t / vh, cb = t - pm * vh;
  const R2<R>* src = U + (size_t)pm * 9 * vs + cb;
  C<R> m[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) m[k] = ld<R>(src + (size_t)k * vs);
  if constexpr (sizeof(R) == 8) {
    R2<R>* dst = Uc + (size_t)pm * 6 * vs + cb;
#pragma unroll
    for (int k = 0; k < 6; ++k) st<R>(dst + (size_t)k * vs, m[k]);
  } else {
    v4f32* dst = reinterpret_cast<v4f32*>(Uc) + (size_t)pm * 3 * vs + cb;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      dst[(size_t)k * vs] = v4f32{m[2 * k].re, m[2 * k].im, m[2 * k + 1].re, m[2 * k + 1].im};
  }
  const C<R> r6 = conj(m[1] * m[5] - m[2] * m[4]);
  const C<R> r7 = conj(m[2] * m[3] - m[0] * m[5]);
  const C<R> r8 = conj(m[0] * m[4] - m[1] * m[3]);
  const R dev = fmax(fmax(fabs(r6.re - m[6].re) + fabs(r6.im - m[6].im),
                          fabs(r7.re - m[7].re) + fabs(r7.im - m[7].im)),
                     fabs(r8.re - m[8].re) + fabs(r8.im - m[8].im));
  if (!(dev <= tol)) *flag = 1;  // also for NaN
}
hipError_t launch_compress_links(const Geom& g, const float2* U32, float2* Uc, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_compress_links<float>, dim3((8 * g.vh + 255) / 256), dim3(256), 0, s, g.vh, g.vs, U32, Uc, flag,
                     1e-5f);
  return hipGetLastError();
}
hipError_t launch_compress_links(const Geom& g, const double2* U64, double2* Uc, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_compress_links<double>, dim3((8 * g.vh + 255) / 256), dim3(256), 0, s, g.vh, g.vs, U64, Uc, flag,
                     kTwoRowTol64);
  return hipGetLastError();
}

// Between FP64 and FP32 (or BF16) fields: a thread takes the four spins of a
// colour, blockIdx.y, at a site (see Planes).
static inline dim3 colour_grid(int vs) { return dim3((vs + 255) / 256, 3); }

// x (FP64) += scale * xs (FP32); xs = 0
__global__ __launch_bounds__(256) void k_mixed_fold(int vs, float2* xs, double2* __restrict__ x,
                                                    const SolverState* st) {
  const int i = blockIdx.x * 256 + threadIdx.x, own = blockIdx.y;
  if (i >= vs) return;
  const double scale = 1.0 / st->sigma;
  C<float> v[4];
  C<double> xv[4];
  Planes<float, float2>::ld(xs, vs, own, i, v);
  ld_colour(x, vs, own, i, xv);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    xv[q].re += scale * (double)v[q].re;
    xv[q].im += scale * (double)v[q].im;
    v[q] = czero<float>();
  }
  st_colour(x, vs, own, i, xv);
  Planes<float, float2>::st(xs, vs, own, i, v);
}
hipError_t launch_mixed_fold(int vs, float2* xs, double2* x, const SolverState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_mixed_fold, colour_grid(vs), dim3(256), 0, s, vs, xs, x, st);
  return hipGetLastError();
}

__global__ __launch_bounds__(1024) void k_reliable_decide(int nblk, const double* __restrict__ partials,
                                                          SolverState* st, Mailbox* mb) {
  double tot[1];
  sum_partials<1024, 1>(partials, nblk, tot);
  if (threadIdx.x != 0) return;
  const double rr64 = tot[0];
  const int entry = st->done;
  st->nupd += 1;
  st->epoch += 1;
  int code = kDoneRunning;
  if (!isfinite(rr64)) {
    code = kDoneFailed;
  } else if (rr64 <= st->rr_target) {
    code = kDoneConverged;
  } else if (entry == kDoneBreakdown && st->restart && st->iter == st->iter_upd) {
    code = kDoneFailed;  // nothing has moved since that restart: another one would repeat it, without end
  } else if (entry == kDoneBreakdown && st->iter >= st->max_iter) {
    code = kDoneMaxIter;  // the recursion looks at the cap only in iterations that do not break down
  } else {
    const double sn = 1.0 / sqrt(rr64);
    st->iter_upd = st->iter;
    st->restart = entry == kDoneBreakdown;
    st->bscale = st->beta * sn / st->sigma;
    st->sigma = sn;
    st->rr = 1.0;
    st->rr0 = 1.0;
    st->rr_max = 1.0;
    st->rr_stop = st->rr_target * sn * sn;
  }
  st->done = code;
  post_progress(mb, st->iter, code != kDoneRunning ? action_word(st->epoch, code) : 0u);
}
hipError_t launch_reliable_decide(int nblk, Reduce red, SolverState* st, hipStream_t s) {
  if (nblk > red.capacity) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_reliable_decide, dim3(1), dim3(1024), 0, s, nblk, red.partials, st, red.mbox);
  return hipGetLastError();
}

// Reliable update of the FP32 recursion: r = sigma r64 (FP64 residual scaled
// to unit norm), and the search direction either restarted (p = r) or
// rescaled to the new units (p *= pscale).
template <typename T>
__device__ __forceinline__ void rescale_site(int vs, const double2* __restrict__ r64, double sigma,
                                             float2* __restrict__ r, T* __restrict__ p, bool restart, double bscale) {
  const int i = blockIdx.x * 256 + threadIdx.x, own = blockIdx.y;
  if (i >= vs) return;
  C<double> v[4];
  C<float> rv[4], pv[4];
  ld_colour(r64, vs, own, i, v);
  if (!restart) Planes<float, T>::ld(p, vs, own, i, pv);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double rx = sigma * v[q].re, ry = sigma * v[q].im;
    rv[q] = {(float)rx, (float)ry};
    pv[q] = restart ? rv[q]
                    : C<float>{(float)(rx + bscale * (double)pv[q].re), (float)(ry + bscale * (double)pv[q].im)};
  }
  Planes<float, float2>::st(r, vs, own, i, rv);
  Planes<float, T>::st(p, vs, own, i, pv);
}
template <typename T>
__global__ __launch_bounds__(256) void k_rescale_residual(int vs, const double2* __restrict__ r64, double sigma,
                                                          float2* __restrict__ r, T* __restrict__ p, int restart,
                                                          double bscale) {
  rescale_site(vs, r64, sigma, r, p, restart != 0, bscale);
}
template <typename T>
hipError_t launch_rescale_residual(int vs, const double2* r64, double sigma, float2* r, T* p, int restart,
                                   double bscale, hipStream_t s) {
  hipLaunchKernelGGL((k_rescale_residual<T>), colour_grid(vs), dim3(256), 0, s, vs, r64, sigma, r, p, restart, bscale);
  return hipGetLastError();
}
template <typename T>
__global__ __launch_bounds__(256) void k_rescale_residual_dev(int vs, const double2* __restrict__ r64,
                                                              float2* __restrict__ r, T* __restrict__ p,
                                                              const SolverState* state) {
  if (state->done != kDoneRunning) return;
  rescale_site(vs, r64, state->sigma, r, p, state->restart != 0, state->bscale);
}
template <typename T>
hipError_t launch_rescale_residual_dev(int vs, const double2* r64, float2* r, T* p, const SolverState* st,
                                       hipStream_t s) {
  hipLaunchKernelGGL((k_rescale_residual_dev<T>), colour_grid(vs), dim3(256), 0, s, vs, r64, r, p, st);
  return hipGetLastError();
}

// FP32 copy of nr FP64 half fields in the batched layout (nr = 1: a half field)
__global__ __launch_bounds__(256) void k_half_64_32(int vs, int nr, const double2* __restrict__ x,
                                                    float2* __restrict__ y) {
  const int i = blockIdx.x * 256 + threadIdx.x, own = blockIdx.y / nr, n = blockIdx.y % nr;
  if (i >= vs) return;
  const size_t ps = (size_t)nr * vs, o = (size_t)n * vs + i;
  C<double> v[4];
  C<float> w[4];
  ld_colour(x, ps, own, o, v);
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = cvt<float>(v[q]);
  Planes<float, float2>::st(y, ps, own, o, w);
}
hipError_t launch_half_64_32(int vs, int nr, const double2* x, float2* y, hipStream_t s) {
  hipLaunchKernelGGL(k_half_64_32, dim3((vs + 255) / 256, 3 * nr), dim3(256), 0, s, vs, nr, x, y);
  return hipGetLastError();
}
template hipError_t launch_rescale_residual_dev<float2>(int, const double2*, float2*, float2*, const SolverState*,
                                                        hipStream_t);
template hipError_t launch_rescale_residual_dev<Bf16c>(int, const double2*, float2*, Bf16c*, const SolverState*,
                                                       hipStream_t);

template hipError_t launch_rescale_residual<float2>(int, const double2*, double, float2*, float2*, int, double,
                                                    hipStream_t);
template hipError_t launch_rescale_residual<Bf16c>(int, const double2*, double, float2*, Bf16c*, int, double,
                                                   hipStream_t);

template hipError_t launch_cg_init<double>(int, const double2*, double2*, double2*, double2*, SolverState*,
                                           Reduce, double, int, hipStream_t);


}  // namespace lgt
