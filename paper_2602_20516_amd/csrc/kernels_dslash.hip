// D psi on the caller's canonical fields, in one launch: the operator of
// lgt_dslash and lgt_dslash_noalloc.
//
// A call that packs U and psi, hops and unpacks moves the links three times
// and the spinors five times, in four launches; each application has new
// links or a new psi from its caller, so nothing of the packing is used
// again.  Here a 256-thread block owns 64 consecutive lexicographic sites and
// wave mu takes both hops along mu for all of them.  A canonical site record
// (192 bytes of spinor, 144 of a link) is read by consecutive lanes -- lane l
// of load i fetches element e = 64 i + l of the wave's 64 records -- and
// transposed through the wave's own strip of LDS to one site a lane; rows of
// 13 (and 9) 16-byte elements keep its reads free of bank conflicts.  Both
// neighbour spinors and the forward link are in flight (33 loads a lane)
// before the first is used, and the backward link follows when the forward
// spinor's registers are free; that hides the latency at two waves per SIMD
// (218 VGPRs: all 42 loads at once take 232 and ran 212 us at 24^3x48 against
// 197; three waves spill, 397 us).  The four directions meet in the same
// strips and the block writes its 64 records as one contiguous span.
// Bound by memory: at 24^3x48 200 us for the 637 MB it cannot do without, of
// 1.13 GB that it moves (neighbour records read again from beyond the L2), 5.6
// TB/s, with the L2's return path busy 80 % of the time (packing, hop and
// unpacking: 454 us); at 4^4, where launches count, 20 -> 11 us a call.
// (Arrays of native vectors: of double2 structs the compiler kept a part in
// scratch, 813 us.)
#include "lgt_internal.h"
#include "lgt_hop.h"

namespace lgt {

namespace {

constexpr int kDS = 64;     // sites per block
constexpr int kPitch = 13;  // LDS row of a spinor record
typedef double v2d __attribute__((ext_vector_type(2)));

// LDS traffic of one wave through its own strip: ordered, no block barrier
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// the wave's 64 spinor records (loads rs, lane-major) -> the lane's own spinor
__device__ __forceinline__ void own_spinor(v2d* strip, int lane, const v2d (&rs)[12], C<double>* psi) {
  wave_sync();
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = 64 * i + lane;
    strip[e + e / 12] = rs[i];
  }
  wave_sync();
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const v2d v = strip[lane * kPitch + k];
    psi[k] = cmk<double>(v.x, v.y);
  }
}
__device__ __forceinline__ M3<double> own_link(v2d* strip, int lane, const v2d (&ru)[9]) {
  wave_sync();
#pragma unroll
  for (int i = 0; i < 9; ++i) strip[64 * i + lane] = ru[i];
  wave_sync();
  M3<double> u;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const v2d v = strip[lane * 9 + k];
    u.m[k] = cmk<double>(v.x, v.y);
  }
  return u;
}

// U h and U^dag h of the two colour vectors of a projected spinor, each
// component as two FMA chains of three products and their sum.  The solves'
// one chain of six (see umul) rounds the growing sum at every step; D psi was
// off by 8.01e-17 with it (against long double, 4^4 to 16^3x12) and by 7.77e-17
// before, with separate complex products.  The two chains, and the directions
// summed in pairs below, give 7.76e-17; the extra instructions are 0.5 % of a
// call at 24^3x48.  S = -1: conj(a).
template <int S>
__device__ __forceinline__ C<double> dot3(C<double> a0, C<double> b0, C<double> a1, C<double> b1, C<double> a2,
                                          C<double> b2) {
  a0.im *= S;
  a1.im *= S;
  a2.im *= S;
  const C<double> p = cmul_f(a0, b0), q = cmul_f(a2, b2);
  return {rfma(a1.re, b1.re, p.re) + rfma(-a1.im, b1.im, q.re), rfma(a1.re, b1.im, p.im) + rfma(a1.im, b1.re, q.im)};
}
__device__ __forceinline__ void link_mul(const M3<double>& U, const C<double>* h, C<double>* w) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const C<double>*u = U.m + 3 * (k % 3), *v = h + 3 * (k / 3);
    w[k] = dot3<1>(u[0], v[0], u[1], v[1], u[2], v[2]);
  }
}
__device__ __forceinline__ void link_mul_dag(const M3<double>& U, const C<double>* h, C<double>* w) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const C<double>*u = U.m + k % 3, *v = h + 3 * (k / 3);
    w[k] = dot3<-1>(u[0], v[0], u[3], v[1], u[6], v[2]);
  }
}

template <int MU, bool DAG, typename F>
__device__ __forceinline__ void both_hops(const Geom& g, int ct, v2d* strip, int lane, const v2d (&pf)[12],
                                          const v2d (&uf)[9], const v2d (&pb)[12], F&& load_ub, C<double>* acc) {
  constexpr int SF = DAG ? +1 : -1;
  C<double> psi[12], h[6], w[6];
  v2d ub[9];
  own_spinor(strip, lane, pf, psi);
  project<double, MU, SF>(psi, h);
  load_ub(ub);
  link_mul(own_link(strip, lane, uf), h, w);
  if (MU == 3 && ct == g.L[3] - 1) apply_bc(g, w);
  reconstruct<double, MU, SF>(w, acc);
  own_spinor(strip, lane, pb, psi);
  project<double, MU, -SF>(psi, h);
  link_mul_dag(own_link(strip, lane, ub), h, w);
  if (MU == 3 && ct == 0) apply_bc(g, w);
  reconstruct<double, MU, -SF>(w, acc);
}

template <bool DAG>
__global__ __launch_bounds__(256, 2) void k_dslash_direct(Geom g, const v2d* __restrict__ U,
                                                          const v2d* __restrict__ psi, v2d* __restrict__ out,
                                                          double kappa, int bps, int tgrp) {
  __shared__ v2d strips[4][kDS * kPitch];
  const int lane = threadIdx.x & 63, mu = threadIdx.x >> 6;
  int blk = xcd_block(blockIdx.x, gridDim.x);
  if (tgrp > 0) {  // t fastest within groups of tgrp slices of bps blocks (see k_hop)
    const int span = tgrp * bps;
    const int grp = blk / span, rem = blk - grp * span;
    const int chunk = rem / tgrp, tl = rem - chunk * tgrp;
    blk = (grp * tgrp + tl) * bps + chunk;
  }
  const int V = 2 * g.vh, s0 = blk * kDS;
  const int s = min(s0 + lane, V - 1);  // lanes past the end repeat the last site
  int c[4];
  lex_coords(g, s, c);
  int st = 1;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (d < mu) st *= g.L[d];
  const int cm = mu == 0 ? c[0] : mu == 1 ? c[1] : mu == 2 ? c[2] : c[3];
  const int lm = mu == 0 ? g.L[0] : mu == 1 ? g.L[1] : mu == 2 ? g.L[2] : g.L[3];
  // the wave's neighbour table lies in its strip until the records need it
  // (a table of its own would cost the third block of a CU)
  v2d* strip = strips[mu];
  int* nbr = reinterpret_cast<int*>(strip);
  nbr[lane] = cm == lm - 1 ? s - (lm - 1) * st : s + st;
  nbr[kDS + lane] = cm == 0 ? s + (lm - 1) * st : s - st;
  wave_sync();
  v2d pf[12], pb[12], uf[9];
  int nj[9];  // sites of the backward links' records
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = 64 * i + lane, j = e / 12, k = e - 12 * j;
    pf[i] = psi[(size_t)nbr[j] * 12 + k];
    pb[i] = psi[(size_t)nbr[kDS + j] * 12 + k];
  }
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    const int e = 64 * i + lane, j = e / 9, k = e - 9 * j;
    uf[i] = U[((size_t)min(s0 + j, V - 1) * 4 + mu) * 9 + k];
    nj[i] = nbr[kDS + j];
  }
  C<double> acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = czero<double>();
  auto load_ub = [&](v2d(&ub)[9]) {
#pragma unroll
    for (int i = 0; i < 9; ++i) ub[i] = U[((size_t)nj[i] * 4 + mu) * 9 + (64 * i + lane) % 9];
  };
  switch (mu) {
    case 0: both_hops<0, DAG>(g, c[3], strip, lane, pf, uf, pb, load_ub, acc); break;
    case 1: both_hops<1, DAG>(g, c[3], strip, lane, pf, uf, pb, load_ub, acc); break;
    case 2: both_hops<2, DAG>(g, c[3], strip, lane, pf, uf, pb, load_ub, acc); break;
    default: both_hops<3, DAG>(g, c[3], strip, lane, pf, uf, pb, load_ub, acc); break;
  }
  wave_sync();
#pragma unroll
  for (int k = 0; k < 12; ++k) strip[lane * kPitch + k] = v2d{acc[k].re, acc[k].im};
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int e = 256 * i + threadIdx.x, j = e / 12;
    if (s0 + j >= V) continue;
    const int o = e + j;  // row j of 13
    const v2d a = strips[0][o], b = strips[1][o], cc = strips[2][o], d = strips[3][o];
    const v2d v = psi[(size_t)s0 * 12 + e];
    const v2d r = {v.x - kappa * ((a.x + b.x) + (cc.x + d.x)), v.y - kappa * ((a.y + b.y) + (cc.y + d.y))};
    __builtin_nontemporal_store(r, out + (size_t)s0 * 12 + e);
  }
}

}  // namespace

hipError_t launch_dslash_direct(const Geom& g, const double2* U, const double2* psi, double2* out, double kappa,
                                bool dag, hipStream_t s) {
  const int V = 2 * g.vh, nb = (V + kDS - 1) / kDS;
  const int slice = V / g.L[3];
  int bps = slice / kDS, tgrp = 0;
  if (slice % kDS == 0 && bps > 0 && g.vh > kHopTOrderMinVh)
    tgrp = g.L[3] % 8 == 0 ? 8 : (g.L[3] % 4 == 0 ? 4 : 2);
  const v2d *u = reinterpret_cast<const v2d*>(U), *in = reinterpret_cast<const v2d*>(psi);
  v2d* o = reinterpret_cast<v2d*>(out);
  if (dag) hipLaunchKernelGGL(k_dslash_direct<true>, dim3(nb), dim3(256), 0, s, g, u, in, o, kappa, bps, tgrp);
  else hipLaunchKernelGGL(k_dslash_direct<false>, dim3(nb), dim3(256), 0, s, g, u, in, o, kappa, bps, tgrp);
  return hipGetLastError();
}

}  // namespace lgt
