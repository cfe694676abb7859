// Two hops of a CG iteration in one launch, for small lattices.
//
// There a hop launch takes about 4 us whatever it computes: the launch, one
// round of loads from beyond the XCD's L2, the LDS exchange and the stores,
// one after the other, on a chip that is mostly idle.  A block here owns the
// eight odd sites of a 2x2x2x2 box.  It applies the first hop at the 40 even
// sites next to them (the box's own eight and four at each of its eight
// faces), exchanges the directions' terms through LDS, and applies the second
// hop from the LDS copy.  The first hop is computed five times over, and the
// iteration is two launches instead of four: FP32 at 8^4 18 -> 12.9 us.
//
// Work split: wave d takes hop direction d = 2 mu + backward, a lane an even
// site (40 of 64); in the second hop a lane takes one of the two spin
// components of the projected spinor of an odd site (16 lanes a wave).  All
// loads but those of the second hop's input are issued before the first
// hop's arithmetic, the block's part of the partial sums included, so that
// one round trip covers them.  With one box a CU the launch is bound by that
// chain (6.2 to 6.7 us, some 2 of them the launch itself), with more by the
// instructions of the first hop (FP32 8^3x16, two boxes a CU: 9.6 us); site
// indices as scalar terms of the box cost 0.6 us more than these per lane.
#include "lgt_hop.h"

namespace lgt {
namespace {

// 16-byte units of a field, as its planes hold them
typedef double v2f64 __attribute__((ext_vector_type(2)));
template <typename R> struct Unit;
template <> struct Unit<double> {
  using V = v2f64;
  static constexpr int N = 12;
  // R2<R> element of a component among the units [N][n] of n sites
  static __device__ __forceinline__ int at(int spin, int colour, int site, int n) {
    return (3 * spin + colour) * n + site;
  }
  static __device__ __forceinline__ double norm2(V v) { return v.x * v.x + v.y * v.y; }
};
template <> struct Unit<float> {
  using V = v4f32;
  static constexpr int N = 6;
  static __device__ __forceinline__ int at(int spin, int colour, int site, int n) {
    return ((2 * colour + (spin >> 1)) * n + site) * 2 + (spin & 1);
  }
  static __device__ __forceinline__ double norm2(V v) {
    return (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
  }
};

constexpr int kBox = 8;    // odd sites of a box
constexpr int kHalo = 40;  // even sites next to them: 8 inside, then [mu][side][4]
constexpr int kPairThreads = 512;

// kPairFresh: t = H p, w = p + k2 H t.  kPairStep: the step of the previous
// iteration first (see EpiStep), t = H r + beta t_old, p = r + beta p.
// kPairSecond: q = w + k2 H t of t = H w, alpha = rr / |w|^2, x += alpha p,
// r -= alpha q.
enum PairMode { kPairFresh, kPairStep, kPairSecond };

// Local coordinates in the box of even site e and of odd site s
__device__ __forceinline__ void halo_local(int e, int l[4]) {
  const int f = (e - kBox) >> 2, mu = f >> 1, side = f & 1;
  const int b0 = e & 1, b1 = (e >> 1) & 1;
  const bool in = e < kBox;
  const int b2 = in ? (e >> 2) & 1 : (b0 + b1 + 1 + side) & 1;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int i = in ? k : (k - mu) & 3;
    l[k] = i == 0 ? (in ? (b0 + b1 + b2) & 1 : side ? 2 : -1) : i == 1 ? b0 : i == 2 ? b1 : b2;
  }
}
__device__ __forceinline__ void odd_local(int s, int l[4]) {
  l[1] = s & 1;
  l[2] = (s >> 1) & 1;
  l[3] = (s >> 2) & 1;
  l[0] = (l[1] + l[2] + l[3] + 1) & 1;
}
// Checkerboard index; it and the extents fit 24 bits (see hop_pair_used)
__device__ __forceinline__ int cb24(const Geom& g, const int c[4]) {
  return (c[0] >> 1) + __mul24(g.hx, c[1] + __mul24(g.L[1], c[2] + __mul24(g.L[2], c[3])));
}
__device__ __forceinline__ int wrap(int v, int L) { return v < 0 ? v + L : v >= L ? v - L : v; }
// the same of the neighbour c + d mu, mu uniform
__device__ __forceinline__ int cb24_shift(const Geom& g, const int c[4], int mu, int d) {
  int n[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) n[k] = mu == k ? wrap(c[k] + d, g.L[k]) : c[k];
  return cb24(g, n);
}

// An even site's index among the block's 40: of the neighbour l + d mu of
// the odd site at l
template <int MU>
__device__ __forceinline__ int halo_index(const int l[4], int d) {
  const int v = l[MU] + d;
  if (v == -1 || v == 2)
    return kBox + 4 * (2 * MU + (v == 2)) + l[(MU + 1) & 3] + 2 * l[(MU + 2) & 3];
  int n[4] = {l[0], l[1], l[2], l[3]};
  n[MU] = v;
  return n[1] + 2 * n[2] + 4 * n[3];
}

// The stored rows of U_mu of parity p at cb (load_link without the rebuilt row)
template <typename R>
__device__ __forceinline__ M3<R> load_rows(const R2<R>* __restrict__ gauge, int nk, const Geom& g, int p, int mu,
                                           int cb) {
  constexpr unsigned E = sizeof(R2<R>);
  const unsigned gs = (unsigned)g.vs * E;
  const BufRsrc ru = make_rsrc(gauge + (size_t)((p * 4 + mu) * nk) * g.vs, (size_t)nk * gs);
  M3<R> U;
  if (nk == 9) {
#pragma unroll
    for (int k = 0; k < 9; ++k) U.m[k] = ld_buf<R>(ru, (unsigned)cb * E, k * gs);
  } else {
    load_two_rows<R, false>(ru, (unsigned)cb * 16u, (unsigned)g.vs * 16u, U);
  }
  return U;
}

template <typename R> struct PairArgs {
  const R2<R>* in;     // odd half the first hop reads: p, r or w
  const R2<R>* t_old;  // even half (step)
  R2<R>* t_new;        // even half (fresh, step)
  R2<R>*p, *w, *x, *r;
  R k2;
  SolverState* st;
  const double* sums;  // block partials the launch sums: |r|^2 (step), |w|^2 (second)
  int nsums;
  double* partials;  // block partials it leaves: |w|^2 (fresh, step), |r|^2 (second)
  Mailbox* mb;
};

// The second hop along MU: lane (site, a) takes component a of the two of
// the projected spinor.  tsh: units [N][kHalo] of the first hop; out: units
// [N][kBox] of this direction's term.
template <typename R, int MU>
__device__ __forceinline__ void second_hop(const Geom& g, const R2<R>* tsh, R2<R>* out, const M3<R>& U, bool bwd, R s,
                                           int site, int a, const int l[4], int ct) {
  using Un = Unit<R>;
  const int e = halo_index<MU>(l, bwd ? -1 : 1);
  const int dn = MU < 2 ? 1 - a : a;  // the lower spin that B_mu joins to upper spin a
  const R sa = a ? s : -s;
  C<R> h[3], w[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const C<R> u = ld<R>(tsh + Un::at(a, i, e, kHalo)), d = ld<R>(tsh + Un::at(2 + dn, i, e, kHalo));
    if constexpr (MU == 0) h[i] = u - s * itimes(d);
    else if constexpr (MU == 1) h[i] = u + sa * d;
    else if constexpr (MU == 2) h[i] = u + sa * itimes(d);
    else h[i] = u + s * d;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (bwd) {
      w[i] = cjmul_f(U.m[i], h[0]);
      w[i] = cjmac(w[i], U.m[3 + i], h[1]);
      w[i] = cjmac(w[i], U.m[6 + i], h[2]);
    } else {
      w[i] = cmul_f(U.m[3 * i], h[0]);
      w[i] = cmac(w[i], U.m[3 * i + 1], h[1]);
      w[i] = cmac(w[i], U.m[3 * i + 2], h[2]);
    }
  }
  if (MU == 3 && ct == (bwd ? 0 : g.L[3] - 1)) {
#pragma unroll
    for (int i = 0; i < 3; ++i) w[i] = R(g.bc) * w[i];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    st<R>(out + Un::at(a, i, site, kBox), w[i]);
    C<R> d;
    if constexpr (MU == 0) d = s * itimes(w[i]);
    else if constexpr (MU == 1) d = sa * w[i];
    else if constexpr (MU == 2) d = -sa * itimes(w[i]);
    else d = s * w[i];
    st<R>(out + Un::at(2 + dn, i, site, kBox), d);
  }
}

template <typename R, bool DAG, int MODE>
__global__ __launch_bounds__(kPairThreads) void k_hop_pair(Geom g, const R2<R>* __restrict__ gauge, int nk,
                                                           PairArgs<R> a) {
  using P = Planes<R, R2<R>>;
  using Un = Unit<R>;
  using V = typename Un::V;
  constexpr int N = Un::N;
  __shared__ V part[8][N][kHalo];
  __shared__ V tsh[N][kHalo];
  __shared__ double wsum[8];
  __shared__ int s_done;
  const int tid = threadIdx.x, lane = tid & 63;
  const int dir = __builtin_amdgcn_readfirstlane(tid >> 6), mu = dir >> 1;
  const bool bwd = dir & 1;
  const R s = R((DAG ? 1 : -1) * (bwd ? -1 : 1));
  const int hy = blockIdx.x / g.hx;
  const int o[4] = {2 * ((int)blockIdx.x - hy * g.hx), 2 * hy, 2 * (int)blockIdx.y, 2 * (int)blockIdx.z};
  const int lb = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  SolverState* st = a.st;

  // ---- loads of the first hop along this wave's direction, at even site e
  const int e = lane < kHalo ? lane : kHalo - 1;
  int c[4];
  halo_local(e, c);
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = wrap(o[k] + c[k], g.L[k]);
  const int cbe = cb24(g, c), nb = cb24_shift(g, c, mu, bwd ? -1 : 1);
  const auto in = make_spinor_in<R, R2<R>>(a.in, g);
  C<R> psi[12], h[6], w[6];
  in.all(in.off(nb), psi);
  M3<R> U = load_rows<R>(gauge, nk, g, bwd ? 1 : 0, mu, bwd ? nb : cbe);

  // ---- every other load but the second hop's input
  // Stopped or not: the step takes what the second launch of its iteration
  // recorded (done itself is block 0's to set below, while other blocks may
  // only be starting); in the second launch block 0 may set a breakdown
  // meanwhile, so one thread reads for its block.
  const int found = MODE == kPairStep ? st->done_prev : st->done;
  if (tid == 0) s_done = found;
  const bool rec = lb == 0 && tid == 0;
  const double rr_in = MODE == kPairSecond ? st->rr : st->rr_prev;
  const int iter_in = MODE == kPairSecond ? st->iter : st->iter_prev;
  const double rr_max0 = st->rr_max, rr_stop = st->rr_stop, delta2 = st->delta2;
  const int max_iter = st->max_iter;
  double sum = 0.0;
  if constexpr (MODE != kPairFresh) {
    for (int i = tid; i < a.nsums; i += kPairThreads) sum += a.sums[i];
  }
  // wave d sums the first hop's units d and d + 8 (if there are any), a lane an even site
  constexpr int kJ = (N + 7) / 8;
  V told[kJ];
#pragma unroll
  for (int j = 0; j < kJ; ++j) {
    if (MODE == kPairStep && dir + 8 * j < N)
      told[j] = reinterpret_cast<const V*>(a.t_old)[(size_t)(dir + 8 * j) * g.vs + cbe];
  }
  // odd site of this lane in the second hop and in the epilogue (48 lanes of
  // wave 0, kK units each)
  const int site = lane & 7;
  int l2[4], c2[4];
  odd_local(site, l2);
#pragma unroll
  for (int k = 0; k < 4; ++k) c2[k] = o[k] + l2[k];
  const int cbo = cb24(g, c2);
  M3<R> U2;
  if (lane < 16) U2 = load_rows<R>(gauge, nk, g, bwd ? 0 : 1, mu, bwd ? cb24_shift(g, c2, mu, -1) : cbo);
  constexpr int kK = N * kBox / 48;
  V ep[kK], er[kK], ew[kK], ex[kK];
  size_t eo[kK];
  const bool epi = dir == 0 && lane < 48;
  if (epi) {
#pragma unroll
    for (int k = 0; k < kK; ++k) {
      eo[k] = (size_t)((lane >> 3) + 6 * k) * g.vs + cbo;
      ep[k] = reinterpret_cast<const V*>(a.p)[eo[k]];
      if constexpr (MODE != kPairFresh) er[k] = reinterpret_cast<const V*>(a.r)[eo[k]];
      if constexpr (MODE == kPairSecond) {
        ew[k] = reinterpret_cast<const V*>(a.w)[eo[k]];
        ex[k] = reinterpret_cast<const V*>(a.x)[eo[k]];
      }
    }
  }

  asm volatile("" ::: "memory");  // the loads are issued before the wait for what was found
  if (found != kDoneRunning && (MODE != kPairSecond || found != kDoneBreakdown)) {
    if (MODE == kPairSecond && rec) st->done_prev = found;
    if (MODE == kPairStep && rec) {
      if (found == kDoneUpdate) st->done = kDoneUpdateHeld;
      post_progress(a.mb, st->iter, action_word(st->epoch, found == kDoneUpdateHeld ? kDoneUpdate : found));
    }
    return;
  }

  // ---- first hop
  switch (mu) {
    case 0: project_s<R, 0>(psi, s, h); break;
    case 1: project_s<R, 1>(psi, s, h); break;
    case 2: project_s<R, 2>(psi, s, h); break;
    default: project_s<R, 3>(psi, s, h); break;
  }
  if (nk == 6) third_row(U);
  if (bwd) umul_dag(U, h, w);
  else umul(U, h, w);
  if (mu == 3 && c[3] == (bwd ? 0 : g.L[3] - 1)) apply_bc(g, w);
  {
    C<R> acc[12];
#pragma unroll
    for (int i = 0; i < 3; ++i) {  // reconstruct
      acc[i] = w[i];
      acc[3 + i] = w[3 + i];
      const C<R> a0 = mu < 2 ? w[3 + i] : w[i], a1 = mu < 2 ? w[i] : w[3 + i];
      const R s0 = s, s1 = mu == 1 || mu == 2 ? -s : s;
      const bool im = mu == 0 || mu == 2;
      acc[6 + i] = s0 * (im ? itimes(a0) : a0);
      acc[9 + i] = s1 * (im ? itimes(a1) : a1);
    }
    if (lane < kHalo) {
#pragma unroll
      for (int own = 0; own < P::kOwners; ++own) {
        C<R> v[P::NC];
#pragma unroll
        for (int q = 0; q < P::NC; ++q) v[q] = acc[P::comp(own, q)];
        P::st(reinterpret_cast<R2<R>*>(&part[dir][0][0]), kHalo, own, lane, v);
      }
    }
  }
  if constexpr (MODE != kPairFresh) {
    sum = wave_sum(sum);
    if (lane == 0) wsum[dir] = sum;
  }
  __syncthreads();

  // ---- the scalars, alike in every thread
  R beta = 0, alpha = 0;
  if (MODE == kPairSecond && s_done != kDoneRunning) {
    if (rec) st->done_prev = s_done;
    return;
  }
  if constexpr (MODE != kPairFresh) {
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) tot += wsum[k];
    if constexpr (MODE == kPairStep) {
      const double b = tot / rr_in, rr_max = fmax(rr_max0, tot);
      const int iter = iter_in + 1;
      int code = kDoneRunning;
      if (!isfinite(tot)) code = kDoneBreakdown;
      else if (tot <= rr_stop) code = delta2 > 0.0 ? kDoneUpdate : kDoneConverged;
      else if (tot <= delta2 * rr_max) code = kDoneUpdate;
      else if (iter >= max_iter) code = kDoneMaxIter;
      if (rec) {
        st->beta = b;
        st->rr = tot;
        st->iter = iter;
        st->rr_max = rr_max;
        if (code != kDoneRunning) st->done = code;
        post_progress(a.mb, iter, code != kDoneRunning ? action_word(st->epoch, code) : 0u);
      }
      if (code != kDoneRunning) return;
      beta = R(b);
    } else {
      const bool ok = tot > 0.0 && isfinite(tot);
      const double al = ok ? rr_in / tot : 0.0;
      if (rec) {
        st->pap = tot;
        st->rr_prev = rr_in;
        st->iter_prev = iter_in;
        st->alpha = al;
        st->done_prev = ok ? kDoneRunning : kDoneBreakdown;
        if (!ok) st->done = kDoneBreakdown;
      }
      if (!ok) return;  // x and r stay as they were (0 times a non-finite p or q is not 0), in every block
      alpha = R(al);
    }
  }

  // ---- t on the 40 even sites
#pragma unroll
  for (int j = 0; j < kJ; ++j) {
    const int u = dir + 8 * j;
    if (u < N && lane < kHalo) {
      V t = part[0][u][lane];
#pragma unroll
      for (int d = 1; d < 8; ++d) t += part[d][u][lane];
      if constexpr (MODE == kPairStep) t += beta * told[j];
      tsh[u][lane] = t;
      if constexpr (MODE != kPairSecond) {
        if (lane < kBox) reinterpret_cast<V*>(a.t_new)[(size_t)u * g.vs + cbe] = t;
      }
    }
  }
  __syncthreads();

  // ---- second hop at the eight odd sites
  if (lane < 16) {
    if (nk == 6) third_row(U2);
    const R2<R>* in = reinterpret_cast<const R2<R>*>(&tsh[0][0]);
    R2<R>* out = reinterpret_cast<R2<R>*>(&part[dir][0][0]);
    const int ah = lane >> 3;
    switch (mu) {
      case 0: second_hop<R, 0>(g, in, out, U2, bwd, s, site, ah, l2, c2[3]); break;
      case 1: second_hop<R, 1>(g, in, out, U2, bwd, s, site, ah, l2, c2[3]); break;
      case 2: second_hop<R, 2>(g, in, out, U2, bwd, s, site, ah, l2, c2[3]); break;
      default: second_hop<R, 3>(g, in, out, U2, bwd, s, site, ah, l2, c2[3]); break;
    }
  }
  __syncthreads();
  if (dir != 0) return;
  double red = 0.0;
  if (epi) {
#pragma unroll
    for (int k = 0; k < kK; ++k) {
      const int u = lane + 48 * k;
      V acc = (&part[0][0][0])[u];
#pragma unroll
      for (int d = 1; d < 8; ++d) acc += (&part[d][0][0])[u];
      if constexpr (MODE == kPairSecond) {
        const V q = ew[k] + a.k2 * acc, r = er[k] - alpha * q;
        reinterpret_cast<V*>(a.x)[eo[k]] = ex[k] + alpha * ep[k];
        reinterpret_cast<V*>(a.r)[eo[k]] = r;
        red += Un::norm2(r);
      } else {
        V p = ep[k];
        if constexpr (MODE == kPairStep) {
          p = er[k] + beta * p;
          reinterpret_cast<V*>(a.p)[eo[k]] = p;
        }
        const V w = p + a.k2 * acc;
        reinterpret_cast<V*>(a.w)[eo[k]] = w;
        red += Un::norm2(w);
      }
    }
  }
  red = wave_sum(red);
  if (lane == 0) a.partials[lb] = red;
}

template <typename R, bool DAG, int MODE>
hipError_t launch(const Geom& g, const R2<R>* gauge, int nk, const PairArgs<R>& a, hipStream_t s) {
  const dim3 grid(g.hx * (g.L[1] / 2), g.L[2] / 2, g.L[3] / 2);
  hipLaunchKernelGGL((k_hop_pair<R, DAG, MODE>), grid, dim3(kPairThreads), 0, s, g, gauge, nk, a);
  return hipGetLastError();
}

}  // namespace

bool hop_pair_used(const Geom& g, size_t elem) {
  return g.hop_ns == 0 && g.vh <= (elem == sizeof(float2) ? kHopPairMaxVh32 : kHopPairMaxVh64);
}

template <typename R, bool DAG>
hipError_t launch_hop_pair_first(const Geom& g, const R2<R>* gauge, int nk, bool fresh, const R2<R>* t_old,
                                 R2<R>* t_new, R2<R>* w, R2<R>* p, const R2<R>* r, double k2, SolverState* st,
                                 Reduce red, hipStream_t s) {
  const int nb = g.vh / kBox;
  if (nb > red.capacity || (size_t)2 * red.capacity > red.ndoubles) return hipErrorInvalidValue;
  PairArgs<R> a{};
  a.in = fresh ? p : r;
  a.t_old = t_old;
  a.t_new = t_new;
  a.p = p;
  a.w = w;
  a.r = const_cast<R2<R>*>(r);
  a.k2 = R(k2);
  a.st = st;
  a.sums = red.partials;
  a.nsums = nb;
  a.partials = red.partials + red.capacity;
  a.mb = red.mbox;
  return fresh ? launch<R, DAG, kPairFresh>(g, gauge, nk, a, s) : launch<R, DAG, kPairStep>(g, gauge, nk, a, s);
}

template <typename R, bool DAG>
hipError_t launch_hop_pair_second(const Geom& g, const R2<R>* gauge, int nk, const R2<R>* w, R2<R>* x, R2<R>* r,
                                  const R2<R>* p, double k2, SolverState* st, Reduce red, hipStream_t s) {
  const int nb = g.vh / kBox;
  if (nb > red.capacity || (size_t)2 * red.capacity > red.ndoubles) return hipErrorInvalidValue;
  PairArgs<R> a{};
  a.in = w;
  a.p = const_cast<R2<R>*>(p);
  a.w = const_cast<R2<R>*>(w);
  a.x = x;
  a.r = r;
  a.k2 = R(k2);
  a.st = st;
  a.sums = red.partials + red.capacity;
  a.nsums = nb;
  a.partials = red.partials;
  return launch<R, DAG, kPairSecond>(g, gauge, nk, a, s);
}

#define LGT_PAIR(R, DAG)                                                                                             \
  template hipError_t launch_hop_pair_first<R, DAG>(const Geom&, const R2<R>*, int, bool, const R2<R>*, R2<R>*,      \
                                                    R2<R>*, R2<R>*, const R2<R>*, double, SolverState*, Reduce,      \
                                                    hipStream_t);                                                    \
  template hipError_t launch_hop_pair_second<R, DAG>(const Geom&, const R2<R>*, int, const R2<R>*, R2<R>*, R2<R>*,   \
                                                     const R2<R>*, double, SolverState*, Reduce, hipStream_t);
LGT_PAIR(float, false)
LGT_PAIR(float, true)
LGT_PAIR(double, false)
LGT_PAIR(double, true)
#undef LGT_PAIR

}  // namespace lgt
