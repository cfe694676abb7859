// Wilson hop H_{p,1-p} on the even/odd lattice, with the epilogues the
// solver fuses into it.
//
//   (H psi)(x) = sum_mu [ (1 - gamma_mu) U~_mu(x) psi(x+mu) + (1 + gamma_mu) U~_mu(x-mu)^dag psi(x-mu) ]
//   (H^dag: the signs of gamma_mu flip)
//
// so that D = 1 - kappa H (the operator of the pseudofermion action, S3.1).
//
// Work decomposition (gfx950): a 256-thread block owns 64 consecutive
// checkerboard sites of one parity; wave w (= direction mu) computes both
// hops along mu for the 64 sites, using the chiral-basis spin projection
// (1 + s gamma_mu) psi = (h ; s B_mu^dag h), h = psi_up + s B_mu psi_dn, so
// only two colour vectors go through each SU(3) multiply.  The four
// per-direction partial spinors meet in LDS and wave w then owns a part of the
// components of the 64 output sites for the epilogue (see Planes: spin w in
// FP64, colour w otherwise), so every global load and store is a unit-stride
// access of 16 bytes a lane.
// Small lattices use 32-site blocks instead, whose half-waves take the
// forward and the backward hop (unit-stride 32-lane halves).
// Blocks are numbered XCD-contiguously (see xcd_block).
#include "lgt_internal.h"
#include "lgt_hop.h"

namespace lgt {

// ---------------------------------------------------------------------------
// Epilogues.  apply() gets the components of owner `own` of the hop result at
// (p, cb) (see Planes); red accumulates this thread's reduction contribution.
// T is the storage type of the spinors t, w, p of the CG (R2<R> or Bf16c);
// x and r are always R2<R>, with the same owners.  vh: plane stride.
// ---------------------------------------------------------------------------
template <typename R, typename T>
struct EpiAxpy {  // out = self + coef * acc
  static constexpr bool kReduce = false;
  static constexpr bool kPrefetch = !std::is_same<T, Bf16c>::value;
  T* out[2];
  const T* self[2];
  R coef;
  int vh;
  SolverState* guard;  // if set, the launch is a no-op once the solve has stopped
  // If set, block 0 also turns the |w|^2 block partials of the previous
  // launch into pap and alpha = rr / pap (the CG step between the two hops
  // of Mhat^dag Mhat, which need no scalar).
  const double* pap_partials;
  int pap_nblk;
  __device__ bool skip() const {
    if (!guard || guard->done == kDoneRunning) return false;
    if (pap_partials && blockIdx.x == 0 && threadIdx.x == 0) guard->done_prev = guard->done;
    return true;
  }
  using P = Planes<R, T>;
  static constexpr int NC = P::NC;
  struct Pre {
    C<R> s[NC];
  };
  __device__ Pre pre(int p, int cb, int own) const {
    Pre q{};
    if (self[p]) P::ld(self[p], vh, own, cb, q.s);
    return q;
  }
  __device__ void apply(int p, int cb, int own, const C<R>* acc, double&, const Pre& q) const {
    C<R> v[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) v[i] = q.s[i] + coef * acc[i];
    P::st(out[p], vh, own, cb, v);
  }
  template <int NT>
  __device__ void tail() const {
    if (!pap_partials || blockIdx.x != 0) return;
    double tot[1];
    sum_partials<NT, 1>(pap_partials, pap_nblk, tot);
    if (threadIdx.x == 0) {
      const double pap = tot[0];
      guard->pap = pap;
      guard->rr_prev = guard->rr;
      guard->iter_prev = guard->iter;
      if (!(pap > 0.0) || !isfinite(pap)) {
        guard->alpha = 0.0;
        guard->done = kDoneBreakdown;
        guard->done_prev = kDoneBreakdown;
      } else {
        guard->alpha = guard->rr / pap;
        guard->done_prev = kDoneRunning;
      }
    }
  }
};

// First hop of a CG iteration with the previous iteration's step folded in
// (FP64 and FP32-stored recursions).  Every block first sums the |r|^2
// partials the previous iteration's last hop wrote (same partials, same
// order: every block takes the same decision) into rr, beta = rr / rr_prev
// and the stop test; block 0 records the state and posts to the mailbox.
// If the recursion goes on, the hop runs on r instead of p, using
// H p_new = H (r + beta p) = H r + beta H p, with H p the t of the previous
// iteration (kept in t, which the iteration's second use of the even half
// does not overwrite), and each thread updates p = r + beta p at the odd
// sites of its own (site, spin): the hop reads only r, so the update races
// with no reader.  One launch and one pass over r and p fewer per iteration
// than a separate step kernel.  A launch finding the solve stopped returns
// (block 0 turns kDoneUpdate into kDoneUpdateHeld and repeats the action).
template <typename R>
struct EpiStep {
  static constexpr bool kReduce = false;
  static constexpr bool kPrefetch = true;
  R2<R>* t;         // even half: H p, updated in place
  R2<R>* p;         // odd half: search direction
  const R2<R>* r;   // odd half: residual (the hop's input)
  int vh;
  SolverState* state;
  const double* partials;
  int nblk;
  Mailbox* mb;
  __device__ static double& beta_sh() {
    __shared__ double b;
    return b;
  }
  __device__ bool skip() const {  // block-collective: every thread of the block calls it
    __shared__ int s_run;
    SolverState* st = state;
    // what the third hop recorded: done itself is block 0's to set below, while
    // other blocks, or waves of them, may only be starting
    const int done0 = st->done_prev;
    if (done0 != kDoneRunning) {
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (done0 == kDoneUpdate) st->done = kDoneUpdateHeld;
        post_progress(mb, st->iter, action_word(st->epoch, done0 == kDoneUpdateHeld ? kDoneUpdate : done0));
      }
      return true;
    }
    double tot[1];
    sum_partials<256, 1>(partials, nblk, tot);
    if (threadIdx.x == 0) {
      const double rr = tot[0];
      const double beta = rr / st->rr_prev;
      const int iter = st->iter_prev + 1;
      const double rr_max = fmax(st->rr_max, rr);
      int code = kDoneRunning;
      if (!isfinite(rr)) code = kDoneBreakdown;
      else if (rr <= st->rr_stop) code = st->delta2 > 0.0 ? kDoneUpdate : kDoneConverged;
      else if (rr <= st->delta2 * rr_max) code = kDoneUpdate;
      else if (iter >= st->max_iter) code = kDoneMaxIter;
      beta_sh() = beta;
      s_run = code == kDoneRunning;
      if (blockIdx.x == 0) {
        st->beta = beta;
        st->rr = rr;
        st->iter = iter;
        st->rr_max = rr_max;
        if (code != kDoneRunning) st->done = code;
        post_progress(mb, iter, code != kDoneRunning ? action_word(st->epoch, code) : 0u);
      }
    }
    __syncthreads();
    return !s_run;
  }
  using P = Planes<R, R2<R>>;
  static constexpr int NC = P::NC;
  struct Pre {
    C<R> t[NC], r[NC], p[NC];
  };
  __device__ Pre pre(int, int cb, int own) const {
    Pre q;
    P::ld(t, vh, own, cb, q.t);
    P::ld(r, vh, own, cb, q.r);
    P::ld(p, vh, own, cb, q.p);
    return q;
  }
  __device__ void apply(int, int cb, int own, const C<R>* acc, double&, const Pre& q) const {
    const R b = R(beta_sh());
    C<R> tn[NC], pn[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      tn[i] = acc[i] + b * q.t[i];
      pn[i] = q.r[i] + b * q.p[i];
    }
    P::st(t, vh, own, cb, tn);
    P::st(p, vh, own, cb, pn);
  }
  template <int NT>
  __device__ void tail() const {}
};

// First hop of a multi-shift iteration: t = H (r + beta p) = H r + beta t and
// p = r + beta p as in EpiStep, with beta and the stop decision from the
// state, where the finalize that advances the shifts has left them.
struct EpiDirection {
  using P = Planes<double, double2>;
  static constexpr bool kReduce = false;
  static constexpr bool kPrefetch = true;
  double2* t;
  double2* p;
  const double2* r;
  int vh;
  const SolverState* state;
  __device__ bool skip() const { return state->done != kDoneRunning; }
  struct Pre {
    C<double> t[3], r[3], p[3];
  };
  __device__ Pre pre(int, int cb, int spin) const {
    Pre q;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const size_t o = (size_t)(3 * spin + i) * vh + cb;
      q.t[i] = ld<double>(t + o);
      q.r[i] = ld<double>(r + o);
      q.p[i] = ld<double>(p + o);
    }
    return q;
  }
  __device__ void apply(int, int cb, int spin, const C<double>* acc, double&, const Pre& q) const {
    const double b = state->beta;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const size_t o = (size_t)(3 * spin + i) * vh + cb;
      lgt::st<double>(t + o, acc[i] + b * q.t[i]);
      lgt::st<double>(p + o, q.r[i] + b * q.p[i]);
    }
  }
  template <int NT>
  __device__ void tail() const {}
};

// Last hop of a shifted true residual: block partials of
// |phi - (w + coef * acc) - sigma x|^2 (odd sites); nothing is stored.
struct EpiShiftResidual {
  using P = Planes<double, double2>;
  static constexpr bool kReduce = true;
  static constexpr bool kPrefetch = true;
  const double2* w;
  const double2* x;
  const double2* phi;
  double sigma, coef;
  int vh;
  __device__ bool skip() const { return false; }
  struct Pre {
    C<double> w[3], x[3], f[3];
  };
  __device__ Pre pre(int, int cb, int spin) const {
    Pre q;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const size_t o = (size_t)(3 * spin + i) * vh + cb;
      q.w[i] = ld<double>(w + o);
      q.x[i] = ld<double>(x + o);
      q.f[i] = ld<double>(phi + o);
    }
    return q;
  }
  __device__ void apply(int, int, int, const C<double>* acc, double& red, const Pre& q) const {
#pragma unroll
    for (int i = 0; i < 3; ++i) red += norm2(q.f[i] - ((q.w[i] + coef * acc[i]) + sigma * q.x[i]));
  }
  template <int NT>
  __device__ void tail() const {}
};

// Last hop of r = phi - Mhat^dag Mhat x (odd sites), block partials of |r|^2:
// the subtraction and the norm of a reliable update were two passes over the
// field (24^3x48: 29 + 13 us, of 93 beside the update's hops).
struct EpiSchurResidual {
  using P = Planes<double, double2>;
  static constexpr bool kReduce = true;
  static constexpr bool kPrefetch = true;
  const double2* w;
  const double2* phi;
  double2* r;
  double coef;
  int vh;
  __device__ bool skip() const { return false; }
  struct Pre {
    C<double> w[3], f[3];
  };
  __device__ Pre pre(int, int cb, int own) const {
    Pre q;
    P::ld(w, vh, own, cb, q.w);
    P::ld(phi, vh, own, cb, q.f);
    return q;
  }
  __device__ void apply(int, int cb, int own, const C<double>* acc, double& red, const Pre& q) const {
    C<double> v[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      v[i] = q.f[i] - (q.w[i] + coef * acc[i]);
      red += norm2(v[i]);
    }
    P::st(r, vh, own, cb, v);
  }
  template <int NT>
  __device__ void tail() const {}
};

template <typename R, typename T>
struct EpiSchurNorm {  // w = x + coef * acc (odd sites), block partials of |w|^2 (of w as stored)
  static constexpr bool kReduce = true;
  static constexpr bool kPrefetch = true;
  T* w;
  const T* x;
  R coef;
  int vh;
  SolverState* state;
  __device__ bool skip() const { return state->done != kDoneRunning; }
  using P = Planes<R, T>;
  static constexpr int NC = P::NC;
  struct Pre {
    C<R> x[NC];
  };
  __device__ Pre pre(int, int cb, int own) const {
    Pre q;
    P::ld(x, vh, own, cb, q.x);
    return q;
  }
  __device__ void apply(int, int cb, int own, const C<R>* acc, double& red, const Pre& q) const {
    C<R> v[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      v[i] = Store<R, T>::round(q.x[i] + coef * acc[i]);
      red += (double)v[i].re * (double)v[i].re + (double)v[i].im * (double)v[i].im;
    }
    P::st(w, vh, own, cb, v);
  }
  template <int NT>
  __device__ void tail() const {}
};

template <typename R, typename T>
struct EpiSchurCG {  // q = w + coef * acc; x += alpha p (if x); ro = r - alpha q; block partials of |ro|^2
  static constexpr bool kReduce = true;
  static constexpr bool kPrefetch = !std::is_same<T, Bf16c>::value;
  const T* w;
  R2<R>* x;
  const R2<R>* r;
  R2<R>* ro;  // may be r
  const T* p;
  R coef;
  int vh;
  SolverState* state;
  __device__ bool skip() const { return state->done != kDoneRunning; }
  using P = Planes<R, T>;        // w, p
  using PR = Planes<R, R2<R>>;   // x, r
  static constexpr int NC = P::NC;
  struct Pre {
    C<R> w[NC], x[NC], r[NC], p[NC];
  };
  __device__ Pre pre(int, int cb, int own) const {
    Pre q;
    P::ld(w, vh, own, cb, q.w);
    PR::ld(r, vh, own, cb, q.r);
    if (x) {
      PR::ld(x, vh, own, cb, q.x);
      P::ld(p, vh, own, cb, q.p);
    }
    return q;
  }
  __device__ void apply(int, int cb, int own, const C<R>* acc, double& red, const Pre& pq) const {
    const R alpha = R(state->alpha);
    C<R> rv[NC], xv[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const C<R> q = pq.w[i] + coef * acc[i];
      rv[i] = pq.r[i] - alpha * q;
      red += (double)rv[i].re * (double)rv[i].re + (double)rv[i].im * (double)rv[i].im;
    }
    if (x) {
#pragma unroll
      for (int i = 0; i < NC; ++i) xv[i] = pq.x[i] + alpha * pq.p[i];
      PR::st(x, vh, own, cb, xv);
    }
    PR::st(ro, vh, own, cb, rv);
  }
  template <int NT>
  __device__ void tail() const {}
};

struct EpiResidual {  // r = phi - (self + coef * acc) over both parities, block partials of |r|^2
  using P = Planes<double, double2>;
  static constexpr bool kReduce = true;
  static constexpr bool kPrefetch = true;
  const double2* self[2];
  const double2* phi[2];
  double2* r[2];
  double coef;
  int vh;
  __device__ bool skip() const { return false; }
  struct Pre {
    C<double> f[3], s[3];
  };
  __device__ Pre pre(int p, int cb, int spin) const {
    Pre q;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const size_t o = (size_t)(3 * spin + i) * vh + cb;
      q.f[i] = ld<double>(phi[p] + o);
      q.s[i] = ld<double>(self[p] + o);
    }
    return q;
  }
  __device__ void apply(int p, int cb, int spin, const C<double>* acc, double& red, const Pre& q) const {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const size_t o = (size_t)(3 * spin + i) * vh + cb;
      C<double> v = q.f[i] - (q.s[i] + coef * acc[i]);
      st<double>(r[p] + o, v);
      red += norm2(v);
    }
  }
  template <int NT>
  __device__ void tail() const {}
};

// ---------------------------------------------------------------------------
// The hop kernel.  Grid: nbp blocks per parity (p_fixed >= 0) or 2*nbp
// (p_fixed < 0, parity = logical block / nbp).  NS = 64: wave mu computes
// both hops along mu for 64 sites.  NS = 32 (small lattices, whose 64-site
// grid would not give every SIMD a wave): wave mu computes the forward hop
// of 32 sites on lanes 0-31 and their backward hop on lanes 32-63, so twice
// as many waves share the latency; waves 0 and 1 then run the epilogue, one
// (site, spin) pair per lane.
//
// Block order (64-site blocks, when a t-slice holds a whole number of
// blocks: bps blocks per slice, tgrp > 0).  Checkerboard sites are x-fastest,
// so in site order a site's t-neighbours are a whole slice away, and on
// large lattices the L2 of an XCD has streamed the slice's links and
// spinors out again before the second read.  The blocks of each group of
// tgrp consecutive slices are therefore taken t-fastest: block j of the
// group covers slice j % tgrp, chunk j / tgrp of that slice, so the t-hops
// of a chunk are a few blocks apart and its z-hops 8 tgrp blocks apart.  A
// bijection of the blocks of a parity: every site is still covered once.
//
// Hops onto odd sites take each XCD's blocks last first.  Hops alternate in
// parity, so a hop starts where the one before it ended, and finds the links
// and spinors of that end in the memory-side cache, which a hop of a large
// lattice has streamed through (FP64 solve at 32^3x64: |w|^2 hop 303 -> 281
// us, CG hop 332 -> 308; FP32 at 16^3x64 15.9 -> 14.4 and 16.9 -> 15.7; BF16
// at 24^3x48 27.9 -> 26.6 and 31.8 -> 30.4; mixed FP32 force at 16^4 5.81 ->
// 5.28 ms, where the XCD's own L2 holds part of that end).
// ---------------------------------------------------------------------------
// A wave's partial hops in LDS: the planes of a half field of 64 sites, which
// are written and read as vectors of 16 bytes (an array of float2 alone is
// only aligned to 8).
template <typename R>
struct alignas(16) HopStrip {
  R2<R> v[12 * 64];
};
// The strip of a wave's hops, and an owner's part of them back.
template <typename R>
__device__ __forceinline__ void put_hops(HopStrip<R>& l, int lane, const C<R>* acc) {
  using P = Planes<R, R2<R>>;
#pragma unroll
  for (int own = 0; own < P::kOwners; ++own) {
    C<R> v[P::NC];
#pragma unroll
    for (int q = 0; q < P::NC; ++q) v[q] = acc[P::comp(own, q)];
    P::st(l.v, 64, own, lane, v);
  }
}
template <typename R>
__device__ __forceinline__ void get_hops(const HopStrip<R>& l, int lane, int own, C<R>* v) {
  Planes<R, R2<R>>::ld(l.v, 64, own, lane, v);
}

template <typename R, bool DAG, typename Epi, typename In, int NS>
__global__ __launch_bounds__(256) void k_hop(Geom g, int nbp, int p_fixed, In hin, Epi epi, double* partials,
                                             int bps, int tgrp) {
  static_assert(NS == 64 || NS == 32, "64 or 32 sites per block");
  if (epi.skip()) return;
  using P = typename Epi::P;
  __shared__ HopStrip<R> lds[4];
  const int lb = xcd_block(blockIdx.x, gridDim.x, p_fixed == 1);
  const int p = p_fixed >= 0 ? p_fixed : lb / nbp;
  int blk = p_fixed >= 0 ? lb : lb % nbp;
  if (NS == 64 && tgrp > 0) {
    const int span = tgrp * bps;
    const int grp = blk / span, rem = blk - grp * span;
    const int chunk = rem / tgrp, tl = rem - chunk * tgrp;
    blk = (grp * tgrp + tl) * bps + chunk;
  }
  const int lane = threadIdx.x & 63;
  const int mu = threadIdx.x >> 6;
  const bool bwd = NS == 32 && lane >= 32;
  const int cb = blk * NS + (NS == 64 ? lane : lane & 31);
  const bool active = cb < g.vh;
  // 64-site blocks: the lane's epilogue operands at its own (site, spin =
  // wave) are independent of the hop, so they are loaded before it and
  // arrive while the neighbour loads are in flight (16^4 mixed force call
  // 5.40 -> 5.15 ms, FP64 at 24^3x48 187 -> 183 ms).  With BF16-stored
  // vectors only where there is one operand: three waves own the
  // components, and holding x, r, p of a third of them across the hop costs
  // registers (24^3x48: EpiSchurCG 31.8 -> 35.9 us, EpiSchurNorm 28.8 -> 27.9).
  typename Epi::Pre pre{};
  if constexpr (NS == 64 && Epi::kPrefetch) {
    if (active && mu < P::kOwners) pre = epi.pre(p, cb, mu);
  }

  C<R> acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = czero<R>();
  if (active) {
    int c[4];
    cb_coords(g, p, cb, c);
    const auto in = make_loader<R>(hin, g, p);
    if constexpr (NS == 64) {
      switch (mu) {
        case 0: hop_dir<R, 0, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc); break;
        case 1: hop_dir<R, 1, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc); break;
        case 2: hop_dir<R, 2, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc); break;
        default: hop_dir<R, 3, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc); break;
      }
    } else {
      switch (mu) {
        case 0: hop_one<R, 0, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc, bwd); break;
        case 1: hop_one<R, 1, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc, bwd); break;
        case 2: hop_one<R, 2, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc, bwd); break;
        default: hop_one<R, 3, DAG>(g, hin.gauge, hin.nk, in, p, cb, c, acc, bwd); break;
      }
    }
  }
  put_hops(lds[mu], lane, acc);
  __syncthreads();
  double red = 0.0;
  if constexpr (NS == 64) {
    // wave `mu` now owns its part of the components of the 64 sites
    if (mu < P::kOwners) {
      C<R> out[P::NC], d1[P::NC], d2[P::NC], d3[P::NC];
      get_hops(lds[0], lane, mu, out);
      get_hops(lds[1], lane, mu, d1);
      get_hops(lds[2], lane, mu, d2);
      get_hops(lds[3], lane, mu, d3);
#pragma unroll
      for (int i = 0; i < P::NC; ++i) out[i] = (out[i] + d1[i]) + (d2[i] + d3[i]);
      if constexpr (!Epi::kPrefetch) {
        if (active) pre = epi.pre(p, cb, mu);
      }
      if (active) epi.apply(p, cb, mu, out, red, pre);
    }
  } else if (mu < 2) {
    // lane -> site lane & 31, owner 2 mu + lane / 32; eight partial hops
    const int site = lane & 31;
    const int own = 2 * mu + (lane >> 5);
    const int cbo = blk * 32 + site;
    C<R> out[P::NC], f[P::NC], b[P::NC], d[4][P::NC];
    if (own < P::kOwners) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        get_hops(lds[m], site, own, f);
        get_hops(lds[m], 32 + site, own, b);
#pragma unroll
        for (int i = 0; i < P::NC; ++i) d[m][i] = f[i] + b[i];
      }
#pragma unroll
      for (int i = 0; i < P::NC; ++i) out[i] = (d[0][i] + d[1][i]) + (d[2][i] + d[3][i]);
      if (cbo < g.vh) epi.apply(p, cbo, own, out, red, epi.pre(p, cbo, own));
    }
  }
  if constexpr (Epi::kReduce) {
    double v[1] = {red};
    block_partials<256, 1>(v, partials, lb);
  }
  epi.template tail<256>();
}

// Sites per hop block: the context's choice, else 32 on small lattices
// (kHopHalfWaveMaxVh sites per parity and below), 64 above.
static inline int hop_sites_per_block(const Geom& g) {
  if (g.hop_ns == 32 || g.hop_ns == 64) return g.hop_ns;
  return g.vh <= kHopHalfWaveMaxVh ? 32 : 64;
}
static inline int nblk_parity(const Geom& g) {
  const int ns = hop_sites_per_block(g);
  return (g.vh + ns - 1) / ns;
}

// t-fastest block groups of the 64-site kernel: (blocks per t-slice, slices
// per group), or tgrp = 0 (site order): by the context's choice, else above
// kHopTOrderMinVh sites per parity (24^3x48: hop 36 -> 32 us, re-read
// traffic 1.29x -> 1.1x; at 16^4, whose fields stay in the caches, site
// order is 3 % faster); never when a slice is not a whole number of blocks.
// Groups of 8 slices where Lt allows, else 4 or 2 (Lt is even).
static inline void hop_block_order(const Geom& g, int& bps, int& tgrp) {
  const int vslice = g.vh / g.L[3];
  bps = vslice / 64;
  tgrp = 0;
  if (vslice % 64 != 0 || bps == 0) return;
  if (g.hop_order == 1 || (g.hop_order == 0 && g.vh <= kHopTOrderMinVh)) return;
  tgrp = g.L[3] % 8 == 0 ? 8 : (g.L[3] % 4 == 0 ? 4 : 2);
}

template <typename R, bool DAG, typename Epi, typename In>
static hipError_t launch(const Geom& g, int p_out, const In& hin, const Epi& epi, double* partials, hipStream_t s,
                         int capacity = 0) {
  const int nbp = nblk_parity(g);
  const int nb = p_out >= 0 ? nbp : 2 * nbp;
  if (Epi::kReduce && nb > capacity) return hipErrorInvalidValue;
  if (hop_sites_per_block(g) == 32) {
    hipLaunchKernelGGL((k_hop<R, DAG, Epi, In, 32>), dim3(nb), dim3(256), 0, s, g, nbp, p_out, hin, epi, partials,
                       0, 0);
  } else {
    int bps, tgrp;
    hop_block_order(g, bps, tgrp);
    hipLaunchKernelGGL((k_hop<R, DAG, Epi, In, 64>), dim3(nb), dim3(256), 0, s, g, nbp, p_out, hin, epi, partials,
                       bps, tgrp);
  }
  return hipGetLastError();
}

int hop_blocks(const Geom& g, int p_out) { return p_out >= 0 ? nblk_parity(g) : 2 * nblk_parity(g); }

template <typename R, bool DAG, typename T>
hipError_t launch_hop_axpy(const Geom& g, int p_out, HopIn<R, T> hin, T* out_even, T* out_odd,
                           const typename NoDeduce<T>::type* self_even, const typename NoDeduce<T>::type* self_odd,
                           double coef, hipStream_t s, SolverState* guard, const double* pap_partials) {
  EpiAxpy<R, T> e;
  e.guard = guard;
  e.pap_partials = pap_partials;
  e.pap_nblk = nblk_parity(g);
  e.out[0] = out_even;
  e.out[1] = out_odd;
  e.self[0] = self_even;
  e.self[1] = self_odd;
  e.coef = R(coef);
  e.vh = g.vs;
  return launch<R, DAG>(g, p_out, hin, e, nullptr, s);
}

template <typename R, typename T, bool DAG>
hipError_t launch_hop_schur_norm(const Geom& g, HopIn<R, T> hin, T* w, const T* x, double coef, SolverState* st,
                                 Reduce red, hipStream_t s) {
  EpiSchurNorm<R, T> e{w, x, R(coef), g.vs, st};
  return launch<R, DAG>(g, 1, hin, e, red.partials, s, red.capacity);
}

template <typename R, typename T, bool DAG>
hipError_t launch_hop_schur_cg(const Geom& g, HopIn<R, T> hin, const T* w, R2<R>* x, const R2<R>* r, R2<R>* ro,
                               const T* p, double coef, SolverState* st, Reduce red, hipStream_t s) {
  EpiSchurCG<R, T> e{w, x, r, ro, p, R(coef), g.vs, st};
  return launch<R, DAG>(g, 1, hin, e, red.partials, s, red.capacity);
}

template <bool DAG>
hipError_t launch_hop_residual(const Geom& g, HopIn<double> hin, const double2* self_full,
                               const double2* phi_full, double2* r_full, double coef, Reduce red,
                               int slot, hipStream_t s) {
  const size_t half = (size_t)12 * g.vs;
  EpiResidual e;
  e.self[0] = self_full;
  e.self[1] = self_full + half;
  e.phi[0] = phi_full;
  e.phi[1] = phi_full + half;
  e.r[0] = r_full;
  e.r[1] = r_full + half;
  e.coef = coef;
  e.vh = g.vs;
  hipError_t err = launch<double, DAG>(g, -1, hin, e, red.partials, s, red.capacity);
  if (err != hipSuccess) return err;
  return launch_finalize(kFinResult1, 2 * nblk_parity(g), red, nullptr, slot, 0.0, 0, s);
}

template <typename R, bool DAG>
hipError_t launch_hop_step(const Geom& g, const R2<R>* gauge, int nk, R2<R>* t, R2<R>* p, const R2<R>* r,
                           SolverState* st, Reduce red, hipStream_t s) {
  EpiStep<R> e;
  e.t = t;
  e.p = p;
  e.r = r;
  e.vh = g.vs;
  e.state = st;
  e.partials = red.partials;
  e.nblk = nblk_parity(g);
  e.mb = red.mbox;
  if (e.nblk > red.capacity) return hipErrorInvalidValue;
  const HopIn<R> hin{gauge, r, r, nk};
  return launch<R, DAG>(g, 0, hin, e, nullptr, s);
}
hipError_t launch_hop_direction(const Geom& g, const double2* gauge, int nk, double2* t, double2* p,
                                const double2* r, const SolverState* st, hipStream_t s) {
  return launch<double, false>(g, 0, HopIn<double>{gauge, r, r, nk}, EpiDirection{t, p, r, g.vs, st}, nullptr, s);
}
hipError_t launch_hop_shift_residual(const Geom& g, HopIn<double> hin, const double2* w, const double2* x,
                                     const double2* phi, double sigma, double coef, double* partials,
                                     hipStream_t s) {
  return launch<double, true>(g, 1, hin, EpiShiftResidual{w, x, phi, sigma, coef, g.vs}, partials, s,
                              hop_blocks(g, 1));
}
template <bool DAG>
hipError_t launch_hop_schur_residual(const Geom& g, HopIn<double> hin, const double2* w, const double2* phi,
                                     double2* r, double coef, Reduce red, hipStream_t s) {
  return launch<double, DAG>(g, 1, hin, EpiSchurResidual{w, phi, r, coef, g.vs}, red.partials, s, red.capacity);
}
template hipError_t launch_hop_schur_residual<false>(const Geom&, HopIn<double>, const double2*, const double2*,
                                                     double2*, double, Reduce, hipStream_t);
template hipError_t launch_hop_schur_residual<true>(const Geom&, HopIn<double>, const double2*, const double2*,
                                                    double2*, double, Reduce, hipStream_t);
template hipError_t launch_hop_step<double, false>(const Geom&, const double2*, int, double2*, double2*,
                                                   const double2*, SolverState*, Reduce, hipStream_t);
template hipError_t launch_hop_step<double, true>(const Geom&, const double2*, int, double2*, double2*,
                                                  const double2*, SolverState*, Reduce, hipStream_t);
template hipError_t launch_hop_step<float, false>(const Geom&, const float2*, int, float2*, float2*,
                                                  const float2*, SolverState*, Reduce, hipStream_t);
template hipError_t launch_hop_step<float, true>(const Geom&, const float2*, int, float2*, float2*, const float2*,
                                                 SolverState*, Reduce, hipStream_t);

#define LGT_INST_AXPY(R, DAG, T)                                                                          \
  template hipError_t launch_hop_axpy<R, DAG, T>(const Geom&, int, HopIn<R, T>, T*, T*, const T*, const T*, \
                                                  double, hipStream_t, SolverState*, const double*);
#define LGT_INST_CG(R, T, DAG)                                                                            \
  template hipError_t launch_hop_schur_norm<R, T, DAG>(const Geom&, HopIn<R, T>, T*, const T*, double,       \
                                                        SolverState*, Reduce, hipStream_t);                 \
  template hipError_t launch_hop_schur_cg<R, T, DAG>(const Geom&, HopIn<R, T>, const T*, R2<R>*,             \
                                                      const R2<R>*, R2<R>*, const T*, double, SolverState*, Reduce, \
                                                      hipStream_t);

LGT_INST_AXPY(double, false, double2)
LGT_INST_AXPY(double, true, double2)
LGT_INST_AXPY(float, false, float2)
LGT_INST_AXPY(float, true, float2)
LGT_INST_AXPY(float, false, Bf16c)
LGT_INST_AXPY(float, true, Bf16c)
LGT_INST_CG(double, double2, false)
LGT_INST_CG(double, double2, true)
LGT_INST_CG(float, float2, false)
LGT_INST_CG(float, float2, true)
LGT_INST_CG(float, Bf16c, false)
LGT_INST_CG(float, Bf16c, true)

template hipError_t launch_hop_residual<false>(const Geom&, HopIn<double>, const double2*, const double2*,
                                               double2*, double, Reduce, int, hipStream_t);
template hipError_t launch_hop_residual<true>(const Geom&, HopIn<double>, const double2*, const double2*,
                                              double2*, double, Reduce, int, hipStream_t);

}  // namespace lgt
