// Multi-right-hand-side kernels: nr spinor fields on one lattice, solved
// together (one pseudofermion per right-hand side, each with its own kappa).
//
// Layout of a multi-RHS half field: the planes of a single half field (see
// Planes), each [nr][vs] (site fastest, vs >= V/2 sites apart; their padding
// holds anything, finite or not, and is never summed, since it moves with
// nr), a full field the even half then the odd half.  Every
// per-component access of a wave is unit stride, as in the single field.
//
// Hop decomposition: a 256-thread block owns 64 consecutive sites of one
// parity and a group of G right-hand sides; wave w (= direction mu) loads
// the two links of its direction once, keeps them in registers and then, for
// each right-hand side of the group in turn, computes both hops along mu,
// meets the other waves in LDS and runs the epilogue for spin component w.
// The link traffic is paid once per group instead of once per field, and
// the neighbour index arithmetic once per block.  G trades link reuse
// (large G) against parallelism (small G gives more blocks); the host picks
// it by timing (see batch.hip).  Per-RHS reductions are deterministic: a
// fixed-order wave reduction, then the four waves in order, one partial per
// (site block, right-hand side), summed by a one-block finalize launch.
#include <type_traits>

#include "lgt_internal.h"
#include "lgt_hop.h"
#include "lgt_mrhs.h"

namespace lgt {

// Per-RHS sums of the partial rows [nblk][kMaxRhs] of an earlier launch, in a
// fixed order; thread n < kMaxRhs of the 256 that call it gets the total of
// right-hand side n.  Thread t adds column t % 16 of every 16th row, so a
// wave reads four whole rows at once and all right-hand sides share one round
// of loads: summed one right-hand side after the other, each with its own
// loads and two barriers, the 12 sums of a 16^4 iteration held the block for
// some 20 us at the end of the third hop, and again in the finalize.
__device__ __forceinline__ double sum_rows(const double* __restrict__ partials, int nblk) {
  static_assert(kMaxRhs == 16, "a quarter wave covers one row");
  __shared__ double sh[4][kMaxRhs];
  const int n = threadIdx.x & 15;
  double v = 0.0;
#pragma unroll 8
  for (int i = threadIdx.x >> 4; i < nblk; i += 16) v += partials[(size_t)i * kMaxRhs + n];
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  if ((threadIdx.x & 63) < 16) sh[threadIdx.x >> 6][n] = v;
  __syncthreads();
  return ((sh[0][n] + sh[1][n]) + sh[2][n]) + sh[3][n];
}

// ---------------------------------------------------------------------------
// Epilogues (owner `own`'s components of right-hand side n at (p, cb), see
// Planes; ps: plane stride nr vs, i = n vs + cb).  rhs_active(n) false:
// nothing of right-hand side n in this launch is used (its CG has stopped:
// converged, or idle until the next reliable update), so the kernel skips its
// hop and writes 0 for its partial.  pre() loads the other operands; the VALU
// kernel calls it before the hop, which they do not depend on.
// ---------------------------------------------------------------------------
template <typename R>
struct MEpiAxpy {  // out = self + coef_n * acc
  static constexpr bool kReduce = false;
  using P = Planes<R, R2<R>>;
  static constexpr int NC = P::NC;
  R2<R>* out[2];
  const R2<R>* self[2];
  const double* coef;  // [NR] device array
  const BatchState* guard;
  const double* mask;  // if set: right-hand side n is computed only where mask[n] != 0
  const double* pap_partials;  // block 0 forms alpha_n (see tail)
  int pap_nblk;
  BatchState* state;
  __device__ bool skip() const { return guard && guard->all_done; }
  __device__ bool rhs_active(int n) const {
    return (!mask || mask[n] != 0.0) && (!guard || guard->done[n] == kDoneRunning);
  }
  struct Pre {
    C<R> s[NC];
  };
  __device__ Pre pre(int p, size_t ps, int own, size_t i) const {
    Pre q{};
    if (self[p]) P::ld(self[p], ps, own, i, q.s);
    return q;
  }
  __device__ void apply(int p, size_t ps, int own, size_t i, int n, const C<R>* a, double&, const Pre& q) const {
    C<R> v[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) v[k] = R(coef[n]) * a[k] + q.s[k];
    P::st(out[p], ps, own, i, v);
  }
  __device__ void tail(int nr) const {
    if (!pap_partials || blockIdx.x != 0) return;
    const double tot = sum_rows(pap_partials, pap_nblk);
    const int n = threadIdx.x;
    if (n < nr && !state->done[n]) {
      state->pap[n] = tot;
      if (!(tot > 0.0) || !isfinite(tot)) {
        state->alpha[n] = 0.0;
        state->done[n] = kDoneBreakdown;
      } else {
        state->alpha[n] = state->rr[n] / tot;
      }
    }
  }
};

template <typename R>
struct MEpiSchurNorm {  // w = x + coef_n acc, per-RHS |w|^2
  static constexpr bool kReduce = true;
  using P = Planes<R, R2<R>>;
  static constexpr int NC = P::NC;
  R2<R>* w;
  const R2<R>* x;
  const double* coef;
  const BatchState* state;
  __device__ bool skip() const { return state->all_done; }
  __device__ bool rhs_active(int n) const { return state->done[n] == kDoneRunning; }
  struct Pre {
    C<R> x[NC];
  };
  __device__ Pre pre(int, size_t ps, int own, size_t i) const {
    Pre q;
    P::ld(x, ps, own, i, q.x);
    return q;
  }
  __device__ void apply(int, size_t ps, int own, size_t i, int n, const C<R>* a, double& red, const Pre& q) const {
    C<R> v[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      v[k] = q.x[k] + R(coef[n]) * a[k];
      red += (double)v[k].re * (double)v[k].re + (double)v[k].im * (double)v[k].im;
    }
    P::st(w, ps, own, i, v);
  }
  __device__ void tail(int) const {}
};

template <typename R>
struct MEpiSchurCG {  // q = w + coef_n acc; r -= alpha_n q (unless converged)
  static constexpr bool kReduce = true;
  using P = Planes<R, R2<R>>;
  static constexpr int NC = P::NC;
  const R2<R>* w;
  R2<R>* r;
  const double* coef;
  const BatchState* state;
  __device__ bool skip() const { return state->all_done; }
  __device__ bool rhs_active(int n) const { return state->done[n] == kDoneRunning; }
  struct Pre {
    C<R> r[NC], w[NC];
  };
  __device__ Pre pre(int, size_t ps, int own, size_t i) const {
    Pre q;
    P::ld(r, ps, own, i, q.r);
    P::ld(w, ps, own, i, q.w);
    return q;
  }
  __device__ void apply(int, size_t ps, int own, size_t i, int n, const C<R>* a, double& red, const Pre& q) const {
    const bool run = !state->done[n];
    const R alpha = R(state->alpha[n]);
    C<R> rv[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      rv[k] = q.r[k];
      if (run) rv[k] = rv[k] - alpha * (q.w[k] + R(coef[n]) * a[k]);
      red += (double)rv[k].re * (double)rv[k].re + (double)rv[k].im * (double)rv[k].im;
    }
    if (run) P::st(r, ps, own, i, rv);
  }
  __device__ void tail(int) const {}
};

struct MEpiResidual {  // r = phi - (self + coef_n acc), per-RHS |r|^2 (FP64)
  static constexpr bool kReduce = true;
  using P = Planes<double, double2>;
  static constexpr int NC = P::NC;
  const double2* self[2];
  const double2* phi[2];
  double2* r[2];
  const double* coef;
  const double* mask;  // if set, only right-hand sides with a nonzero entry
  __device__ bool skip() const { return false; }
  __device__ bool rhs_active(int n) const { return !mask || mask[n] != 0.0; }
  struct Pre {
    C<double> f[NC], s[NC];
  };
  __device__ Pre pre(int p, size_t ps, int own, size_t i) const {
    Pre q;
    P::ld(phi[p], ps, own, i, q.f);
    P::ld(self[p], ps, own, i, q.s);
    return q;
  }
  __device__ void apply(int p, size_t ps, int own, size_t i, int n, const C<double>* a, double& red,
                        const Pre& q) const {
    C<double> v[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      v[k] = q.f[k] - (q.s[k] + coef[n] * a[k]);
      red += norm2(v[k]);
    }
    P::st(r[p], ps, own, i, v);
  }
  __device__ void tail(int) const {}
};


// Loader of one right-hand side of a multi-RHS field: a plane is [nr][vs]
// vectors of 16 bytes; the per-lane offset carries site and n, the plane
// offset is uniform.
template <typename R>
struct MrhsIn {
  BufRsrc rs;
  unsigned ks;  // plane stride in bytes (nr * vs vectors)
  unsigned ns;  // right-hand-side stride in bytes (vs vectors)
  __device__ __forceinline__ unsigned off(int site, int n) const { return (unsigned)site * 16u + (unsigned)n * ns; }
  __device__ __forceinline__ void all(unsigned o, C<R>* psi) const { Planes<R, R2<R>>::all(rs, o, ks, psi); }
};
template <typename R>
__device__ __forceinline__ MrhsIn<R> make_mrhs_in(const R2<R>* half, const Geom& g, int nr) {
  const unsigned ns = (unsigned)g.vs * 16u, ks = (unsigned)nr * ns;
  return {make_rsrc(half, (size_t)Planes<R, R2<R>>::kPlanes * ks), ks, ns};
}

// The partial hops of wave MU for the other owners: strip [owner][source] of
// the exchange, the source counted without the owner's own wave, which keeps
// its part in registers.
template <typename R>
struct Exchange {
  using P = Planes<R, R2<R>>;
  static constexpr int kStrip = P::NC * 64;  // R2<R> of an owner's part for 64 sites
  static constexpr int kSize = P::kOwners * 3 * kStrip;
  static __device__ __forceinline__ R2<R>* strip(R2<R>* ex, int own, int src) { return ex + (own * 3 + src) * kStrip; }
  // place (0, plane q) of a strip: an owner's planes, 64 vectors each
  template <int MU>
  static __device__ __forceinline__ void share(const C<R>* acc, R2<R>* ex, int lane, C<R>* mine) {
#pragma unroll
    for (int own = 0; own < P::kOwners; ++own) {
      C<R> v[P::NC];
#pragma unroll
      for (int q = 0; q < P::NC; ++q) v[q] = acc[P::comp(own, q)];
      if (own == MU) {
#pragma unroll
        for (int q = 0; q < P::NC; ++q) mine[q] = v[q];
      } else {
        P::st(strip(ex, own, MU < own ? MU : MU - 1), 64, 0, lane, v);
      }
    }
  }
};

template <typename R, bool DAG, typename Epi>
__global__ __launch_bounds__(256, 2) void k_hop_mrhs(Geom g, int nr, int G, int nbp, int ngrp, int p_fixed,
                                                  HopIn<R> hin, Epi epi, double* partials) {
  if (epi.skip()) return;
  // two buffers, so that one barrier a right-hand side is enough
  using P = typename Epi::P;
  using X = Exchange<R>;
  __shared__ __align__(16) R2<R> lds[2][X::kSize];
  __shared__ double wred[4][kMaxRhs];
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int per_par = nbp * ngrp;
  const int p = p_fixed >= 0 ? p_fixed : lb / per_par;
  const int rem = p_fixed >= 0 ? lb : lb % per_par;
  const int blk = rem / ngrp, grp = rem - blk * ngrp;  // neighbouring blocks share a site block
  const int n0 = grp * G, n1 = min(nr, n0 + G);
  const int lane = threadIdx.x & 63;
  const int mu = threadIdx.x >> 6;
  const int cb = blk * 64 + lane;
  const bool active = cb < g.vh;
  // the group's running right-hand sides, read once per block so that every
  // thread skips the same ones (a later write to the state by another block
  // concerns a right-hand side whose results this launch no longer needs)
  __shared__ unsigned s_act;
  if (threadIdx.x == 0) {
    unsigned m = 0;
    for (int n = n0; n < n1; ++n) m |= (epi.rhs_active(n) ? 1u : 0u) << (n - n0);
    s_act = m;
  }
  if (threadIdx.x < 4 * kMaxRhs) wred[threadIdx.x / kMaxRhs][threadIdx.x % kMaxRhs] = 0.0;
  __syncthreads();
  const unsigned act = s_act;
  constexpr unsigned E = sizeof(R2<R>);
  const unsigned gs = (unsigned)g.vs * E;
  const auto in = make_mrhs_in<R>(p ? hin.in_even : hin.in_odd, g, nr);
  const size_t ps = (size_t)nr * g.vs;
  int c[4] = {0, 0, 0, 0};
  int nf = 0, nb = 0;
  if (active) {
    cb_coords(g, p, cb, c);
    nf = cb_shift(g, c, mu, +1);
    nb = cb_shift(g, c, mu, -1);
  }
  // links [2][4][nk][vh]: all nine components, or (FP32) the first two rows
  // of SU(3) links with the third rebuilt in registers (a third less link
  // traffic per group, as in the single-field hop)
  const int nk = hin.nk;
  const BufRsrc ruf = make_rsrc(hin.gauge + (size_t)((p * 4 + mu) * nk) * g.vs, (size_t)nk * gs);
  const BufRsrc rub = make_rsrc(hin.gauge + (size_t)(((1 - p) * 4 + mu) * nk) * g.vs, (size_t)nk * gs);
  // The links stay in registers for the whole group.  FP64 read them again for
  // every right-hand side, 18 of its 42 loads, and the L2's return path bounds
  // the launch: 16^4 x 12 69.6 -> 49.3 us in a mixed solve, 59 -> 35 us where
  // all right-hand sides run; two waves a SIMD, as the exchange allows, leave
  // 256 registers for them.
  M3<R> Uf, Ub;
#pragma unroll
  for (int k = 0; k < 9; ++k) Uf.m[k] = Ub.m[k] = czero<R>();
  if (active && act) {
    if (nk == 9) {
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        Uf.m[k] = ld_buf<R>(ruf, (unsigned)cb * E, k * gs);
        Ub.m[k] = ld_buf<R>(rub, (unsigned)nb * E, k * gs);
      }
    } else {
      load_two_rows<R, false>(ruf, (unsigned)cb * 16u, (unsigned)g.vs * 16u, Uf);
      load_two_rows<R, false>(rub, (unsigned)nb * 16u, (unsigned)g.vs * 16u, Ub);
      third_row(Uf);
      third_row(Ub);
    }
  }
  int buf = 0;
  for (int n = n0; n < n1; ++n) {
    if (!((act >> (n - n0)) & 1u)) continue;  // uniform: the block's mask
    typename Epi::Pre pre{};
    C<R> acc[12], sum[P::NC];
    const size_t at = (size_t)n * g.vs + cb;
    const bool owner = active && mu < P::kOwners;
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = czero<R>();
    if (owner) pre = epi.pre(p, ps, mu, at);
    if (active) {
      const unsigned of = in.off(nf, n), ob = in.off(nb, n);
      switch (mu) {
        case 0: hop_dir_u<R, 0, DAG>(g, Uf, Ub, in, of, ob, c, acc); break;
        case 1: hop_dir_u<R, 1, DAG>(g, Uf, Ub, in, of, ob, c, acc); break;
        case 2: hop_dir_u<R, 2, DAG>(g, Uf, Ub, in, of, ob, c, acc); break;
        default: hop_dir_u<R, 3, DAG>(g, Uf, Ub, in, of, ob, c, acc); break;
      }
    }
    switch (mu) {
      case 0: X::template share<0>(acc, lds[buf], lane, sum); break;
      case 1: X::template share<1>(acc, lds[buf], lane, sum); break;
      case 2: X::template share<2>(acc, lds[buf], lane, sum); break;
      default: X::template share<3>(acc, lds[buf], lane, sum); break;
    }
    __syncthreads();
    double red = 0.0;
    if (owner) {
#pragma unroll
      for (int src = 0; src < 3; ++src) {
        C<R> b[P::NC];
        P::ld(X::strip(lds[buf], mu, src), 64, 0, lane, b);
#pragma unroll
        for (int q = 0; q < P::NC; ++q) sum[q] += b[q];
      }
      epi.apply(p, ps, mu, at, n, sum, red, pre);
    }
    if constexpr (Epi::kReduce) {
      red = wave_sum(red);
      if (lane == 0) wred[mu][n - n0] = red;
    }
    buf ^= 1;
  }
  if constexpr (Epi::kReduce) __syncthreads();
  if constexpr (Epi::kReduce) {
    const int t = threadIdx.x;
    if (t < n1 - n0) {
      const int row = p_fixed >= 0 ? blk : p * nbp + blk;
      partials[(size_t)row * kMaxRhs + n0 + t] = ((wred[0][t] + wred[1][t]) + wred[2][t]) + wred[3][t];
    }
  }
  epi.tail(nr);
}

// ---------------------------------------------------------------------------
// MFMA form of the FP32 batched hop.  Per site x, direction mu and sign, the
// hop applies one link to the projected half spinors of every right-hand
// side of the group: W = U H, a complex 3 x (2 G) product, i.e. the real
// product [[Ur, -Ui], [Ui, Ur]] (6 x 6) times [Hr; Hi] (6 x 2G).  Every
// site has its own U, so the product runs on v_mfma_f32_4x4x1_16b_f32,
// whose 16 independent 4x4 blocks take 16 sites per instruction: block b
// (lanes 4b..4b+3) is site b of the wave's 16; its output rows are the
// real-form rows (Re W_0, Re W_1, Re W_2, Im W_0 | Im W_1, Im W_2, -, -)
// in two row tiles, its columns (spin, right-hand side) in 2G/4 column
// tiles, and the six real input components are six rank-1 steps.  Lane j
// of a block feeds row j of the link operand and column j of the spinor
// operand, and receives column j of every output tile: the whole W of
// right-hand sides j (and j + 4 for G = 8), both spins.  So the lane that
// projects a right-hand side's neighbour spinor is also the lane that
// reconstructs its W, and the link is loaded once per site (each lane one
// or two of its rows).  A 256-thread block takes 16 sites of one parity
// and a group of G right-hand sides; wave w takes direction mu = w (both
// hops); the four directions meet in LDS as in k_hop_mrhs and the same
// epilogues run.  Reductions: per right-hand side, a fixed-order sum over
// the threads that own it, then one partial per (block, right-hand side).
// ---------------------------------------------------------------------------
typedef float v4f __attribute__((ext_vector_type(4)));

// Rows of the real-form link operand fed by lane j (0..3): tile 0 row j,
// tile 1 row j, as six values over the input components (Re h_c, Im h_c).
// Forward: the link U; backward: U^dag (rows of U^dag = conjugated columns).
template <bool ADJ>
__device__ __forceinline__ void link_rows(const BufRsrc& ru, unsigned o, unsigned gs, int j, float* a0,
                                          float* a1) {
  // element (i, c) of the operator and its real and imaginary parts
  auto el = [&](int i, int c) -> C<float> {
    const C<float> u = ADJ ? ld_buf<float>(ru, o, (3 * c + i) * gs) : ld_buf<float>(ru, o, (3 * i + c) * gs);
    return ADJ ? conj(u) : u;
  };
  if (j < 3) {  // tile 0: Re W_j = sum_c Re u_jc Re h_c - Im u_jc Im h_c
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const C<float> u = el(j, c);
      a0[c] = u.re;
      a0[3 + c] = -u.im;
    }
  } else {      // tile 0 row 3: Im W_0 = sum_c Im u_0c Re h_c + Re u_0c Im h_c
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const C<float> u = el(0, c);
      a0[c] = u.im;
      a0[3 + c] = u.re;
    }
  }
  if (j < 2) {  // tile 1 rows 0, 1: Im W_1, Im W_2
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const C<float> u = el(j + 1, c);
      a1[c] = u.im;
      a1[3 + c] = u.re;
    }
  } else {
#pragma unroll
    for (int c = 0; c < 6; ++c) a1[c] = 0.f;
  }
}

// W (2 spins x 3 colours) of the right-hand side in column tiles (c0, c1)
// (spin 0, spin 1) from the accumulators
__device__ __forceinline__ void tile_w(const v4f (*acc)[4], int c0, int c1, C<float>* w) {
  const int cs[2] = {c0, c1};
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int c = cs[a];
    w[3 * a + 0] = cmk<float>(acc[0][c][0], acc[0][c][3]);
    w[3 * a + 1] = cmk<float>(acc[0][c][1], acc[1][c][0]);
    w[3 * a + 2] = cmk<float>(acc[0][c][2], acc[1][c][1]);
  }
}

// One hop (forward: U_mu(x) psi(x + mu) with projector 1 + S gamma_mu;
// backward: U_mu(x - mu)^dag psi(x - mu) with 1 + S gamma_mu) of the lane's
// right-hand sides, added to out[0..NL-1][12].
template <int MU, int S, bool ADJ, int G>
__device__ __forceinline__ void mfma_hop(const MrhsIn<float>& in, unsigned osite, const BufRsrc& ru, unsigned olink,
                                         unsigned gs, int j, int n0, unsigned live, bool bc, float bcs,
                                         C<float> (*out)[12]) {
  constexpr int NL = G / 4;       // right-hand sides per lane
  constexpr int NCT = 2 * G / 4;  // column tiles
  float a0[6], a1[6];
  link_rows<ADJ>(ru, olink, gs, j, a0, a1);
  C<float> h[NL][6];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int nl = j + 4 * q;
    if ((live >> nl) & 1u) {
      C<float> psi[12];
      in.all(in.off(0, n0 + nl) + osite, psi);
      project<float, MU, S>(psi, h[q]);
    } else {
#pragma unroll
      for (int k = 0; k < 6; ++k) h[q][k] = czero<float>();
    }
  }
  v4f acc[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = v4f{0.f, 0.f, 0.f, 0.f};
  // column tile c: spin c / NL, right-hand side (lane's) c % NL
#pragma unroll
  for (int k = 0; k < 6; ++k) {
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
      const C<float> hv = h[c % NL][3 * (c / NL) + (k % 3)];
      const float b = k < 3 ? hv.re : hv.im;
      acc[0][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(a0[k], b, acc[0][c], 0, 0, 0);
      acc[1][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(a1[k], b, acc[1][c], 0, 0, 0);
    }
  }
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    C<float> w[6];
    tile_w(acc, q, NL + q, w);
    if (bc) {
#pragma unroll
      for (int k = 0; k < 6; ++k) w[k] = bcs * w[k];
    }
    reconstruct<float, MU, S>(w, out[q]);
  }
}

template <int MU, bool DAG, int G>
__device__ __forceinline__ void mfma_dir(const Geom& g, const MrhsIn<float>& in, const float2* gauge, int p, int cb,
                                         const int c[4], int j, int n0, unsigned live, C<float> (*out)[12]) {
  constexpr int SF = DAG ? +1 : -1;
  constexpr unsigned E = sizeof(float2);
  const unsigned gs = (unsigned)g.vs * E;
  const int nf = cb_shift(g, c, MU, +1), nb = cb_shift(g, c, MU, -1);
  const BufRsrc ruf = make_rsrc(gptr<float>(gauge, g, p, MU), (size_t)9 * gs);
  const BufRsrc rub = make_rsrc(gptr<float>(gauge, g, 1 - p, MU), (size_t)9 * gs);
  const float bcs = (float)g.bc;
  mfma_hop<MU, SF, false, G>(in, (unsigned)nf * 16u, ruf, (unsigned)cb * E, gs, j, n0, live,
                             MU == 3 && c[3] == g.L[3] - 1, bcs, out);
  mfma_hop<MU, -SF, true, G>(in, (unsigned)nb * 16u, rub, (unsigned)nb * E, gs, j, n0, live, MU == 3 && c[3] == 0,
                             bcs, out);
}

template <bool DAG, typename Epi, int G>
__global__ __launch_bounds__(256) void k_hop_mrhs_mfma(Geom g, int nr, int nbp, int ngrp, int p_fixed,
                                                       HopIn<float> hin, Epi epi, double* partials) {
  if (epi.skip()) return;
  constexpr int NL = G / 4;
  __shared__ float2 lds[4][G][12][16];
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const int per_par = nbp * ngrp;
  const int p = p_fixed >= 0 ? p_fixed : lb / per_par;
  const int rem = p_fixed >= 0 ? lb : lb % per_par;
  const int blk = rem / ngrp, grp = rem - blk * ngrp;
  const int n0 = grp * G, ng = min(G, nr - n0);
  const int lane = threadIdx.x & 63;
  const int mu = threadIdx.x >> 6;
  const int j = lane & 3, sb = lane >> 2;
  const int cb = blk * 16 + sb;
  const bool active = cb < g.vh;
  __shared__ unsigned s_act;
  if (threadIdx.x == 0) {
    unsigned m = 0;
    for (int n = 0; n < ng; ++n) m |= (epi.rhs_active(n0 + n) ? 1u : 0u) << n;
    s_act = m;
  }
  __syncthreads();
  const unsigned act = s_act;
  const auto in = make_mrhs_in<float>(p ? hin.in_even : hin.in_odd, g, nr);
  C<float> out[NL][12];
#pragma unroll
  for (int q = 0; q < NL; ++q)
#pragma unroll
    for (int k = 0; k < 12; ++k) out[q][k] = czero<float>();
  // every lane of the wave runs the MFMA (inactive sites read site 0 and
  // are not stored); a block whose group has no running right-hand side
  // skips the work
  if (act) {
    int c[4] = {0, 0, 0, 0};
    cb_coords(g, p, active ? cb : 0, c);
    switch (mu) {
      case 0: mfma_dir<0, DAG, G>(g, in, hin.gauge, p, active ? cb : 0, c, j, n0, act, out); break;
      case 1: mfma_dir<1, DAG, G>(g, in, hin.gauge, p, active ? cb : 0, c, j, n0, act, out); break;
      case 2: mfma_dir<2, DAG, G>(g, in, hin.gauge, p, active ? cb : 0, c, j, n0, act, out); break;
      default: mfma_dir<3, DAG, G>(g, in, hin.gauge, p, active ? cb : 0, c, j, n0, act, out); break;
    }
  }
#pragma unroll
  for (int q = 0; q < NL; ++q)
#pragma unroll
    for (int k = 0; k < 12; ++k) lds[mu][j + 4 * q][k][sb] = make_float2(out[q][k].re, out[q][k].im);
  __syncthreads();
  // epilogue: thread t owns right-hand side nl = t / (256 / G) of the group
  // and colours kq, kq + KS, ... of site t % 16
  constexpr int TPR = 256 / G;   // threads per right-hand side (32 or 64)
  constexpr int KS = TPR / 16;   // colour stride (2 or 4)
  const int nl = threadIdx.x / TPR, q = threadIdx.x % TPR;
  const int site = q & 15, kq = q >> 4;
  const int ocb = blk * 16 + site;
  const bool run = nl < ng && ((act >> nl) & 1u) && ocb < g.vh;
  double red = 0.0;
  if (run) {
    const int n = n0 + nl;
    const size_t ps = (size_t)nr * g.vs, at = (size_t)n * g.vs + ocb;
    for (int own = kq; own < 3; own += KS) {
      C<float> sum[4];
#pragma unroll
      for (int j4 = 0; j4 < 4; ++j4) {
        const int k = 3 * j4 + own;
        const float2 a = lds[0][nl][k][site], b = lds[1][nl][k][site], cc = lds[2][nl][k][site],
                     d = lds[3][nl][k][site];
        sum[j4] = cmk<float>(((a.x + b.x) + cc.x) + d.x, ((a.y + b.y) + cc.y) + d.y);
      }
      epi.apply(p, ps, own, at, n, sum, red, epi.pre(p, ps, own, at));
    }
  }
  if constexpr (Epi::kReduce) {
#pragma unroll
    for (int o = TPR / 2; o > 0; o >>= 1) red += __shfl_xor(red, o, 64);
    if (q == 0 && nl < ng) {
      const int row = p_fixed >= 0 ? blk : p * nbp + blk;
      partials[(size_t)row * kMaxRhs + n0 + nl] = red;
    }
  }
  epi.tail(nr);
}

// site blocks per parity of the batched hop: 64 sites (VALU kernel, G > 0)
// or 16 sites (MFMA kernel, G = -4 or -8)
static inline int mrhs_nbp(const Geom& g, int G = 1) { return G < 0 ? (g.vh + 15) / 16 : (g.vh + 63) / 64; }

template <typename R, bool DAG, typename Epi>
static hipError_t mlaunch(const Geom& g, int nr, int G, int p_out, const HopIn<R>& hin, const Epi& epi, Reduce red,
                          hipStream_t s) {
  if (nr < 1 || nr > kMaxRhs) return hipErrorInvalidValue;
  if (hin.nk != 9 && (hin.nk != 6 || sizeof(R) != 4)) return hipErrorInvalidValue;  // two-row links: FP32 only
  const int gs = G < 0 ? -G : G;
  if (gs < 1 || gs > kMaxRhs || (G < 0 && gs != 4 && gs != 8)) return hipErrorInvalidValue;
  const int nbp = mrhs_nbp(g, G);
  const int ngrp = (nr + gs - 1) / gs;
  const int rows = p_out >= 0 ? nbp : 2 * nbp;
  if (Epi::kReduce && (size_t)rows * kMaxRhs > red.ndoubles) return hipErrorInvalidValue;
  if (G < 0) {
    if (hin.nk != 9) return hipErrorInvalidValue;  // the MFMA form reads full links
    if constexpr (std::is_same<R, float>::value) {
      if (gs == 8)
        hipLaunchKernelGGL((k_hop_mrhs_mfma<DAG, Epi, 8>), dim3(rows * ngrp), dim3(256), 0, s, g, nr, nbp, ngrp,
                           p_out, hin, epi, red.partials);
      else
        hipLaunchKernelGGL((k_hop_mrhs_mfma<DAG, Epi, 4>), dim3(rows * ngrp), dim3(256), 0, s, g, nr, nbp, ngrp,
                           p_out, hin, epi, red.partials);
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;  // the MFMA form is FP32 only
    }
  }
  hipLaunchKernelGGL((k_hop_mrhs<R, DAG, Epi>), dim3(rows * ngrp), dim3(256), 0, s, g, nr, G, nbp, ngrp, p_out, hin,
                     epi, red.partials);
  return hipGetLastError();
}

// largest number of partial rows a reducing batched hop writes (the 16-site MFMA blocks)
int mrhs_hop_blocks(const Geom& g, int p_out) { return p_out >= 0 ? mrhs_nbp(g, -8) : 2 * mrhs_nbp(g, -8); }

template <typename R, bool DAG>
hipError_t launch_mhop_axpy(const Geom& g, int nr, int G, int p_out, HopIn<R> hin, R2<R>* out_e, R2<R>* out_o,
                            const R2<R>* self_e, const R2<R>* self_o, const double* coef, hipStream_t s,
                            BatchState* guard, const double* pap_partials, Reduce red, const double* mask) {
  MEpiAxpy<R> e;
  e.mask = mask;
  e.out[0] = out_e;
  e.out[1] = out_o;
  e.self[0] = self_e;
  e.self[1] = self_o;
  e.coef = coef;
  e.guard = guard;
  e.pap_partials = pap_partials;
  e.pap_nblk = mrhs_nbp(g, G);
  e.state = guard;
  return mlaunch<R, DAG>(g, nr, G, p_out, hin, e, red, s);
}

template <typename R, bool DAG>
hipError_t launch_mhop_schur_norm(const Geom& g, int nr, int G, HopIn<R> hin, R2<R>* w, const R2<R>* x,
                                  const double* coef, BatchState* st, Reduce red, hipStream_t s) {
  MEpiSchurNorm<R> e{w, x, coef, st};
  return mlaunch<R, DAG>(g, nr, G, 1, hin, e, red, s);
}

template <typename R, bool DAG>
hipError_t launch_mhop_schur_cg(const Geom& g, int nr, int G, HopIn<R> hin, const R2<R>* w, R2<R>* r,
                                const double* coef, BatchState* st, Reduce red, hipStream_t s) {
  MEpiSchurCG<R> e{w, r, coef, st};
  hipError_t err = mlaunch<R, DAG>(g, nr, G, 1, hin, e, red, s);
  if (err != hipSuccess) return err;
  return launch_mfinalize(kFinCgStep, mrhs_nbp(g, G), nr, red, st, 0.0, 0, s);
}

template <bool DAG>
hipError_t launch_mhop_residual(const Geom& g, int nr, int G, HopIn<double> hin, const double2* self_full,
                                const double2* phi_full, double2* r_full, const double* coef, Reduce red,
                                hipStream_t s) {
  const size_t half = (size_t)12 * g.vs * nr;
  MEpiResidual e;
  e.self[0] = self_full;
  e.self[1] = self_full + half;
  e.phi[0] = phi_full;
  e.phi[1] = phi_full + half;
  e.r[0] = r_full;
  e.r[1] = r_full + half;
  e.coef = coef;
  e.mask = nullptr;
  hipError_t err = mlaunch<double, DAG>(g, nr, G, -1, hin, e, red, s);
  if (err != hipSuccess) return err;
  return launch_mfinalize(kFinResult1, 2 * mrhs_nbp(g, G), nr, red, nullptr, 0.0, 0, s);
}
// (subtraction and norm were passes of their own: 16^4 x 12 46 + 33 us beside
// four hops of 49 us)
template <bool DAG>
hipError_t launch_mhop_schur_residual(const Geom& g, int nr, int G, HopIn<double> hin, const double2* w,
                                      const double2* phi, double2* r, const double* coef, const double* mask,
                                      Reduce red, hipStream_t s) {
  const MEpiResidual e{{nullptr, w}, {nullptr, phi}, {nullptr, r}, coef, mask};
  hipError_t err = mlaunch<double, DAG>(g, nr, G, 1, hin, e, red, s);
  if (err != hipSuccess) return err;
  return launch_mfinalize(kFinResult1, mrhs_nbp(g, G), nr, red, nullptr, 0.0, 0, s);
}

#define LGT_INST_MHOP(R, DAG)                                                                                   \
  template hipError_t launch_mhop_axpy<R, DAG>(const Geom&, int, int, int, HopIn<R>, R2<R>*, R2<R>*,             \
                                                const R2<R>*, const R2<R>*, const double*, hipStream_t,          \
                                                BatchState*, const double*, Reduce, const double*);              \
  template hipError_t launch_mhop_schur_norm<R, DAG>(const Geom&, int, int, HopIn<R>, R2<R>*, const R2<R>*,      \
                                                      const double*, BatchState*, Reduce, hipStream_t);         \
  template hipError_t launch_mhop_schur_cg<R, DAG>(const Geom&, int, int, HopIn<R>, const R2<R>*, R2<R>*,         \
                                                    const double*, BatchState*, Reduce, hipStream_t);

LGT_INST_MHOP(double, false)
LGT_INST_MHOP(double, true)
LGT_INST_MHOP(float, false)
LGT_INST_MHOP(float, true)
template hipError_t launch_mhop_schur_residual<false>(const Geom&, int, int, HopIn<double>, const double2*,
                                                      const double2*, double2*, const double*, const double*, Reduce,
                                                      hipStream_t);
template hipError_t launch_mhop_schur_residual<true>(const Geom&, int, int, HopIn<double>, const double2*,
                                                     const double2*, double2*, const double*, const double*, Reduce,
                                                     hipStream_t);
template hipError_t launch_mhop_residual<false>(const Geom&, int, int, HopIn<double>, const double2*,
                                                const double2*, double2*, const double*, Reduce, hipStream_t);
template hipError_t launch_mhop_residual<true>(const Geom&, int, int, HopIn<double>, const double2*,
                                               const double2*, double2*, const double*, Reduce, hipStream_t);

// ---------------------------------------------------------------------------
// Vector kernels over multi-RHS fields (padding included, except in sums):
// grid (site blocks, planes * nr slabs); slab s of a half field holds plane
// s / nr of right-hand side s % nr.
// ---------------------------------------------------------------------------
template <typename R> static inline dim3 plane_grid(int vs, int nr) {
  return dim3((vs + 255) / 256, Planes<R, R2<R>>::kPlanes * nr);
}
// a thread takes the four spins of a colour (FP64 beside FP32 fields, see Planes)
static inline dim3 colour_grid(int vs, int nr) { return dim3((vs + 255) / 256, 3 * nr); }

// per-RHS |a|^2 over ncomp components (12: half field, 24: full field):
// grid (nbx, nr), block (bx, n) sums its sites over all components into
// partials [bx][kMaxRhs]
template <typename R>
__global__ __launch_bounds__(256) void k_mnorm(int vh, int vs, int ncomp, int nr, const R2<R>* __restrict__ a,
                                               double* partials) {
  __shared__ double sh[4];
  const int n = blockIdx.y;
  double acc = 0.0;
  for (int s = blockIdx.x * 256 + threadIdx.x; s < vh; s += gridDim.x * 256) {
    for (int k = 0; k < ncomp; ++k) {
      const R2<R> v = a[((size_t)k * nr + n) * vs + s];
      acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
    }
  }
  const double t = block_sum<256>(acc, sh);
  if (threadIdx.x == 0) partials[(size_t)blockIdx.x * kMaxRhs + n] = t;
}

static inline int mnorm_blocks(int vh) {
  const int nb = (vh + 255) / 256;
  return nb > 1024 ? 1024 : nb;
}

template <typename R>
hipError_t launch_mnorm(int vh, int vs, int ncomp, int nr, const R2<R>* a, Reduce red, hipStream_t s) {
  const int nb = mnorm_blocks(vh);
  hipLaunchKernelGGL((k_mnorm<R>), dim3(nb, nr), dim3(256), 0, s, vh, vs, ncomp, nr, a, red.partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_mfinalize(kFinResult1, nb, nr, red, nullptr, 0.0, 0, s);
}
template hipError_t launch_mnorm<double>(int, int, int, int, const double2*, Reduce, hipStream_t);

// After the finalize of an iteration: x += alpha_n p for every right-hand
// side whose recursion ran it (still running, or stopped by this finalize:
// conv_iter == iter; nothing in an iteration queued after the whole batch
// stopped, whose finalize leaves iter as it was and sets idle), then
// p = r + beta_n p where the recursion goes on or waits for the update.  The x update is here rather than in the Schur-CG
// epilogue because this kernel reads p anyway.
template <typename R>
__global__ __launch_bounds__(256) void k_mxpay(int vs, int nr, const R2<R>* __restrict__ r, R2<R>* __restrict__ p,
                                               R2<R>* __restrict__ x, const BatchState* st) {
  if (st->idle) return;  // a queued iteration after the batch stopped: nothing ran
  const int n = blockIdx.y % nr;
  const int d = st->done[n];
  const bool ran = d == kDoneRunning || st->conv_iter[n] == st->iter;
  const bool upd = d == kDoneRunning || d == kDoneUpdate;
  if (!ran && !upd) return;
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= vs) return;
  using V = R __attribute__((ext_vector_type(16 / sizeof(R))));
  const size_t i = (size_t)blockIdx.y * vs + s;
  V* __restrict__ pp = reinterpret_cast<V*>(p) + i;
  V* __restrict__ xp = reinterpret_cast<V*>(x) + i;
  V pv = *pp;
  if (ran) *xp += R(st->alpha[n]) * pv;
  if (upd) *pp = reinterpret_cast<const V*>(r)[i] + R(st->beta[n]) * pv;
}
template <typename R>
hipError_t launch_mxpay(int vs, int nr, const R2<R>* r, R2<R>* p, R2<R>* x, BatchState* st, hipStream_t s) {
  hipLaunchKernelGGL((k_mxpay<R>), plane_grid<R>(vs, nr), dim3(256), 0, s, vs, nr, r, p, x, st);
  return hipGetLastError();
}
template hipError_t launch_mxpay<double>(int, int, const double2*, double2*, double2*, BatchState*, hipStream_t);
template hipError_t launch_mxpay<float>(int, int, const float2*, float2*, float2*, BatchState*, hipStream_t);

// x64 += scale_n * xs; xs = 0
__global__ __launch_bounds__(256) void k_mmixed_update(int vs, int nr, float2* xs, double2* __restrict__ x,
                                                       const double* __restrict__ scale) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= vs) return;
  const int own = blockIdx.y / nr, n = blockIdx.y % nr;
  const size_t ps = (size_t)nr * vs, i = (size_t)n * vs + s;
  const double sc = scale[n];
  C<float> v[4];
  C<double> xv[4];
  Planes<float, float2>::ld(xs, ps, own, i, v);
  ld_colour(x, ps, own, i, xv);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    xv[q].re += sc * (double)v[q].re;
    xv[q].im += sc * (double)v[q].im;
    v[q] = czero<float>();
  }
  st_colour(x, ps, own, i, xv);
  Planes<float, float2>::st(xs, ps, own, i, v);
}
hipError_t launch_mmixed_update(int vs, int nr, float2* xs, double2* x, const double* scale, hipStream_t s) {
  hipLaunchKernelGGL(k_mmixed_update, colour_grid(vs, nr), dim3(256), 0, s, vs, nr, xs, x, scale);
  return hipGetLastError();
}

// r = sigma_n r64; p = r (restart_n) or p *= pscale_n
__global__ __launch_bounds__(256) void k_mrescale(int vs, int nr, const double2* __restrict__ r64,
                                                  const double* __restrict__ sigma, float2* __restrict__ r,
                                                  float2* __restrict__ p, const int* __restrict__ restart,
                                                  const double* __restrict__ pscale) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= vs) return;
  const int own = blockIdx.y / nr, n = blockIdx.y % nr;
  const size_t ps = (size_t)nr * vs, i = (size_t)n * vs + s;
  const double sg = sigma[n], sp = pscale[n];
  C<double> v[4];
  C<float> w[4], q[4];
  ld_colour(r64, ps, own, i, v);
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = {(float)(sg * v[k].re), (float)(sg * v[k].im)};
  Planes<float, float2>::st(r, ps, own, i, w);
  if (!restart[n]) {
    Planes<float, float2>::ld(p, ps, own, i, q);
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = {(float)(sp * (double)q[k].re), (float)(sp * (double)q[k].im)};
  }
  Planes<float, float2>::st(p, ps, own, i, w);
}
hipError_t launch_mrescale(int vs, int nr, const double2* r64, const double* sigma, float2* r, float2* p,
                           const int* restart, const double* pscale, hipStream_t s) {
  hipLaunchKernelGGL(k_mrescale, colour_grid(vs, nr), dim3(256), 0, s, vs, nr, r64, sigma, r, p, restart, pscale);
  return hipGetLastError();
}

// r = b, p = b, x = 0 (FP64 multi-RHS CG start); per-RHS |b|^2 to state
__global__ __launch_bounds__(256) void k_mcg_init64(size_t n, const double2* __restrict__ b, double2* __restrict__ r,
                                                    double2* __restrict__ p, double2* __restrict__ x) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const double2 v = b[i];
    r[i] = v;
    p[i] = v;
    x[i] = make_double2(0.0, 0.0);
  }
}
hipError_t launch_mcg_init64(int vh, int vs, int nr, const double2* b, double2* r, double2* p, double2* x, BatchState* st,
                             Reduce red, double tol, int max_iter, hipStream_t s) {
  const size_t n = (size_t)12 * vs * nr;
  hipLaunchKernelGGL(k_mcg_init64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, b, r, p, x);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int nb = mnorm_blocks(vh);
  hipLaunchKernelGGL((k_mnorm<double>), dim3(nb, nr), dim3(256), 0, s, vh, vs, 12, nr, b, red.partials);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_mfinalize(kFinCgInit, nb, nr, red, st, tol, max_iter, s);
}

// One block: per-RHS sums of the partials of the previous launch, then thread
// n updates right-hand side n (the decisions that take all of them together
// come from votes of the first wave, which holds them).  With the sums taken
// together (sum_rows) and the scalars updated side by side instead of by one
// thread in turn, a 12-RHS finalize at 16^4 went from 21 us (in a batch over
// three lattices) to 6.9 us.
__global__ __launch_bounds__(256) void k_mfinalize(int mode, int nblk, int nr, const double* __restrict__ partials,
                                                   BatchState* st, double* result, double tol, int max_iter,
                                                   Mailbox* mb) {
  const int n = threadIdx.x;
  const bool mine = n < nr;
  if (mode == kFinCgStep && st->all_done) {  // the iteration was skipped
    if (mine && st->done[n] == kDoneUpdate) st->done[n] = kDoneUpdateHeld;
    if (n == 0) {
      st->any_update = 0;
      st->idle = 1;
      post_progress(mb, st->iter, 1);
    }
    return;
  }
  const double tot = sum_rows(partials, nblk);
  if (n >= 64) return;  // the first wave goes on
  if (mode == kFinResult1) {
    if (mine) result[n] = tot;
    return;
  }
  if (mode == kFinCgInit) {
    int done = kDoneConverged;
    if (mine) {
      done = !isfinite(tot) ? kDoneBreakdown : (tot == 0.0 ? kDoneConverged : kDoneRunning);
      st->rr[n] = tot;
      st->rr_max[n] = tot;
      st->rr_stop[n] = tol * tol * tot;
      st->alpha[n] = st->beta[n] = st->pap[n] = 0.0;
      st->done[n] = done;
      st->conv_iter[n] = 0;
      st->work[n] = 0;
    }
    const bool all = __ballot(done == kDoneRunning) == 0;
    if (n == 0) {
      st->nr = nr;
      st->iter = 0;
      st->max_iter = max_iter;
      st->delta2 = 0.0;
      st->any_update = 0;
      st->idle = 0;
      st->all_done = all;
    }
    return;
  }
  // kFinCgStep
  const int iter = st->iter + 1;
  const double d2 = st->delta2;
  int done = kDoneConverged;
  if (mine) {
    done = st->done[n];
    if (done == kDoneUpdate) done = kDoneUpdateHeld;
    if (done == kDoneRunning) {  // the iteration ran for this right-hand side
      const double rr = tot, rr_max = fmax(st->rr_max[n], rr);
      st->work[n] += 1;
      st->beta[n] = rr / st->rr[n];
      st->rr[n] = rr;
      st->rr_max[n] = rr_max;
      if (!isfinite(rr)) done = kDoneBreakdown;
      else if (rr <= st->rr_stop[n]) done = d2 > 0.0 ? kDoneUpdate : kDoneConverged;
      else if (rr <= d2 * rr_max) done = kDoneUpdate;
      else if (iter >= st->max_iter) done = kDoneMaxIter;
      if (done != kDoneRunning) st->conv_iter[n] = iter;
    }
    st->done[n] = done;
  }
  const unsigned long long running = __ballot(done == kDoneRunning);
  const unsigned long long open = __ballot(done != kDoneConverged);  // not yet verified (reliable updates on)
  const bool any_update = __ballot(done == kDoneUpdate) != 0;
  if (n == 0) {
    st->idle = 0;
    st->iter = iter;
    st->all_done = running == 0;
    st->any_update = any_update;
    // the host has to act once every right-hand side is done or, with reliable
    // updates on (delta2 > 0), once half of those not yet verified have
    // stopped (a stopped one idles until the update)
    const int active = __popcll(open), stopped = active - __popcll(running);
    post_progress(mb, iter, running == 0 || (d2 > 0.0 && 2 * stopped >= active));
  }
}

hipError_t launch_mfinalize(int mode, int nblk, int nr, Reduce red, BatchState* st, double tol, int max_iter,
                            hipStream_t s) {
  if ((size_t)nblk * kMaxRhs > red.ndoubles) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mfinalize, dim3(1), dim3(256), 0, s, mode, nblk, nr, red.partials, st, red.result, tol,
                     max_iter, red.mbox);
  return hipGetLastError();
}

// element (k, n, site) of a multi-RHS FP64 field is at (k nr + n) vs + site
__global__ __launch_bounds__(256) void k_mzero_rhs(size_t tot, int vs, int nr, double2* __restrict__ f,
                                                   unsigned mask) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= tot) return;
  const int n = (int)((t / (size_t)vs) % (size_t)nr);
  if ((mask >> n) & 1u) f[t] = make_double2(0.0, 0.0);
}
hipError_t launch_mzero_rhs(int vs, int ncomp, int nr, double2* f, unsigned mask, hipStream_t s) {
  if (!mask) return hipSuccess;
  const size_t tot = (size_t)ncomp * nr * vs;
  hipLaunchKernelGGL(k_mzero_rhs, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, tot, vs, nr, f, mask);
  return hipGetLastError();
}

// canonical spinor [V][4][3] of right-hand side n <-> full multi-RHS field
__global__ __launch_bounds__(256) void k_mpack(Geom g, int nr, int n, const double2* __restrict__ canon,
                                               double2* __restrict__ packed) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= 2 * (size_t)g.vh * 12) return;
  const int s = (int)(t / 12), k = (int)(t % 12);
  int c[4];
  lex_coords(g, s, c);
  packed[(((size_t)parity_of(c) * 12 + k) * nr + n) * g.vs + (s >> 1)] = canon[t];
}
__global__ __launch_bounds__(256) void k_munpack(Geom g, int nr, int n, const double2* __restrict__ packed,
                                                 double2* __restrict__ canon) {
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= 2 * (size_t)g.vh * 12) return;
  const int s = (int)(t / 12), k = (int)(t % 12);
  int c[4];
  lex_coords(g, s, c);
  canon[t] = packed[(((size_t)parity_of(c) * 12 + k) * nr + n) * g.vs + (s >> 1)];
}
hipError_t launch_mpack(const Geom& g, int nr, int n, const double2* canon, double2* packed, hipStream_t s) {
  const size_t tot = 2 * (size_t)g.vh * 12;
  hipLaunchKernelGGL(k_mpack, dim3((tot + 255) / 256), dim3(256), 0, s, g, nr, n, canon, packed);
  return hipGetLastError();
}
hipError_t launch_munpack(const Geom& g, int nr, int n, const double2* packed, double2* canon, hipStream_t s) {
  const size_t tot = 2 * (size_t)g.vh * 12;
  hipLaunchKernelGGL(k_munpack, dim3((tot + 255) / 256), dim3(256), 0, s, g, nr, n, packed, canon);
  return hipGetLastError();
}

}  // namespace lgt
