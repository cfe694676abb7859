// Multi-shift CG on the even/odd Schur normal operator A = Mhat^dag Mhat
// (Mhat = 1 - kappa^2 H_oe H_eo, odd sites): X_i = (A + sigma_i)^-1 phi_o for
// several shifts sigma_i >= 0 from one Krylov space, the building block of
// rational (RHMC) pseudofermion actions (Sec. I names RHMC among the targets).
//
// The base CG runs on A itself with the usual four hop launches per
// iteration (the base solution is not tracked).  The shifted residuals stay
// collinear with the base one, r_i = zeta_i r, and the shifted iterates
// follow from scalar recurrences (Jegerlehner's shifted CG):
//   zeta_i' = zeta_i zeta_i^- alpha^- / (alpha beta^- (zeta_i^- - zeta_i)
//                                        + zeta_i^- alpha^- (1 + sigma_i alpha))
//   alpha_i = alpha zeta_i' / zeta_i,  beta_i = beta (zeta_i' / zeta_i)^2
//   x_i += alpha_i p_i;  p_i = zeta_i' r + beta_i p_i
// (^-: previous iteration, ': next).  A one-block finalize forms them and
// the stopping test.  Shift i stops updating once |zeta_i|^2 |r|^2 <= tol^2
// |phi_o|^2; the solve stops when all have.  FP64 throughout.
//
// The recurrences couple neither the shifts' vectors to the base recursion
// nor the shifts to each other, so the vectors may lag: the last kGroup
// residuals r are kept in a ring and the iterations' coefficients in the
// state, and one kernel carries every x_i, p_i through up to kGroup
// iterations in registers.  Updated in every iteration, the 12 pairs of 16^4
// were 302 MB each time, 30 us of a 98 us iteration (10 TB/s); in groups of
// eight 50 us a group.  The base direction moves into the first hop
// (EpiDirection), and the hops of the true residual leave the fields of a
// rational force's term behind, so the force takes them from there: 12 terms
// at 16^4 8.47 -> 5.30 ms.
#include <algorithm>
#include <cmath>

#include "lgt_ctx.h"

using namespace lgt;

namespace {

constexpr int kMaxShift = 32;  // two result slots per shift fill the context's 64
constexpr int kGroup = 8;      // iterations a pass over the shifts' vectors takes (fewer if the ring did not fit)

struct ShiftState {
  int ns, pad;
  double alpha_prev, beta_prev;
  double rr_stop;
  double sigma[kMaxShift], zeta[kMaxShift], zeta_prev[kMaxShift];
  int done[kMaxShift];
  // coefficients of the iterations since the last update, by their place in the group
  double alpha_s[kGroup][kMaxShift], beta_s[kGroup][kMaxShift], zeta_s[kGroup][kMaxShift];
  int upd[kGroup][kMaxShift];
};

// rr = sum of the |r|^2 partials of the last hop; beta; the shift
// recurrences (thread i: shift i) and the stop test; slot: the iteration's
// place in its group.
__global__ __launch_bounds__(256) void k_msfinalize(int nblk, const double* __restrict__ partials, SolverState* st,
                                                    ShiftState* ss, int slot, Mailbox* mb) {
  const int i = threadIdx.x;
  const int ns = ss->ns;
  if (st->done != kDoneRunning) {  // the iteration was skipped
    if (i < ns) ss->upd[slot][i] = 0;
    if (i == 0) post_progress(mb, st->iter, 1);
    return;
  }
  __shared__ double s_rr;
  double tot[1];
  sum_partials<256, 1>(partials, nblk, tot);
  if (i == 0) s_rr = tot[0];
  __syncthreads();
  const double rr = s_rr;
  const double a = st->alpha;  // alpha of this iteration (formed by the third hop)
  const double b = rr / st->rr;
  int open = 0;
  if (i < ns) {
    int upd = 0;
    if (!ss->done[i]) {
      const double z = ss->zeta[i], zp = ss->zeta_prev[i];
      const double zn = z * zp * ss->alpha_prev /
                        (a * ss->beta_prev * (zp - z) + zp * ss->alpha_prev * (1.0 + ss->sigma[i] * a));
      ss->alpha_s[slot][i] = a * zn / z;
      ss->beta_s[slot][i] = b * (zn / z) * (zn / z);
      ss->zeta_s[slot][i] = zn;
      ss->zeta_prev[i] = z;
      ss->zeta[i] = zn;
      upd = 1;
      if (zn * zn * rr <= ss->rr_stop) ss->done[i] = 1;
      else open = 1;
    }
    ss->upd[slot][i] = upd;
  }
  const int all = __syncthreads_and(!open);
  if (i != 0) return;
  ss->alpha_prev = a;
  ss->beta_prev = b;
  st->beta = b;
  st->rr = rr;
  st->iter += 1;
  if (!isfinite(rr)) st->done = kDoneBreakdown;
  else if (all) st->done = kDoneConverged;
  else if (st->iter >= st->max_iter) st->done = kDoneMaxIter;
  post_progress(mb, st->iter, st->done != kDoneRunning);
}

// The residuals of a group's iterations.
struct Ring {
  double2* r[kGroup];
};

// Iterations 0 .. m-1 of the group for the kUpdShifts shifts from kUpdShifts
// blockIdx.y on, one element a thread: x_i += alpha_i p_i, p_i = zeta_i r +
// beta_i p_i for each iteration in which the shift was updated (its updates
// end with its convergence, so they are the first ones).  Shift fields are
// contiguous: x_i = X + i n, p_i = Pn + i n.  Four shifts share the group's
// residuals in registers: with a shift a block the residuals, read once per
// shift, were two thirds of the traffic (76 us a group at 16^4 with 12 shifts,
// 50 us like this).
constexpr int kUpdShifts = 4;
__global__ __launch_bounds__(256) void k_msupdate(int n, int ns, int m, Ring ring, double2* __restrict__ X,
                                                  double2* __restrict__ Pn, const ShiftState* __restrict__ ss) {
  const int s0 = blockIdx.y * kUpdShifts;
  int cnt[kUpdShifts], most = 0;
#pragma unroll
  for (int q = 0; q < kUpdShifts; ++q) {
    cnt[q] = 0;
    while (s0 + q < ns && cnt[q] < m && ss->upd[cnt[q]][s0 + q]) ++cnt[q];
    most = max(most, cnt[q]);
  }
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (most == 0 || i >= n) return;
  C<double> x[kUpdShifts], p[kUpdShifts], r[kGroup];
#pragma unroll
  for (int q = 0; q < kUpdShifts; ++q) {
    if (cnt[q] == 0) continue;
    p[q] = ld<double>(Pn + (size_t)(s0 + q) * n + i);
    x[q] = ld<double>(X + (size_t)(s0 + q) * n + i);
  }
#pragma unroll
  for (int j = 0; j < kGroup; ++j)
    if (j < most) r[j] = ld<double>(ring.r[j] + i);
#pragma unroll
  for (int j = 0; j < kGroup; ++j) {
#pragma unroll
    for (int q = 0; q < kUpdShifts; ++q) {
      if (j >= cnt[q]) continue;
      x[q] += ss->alpha_s[j][s0 + q] * p[q];
      p[q] = ss->zeta_s[j][s0 + q] * r[j] + ss->beta_s[j][s0 + q] * p[q];
    }
  }
#pragma unroll
  for (int q = 0; q < kUpdShifts; ++q) {
    if (cnt[q] == 0) continue;
    st<double>(X + (size_t)(s0 + q) * n + i, x[q]);
    st<double>(Pn + (size_t)(s0 + q) * n + i, p[q]);
  }
}

__global__ __launch_bounds__(256) void k_msinit(int n, int ns, const double2* __restrict__ b, double2* __restrict__ r,
                                                double2* __restrict__ p, double2* __restrict__ X,
                                                double2* __restrict__ Pn) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double2 v = b[i];
    r[i] = v;
    p[i] = v;
    for (int s = 0; s < ns; ++s) {
      X[(size_t)s * n + i] = make_double2(0.0, 0.0);
      Pn[(size_t)s * n + i] = v;
    }
  }
}

// |x|^2, Re <x, phi> and |y|^2 of shift blockIdx.y: block partials [shift][value][block]
__global__ __launch_bounds__(256) void k_msterms(int n, const double2* __restrict__ phi, const double2* __restrict__ X,
                                                 const double2* __restrict__ Y, double* __restrict__ partials) {
  const double2* __restrict__ x = X + (size_t)blockIdx.y * n;
  const double2* __restrict__ y = Y + (size_t)blockIdx.y * n;
  double v[3] = {0.0, 0.0, 0.0};
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const double2 a = x[i], f = phi[i], b = y[i];
    v[0] += a.x * a.x + a.y * a.y;
    v[1] += a.x * f.x + a.y * f.y;
    v[2] += b.x * b.x + b.y * b.y;
  }
  __shared__ double sh[4];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double t = block_sum<256>(v[k], sh);
    if (threadIdx.x == 0) partials[((size_t)blockIdx.y * 3 + k) * gridDim.x + blockIdx.x] = t;
  }
}

// result[b] = sum of the nblk partials of row b, a block each
__global__ __launch_bounds__(256) void k_mssums(int nblk, const double* __restrict__ partials, double* result) {
  double tot[1];
  sum_partials<256, 1>(partials + (size_t)blockIdx.x * nblk, nblk, tot);
  if (threadIdx.x == 0) result[blockIdx.x] = tot[0];
}

constexpr int kTermBlocks = 128;  // blocks a shift of k_msterms

}  // namespace

struct MultiShiftWork {
  int ns = 0;
  double2* X = nullptr;   // ns odd halves
  double2* Pn = nullptr;  // ns odd halves; after the solve, the force fields of a group of terms
  int group = 0;          // residuals the ring holds (1: a single one, updated in place)
  Ring ring{};            // odd halves
  double2* p = nullptr;   // base direction
  double* partials = nullptr;  // [ns][hop blocks] residual norms, [ns][3][kTermBlocks] action terms
  double* sums = nullptr;      // their sums: ns and 3 ns
  double* hsums = nullptr;     // pinned
  ShiftState* ss = nullptr;
  ShiftState* hss = nullptr;  // pinned
};

void lgt_ctx_free_multishift(lgt_ctx* c) {
  MultiShiftWork* w = c->mshift;
  if (!w) return;
  (void)hipFree(w->X);
  (void)hipFree(w->Pn);
  for (int k = 0; k < w->group; ++k) (void)hipFree(w->ring.r[k]);
  (void)hipFree(w->p);
  (void)hipFree(w->partials);
  (void)hipFree(w->sums);
  if (w->hsums) (void)hipHostFree(w->hsums);
  (void)hipFree(w->ss);
  if (w->hss) (void)hipHostFree(w->hss);
  delete w;
  c->mshift = nullptr;
}

static MultiShiftWork* mshift_work(lgt_ctx* c, int ns) {
  if (c->mshift && c->mshift->ns >= ns) return c->mshift;
  lgt_ctx_free_multishift(c);
  MultiShiftWork* w = new MultiShiftWork();
  c->mshift = w;
  try {
    const size_t hb = c->half_elems() * sizeof(double2);
    const size_t np = (size_t)ns * (reduce_capacity(c->vh) + 3 * kTermBlocks);
    LGT_HIP(hipMalloc(&w->X, ns * hb));
    LGT_HIP(hipMalloc(&w->Pn, ns * hb));
    LGT_HIP(hipMalloc(&w->p, hb));
    LGT_HIP(hipMalloc(&w->partials, np * sizeof(double)));
    LGT_HIP(hipMalloc(&w->sums, (size_t)4 * ns * sizeof(double)));
    LGT_HIP(hipHostMalloc(&w->hsums, (size_t)4 * ns * sizeof(double), hipHostMallocDefault));
    LGT_HIP(hipMalloc(&w->ss, sizeof(ShiftState)));
    LGT_HIP(hipHostMalloc(&w->hss, sizeof(ShiftState), hipHostMallocDefault));
    LGT_HIP(hipMalloc(&w->ring.r[0], hb));
    w->group = 1;
    LGT_HIP(hipMemsetAsync(w->ring.r[0], 0, hb, c->stream));
  } catch (...) {
    lgt_ctx_free_multishift(c);
    throw;
  }
  w->ns = ns;
  return w;
}

// Residuals of the ring beyond the first, which only save traffic: taken once
// everything else that the call allocates is there, and only while an eighth
// of the device memory stays free for what comes after it (the reserve of the
// smearing's checkpoints).  The results have the same bits for any number.
static void grow_ring(lgt_ctx* c, MultiShiftWork* w) {
  const size_t hb = c->half_elems() * sizeof(double2);
  for (; w->group < kGroup; ++w->group) {
    size_t avail = 0, total = 0;
    LGT_HIP(hipMemGetInfo(&avail, &total));
    if (avail < total / 8 + hb) return;
    const hipError_t e = hipMalloc(&w->ring.r[w->group], hb);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      return;
    }
    LGT_HIP(e);
    LGT_HIP(hipMemsetAsync(w->ring.r[w->group], 0, hb, c->stream));
  }
}

int lgt_ctx_max_shifts() { return kMaxShift; }

// phi: packed full field (odd half read).  Xout[i]: the caller's canonical
// full fields, written with X_i on the odd sites and zero on the even ones
// (Xout null: the solutions stay in the workspace, mshift->X + i V/2 * 12).
// The shifted recursions stop at half the tolerance; the returned true_res
// is the largest FP64 true residual ||phi_o - (A + sigma_i) X_i|| / ||phi_o||
// over the shifts, and converged is false if it exceeds the tolerance.
// force (or null): called for every group of terms [i0, i0 + c) while X_e =
// H_eo X_i, Y_o = Mhat X_i and A_e = H_oe^dag Y_o, which the true residual
// passes through, are at hand, c odd or even halves each, n elements apart.
SolveStats lgt_ctx::solve_multishift(const double2* phi, int ns, const double* shifts, void* const* Xout,
                                     const SolverOpts& o, const MultiShiftTerms& force) {
  SolveStats st;
  MultiShiftWork* w = mshift_work(this, ns);
  const size_t h = half_elems();
  const int n = (int)h;
  const double2* phio = phi + h;
  double2* stage = f64(kStageB);  // packed full field holding one output at a time
  LGT_HIP(launch_zero64(n, stage, stream));
  auto emit = [&](int i, const double2* xo) {
    if (!Xout) return;
    LGT_HIP(launch_copy64(n, xo, stage + h, stream));
    LGT_HIP(launch_unpack(g, 12, stage, (double2*)Xout[i], stream));
  };
  LGT_HIP(launch_norm_dot(n, phio, nullptr, red(), 0, stream));
  read_results(1);
  const double bb = host_result[0];
  if (!std::isfinite(bb)) throw Error(LGT_ERR_NONFINITE, "phi holds NaN or Inf");
  if (bb == 0.0) {
    LGT_HIP(launch_zero64(n, stage + h, stream));
    LGT_HIP(launch_zero64((int)(ns * h), w->X, stream));
    for (int i = 0; i < ns; ++i)
      if (Xout) LGT_HIP(launch_unpack(g, 12, stage, (double2*)Xout[i], stream));
    st.true_res = 0.0;
    return st;
  }
  double2* p = w->p;
  double2* t = f64(kW0);  // even-half scratch, as the FP64 CG's: H p, kept for the next iteration
  double2* t2 = t + h;
  double2* wv = f64(kW4) + h;  // odd-half scratch, as the FP64 CG's
  // the recursion's hops read two-row links when the links are SU(3) to FP64
  // rounding, as the single-shift FP64 CG's; the true residuals below use the
  // full links
  compress_links64();
  grow_ring(this, w);
  const int m = w->group;
  const int nb = std::min((n + 255) / 256, 2048);
  hipLaunchKernelGGL(k_msinit, dim3(nb), dim3(256), 0, stream, n, ns, phio, w->ring.r[m - 1], p, w->X, w->Pn);
  LGT_HIP(hipGetLastError());
  ShiftState& s = *w->hss;
  s = ShiftState{};
  s.ns = ns;
  s.alpha_prev = 1.0;
  s.beta_prev = 0.0;
  const double tol_in = 0.5 * o.tol;
  s.rr_stop = tol_in * tol_in * bb;
  for (int i = 0; i < ns; ++i) {
    s.sigma[i] = shifts[i];
    s.zeta[i] = s.zeta_prev[i] = 1.0;
  }
  LGT_HIP(hipMemcpyAsync(w->ss, w->hss, sizeof(ShiftState), hipMemcpyHostToDevice, stream));
  SolverState& b0 = *host_state;
  b0 = SolverState{};
  b0.rr = bb;
  b0.rr0 = bb;
  b0.rr_max = bb;
  b0.rr_stop = 0.0;  // the base recursion never stops on its own: the shifts decide
  b0.max_iter = o.max_iter;
  b0.done = kDoneRunning;
  LGT_HIP(hipMemcpyAsync(state, host_state, sizeof(SolverState), hipMemcpyHostToDevice, stream));
  const double k2 = -kappa * kappa;
  const Reduce rd = red();
  sync();
  const int nk = host_flags[2] == 0 ? 6 : 9;
  const double2* links = nk == 6 ? U64c : U64;
  int queued = 0;
  auto update = [&](int slots) {
    hipLaunchKernelGGL(k_msupdate, dim3((n + 255) / 256, (ns + kUpdShifts - 1) / kUpdShifts), dim3(256), 0, stream, n,
                       ns, slots, w->ring, w->X, w->Pn, w->ss);
    LGT_HIP(hipGetLastError());
  };
  auto iteration = [&] {
    const int slot = queued % m;
    const double2* r = w->ring.r[(slot + m - 1) % m];
    if (queued == 0)
      LGT_HIP((launch_hop_axpy<double, false>(g, 0, HopIn<double>{links, p, p, nk}, t, t, nullptr, nullptr, 1.0,
                                               stream, state)));
    else
      LGT_HIP(launch_hop_direction(g, links, nk, t, p, r, state, stream));
    LGT_HIP((launch_hop_schur_norm<double, double2, false>(g, HopIn<double>{links, t, t, nk}, wv, p, k2, state, rd,
                                                            stream)));
    // block 0 also forms alpha = |r|^2 / |Mhat p|^2 from the partials
    LGT_HIP((launch_hop_axpy<double, true>(g, 0, HopIn<double>{links, wv, wv, nk}, t2, t2, nullptr, nullptr, 1.0,
                                            stream, state, rd.partials)));
    // the next residual r - alpha A p, |r|^2 partials; the base solution is not formed
    LGT_HIP((launch_hop_schur_cg<double, double2, true>(g, HopIn<double>{links, t2, t2, nk}, wv, nullptr, r,
                                                         w->ring.r[slot], p, k2, state, rd, stream)));
    hipLaunchKernelGGL(k_msfinalize, dim3(1), dim3(256), 0, stream, hop_blocks(g, 1), rd.partials, state, w->ss, slot,
                       rd.mbox);
    LGT_HIP(hipGetLastError());
    ++queued;
    if (slot == m - 1) update(m);
  };
  for (int iter0 = 0;;) {
    drive(iter0, iteration);
    LGT_HIP(hipMemcpyAsync(host_state, state, sizeof(SolverState), hipMemcpyDeviceToHost, stream));
    sync();
    if (b0.done != kDoneRunning) break;
    iter0 = b0.iter;
  }
  st.iters = b0.iter;
  if (b0.done == kDoneBreakdown) throw Error(LGT_ERR_NONFINITE, "multi-shift CG breakdown");
  if (b0.done == kDoneMaxIter) st.converged = false;
  if (queued % m != 0) update(queued % m);
  // true residuals phi_o - (A + sigma_i) X_i with the full links, all norms read back at once
  const int nres = hop_blocks(g, 1);
  // the force's fields of a group of terms: in the shifts' directions, which
  // are done with, three halves a term (fewer than three shifts: in the scratch)
  const bool in_dirs = force && ns >= 3;
  const int gc = in_dirs ? std::min(kBilinearTerms, ns / 3) : 1;
  double2* xe = in_dirs ? w->Pn : t;
  double2* yo = in_dirs ? w->Pn + gc * h : wv;
  double2* ae = in_dirs ? w->Pn + 2 * gc * h : t2;
  for (int i0 = 0; i0 < ns; i0 += gc) {
    const int c = std::min(gc, ns - i0);
    for (int i = 0; i < c; ++i) {
      const double2* xi = w->X + (size_t)(i0 + i) * h;
      double2 *e = xe + i * h, *y = yo + i * h, *a = ae + i * h;
      LGT_HIP((launch_hop_axpy<double, false>(g, 0, HopIn<double>{U64, xi, xi}, e, e, nullptr, nullptr, 1.0, stream)));
      LGT_HIP((launch_hop_axpy<double, false>(g, 1, HopIn<double>{U64, e, e}, y, y, xi, xi, k2, stream)));
      LGT_HIP((launch_hop_axpy<double, true>(g, 0, HopIn<double>{U64, y, y}, a, a, nullptr, nullptr, 1.0, stream)));
      LGT_HIP(launch_hop_shift_residual(g, HopIn<double>{U64, a, a}, y, xi, phio, shifts[i0 + i], k2,
                                        w->partials + (size_t)(i0 + i) * nres, stream));
      emit(i0 + i, xi);
    }
    if (force) force(i0, c, xe, yo, ae);
  }
  hipLaunchKernelGGL(k_mssums, dim3(ns), dim3(256), 0, stream, nres, w->partials, w->sums);
  LGT_HIP(hipGetLastError());
  LGT_HIP(hipMemcpyAsync(w->hsums, w->sums, 4 * ns * sizeof(double), hipMemcpyDeviceToHost, stream));
  sync();
  double worst = 0.0;
  for (int i = 0; i < ns; ++i) {
    const double tr = std::sqrt(w->hsums[i] / bb);
    if (!std::isfinite(tr)) throw Error(LGT_ERR_NONFINITE, "non-finite residual");
    worst = std::max(worst, tr);
  }
  st.true_res = worst;
  if (worst > o.tol) st.converged = false;
  return st;
}

// Rational (RHMC) even/odd pseudofermion action S_R = phi_o^dag R(A) phi_o,
// R(A) = a0 + sum_i a_i (A + sigma_i)^-1, A = Mhat^dag Mhat, and its force.
// With X_i = (A + sigma_i)^-1 phi_o from one multi-shift solve, the term i
// varies as -a_i X_i^dag dA X_i = -2 a_i Re[Y_i^dag dMhat X_i], Y_i = Mhat X_i
// (the shift is constant): the even/odd bilinear of each X_i with the
// coefficient -2 kappa a_i, summed into one gradient.  S_R is evaluated as
// a0 |phi_o|^2 + sum_i a_i (2 Re phi_o^dag X_i - |Y_i|^2 - sigma_i |X_i|^2),
// equal to the action at the solutions and second order in their error.
SolveStats lgt_ctx::rational_force(const double2* phi, int ns, const double* shifts, const double* residues,
                                   double a0, const SolverOpts& o, int mode, double dt, void* out, double* S) {
  const size_t h = half_elems();
  const int n = (int)h;
  const double2* phio = phi + h;
  double2* zsum = g64(12);
  bool emitted = false;
  auto force = [&](int i0, int c, const double2* xe, const double2* yo, const double2* ae) {
    MultiShiftWork* w = mshift;
    const double2* xo = w->X + (size_t)i0 * h;
    BilinearSum t{ae, yo, xe, xo, h, h, c, {}};
    for (int i = 0; i < c; ++i) t.weight[i] = residues[i0 + i];
    emitted = i0 + c == ns;
    LGT_HIP(launch_bilinear_sum(g, U64, t, zsum, i0 == 0, emitted, kappa, -2.0 * kappa, mode, dt, out, stream));
    if (S) {
      double* part = w->partials + (size_t)w->ns * reduce_capacity(vh) + (size_t)i0 * 3 * kTermBlocks;
      hipLaunchKernelGGL(k_msterms, dim3(kTermBlocks, c), dim3(256), 0, stream, n, phio, xo, yo, part);
      LGT_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_mssums, dim3(3 * c), dim3(256), 0, stream, kTermBlocks, part, w->sums + ns + 3 * i0);
      LGT_HIP(hipGetLastError());
    }
  };
  SolveStats st = solve_multishift(phi, ns, shifts, nullptr, o, force);
  if (!emitted) {  // phi_o = 0: every term is zero
    BilinearSum none{zsum, zsum, zsum, zsum, 0, 0, 0, {}};
    LGT_HIP(launch_bilinear_sum(g, U64, none, zsum, true, true, kappa, -2.0 * kappa, mode, dt, out, stream));
    if (S) *S = 0.0;
    return st;
  }
  if (S) {
    LGT_HIP(launch_norm_dot(n, phio, nullptr, red(), 0, stream));
    read_results(1);
    double sr = a0 * host_result[0];
    for (int i = 0; i < ns; ++i) {
      const double* q = mshift->hsums + ns + 3 * i;  // |X_i|^2, Re <X_i, phi_o>, |Y_i|^2
      sr += residues[i] * (2.0 * q[1] - q[2] - shifts[i] * q[0]);
    }
    *S = sr;
  }
  return st;
}
