// SU(3) device functions shared by the force and stout kernels: link access
// by coordinates, the plaquette staple sum, exp of su(3) and reunitarization.
#pragma once

#include "lgt_device.h"

namespace lgt {

// Order of the 64-site blocks of the gauge-link kernels (staple force,
// stout levels; logical block lb, parity lb & 1, so the two parities of a
// site block run side by side).  On lattices above 131072 sites per parity
// whose t-slice holds whole blocks: where the (x, y) plane holds nyc whole
// blocks and Lz, Lt are multiples of 4, t fastest within groups of 4
// t-slices, then z within groups of 4 planes, then the nyc blocks of a
// plane, then the z groups, then the t groups; otherwise t fastest within
// groups of tgrp t-slices of bps blocks.  A block's neighbours in t and z
// were then read a few dozen blocks earlier on the same XCD (32^3x64, staple
// force: 1501 -> 1374 us; stout levels 9.3 -> 8.0 ms).
struct BlockOrder {
  int bps, tgrp, nyc;
};
__host__ __device__ inline BlockOrder gauge_block_order(const Geom& g) {
  BlockOrder o{0, 0, 0};
  const int vslice = g.vh / g.L[3];
  o.bps = vslice / 64;
  if (vslice % 64 != 0 || o.bps == 0 || g.vh <= 131072) return o;
  o.tgrp = g.L[3] % 8 == 0 ? 8 : (g.L[3] % 4 == 0 ? 4 : 2);
  const int plane = g.hx * g.L[1];
  if (plane % 64 == 0 && g.L[2] % 4 == 0 && g.L[3] % 4 == 0) o.nyc = plane / 64;
  return o;
}
__device__ __forceinline__ int gauge_site_block(int lb, const BlockOrder& o, int lz) {
  int r = lb >> 1;
  if (o.nyc > 0) {
    const int t_in = r & 3;
    r >>= 2;
    const int z_in = r & 3;
    r >>= 2;
    const int yc = r % o.nyc;
    r /= o.nyc;
    const int nzg = lz >> 2;
    const int zo = r % nzg, to = r / nzg;
    return ((to * 4 + t_in) * lz + zo * 4 + z_in) * o.nyc + yc;
  }
  if (o.tgrp > 0) {
    const int span = o.tgrp * o.bps;
    const int grp = r / span, rem = r - grp * span;
    const int chunk = rem / o.tgrp, tl = rem - chunk * o.tgrp;
    return (grp * o.tgrp + tl) * o.bps + chunk;
  }
  return r;
}

__device__ __forceinline__ M3<double> link_at(const double2* U, const Geom& g, const int c[4], int mu) {
  return load_m3<double>(gptr<double>(U, g, parity_of(c), mu), g.vs, cb_of(g, c));
}


// The link U_mu of parity p at checkerboard site cb.  p and mu must be the
// same for the whole wave: the load then takes one 32-bit offset a lane and
// the component planes' offsets from scalar registers, no address arithmetic.
__device__ __forceinline__ M3<double> link_uni(const double2* U, const Geom& g, int p, int mu, int cb) {
  const unsigned gs = (unsigned)g.vs * (unsigned)sizeof(double2);
  const BufRsrc r = make_rsrc(U + (size_t)((p * 4 + mu) * 9) * g.vs, (size_t)9 * gs);
  M3<double> u;
#pragma unroll
  for (int k = 0; k < 9; ++k) u.m[k] = ld_buf<double>(r, (unsigned)cb * (unsigned)sizeof(double2), k * gs);
  return u;
}

// A traceless anti-Hermitian matrix Q as its eight real numbers: the upper
// off-diagonal elements and the imaginary parts of the first two diagonal
// ones.  Stored as four complex planes, [parity][mu][4][vs].
struct Su3Alg {
  C<double> o01, o02, o12;
  double d0, d1;
};
__device__ __forceinline__ Su3Alg operator-(const Su3Alg& a, const Su3Alg& b) {
  return {a.o01 - b.o01, a.o02 - b.o02, a.o12 - b.o12, a.d0 - b.d0, a.d1 - b.d1};
}
__device__ __forceinline__ Su3Alg operator-(const Su3Alg& a) { return {-a.o01, -a.o02, -a.o12, -a.d0, -a.d1}; }
__device__ __forceinline__ void store_alg(double2* f, const Geom& g, int p, int mu, int cb, const M3<double>& q) {
  double2* t = f + (size_t)((p * 4 + mu) * 4) * g.vs + cb;
  st<double>(t, q.m[1]);
  st<double>(t + g.vs, q.m[2]);
  st<double>(t + 2 * (size_t)g.vs, q.m[5]);
  st<double>(t + 3 * (size_t)g.vs, cmk<double>(q.m[0].im, q.m[4].im));
}
// p and mu uniform over the wave, as link_uni
__device__ __forceinline__ Su3Alg alg_uni(const double2* f, const Geom& g, int p, int mu, int cb) {
  const unsigned gs = (unsigned)g.vs * (unsigned)sizeof(double2), o = (unsigned)cb * (unsigned)sizeof(double2);
  const BufRsrc r = make_rsrc(f + (size_t)((p * 4 + mu) * 4) * g.vs, (size_t)4 * gs);
  const C<double> d = ld_buf<double>(r, o, 3 * gs);
  return {ld_buf<double>(r, o, 0), ld_buf<double>(r, o, gs), ld_buf<double>(r, o, 2 * gs), d.re, d.im};
}
// s + i d b
__device__ __forceinline__ C<double> cimac(C<double> s, double d, C<double> b) {
  return {rfma(-d, b.im, s.re), rfma(d, b.re, s.im)};
}
// acc + Q b and acc + b Q
__device__ __forceinline__ M3<double> qmac(const M3<double>& acc, const Su3Alg& q, const M3<double>& b) {
  const C<double> l01 = -conj(q.o01), l02 = -conj(q.o02), l12 = -conj(q.o12);
  M3<double> c;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const C<double> b0 = b.m[k], b1 = b.m[3 + k], b2 = b.m[6 + k];
    c.m[k] = cmac(cmac(cimac(acc.m[k], q.d0, b0), q.o01, b1), q.o02, b2);
    c.m[3 + k] = cmac(cimac(cmac(acc.m[3 + k], l01, b0), q.d1, b1), q.o12, b2);
    c.m[6 + k] = cimac(cmac(cmac(acc.m[6 + k], l02, b0), l12, b1), -(q.d0 + q.d1), b2);
  }
  return c;
}
__device__ __forceinline__ M3<double> macq(const M3<double>& acc, const M3<double>& b, const Su3Alg& q) {
  const C<double> l01 = -conj(q.o01), l02 = -conj(q.o02), l12 = -conj(q.o12);
  M3<double> c;
#pragma unroll
  for (int i = 0; i < 9; i += 3) {
    const C<double> b0 = b.m[i], b1 = b.m[i + 1], b2 = b.m[i + 2];
    c.m[i] = cmac(cmac(cimac(acc.m[i], q.d0, b0), b1, l01), b2, l02);
    c.m[i + 1] = cmac(cimac(cmac(acc.m[i + 1], b0, q.o01), q.d1, b1), b2, l12);
    c.m[i + 2] = cimac(cmac(cmac(acc.m[i + 2], b0, q.o02), b1, q.o12), -(q.d0 + q.d1), b2);
  }
  return c;
}
__device__ __forceinline__ M3<double> mzero() {
  M3<double> c;
#pragma unroll
  for (int k = 0; k < 9; ++k) c.m[k] = czero<double>();
  return c;
}

// wave index in the block as a scalar
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Plaquette staple sum of the link U_mu(x):
//   A = sum_{nu != mu} [ U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//                      + U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu) ],
// so that the plaquettes through U_mu(x) sum to Re tr(U_mu(x) A).
__device__ __forceinline__ M3<double> staple_A(const double2* U, const Geom& g, const int c[4], int mu) {
  int xpm[4];
  shifted(g, c, mu, +1, xpm);
  M3<double> A;
#pragma unroll
  for (int k = 0; k < 9; ++k) A.m[k] = czero<double>();
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    const int nu = (mu + k) & 3;
    int xpn[4], xmn[4], xpmmn[4];
    shifted(g, c, nu, +1, xpn);
    shifted(g, c, nu, -1, xmn);
    shifted(g, xpm, nu, -1, xpmmn);
    {
      const M3<double> u1 = link_at(U, g, xpm, nu), u2 = link_at(U, g, xpn, mu), u3 = link_at(U, g, c, nu);
      A = mmac_nd(A, mmul_nd(u1, u2), u3);
    }
    {
      const M3<double> v1 = link_at(U, g, xpmmn, nu), v2 = link_at(U, g, xmn, mu), v3 = link_at(U, g, xmn, nu);
      A = mmac_dn(A, mmul(v2, v1), v3);
    }
  }
  return A;
}

// The same by a block of 256 threads, wave mu at the sites cb (of parity p,
// coordinates c) of its 64 lanes, with the links that several of the waves
// read, U_mu(x) and U_mu(x-mu), exchanged through LDS.
struct StapleLinks {
  double2 own[4][9][64], low[4][9][64];
};
__device__ __forceinline__ void lds_put(double2 (*s)[64], int lane, const M3<double>& u) {
#pragma unroll
  for (int k = 0; k < 9; ++k) st<double>(&s[k][lane], u.m[k]);
}
__device__ __forceinline__ M3<double> lds_link(const double2 (*s)[64], int lane) {
  M3<double> u;
#pragma unroll
  for (int k = 0; k < 9; ++k) u.m[k] = ld<double>(&s[k][lane]);
  return u;
}
__device__ __forceinline__ M3<double> staple_block(const double2* U, const Geom& g, int p, int cb, const int c[4],
                                                   int mu, int lane, StapleLinks& s) {
  lds_put(s.own[mu], lane, link_uni(U, g, p, mu, cb));
  lds_put(s.low[mu], lane, link_uni(U, g, 1 - p, mu, cb_shift(g, c, mu, -1)));
  __syncthreads();
  int xpm[4];
  shifted(g, c, mu, +1, xpm);
  const int cpm = cb_of(g, xpm);
  M3<double> A = mzero();
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    const int nu = (mu + k) & 3;
    const int xpn = cb_shift(g, c, nu, +1), xmn = cb_shift(g, c, nu, -1), xpmmn = cb_shift(g, xpm, nu, -1);
    M3<double> t = mmul_nd(link_uni(U, g, 1 - p, nu, cpm), link_uni(U, g, 1 - p, mu, xpn));
    A = mmac_nd(A, t, lds_link(s.own[nu], lane));
    t = mmul(link_uni(U, g, 1 - p, mu, xmn), link_uni(U, g, p, nu, xpmmn));
    A = mmac_dn(A, t, lds_link(s.low[nu], lane));
  }
  return A;
}

// ---------------------------------------------------------------------------
// exp(X) for traceless anti-Hermitian X, by Cayley-Hamilton: with Q = -iX
// (Hermitian, traceless), exp(iQ) = f0 + f1 Q + f2 Q^2 and the f_j of
// Morningstar & Peardon (Phys. Rev. D 69, 054501), using
// c0 = det Q = tr(Q^3)/3, c1 = tr(Q^2)/2 and the symmetry
// f_j(-c0) = (-1)^j conj(f_j(c0)).  Below c1 = 1e-10 a 4th-order series
// through Q^3 = c1 Q + c0 is used instead (error < 1e-25).
// ---------------------------------------------------------------------------
__device__ __forceinline__ M3<double> exp_ah(const M3<double>& X) {
  M3<double> Q;
#pragma unroll
  for (int k = 0; k < 9; ++k) Q.m[k] = cmk<double>(X.m[k].im, -X.m[k].re);  // -i X
  const M3<double> Q2 = mmul(Q, Q);
  const double c1 = 0.5 * (Q2.m[0].re + Q2.m[4].re + Q2.m[8].re);
  double c0 = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) c0 += (Q2.m[3 * i + j] * Q.m[3 * j + i]).re;
  c0 *= (1.0 / 3.0);
  C<double> f0, f1, f2;
  if (c1 < 1e-10) {
    f0 = cmk(1.0, -c0 / 6.0);
    f1 = cmk(c0 / 24.0, 1.0 - c1 / 6.0);
    f2 = cmk(-0.5 + c1 / 24.0, 0.0);
  } else {
    const bool neg = c0 < 0.0;
    const double c0a = fabs(c0);
    const double c0max = 2.0 * c1 / 3.0 * sqrt(c1 / 3.0);
    double ratio = c0a / c0max;
    ratio = ratio > 1.0 ? 1.0 : ratio;
    const double theta = acos(ratio);
    const double u = sqrt(c1 / 3.0) * cos(theta / 3.0);
    const double w = sqrt(c1) * sin(theta / 3.0);
    const double w2 = w * w, u2 = u * u;
    const double xi0 = fabs(w) < 0.05 ? 1.0 - w2 / 6.0 * (1.0 - w2 / 20.0 * (1.0 - w2 / 42.0)) : sin(w) / w;
    const double cw = cos(w);
    const C<double> e2iu = cmk(cos(2.0 * u), sin(2.0 * u));
    const C<double> emiu = cmk(cos(u), -sin(u));
    const C<double> h0 = (u2 - w2) * e2iu + emiu * cmk(8.0 * u2 * cw, 2.0 * u * (3.0 * u2 + w2) * xi0);
    const C<double> h1 = (2.0 * u) * e2iu - emiu * cmk(2.0 * u * cw, -(3.0 * u2 - w2) * xi0);
    const C<double> h2 = e2iu - emiu * cmk(cw, 3.0 * u * xi0);
    const double inv = 1.0 / (9.0 * u2 - w2);
    f0 = inv * h0;
    f1 = inv * h1;
    f2 = inv * h2;
    if (neg) {
      f0 = conj(f0);
      f1 = -conj(f1);
      f2 = conj(f2);
    }
  }
  M3<double> E;
#pragma unroll
  for (int k = 0; k < 9; ++k) E.m[k] = f1 * Q.m[k] + f2 * Q2.m[k];
  E.m[0] += f0;
  E.m[4] += f0;
  E.m[8] += f0;
  return E;
}

// Row Gram-Schmidt on rows 1 and 2, row 3 = conj(row1 x row2).
__device__ __forceinline__ M3<double> reunitarize(const M3<double>& a) {
  C<double> r1[3], r2[3];
  double n1 = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) n1 += norm2(a.m[j]);
  n1 = 1.0 / sqrt(n1);
#pragma unroll
  for (int j = 0; j < 3; ++j) r1[j] = n1 * a.m[j];
  C<double> d = czero<double>();
#pragma unroll
  for (int j = 0; j < 3; ++j) d += cjmul(r1[j], a.m[3 + j]);
#pragma unroll
  for (int j = 0; j < 3; ++j) r2[j] = a.m[3 + j] - d * r1[j];
  double n2 = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) n2 += norm2(r2[j]);
  n2 = 1.0 / sqrt(n2);
#pragma unroll
  for (int j = 0; j < 3; ++j) r2[j] = n2 * r2[j];
  M3<double> o;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    o.m[j] = r1[j];
    o.m[3 + j] = r2[j];
  }
  o.m[6] = conj(r1[1] * r2[2] - r1[2] * r2[1]);
  o.m[7] = conj(r1[2] * r2[0] - r1[0] * r2[2]);
  o.m[8] = conj(r1[0] * r2[1] - r1[1] * r2[0]);
  return o;
}

}  // namespace lgt
