// Double-precision |M|^2 of the electroweak processes (two massless fermion
// lines joined by a photon and a Z, one of them with or without a gluon) from
// two kinematic weights per event.
//
// Every helicity amplitude is K_h(p) F_chi(card, s): chi the chiralities of
// the two lines, s the invariant mass squared of the lepton pair,
//   F_chi = A / s + B_chi / (s - M_Z^2 + i M_Z Gamma_Z),
// A the product of the lines' photon couplings and B_chi of their Z couplings
// (a Z propagator's q^mu q^nu term meets a conserved current).  For real
// momenta reversing every helicity conjugates K_h up to a sign, so the
// weights of LL and RR are equal and so are those of LR and RL:
//   |M|^2 = N g_s^(2p) [W_same (|F_LL|^2 + |F_RR|^2) + W_opp (|F_LR|^2 + |F_RL|^2)],
// W a sum over the gluon's helicities.  With two-component spinors chi (the
// right-handed one times sqrt(E + |p|), as ixx and oxx of helas.h build them)
// the contraction of two currents is a product of two 2x2 determinants or two
// dot products (Fierz).
//
// The weights are an event's, so any number of cards costs a few operations
// each.  The plain, batched and re-evaluation kernels of double precision share
// this code and its roundings are fixed (no contraction but the written fma),
// so they agree to the bit; the scan forms s in another way (pair_mass) and
// agrees to 5e-12; the card-per-event path (batch.hip) keeps the generated
// amplitudes, which agree to a few ulp.
#pragma once

#include "card.h"
#include "helas.h"

namespace rwgt {
namespace ew {

#pragma clang fp contract(off)

typedef cx<double> C;
RWGT_HD double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
RWGT_HD C mul(C a, C b) { return {fma_(-a.im, b.im, a.re * b.re), fma_(a.im, b.re, a.re * b.im)}; }
RWGT_HD C mul(C a, double s) { return {a.re * s, a.im * s}; }
// c + a b, c - a b
RWGT_HD C add_mul(C c, C a, C b) {
  return {fma_(-a.im, b.im, fma_(a.re, b.re, c.re)), fma_(a.im, b.re, fma_(a.re, b.im, c.im))};
}
RWGT_HD C sub_mul(C c, C a, C b) {
  return {fma_(a.im, b.im, fma_(-a.re, b.re, c.re)), fma_(-a.im, b.re, fma_(-a.re, b.im, c.im))};
}
RWGT_HD C add_mul(C c, C a, double s) { return {fma_(a.re, s, c.re), fma_(a.im, s, c.im)}; }
RWGT_HD double norm(C a) { return fma_(a.im, a.im, a.re * a.re); }

struct Chi { C a, b; };                         // two components
RWGT_HD C det(const Chi& x, const Chi& y) { return sub_mul(mul(x.a, y.b), x.b, y.a); }
RWGT_HD C dot(const Chi& x, const Chi& y) { return add_mul(mul(x.a, y.a), x.b, y.b); }
RWGT_HD Chi conj(const Chi& x) { return {rwgt::conj(x.a), rwgt::conj(x.b)}; }
RWGT_HD Chi flip(const Chi& x) { return {C{-x.b.re, x.b.im}, rwgt::conj(x.a)}; }   // chi_- of chi_+

// sqrt(E + |p|) chi_+(p); along -z chi_+ = (0, 1)
RWGT_HD Chi spinor(const double* p) {
  const double pt2 = fma_(p[1], p[1], p[2] * p[2]), pabs = sqrt(fma_(p[3], p[3], pt2));
  const double ppz = p[3] >= 0.0 ? pabs + p[3] : quot(pt2, pabs - p[3]);
  const double big = p[0] + pabs;
  const bool along = ppz <= 0.0;                // false for NaN
  const double c = sqrt(along ? big : quot(big, 2.0 * pabs * ppz));
  return {C{along ? 0.0 : ppz * c, 0.0}, along ? C{c, 0.0} : C{p[1] * c, p[2] * c}};
}

struct Weights { double inv_s, s, same, opp; };
// k^2: the rounded product is the smallest one of a boosted pair (transverse),
// as in the generated code.
RWGT_HD double square(const double* k) {
  return fma_(-k[3], k[3], fma_(-k[2], k[2], fma_(k[0], k[0], -(k[1] * k[1]))));
}
// s = (a + b)^2, or with PRODUCT 2 a.b: the same for massless momenta, without
// the cancellation of a boosted pair's energy and momentum, which the many
// cards of a scan, all close to the pole, would carry.
template <bool PRODUCT> RWGT_HD void pair_mass(const double* a, const double* b, Weights& w) {
  const double q[4] = {a[0] + b[0], a[1] + b[1], a[2] + b[2], a[3] + b[3]};
  w.s = PRODUCT ? 2.0 * fma_(-a[3], b[3], fma_(-a[2], b[2], fma_(-a[1], b[1], a[0] * b[0]))) : square(q);
  w.inv_s = quot(1.0, w.s);
}

// e+(p0) e-(p1) -> mu+(p2) mu-(p3), and any such pair of lines: row and column
// of the first, row and column of the second.
RWGT_HD void pair_weights(const Chi& row, const Chi& col, const Chi& lrow, const Chi& lcol, C& same, C& opp) {
  const Chi a = conj(row), al = conj(lrow);
  same = mul(det(a, al), det(col, lcol));
  opp = mul(dot(a, flip(lcol)), dot(conj(flip(lrow)), col));
}

template <int NPART> struct Process;

template <> struct Process<4> {                 // two lines
  static constexpr int kLine1 = 0, kLine2 = 1;  // species of the lines
  static constexpr double kColour = 1.0;
  static RWGT_HD double coupling(const Card<double>&) { return 1.0; }
  template <bool PRODUCT> static RWGT_HD Weights weights(const double (&P)[4][4]) {
    Weights w;
    pair_mass<PRODUCT>(P[2], P[3], w);
    C same, opp;
    pair_weights(spinor(P[0]), spinor(P[1]), spinor(P[3]), spinor(P[2]), same, opp);
    w.same = 4.0 * norm(same);
    w.opp = 4.0 * norm(opp);
    return w;
  }
};

template <> struct Process<5> {                 // u(p0) u~(p1) -> e+(p2) e-(p3) g(p4)
  static constexpr int kLine1 = 2, kLine2 = 0;
  static constexpr double kColour = 4.0;
  static RWGT_HD double coupling(const Card<double>& c) { return c.gqq * c.gqq; }
  template <bool PRODUCT> static RWGT_HD Weights weights(const double (&P)[5][4]) {
    Weights w;
    pair_mass<PRODUCT>(P[2], P[3], w);
    // quark momenta after the gluon and after the lepton pair have left it
    double ka[4], kb[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      ka[m] = P[0][m] - P[4][m];
      kb[m] = P[0][m] - P[2][m] - P[3][m];
    }
    const double ia = quot(1.0, square(ka)), ib = quot(1.0, square(kb));
    const Chi col = spinor(P[0]), row = conj(spinor(P[1])), lcol = spinor(P[2]), lrow = spinor(P[3]);
    const Chi al = conj(lrow), bl = conj(flip(lrow)), ll = flip(lcol);
    const C d_row = det(row, al), d_col = det(col, lcol), p_row = dot(row, ll), p_col = dot(bl, col);
    // eps*(p4, h): u = h st r, p = -(1 + h ct) r e^{i f}, m = (1 - h ct) r e^{-i f}
    const double* g = P[4];
    const double pt = sqrt(fma_(g[1], g[1], g[2] * g[2])), pabs = sqrt(fma_(g[3], g[3], pt * pt));
    double cf = 1.0, sf = 0.0, ct = g[3] >= 0.0 ? 1.0 : -1.0, st = 0.0;
    if (!(pt <= 0.0)) { cf = quot(g[1], pt); sf = quot(g[2], pt); ct = quot(g[3], pabs); st = quot(pt, pabs); }
    const double r = 0.70710678118654752440;
    w.same = w.opp = 0.0;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const double h = n ? 1.0 : -1.0;
      const double u = h * (st * r), fp = -r * fma_(h, ct, 1.0), fm = r * fma_(-h, ct, 1.0);
      const C ep = {fp * cf, fp * sf}, em = {fm * cf, -(fm * sf)};
      // column: k-sigmabar (eps.sigma chi) / k^2; eps.sigma = [[-u, -m], [-p, u]]
      const C y0 = sub_mul(mul(col.a, -u), em, col.b), y1 = sub_mul(mul(col.b, u), ep, col.a);
      const Chi z = {mul(add_mul(mul(y0, ka[0] + ka[3]), y1, C{ka[1], -ka[2]}), ia),
                     mul(add_mul(mul(y1, ka[0] - ka[3]), y0, C{ka[1], ka[2]}), ia)};
      // row: (chi eps.sigma) k-sigmabar / k^2
      const C x0 = sub_mul(mul(row.a, -u), row.b, ep), x1 = sub_mul(mul(row.b, u), row.a, em);
      const Chi v = {mul(add_mul(mul(x0, kb[0] + kb[3]), x1, C{kb[1], kb[2]}), ib),
                     mul(add_mul(mul(x1, kb[0] - kb[3]), x0, C{kb[1], -kb[2]}), ib)};
      w.same += norm(add_mul(mul(d_row, det(z, lcol)), det(v, al), d_col));
      w.opp += norm(add_mul(mul(p_row, dot(bl, z)), dot(v, ll), p_col));
    }
    w.same *= 4.0;
    w.opp *= 4.0;
    return w;
  }
};

// What one card brings to |M|^2: the products of the lines' photon and Z
// couplings, M_Z, M_Z Gamma_Z and the factor in front (average: over initial
// spins and colours).
struct Couplings { double a, ll, rr, lr, rl, mz, y, front; };
template <int NPART> RWGT_HD Couplings couplings(const Card<double>& cd, double average) {
  typedef Process<NPART> P;
  const double l1 = cd.zL[P::kLine1], r1 = cd.zR[P::kLine1], l2 = cd.zL[P::kLine2], r2 = cd.zR[P::kLine2];
  return {cd.a[P::kLine1] * cd.a[P::kLine2], l1 * l2, r1 * r2, l1 * r2, r1 * l2, cd.mz, cd.mz * cd.wz,
          average * P::kColour * P::coupling(cd)};
}
// |M|^2 under one card.
RWGT_HD double me2(const Weights& w, const Couplings& c) {
  const double ga = c.a * w.inv_s;
  const double x = fma_(-c.mz, c.mz, w.s), inv = quot(1.0, fma_(c.y, c.y, x * x));
  const double gr = x * inv, gi = c.y * inv;
  auto f2 = [&](double b) {
    const double re = fma_(b, gr, ga), im = b * gi;
    return fma_(im, im, re * re);
  };
  const double sum = fma_(w.same, f2(c.ll) + f2(c.rr), w.opp * (f2(c.lr) + f2(c.rl)));
  return sum * c.front;
}
template <int NPART> RWGT_HD double me2(const Weights& w, const Card<double>& cd, double average) {
  return me2(w, couplings<NPART>(cd, average));
}

#pragma clang fp contract(fast)
}  // namespace ew
}  // namespace rwgt
