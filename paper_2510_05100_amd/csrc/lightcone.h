// Complex vectors by their light-cone components and the vertices of the
// ordered recursions (ordered.h, ordered_pairs.h) on them.
//
// A vector is kept as u = V0 + V3, d = V0 - V3, p = V1 + i V2, m = V1 - i V2: the
// entries of V.sigma and V.sigmabar, so V-slash on a spinor is eight complex
// products, and 2 V.W = u d' + d u' - p m' - m p'.  Overall factors are real: the
// phases of the textbook vertices and propagators (helas.h) combine to one
// common i per flow, which drops out of |M|^2.
#pragma once

#include "card.h"
#include "helas.h"

namespace rwgt {
namespace ordered {

template <class R> struct Lc { cx<R> u, d, p, m; };     // complex vector
template <class R> struct LcK { R u, d; cx<R> p; };     // real momentum (m = conj p)

// a += b c, a -= b c, written so that each real product is one FMA
template <class R> RWGT_HD void mac(cx<R>& a, cx<R> b, cx<R> c) {
  a.re += b.re * c.re; a.re -= b.im * c.im;
  a.im += b.re * c.im; a.im += b.im * c.re;
}
template <class R> RWGT_HD void msc(cx<R>& a, cx<R> b, cx<R> c) {
  a.re -= b.re * c.re; a.re += b.im * c.im;
  a.im -= b.re * c.im; a.im -= b.im * c.re;
}
template <class R> RWGT_HD void mac(cx<R>& a, cx<R> b, R s) { a.re += b.re * s; a.im += b.im * s; }

template <class R> RWGT_HD LcK<R> operator+(const LcK<R>& a, const LcK<R>& b) {
  return {a.u + b.u, a.d + b.d, a.p + b.p};
}
template <class R> RWGT_HD LcK<R> operator-(const LcK<R>& a, const LcK<R>& b) {
  return {a.u - b.u, a.d - b.d, a.p - b.p};
}
template <class R> RWGT_HD R square(const LcK<R>& k) { return k.u * k.d - (k.p.re * k.p.re + k.p.im * k.p.im); }
template <class R> RWGT_HD LcK<R> lc_momentum(const R* p, R sign) {
  return {sign * (p[0] + p[3]), sign * (p[0] - p[3]), {sign * p[1], sign * p[2]}};
}

// 2 a.b
template <class R> RWGT_HD cx<R> dot2(const Lc<R>& a, const Lc<R>& b) {
  cx<R> s = a.u * b.d;
  mac(s, a.d, b.u); msc(s, a.p, b.m); msc(s, a.m, b.p);
  return s;
}
template <class R> RWGT_HD void settle(Lc<R>& a) {
  rwgt::settle(a.u); rwgt::settle(a.d); rwgt::settle(a.p); rwgt::settle(a.m);
}
template <class R> RWGT_HD cx<R> dot2(const LcK<R>& k, const Lc<R>& a) {
  cx<R> s = a.d * k.u;
  mac(s, a.u, k.d); msc(s, a.m, k.p); msc(s, a.p, conj(k.p));
  return s;
}
template <class R> RWGT_HD void axpy(Lc<R>& o, cx<R> s, const Lc<R>& a) {
  mac(o.u, s, a.u); mac(o.d, s, a.d); mac(o.p, s, a.p); mac(o.m, s, a.m);
}
template <class R> RWGT_HD void axmy(Lc<R>& o, cx<R> s, const Lc<R>& a) {
  msc(o.u, s, a.u); msc(o.d, s, a.d); msc(o.p, s, a.p); msc(o.m, s, a.m);
}
template <class R> RWGT_HD Lc<R> operator*(const Lc<R>& a, R s) { return {a.u * s, a.d * s, a.p * s, a.m * s}; }
template <class R> RWGT_HD Lc<R> lincomb(const Lc<R>& a, R s, const Lc<R>& b, R t) {
  Lc<R> o = a * s;
  mac(o.u, b.u, t); mac(o.d, b.d, t); mac(o.p, b.p, t); mac(o.m, b.m, t);
  return o;
}

// Three-gluon vertex of two conserved currents (k.J(k) = 0):
// o += (a.b)(ka - kb) + 2 (kb.a) b - 2 (ka.b) a
template <class R>
RWGT_HD void add_v3(Lc<R>& o, const Lc<R>& a, const LcK<R>& ka, const Lc<R>& b, const LcK<R>& kb) {
  const cx<R> ab = dot2(a, b), y = dot2(kb, a), z = dot2(ka, b);
  const LcK<R> h = {R(0.5) * (ka.u - kb.u), R(0.5) * (ka.d - kb.d),
                    {R(0.5) * (ka.p.re - kb.p.re), R(0.5) * (ka.p.im - kb.p.im)}};
  mac(o.u, ab, h.u); mac(o.d, ab, h.d); mac(o.p, ab, h.p); mac(o.m, ab, conj(h.p));
  axpy(o, y, b);
  axmy(o, z, a);
}
// Four-gluon vertex of ordered currents: o += 2 b (a.c) - a (b.c) - c (a.b),
// from the doubled products ab2 = 2 a.b etc.
template <class R>
RWGT_HD void add_v4(Lc<R>& o, const Lc<R>& a, const Lc<R>& b, const Lc<R>& c, cx<R> ab2, cx<R> ac2, cx<R> bc2) {
  axpy(o, ac2, b);
  axmy(o, bc2 * R(0.5), a);
  axmy(o, ab2 * R(0.5), c);
}

// Polarisation of a gluon with momentum k flowing in (sign -1: outgoing, eps*),
// the components of vxx up to rounding.
template <class R> RWGT_HD Lc<R> polarisation(const LcK<R>& k, int h, bool outgoing) {
  const R s = outgoing ? R(-1) : R(1), half = R(0.5);
  const R x = s * k.p.re, y = s * k.p.im, z = s * half * (k.u - k.d);
  const R pt = sqrt(x * x + y * y), pabs = sqrt(x * x + y * y + z * z);
  R cf = R(1), sf = R(0), ct = z >= R(0) ? R(1) : R(-1), st = R(0);
  // not (pt <= 0), so that NaN momenta give NaN polarisations
  if (!(pt <= R(0))) { cf = quot(x, pt); sf = quot(y, pt); ct = quot(z, pabs); st = quot(pt, pabs); }
  const R r = R(0.70710678118654752440), hh = R(h);
  const R a = r * (R(1) - hh * ct), b = -r * (R(1) + hh * ct);
  const cx<R> p = {a * cf, a * sf}, m = {b * cf, -b * sf};
  const cx<R> u = {hh * r * st, R(0)};
  return outgoing ? Lc<R>{u, -u, conj(m), conj(p)} : Lc<R>{u, -u, p, m};
}

// row V-slash, V-slash column
template <class R> RWGT_HD Spinor<R> row_slash(const Spinor<R>& r, const Lc<R>& v) {
  Spinor<R> o;
  o.c[0] = r.c[2] * v.u; mac(o.c[0], r.c[3], v.p);
  o.c[1] = r.c[2] * v.m; mac(o.c[1], r.c[3], v.d);
  o.c[2] = r.c[0] * v.d; msc(o.c[2], r.c[1], v.p);
  o.c[3] = r.c[1] * v.u; msc(o.c[3], r.c[0], v.m);
  return o;
}
template <class R> RWGT_HD void add_row_slash(Spinor<R>& o, const Spinor<R>& r, const Lc<R>& v) {
  mac(o.c[0], r.c[2], v.u); mac(o.c[0], r.c[3], v.p);
  mac(o.c[1], r.c[2], v.m); mac(o.c[1], r.c[3], v.d);
  mac(o.c[2], r.c[0], v.d); msc(o.c[2], r.c[1], v.p);
  mac(o.c[3], r.c[1], v.u); msc(o.c[3], r.c[0], v.m);
}
template <class R> RWGT_HD Spinor<R> slash_col(const Lc<R>& v, const Spinor<R>& c) {
  Spinor<R> o;
  o.c[0] = v.d * c.c[2]; msc(o.c[0], v.m, c.c[3]);
  o.c[1] = v.u * c.c[3]; msc(o.c[1], v.p, c.c[2]);
  o.c[2] = v.u * c.c[0]; mac(o.c[2], v.m, c.c[1]);
  o.c[3] = v.p * c.c[0]; mac(o.c[3], v.d, c.c[1]);
  return o;
}
template <class R> RWGT_HD void add_slash_col(Spinor<R>& o, const Lc<R>& v, const Spinor<R>& c) {
  mac(o.c[0], v.d, c.c[2]); msc(o.c[0], v.m, c.c[3]);
  mac(o.c[1], v.u, c.c[3]); msc(o.c[1], v.p, c.c[2]);
  mac(o.c[2], v.u, c.c[0]); mac(o.c[2], v.m, c.c[1]);
  mac(o.c[3], v.p, c.c[0]); mac(o.c[3], v.d, c.c[1]);
}
template <class R> RWGT_HD void add_dot(cx<R>& a, const Spinor<R>& r, const Spinor<R>& c) {
  for (int i = 0; i < 4; ++i) mac(a, r.c[i], c.c[i]);
}
template <class R> RWGT_HD cx<R> dot(const Spinor<R>& r, const Spinor<R>& c) {
  cx<R> s = r.c[0] * c.c[0];
  for (int i = 1; i < 4; ++i) mac(s, r.c[i], c.c[i]);
  return s;
}

// Coefficients of V-slash between a row and a column: row V-slash col =
// u w.u + d w.d + p w.p + m w.m.
template <class R> RWGT_HD Lc<R> pair_coeffs(const Spinor<R>& r, const Spinor<R>& c) {
  Lc<R> w;
  w.d = r.c[0] * c.c[2]; mac(w.d, r.c[3], c.c[1]);
  w.u = r.c[1] * c.c[3]; mac(w.u, r.c[2], c.c[0]);
  w.m = r.c[2] * c.c[1]; msc(w.m, r.c[0], c.c[3]);
  w.p = r.c[3] * c.c[0]; msc(w.p, r.c[1], c.c[2]);
  return w;
}
template <class R> RWGT_HD cx<R> apply(const Lc<R>& w, const Lc<R>& v) {
  cx<R> s = w.u * v.u;
  mac(s, w.d, v.d); mac(s, w.p, v.p); mac(s, w.m, v.m);
  return s;
}

// Quark propagator with its vertex factor, -g (q-slash + m)/(q^2 - m^2).
template <class R> RWGT_HD Spinor<R> prop_row(const Spinor<R>& r, const LcK<R>& q, R m, R g) {
  const R s = quot(-g, square(q) - m * m);
  const R u = q.u * s, d = q.d * s, ms = m * s;
  const cx<R> p = q.p * s, pc = conj(p);
  Spinor<R> o;
  o.c[0] = r.c[2] * u; mac(o.c[0], r.c[3], p);  mac(o.c[0], r.c[0], ms);
  o.c[1] = r.c[3] * d; mac(o.c[1], r.c[2], pc); mac(o.c[1], r.c[1], ms);
  o.c[2] = r.c[0] * d; msc(o.c[2], r.c[1], p);  mac(o.c[2], r.c[2], ms);
  o.c[3] = r.c[1] * u; msc(o.c[3], r.c[0], pc); mac(o.c[3], r.c[3], ms);
  return o;
}
template <class R> RWGT_HD Spinor<R> prop_col(const Spinor<R>& c, const LcK<R>& q, R m, R g) {
  const R s = quot(-g, square(q) - m * m);
  const R u = q.u * s, d = q.d * s, ms = m * s;
  const cx<R> p = q.p * s, pc = conj(p);
  Spinor<R> o;
  o.c[0] = c.c[2] * d; msc(o.c[0], pc, c.c[3]); mac(o.c[0], c.c[0], ms);
  o.c[1] = c.c[3] * u; msc(o.c[1], p, c.c[2]);  mac(o.c[1], c.c[1], ms);
  o.c[2] = c.c[0] * u; mac(o.c[2], pc, c.c[1]); mac(o.c[2], c.c[2], ms);
  o.c[3] = c.c[1] * d; mac(o.c[3], p, c.c[0]);  mac(o.c[3], c.c[3], ms);
  return o;
}

// Three-gluon vertex without the currents' conservation:
// o += (a.b)(ka - kb) + ((ka + 2 kb).a) b - ((2 ka + kb).b) a
template <class R>
RWGT_HD void add_v3_full(Lc<R>& o, const Lc<R>& a, const LcK<R>& ka, const Lc<R>& b, const LcK<R>& kb) {
  const cx<R> ab = dot2(a, b), y = dot2(ka + kb + kb, a) * R(0.5), z = dot2(ka + ka + kb, b) * R(0.5);
  const LcK<R> h = {R(0.5) * (ka.u - kb.u), R(0.5) * (ka.d - kb.d),
                    {R(0.5) * (ka.p.re - kb.p.re), R(0.5) * (ka.p.im - kb.p.im)}};
  mac(o.u, ab, h.u); mac(o.d, ab, h.d); mac(o.p, ab, h.p); mac(o.m, ab, conj(h.p));
  axpy(o, y, b);
  axmy(o, z, a);
}

// The vector V with 2 V.W = 2 apply(w, W): s times row gamma^mu col from its
// coefficients.
template <class R> RWGT_HD Lc<R> as_vector(const Lc<R>& w, R s) {
  const R t = R(2) * s;
  return {w.d * t, w.u * t, w.m * -t, w.p * -t};
}

}  // namespace ordered
}  // namespace rwgt
