// Colour-ordered recursion for two massive quark lines of one flavour and two
// gluons, g g -> Q Q~ Q Q~: the double-precision path of that process.
//
// The quarks r = 0, 1 (rows ubar) and antiquarks c = 0, 1 (columns v) form
// the lines (r c); pairing b joins quark 0 with antiquark b and quark 1 with
// the other one, and the two pairings enter with opposite sign.  In a pairing
// the second line emits a gluon that the first absorbs.  With
//   chi(x), psi(x)      the row and column with gluon x absorbed, propagated,
//   chi(xy), psi(xy)    with both, x nearest the row end, J(01) among them,
//   C[X|Y]              the line's current with the gluons X between its quark
//                       and the emission and Y between that and its antiquark,
//   G, G'(X|Y)          the second line's currents, propagated,
//   J(0G), J(01G), ...  gluon currents with G as a leg,
// the first line's ordered amplitudes are
//   A(0 1 G) = C[01|].G + C[0|].J(1G) + C[|].J(01G)
//   A(0 G 1) = C[0|1].G + C[|1].J(0G) - C[0|].J(1G) + C[|].J(0G1)
//   A(G 0 1) = C[|01].G - C[|1].J(0G) + C[|].J(10G)         and 0 <-> 1,
//   A(0 G') = C[0|].G' + C[|].J(0G'),  A(G' 0) = C[|0].G' - C[|].J(0G')
// for G' with gluon 1 absorbed by the second line, 0 <-> 1, and C[|].G'' with
// both.  Each multiplies the generator strings (X a Y)(X' a Y') of the two
// lines, which the Fierz identity turns into 3 (X Y')(X' Y) with the antiquarks
// exchanged minus (X Y)(X' Y'), in units of 1/6: the twelve flows of the
// generated colour matrix.
//
// As in ordered.h an event is the work of 32 lanes, one per helicity
// combination (gluon 0 always -1), and every current is computed once per
// helicity of its own legs; J(01) and the currents of the gluons absorbed by
// one line are not conserved, so the vertices are the full ones.
#pragma once

#include "lightcone.h"

namespace rwgt {
namespace ordered {
namespace pairs {

// Slots of one event's vectors and spinors.
constexpr int kLanes = 32;
constexpr int kRow = 0, kCol = 4;                      // ubar, v: 2 r + spin
constexpr int kChi = 8, kPsi = kChi + 12;              // chi(0): 2 r + spin; chi(1): 4 + 4 r + 2 h + spin
constexpr int kGluon = kPsi + 12;                      // J(01) by h
constexpr int kChi2 = kGluon + 2, kPsi2 = kChi2 + 16;  // chi(01), chi(10): 8 o + 4 r + 2 h + spin
constexpr int kWork = kPsi2 + 16;
// first: currents with G for both pairings, by b and the second line's spins s = spin(row) + 2 spin(column)
constexpr int kG = kWork, kJ0 = kG + 8, kJ1 = kJ0 + 8, kE = kJ1 + 16;   // 4 b + s; J(1G), E: 8 b + 4 h + s (E: + 16 o)
// then, one pairing at a time: the second line with one gluon, and the other gluon on its current
constexpr int kOne = kWork;                            // G'(1|), G'(|1): 8 y + 4 h + s; G'(0|), G'(|0): 16 + 4 y + s
constexpr int kJOne = kOne + 24;                       // J(0 G'(1)): 8 y + 4 h + s; J(1 G'(0)): 16 + 8 y + 4 h + s
constexpr int kSlots = kE + 32;
static_assert(kJOne + 32 <= kSlots, "the second use of the work slots fits the first");
constexpr int kPols = 3;                               // gluon 0, gluon 1 by h

RWGT_HD constexpr int chi_slot(int x, int r, int h, int spin) {
  return kChi + (x == 0 ? 2 * r + spin : 4 + 4 * r + 2 * h + spin);
}
RWGT_HD constexpr int psi_slot(int x, int c, int h, int spin) { return chi_slot(x, c, h, spin) - kChi + kPsi; }
RWGT_HD constexpr int chi2_slot(int o, int r, int h, int spin) { return kChi2 + 8 * o + 4 * r + 2 * h + spin; }
RWGT_HD constexpr int psi2_slot(int o, int c, int h, int spin) { return kPsi2 + 8 * o + 4 * c + 2 * h + spin; }

// A Memory provides mom(a) of the particles g g Q Q~ Q Q~ (the gluons' flowing
// in, the quarks' their own), pol(slot), set_pol, vec, set_vec, spin, set_spin.
RWGT_HD constexpr int row_particle(int r) { return 2 + 2 * r; }
RWGT_HD constexpr int col_particle(int c) { return 3 + 2 * c; }

// ubar (t < 4) and v of slot t; p: the particle's momentum (E px py pz)
RWGT_HD constexpr int spinor_particle(int t) { return t < 4 ? row_particle(t >> 1) : col_particle((t - 4) >> 1); }
template <class R, class M> RWGT_HD void spinor_task(M& m, int t, const R* p, R mass) {
  const bool row = t < 4;
  const Spinor<R> s = ixx<R>(p, mass, t & 1 ? 1 : -1, row ? 1 : -1);
  Spinor<R> o;
#pragma unroll
  for (int n = 0; n < 4; ++n) {                        // a row is u^dagger gamma^0
    const cx<R> a = s.c[n], b = conj(s.c[n ^ 2]);
    o.c[n] = {row ? b.re : a.re, row ? b.im : a.im};
  }
  m.set_spin(t, o);
}

// chi and psi of slot t (of 12)
template <class R, class M> RWGT_HD void single_task(M& m, int t, R mass, R gq) {
  const int x = t < 4 ? 0 : 1, r = t < 4 ? t >> 1 : (t - 4) >> 2, h = t < 4 ? 0 : (t >> 1) & 1, spin = t & 1;
  const Lc<R> e = m.pol(x == 0 ? 0 : 1 + h);
  const LcK<R> k = m.mom(x);
  m.set_spin(kChi + t, prop_row(row_slash(m.spin(kRow + 2 * r + spin), e), m.mom(row_particle(r)) - k, mass, gq));
  load_fence();
  m.set_spin(kPsi + t, prop_col(slash_col(e, m.spin(kCol + 2 * r + spin)), k - m.mom(col_particle(r)), mass, gq));
}

template <class R, class M> RWGT_HD void gluon_task(M& m, int h, R g3) {
  const LcK<R> k0 = m.mom(0), k1 = m.mom(1);
  Lc<R> o = {};
  add_v3(o, m.pol(0), k0, m.pol(1 + h), k1);
  m.set_vec(kGluon + h, o * quot(-g3, square(k0 + k1)));
}

// chi(xy) and psi(xy) of slot t (of 16): o = 0: xy = 01, 1: 10
template <class R, class M> RWGT_HD void double_task(M& m, int t, R mass, R gq) {
  const int o = t >> 3, r = (t >> 2) & 1, h = (t >> 1) & 1, spin = t & 1;
  const R sign = o ? R(-1) : R(1);
  const LcK<R> k = m.mom(0) + m.mom(1);
  Spinor<R> a = row_slash(m.spin(kRow + 2 * r + spin), m.vec(kGluon + h) * sign);
  add_row_slash(a, m.spin(chi_slot(o ? 1 : 0, r, h, spin)), m.pol(o ? 0 : 1 + h));
  m.set_spin(kChi2 + t, prop_row(a, m.mom(row_particle(r)) - k, mass, gq));
  load_fence();
  Spinor<R> b = slash_col(m.vec(kGluon + h) * sign, m.spin(kCol + 2 * r + spin));
  add_slash_col(b, m.pol(o ? 1 + h : 0), m.spin(psi_slot(o ? 0 : 1, r, h, spin)));
  m.set_spin(kPsi2 + t, prop_col(b, k - m.mom(col_particle(r)), mass, gq));
}

// Momentum the second line of pairing b sends into the first, without gluons.
template <class R, class M> RWGT_HD LcK<R> second_momentum(M& m, int b) {
  const LcK<R> p = m.mom(row_particle(1)) + m.mom(col_particle(1 - b));
  return {-p.u, -p.d, {-p.p.re, -p.p.im}};
}

// G of slot t (of 8)
template <class R, class M> RWGT_HD void line_task(M& m, int t, R gq) {
  const int b = t >> 2, s = t & 3;
  const Lc<R> w = pair_coeffs(m.spin(kRow + 2 + (s & 1)), m.spin(kCol + 2 * (1 - b) + (s >> 1)));
  m.set_vec(kG + t, as_vector(w, quot(gq, square(second_momentum<R>(m, b)))));
}

// J(0G) and J(1G): slot t of 24
template <class R, class M> RWGT_HD void attach_task(M& m, int t, R g3) {
  const int x = t < 8 ? 0 : 1, b = t < 8 ? t >> 2 : (t - 8) >> 3, h = t < 8 ? 0 : (t >> 2) & 1, s = t & 3;
  const LcK<R> k = m.mom(x), q = second_momentum<R>(m, b);
  Lc<R> o = {};
  add_v3_full(o, m.pol(x == 0 ? 0 : 1 + h), k, m.vec(kG + 4 * b + s), q);
  m.set_vec(kJ0 + t, o * quot(-g3, square(k + q)));
}

// J(01G) (o = 0) and J(10G) before their propagator: slot t of 32
template <class R, class M> RWGT_HD void both_task(M& m, int t, R g3, R g4) {
  const int o = t >> 4, b = (t >> 3) & 1, h = (t >> 2) & 1, s = t & 3;
  const int x = o, y = 1 - o;
  const LcK<R> kx = m.mom(x), ky = m.mom(y), q = second_momentum<R>(m, b);
  const Lc<R> jx = m.pol(x == 0 ? 0 : 1 + h), jy = m.pol(y == 0 ? 0 : 1 + h), g = m.vec(kG + 4 * b + s);
  const Lc<R> jxy = m.vec(kGluon + h) * (o ? R(-1) : R(1));
  const Lc<R> jyg = m.vec(y == 0 ? kJ0 + 4 * b + s : kJ1 + 8 * b + 4 * h + s);
  Lc<R> v = {}, f = {};
  add_v3_full(v, jx, kx, jyg, ky + q);
  settle(v); load_fence();
  add_v3_full(v, jxy, kx + ky, g, q);
  settle(v); load_fence();
  add_v4(f, jx, jy, g, dot2(jx, jy), dot2(jx, g), dot2(jy, g));
  m.set_vec(kE + t, lincomb(v, -g3, f, g4));
}

// G'(1|), G'(|1), G'(0|), G'(|0) of the second line of pairing b: slot t of 24
template <class R, class M> RWGT_HD void line_one_task(M& m, int b, int t, R gq) {
  const int x = t < 16 ? 1 : 0, y = t < 16 ? t >> 3 : (t >> 2) & 1, h = t < 16 ? (t >> 2) & 1 : 0;
  const int sr = t & 1, sc = (t >> 1) & 1, c = 1 - b;
  // y = 0: chi(x) and v; 1: ubar and psi(x)
  const Lc<R> w = pair_coeffs(m.spin(y == 0 ? chi_slot(x, 1, h, sr) : kRow + 2 + sr),
                              m.spin(y == 0 ? kCol + 2 * c + sc : psi_slot(x, c, h, sc)));
  m.set_vec(kOne + t, as_vector(w, quot(gq, square(second_momentum<R>(m, b) + m.mom(x)))));
}

// J(0 G'(1)) and J(1 G'(0)) before their propagator: slot t of 32
template <class R, class M> RWGT_HD void attach_one_task(M& m, int b, int t, R g3) {
  const int x = t >> 4, y = (t >> 3) & 1, h = (t >> 2) & 1, s = t & 3;   // gluon x on the current of the other one
  const Lc<R> g = m.vec(kOne + (x == 0 ? 8 * y + 4 * h + s : 16 + 4 * y + s));
  Lc<R> o = {};
  add_v3_full(o, m.pol(x == 0 ? 0 : 1 + h), m.mom(x), g, second_momentum<R>(m, b) + m.mom(1 - x));
  m.set_vec(kJOne + t, o * -g3);
}

// ------------------------------------------------------------------ one lane
struct LaneHel { int h, row[2], col[2]; };
RWGT_HD LaneHel lane_hel(int t) { return {t & 1, {(t >> 1) & 1, (t >> 2) & 1}, {(t >> 3) & 1, (t >> 4) & 1}}; }

// Generator strings of the two gluons: "", "0", "1", "01", "10".
enum { kNone, k0, k1, k01, k10 };
RWGT_HD constexpr int joined(int a, int b) { return a == kNone ? b : b == kNone ? a : a == k0 ? k01 : k10; }
// Position of the strings (alpha, beta) of the two quarks among a joining's six flows.
RWGT_HD constexpr int strings(int alpha, int beta) {
  return alpha == kNone ? (beta == k01 ? 0 : 1) : alpha == k0 ? 2 : alpha == k1 ? 3 : alpha == k01 ? 4 : 5;
}

// Flows of the ordered amplitude p of pairing b with strings (X a Y)(X' a Y').
template <class R>
RWGT_HD void add_flows(cx<R> (&f)[12], int b, int x, int y, int x2, int y2, cx<R> p) {
  const R s = b ? R(-1) : R(1);
  cx<R>& direct = f[6 * b + strings(joined(x, y), joined(x2, y2))];
  cx<R>& swapped = f[6 * (1 - b) + strings(joined(x, y2), joined(x2, y))];
  direct.re -= s * p.re; direct.im -= s * p.im;
  mac(swapped, p, R(3) * s);
}

// C[01|].V, C[10|].V, C[0|1].V, C[1|0].V, C[|01].V, C[|10].V of the line (r c).
template <class R, class M>
RWGT_HD void both_on_line(M& m, const LaneHel& h, int r, int c, const Lc<R>& g, cx<R> (&a)[6]) {
  {
    const Spinor<R> col = slash_col(g, m.spin(kCol + 2 * c + h.col[c]));
    a[0] = dot(m.spin(chi2_slot(0, r, h.h, h.row[r])), col);
    a[1] = dot(m.spin(chi2_slot(1, r, h.h, h.row[r])), col);
  }
  settle(a[0]); settle(a[1]); load_fence();
  {
    const Spinor<R> row = row_slash(m.spin(kRow + 2 * r + h.row[r]), g);
    a[4] = dot(row, m.spin(psi2_slot(0, c, h.h, h.col[c])));
    a[5] = dot(row, m.spin(psi2_slot(1, c, h.h, h.col[c])));
  }
  settle(a[4]); settle(a[5]); load_fence();
  a[2] = dot(row_slash(m.spin(chi_slot(0, r, h.h, h.row[r])), g), m.spin(psi_slot(1, c, h.h, h.col[c])));
  a[3] = dot(row_slash(m.spin(chi_slot(1, r, h.h, h.row[r])), g), m.spin(psi_slot(0, c, h.h, h.col[c])));
  settle(a[2]); settle(a[3]); load_fence();
}

// The terms with no gluon or both on the second line: L = (0 b), L' = (1 1-b).
template <class R, class M> RWGT_HD void pairing_terms(M& m, int t, int b, R gq, cx<R> (&f)[12]) {
  load_fence();
  const LaneHel h = lane_hel(opq_index(t));
  const int c = 1 - b, s = h.row[1] + 2 * h.col[c];
  const LcK<R> p = m.mom(row_particle(0)) + m.mom(col_particle(b));
  const Lc<R> w = pair_coeffs(m.spin(kRow + h.row[0]), m.spin(kCol + 2 * b + h.col[b])) * quot(R(1), square(p));
  cx<R> a[6];
  both_on_line(m, h, 1, c, as_vector(w, gq), a);
  add_flows(f, b, kNone, kNone, k01, kNone, a[0]);
  add_flows(f, b, kNone, kNone, k10, kNone, a[1]);
  add_flows(f, b, kNone, kNone, k0, k1, a[2]);
  add_flows(f, b, kNone, kNone, k1, k0, a[3]);
  add_flows(f, b, kNone, kNone, kNone, k01, a[4]);
  add_flows(f, b, kNone, kNone, kNone, k10, a[5]);
  both_on_line(m, h, 0, b, m.vec(kG + 4 * b + s), a);
  {
    const cx<R> e0 = apply(w, m.vec(kE + 8 * b + 4 * h.h + s)), e1 = apply(w, m.vec(kE + 16 + 8 * b + 4 * h.h + s));
    const cx<R> e2 = e0 + e1;
    a[0] = a[0] + e0; a[1] = a[1] + e1; a[2] = a[2] - e2; a[3] = a[3] - e2; a[4] = a[4] + e1; a[5] = a[5] + e0;
  }
#pragma unroll
  for (int n = 0; n < 6; ++n) settle(a[n]);
  load_fence();
  {
    const Lc<R> j1 = m.vec(kJ1 + 8 * b + 4 * h.h + s);
    const cx<R> x = apply(pair_coeffs(m.spin(chi_slot(0, 0, h.h, h.row[0])), m.spin(kCol + 2 * b + h.col[b])), j1);
    const cx<R> y = apply(pair_coeffs(m.spin(kRow + h.row[0]), m.spin(psi_slot(0, b, h.h, h.col[b]))), j1);
    a[0] = a[0] + x; a[2] = a[2] - x; a[3] = a[3] + y; a[5] = a[5] - y;
  }
#pragma unroll
  for (int n = 0; n < 6; ++n) settle(a[n]);
  load_fence();
  {
    const Lc<R> j0 = m.vec(kJ0 + 4 * b + s);
    const cx<R> x = apply(pair_coeffs(m.spin(chi_slot(1, 0, h.h, h.row[0])), m.spin(kCol + 2 * b + h.col[b])), j0);
    const cx<R> y = apply(pair_coeffs(m.spin(kRow + h.row[0]), m.spin(psi_slot(1, b, h.h, h.col[b]))), j0);
    a[1] = a[1] + x; a[3] = a[3] - x; a[2] = a[2] + y; a[4] = a[4] - y;
  }
  add_flows(f, b, k01, kNone, kNone, kNone, a[0]);
  add_flows(f, b, k10, kNone, kNone, kNone, a[1]);
  add_flows(f, b, k0, k1, kNone, kNone, a[2]);
  add_flows(f, b, k1, k0, kNone, kNone, a[3]);
  add_flows(f, b, kNone, k01, kNone, kNone, a[4]);
  add_flows(f, b, kNone, k10, kNone, kNone, a[5]);
#pragma unroll
  for (int n = 0; n < 12; ++n) settle(f[n]);
}

// The terms with one gluon on each line or its current.
template <class R, class M> RWGT_HD void shared_terms(M& m, int t, int b, cx<R> (&f)[12]) {
  load_fence();
  const LaneHel h = lane_hel(opq_index(t));
  const int s = h.row[1] + 2 * h.col[1 - b];
  const LcK<R> p = m.mom(row_particle(0)) + m.mom(col_particle(b));
  const Lc<R> w = pair_coeffs(m.spin(kRow + h.row[0]), m.spin(kCol + 2 * b + h.col[b])) * quot(R(1), square(p));
#pragma unroll
  for (int x = 0; x < 2; ++x) {                        // gluon x on the first line, the other one on the second
    const Lc<R> wr = pair_coeffs(m.spin(chi_slot(x, 0, h.h, h.row[0])), m.spin(kCol + 2 * b + h.col[b]));
    const Lc<R> wc = pair_coeffs(m.spin(kRow + h.row[0]), m.spin(psi_slot(x, b, h.h, h.col[b])));
#pragma unroll
    for (int y = 0; y < 2; ++y) {                      // the other one before or after the emission
      const Lc<R> g = m.vec(kOne + (x == 0 ? 8 * y + 4 * h.h + s : 16 + 4 * y + s));
      const cx<R> j = apply(w, m.vec(kJOne + 16 * x + 8 * y + 4 * h.h + s));
      const int mine = x == 0 ? k0 : k1, other = x == 0 ? k1 : k0;
      const int x2 = y == 0 ? other : kNone, y2 = y == 0 ? kNone : other;
      add_flows(f, b, mine, kNone, x2, y2, apply(wr, g) + j);
      add_flows(f, b, kNone, mine, x2, y2, apply(wc, g) - j);
#pragma unroll
      for (int n = 0; n < 12; ++n) settle(f[n]);
      load_fence();
    }
  }
}

// One lane's part of an event: |M_h|^2 summed over colours, without g^2 of the
// last vertices.  momentum(a, p) loads particle a's momentum (E px py pz).
template <class R, class M, class Load, class Cd, class Sync, class Colour>
RWGT_HD R lane_me2(M& m, int t, Load momentum, const Cd& cd, Sync sync, Colour colour) {
  auto clamp = [&](int n) { const int x = opq_index(t); return x < n ? x : n - 1; };   // idle lanes repeat the last task
  {
    const int n = clamp(8);
    R p[4];
    momentum(spinor_particle(n), p);
    spinor_task(m, n, p, cd.mt);
    const int g = clamp(kPols);
    m.set_pol(g, polarisation(m.mom(g == 0 ? 0 : 1), g == 2 ? 1 : -1, false));
  }
  sync();
  single_task(m, clamp(12), cd.mt, cd.gqq);
  gluon_task(m, clamp(2), cd.g3);
  sync();
  double_task(m, clamp(16), cd.mt, cd.gqq);
  line_task(m, clamp(8), cd.gqq);
  sync();
  attach_task(m, clamp(24), cd.g3);
  sync();
  both_task(m, opq_index(t), cd.g3, cd.g4);
  sync();
  cx<R> f[12];
#pragma unroll
  for (int n = 0; n < 12; ++n) f[n] = {R(0), R(0)};
  pairing_terms(m, t, 0, cd.gqq, f);
  pairing_terms(m, t, 1, cd.gqq, f);
  sync();
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    line_one_task(m, b, clamp(24), cd.gqq);
    sync();
    attach_one_task(m, b, opq_index(t), cd.g3);
    sync();
    shared_terms(m, t, b, f);
    sync();
  }
  return colour(f);
}

}  // namespace pairs

}  // namespace ordered
}  // namespace rwgt
