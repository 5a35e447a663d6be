// Colour-ordered recursion for one massive quark line and four gluons,
// g g -> Q Q~ g g: the double-precision path of that process.
//
// Every off-shell current is a sum over the diagrams that share its ordered
// legs (Berends and Giele, Nucl. Phys. B306 (1988) 759) and is computed once
// for each helicity of its own legs:
//
//   J(ab), J(abc)   gluon currents (6 pairs, 2 of 3 orderings of each triple:
//                   J(ab) = -J(ba), J(cba) = J(abc), and the three orderings
//                   with different middle legs add to zero),
//   J(0abc)         the six orderings that start with gluon 0, contracted with
//                   the quark pair; the other 18 are sums of these (the
//                   current vanishes on shuffles; J(dcba) = -J(abcd)),
//   chi(i), chi(ij) rows ubar(t) with one or two gluons absorbed, propagated,
//   psi(l)          columns v(t~) with one gluon absorbed, propagated,
//   phi(kl)         J(k) psi(l) + J(kl) v,
//
//   A(ijkl) = chi(ij) phi(kl) + chi(i) J(jk) psi(l)
//           + ubar J(ijk) psi(l) + chi(i) J(jkl) v + ubar J(ijkl) v
//
// with J standing for J-slash and i the gluon nearest the outgoing quark.  The
// last vertex's g_s is left out of A.
//
// An event is the work of 32 lanes, one per helicity combination evaluated
// (gluon 0 always -1: the combinations with every helicity reversed have the
// same |M|^2).  The currents are tasks dealt to the lanes and shared through
// a Memory (LDS on the device); the sums over flows are each lane's own.
#pragma once

#include "lightcone.h"

namespace rwgt {
namespace ordered {

// ------------------------------------------------------------ shared memory
// Slots of the vectors and spinors of one event (four complex numbers each),
// by the helicity bits (0: -1, 1: +1) of their legs.
constexpr int kLanes = 32;
constexpr int kPair = 0, kPairSlots = 18;
constexpr int kTriple = kPair + kPairSlots, kTripleSlots = 20;   // two orderings: slots s and s + 20
constexpr int kHalf = kTriple;                                   // chi(ij) and phi(kl), once the triples are used up
constexpr int kHalfSlots = 72;
constexpr int kFour = kHalf + kHalfSlots;                        // 32 of the 48 J(0abc) at a time
constexpr int kChi = kFour, kPsi = kChi + 14;                    // chi(i) and psi(l), once those are used up
constexpr int kUbar = kFour + kLanes, kV = kUbar + 2;
constexpr int kSlots = kV + 2;
constexpr int kPols = 7;

RWGT_HD constexpr int pol_slot(int g, int h) { return g == 0 ? 0 : 2 * g - 1 + h; }
// J(ab), a < b
RWGT_HD constexpr int pair_slot(int a, int b, int ha, int hb) {
  return kPair + (a == 0 ? 2 * (b - 1) + hb : 4 * (a + b) - 6 + ha + 2 * hb);
}
// The triple without gluon g, sorted, has the legs member(g, 0..2).
RWGT_HD constexpr int member(int g, int n) { return n < g ? n : n + 1; }
RWGT_HD constexpr int triple_slot(int g, int ha, int hb, int hc) {
  return kTriple + (g == 0 ? ha + 2 * hb + 4 * hc : 4 + 4 * g + hb + 2 * hc);
}
RWGT_HD constexpr int single_slot(int g, int h, int spin) { return g == 0 ? spin : 4 * g - 2 + h + 2 * spin; }
// chi(ij) or phi(ij) for a pair a < b; o = 0: (i j) = (a b), 1: (b a)
RWGT_HD constexpr int half_index(int a, int b, int o, int ha, int hb, int spin) {
  return a == 0 ? 8 * (b - 1) + hb + 2 * spin + 4 * o : 16 * (a + b) - 24 + ha + 2 * hb + 4 * spin + 8 * o;
}
// Position of the flow (i j k l) in the lexicographic order of permutations.
RWGT_HD constexpr int flow(int i, int j, int k) { return 6 * i + 2 * (j - (j > i)) + k - (k > i) - (k > j); }

// J of a triple by the rank of its middle leg, from the two stored orderings
// x (middle leg of rank 1) and y (rank 0): the third is -x - y.
template <class R> RWGT_HD Lc<R> by_middle(const Lc<R>& x, const Lc<R>& y, int rank) {
  return lincomb(x, rank == 1 ? R(1) : rank == 0 ? R(0) : R(-1), y, rank == 0 ? R(1) : rank == 1 ? R(0) : R(-1));
}

// A Memory provides mom(g), set_mom, pol(slot), set_pol, vec(slot), set_vec,
// spin(slot), set_spin.  Each task function below is one lane's task; between
// a group of tasks and the next the Memory is synchronised.

// ------------------------------------------------------------ gluon currents
constexpr int kPolTasks = kPols, kPairTasks = kPairSlots, kTripleTasks = kTripleSlots;

template <class R, class M> RWGT_HD void pol_task(M& m, int t) {
  const int g = (t + 1) >> 1, h = t == 0 ? 0 : (t + 1) & 1;
  m.set_pol(t, polarisation(m.mom(g), h ? 1 : -1, g >= 2));
}

template <class R, class M> RWGT_HD void pair_task(M& m, int t, R g3) {
  const int q = (t - 6) >> 2, r = t - 6;
  const int a = t < 6 ? 0 : q == 2 ? 2 : 1, b = t < 6 ? 1 + (t >> 1) : q == 0 ? 2 : 3;
  const int ha = t < 6 ? 0 : r & 1, hb = t < 6 ? t & 1 : (r >> 1) & 1;
  const LcK<R> ka = m.mom(a), kb = m.mom(b);
  Lc<R> o = {};
  add_v3(o, m.pol(pol_slot(a, ha)), ka, m.pol(pol_slot(b, hb)), kb);
  m.set_vec(kPair + t, o * quot(-g3, square(ka + kb)));
}

template <class R, class M> RWGT_HD void triple_task(M& m, int t, R g3, R g4) {
  const int g = t < 8 ? 0 : (t - 4) >> 2, r = t < 8 ? t : (t & 3) << 1;
  const int a = member(g, 0), b = member(g, 1), c = member(g, 2), ha = r & 1, hb = (r >> 1) & 1, hc = r >> 2;
  const LcK<R> ka = m.mom(a), kb = m.mom(b), kc = m.mom(c);
  const Lc<R> ja = m.pol(pol_slot(a, ha)), jb = m.pol(pol_slot(b, hb)), jc = m.pol(pol_slot(c, hc));
  const Lc<R> jab = m.vec(pair_slot(a, b, ha, hb)), jbc = m.vec(pair_slot(b, c, hb, hc));
  const Lc<R> jac = m.vec(pair_slot(a, c, ha, hc));
  const cx<R> ab = dot2(ja, jb), ac = dot2(ja, jc), bc = dot2(jb, jc);
  const LcK<R> kab = ka + kb;
  const R inv = quot(R(1), square(kab + kc)), s3 = -g3 * inv, s4 = g4 * inv;
  Lc<R> v = {}, q = {};                         // J(abc)
  add_v3(v, ja, ka, jbc, kb + kc);
  add_v3(v, jab, kab, jc, kc);
  add_v4(q, ja, jb, jc, ab, ac, bc);
  m.set_vec(kTriple + t, lincomb(v, s3, q, s4));
  load_fence();
  v = {}; q = {};                               // J(bac)
  add_v3(v, jc, kc, jab, kab);                  // V3(J(ba), J(c)) = V3(J(c), J(ab))
  add_v3(v, jb, kb, jac, ka + kc);
  add_v4(q, jb, ja, jc, ab, bc, ac);
  m.set_vec(kTriple + kTripleSlots + t, lincomb(v, s3, q, s4));
}

// J(0abc) before its propagator for the n-th ordering of 1 2 3 (123 132 213
// 231 312 321) and the gluon helicities cfg (bits h1 h2 h3).
template <class R, class M> RWGT_HD Lc<R> four_task(M& m, int n, int cfg, R g3, R g4) {
  const int a = 1 + (n >> 1), lo = a == 1 ? 2 : 1, hi = a == 3 ? 2 : 3, swap = n & 1;
  const int b = swap ? hi : lo, c = swap ? lo : hi;
  const int ha = (cfg >> (a - 1)) & 1, hb = (cfg >> (b - 1)) & 1, hc = (cfg >> (c - 1)) & 1;
  const LcK<R> k0 = m.mom(0), ka = m.mom(a), kb = m.mom(b), kc = m.mom(c);
  const Lc<R> j0 = m.pol(0), ja = m.pol(pol_slot(a, ha)), jb = m.pol(pol_slot(b, hb)), jc = m.pol(pol_slot(c, hc));
  const Lc<R> j0a = m.vec(pair_slot(0, a, 0, ha));
  const Lc<R> jbc = m.vec(pair_slot(lo, hi, swap ? hc : hb, swap ? hb : hc)) * (swap ? R(-1) : R(1));
  const bool up = a < b;
  const Lc<R> jab = m.vec(up ? pair_slot(a, b, ha, hb) : pair_slot(b, a, hb, ha)) * (up ? R(1) : R(-1));
  Lc<R> v = {}, q = {};
  const int s = triple_slot(0, cfg & 1, (cfg >> 1) & 1, cfg >> 2);
  add_v3(v, j0, k0, by_middle(m.vec(s), m.vec(s + kTripleSlots), b - 1), ka + kb + kc);
  settle(v); settle(q); load_fence();
  add_v3(v, j0a, k0 + ka, jbc, kb + kc);
  settle(v); settle(q); load_fence();
  // J(0ab), of the triple without c: a has rank 1 if a < b, else 2
  const int s2 = triple_slot(c, 0, up ? ha : hb, up ? hb : ha);
  add_v3(v, by_middle(m.vec(s2), m.vec(s2 + kTripleSlots), up ? 1 : 2), k0 + ka + kb, jc, kc);
  settle(v); settle(q); load_fence();
  add_v4(q, j0, ja, jbc, dot2(j0, ja), dot2(j0, jbc), dot2(ja, jbc));
  settle(v); settle(q); load_fence();
  add_v4(q, j0, jab, jc, dot2(j0, jab), dot2(j0, jc), dot2(jab, jc));
  settle(v); settle(q); load_fence();
  add_v4(q, j0a, jb, jc, dot2(j0a, jb), dot2(j0a, jc), dot2(jb, jc));
  return lincomb(v, -g3, q, g4);
}

// ------------------------------------------------------------ the quark line
constexpr int kSingleTasks = 14, kHalfSmall = 24;   // half tasks of pairs with gluon 0 (48 more without)

template <class R> struct Quarks { LcK<R> pt, ptb; R m; };

// chi(g) and psi(g) of slot t
template <class R, class M> RWGT_HD void single_task(M& m, int t, const Quarks<R>& q, R gq) {
  const int g = t < 2 ? 0 : (t + 2) >> 2, r = t + 2, h = t < 2 ? 0 : r & 1, spin = t < 2 ? t : (r >> 1) & 1;
  const Lc<R> e = m.pol(pol_slot(g, h));
  const LcK<R> k = m.mom(g);
  m.set_spin(kChi + t, prop_row(row_slash(m.spin(kUbar + spin), e), q.pt - k, q.m, gq));
  load_fence();
  m.set_spin(kPsi + t, prop_col(slash_col(e, m.spin(kV + spin)), k - q.ptb, q.m, gq));
}

// Legs of half task t: (i j) = (a b) for o = 0, (b a) for o = 1.
struct HalfTask { int i, j, hi, hj, spin, pair; bool o; };
RWGT_HD HalfTask half_task(int t) {
  const bool small = t < kHalfSmall;
  const int r = t - kHalfSmall, q = r >> 4;
  const int a = small ? 0 : q == 2 ? 2 : 1, b = small ? 1 + (t >> 3) : q == 0 ? 2 : 3;
  const int ha = small ? 0 : r & 1, hb = small ? t & 1 : (r >> 1) & 1;
  const int spin = small ? (t >> 1) & 1 : (r >> 2) & 1;
  const bool o = ((small ? t >> 2 : r >> 3) & 1) != 0;
  return {o ? b : a, o ? a : b, o ? hb : ha, o ? ha : hb, spin, pair_slot(a, b, ha, hb), o};
}
template <class R, class M> RWGT_HD Spinor<R> chi2_task(M& m, const HalfTask& h, const Quarks<R>& q, R gq) {
  const R sign = h.o ? R(-1) : R(1);
  Spinor<R> r = row_slash(m.spin(kUbar + h.spin), m.vec(h.pair) * sign);
  for (int n = 0; n < 4; ++n) settle(r.c[n]);
  load_fence();
  add_row_slash(r, m.spin(kChi + single_slot(h.i, h.hi, h.spin)), m.pol(pol_slot(h.j, h.hj)));
  return prop_row(r, q.pt - m.mom(h.i) - m.mom(h.j), q.m, gq);
}
template <class R, class M> RWGT_HD Spinor<R> phi2_task(M& m, const HalfTask& h) {
  const R sign = h.o ? R(-1) : R(1);
  Spinor<R> c = slash_col(m.vec(h.pair) * sign, m.spin(kV + h.spin));
  add_slash_col(c, m.pol(pol_slot(h.i, h.hi)), m.spin(kPsi + single_slot(h.j, h.hj, h.spin)));
  return c;
}

// ------------------------------------------------------------------ one lane
// Helicities of lane t: gluons 1 2 3, antiquark, quark.
struct LaneHel { int h[4], anti, quark; };
RWGT_HD LaneHel lane_hel(int t) {
  return {{0, t & 1, (t >> 1) & 1, (t >> 2) & 1}, (t >> 3) & 1, (t >> 4) & 1};
}

// The J(ijkl) term of every flow from the six that start with gluon 0, in the
// order (a b c) = 123 132 213 231 312 321.
template <class R> RWGT_HD void spread_four(cx<R> (&f)[24], const cx<R> (&b)[6]) {
  constexpr int perm[6][3] = {{1, 2, 3}, {1, 3, 2}, {2, 1, 3}, {2, 3, 1}, {3, 1, 2}, {3, 2, 1}};
  auto at = [](int x, int y, int z) constexpr { return 2 * (x - 1) + (y > z ? 1 : 0); };
#pragma unroll
  for (int n = 0; n < 6; ++n) {
    const int x = perm[n][0], y = perm[n][1], z = perm[n][2];
    const cx<R> t = b[at(x, y, z)] + b[at(y, x, z)] + b[at(y, z, x)];
    f[flow(0, x, y)] = b[at(x, y, z)];
    f[flow(z, y, x)] = -b[at(x, y, z)];          // (z y x 0)
    f[flow(x, 0, y)] = -t;                       // (x 0 y z)
    f[flow(z, y, 0)] = t;                        // (z y 0 x)
    settle(f[flow(x, 0, y)]);
  }
}

// ubar J(ijk) psi(l) and chi(i) J(jkl) v
template <class R, class M>
RWGT_HD void triple_terms(M& m, int t,  const Spinor<R>& ubar, const Spinor<R>& v, cx<R> (&f)[24]) {
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    load_fence();
    const LaneHel h = lane_hel(opq_index(t));
    const int a = member(g, 0), b = member(g, 1), c = member(g, 2);
    const int s = triple_slot(g, h.h[a], h.h[b], h.h[c]);
    const Lc<R> x = m.vec(s), y = m.vec(s + kTripleSlots);
    const Lc<R> wl = pair_coeffs(ubar, m.spin(kPsi + single_slot(g, h.h[g], h.anti)));
    const Lc<R> wi = pair_coeffs(m.spin(kChi + single_slot(g, h.h[g], h.quark)), v);
    const cx<R> tx = apply(wl, x), ty = apply(wl, y), tz = tx + ty;
    const cx<R> sx = apply(wi, x), sy = apply(wi, y), sz = sx + sy;
    auto add = [&](int n, cx<R> t) { f[n] = f[n] + t; settle(f[n]); };
    auto sub = [&](int n, cx<R> t) { f[n] = f[n] - t; settle(f[n]); };
    add(flow(a, b, c), tx); add(flow(c, b, a), tx);
    add(flow(b, a, c), ty); add(flow(c, a, b), ty);
    sub(flow(a, c, b), tz); sub(flow(b, c, a), tz);
    add(flow(g, a, b), sx); add(flow(g, c, b), sx);
    add(flow(g, b, a), sy); add(flow(g, c, a), sy);
    sub(flow(g, a, c), sz); sub(flow(g, b, c), sz);
  }
}

// chi(i) J(jk) psi(l)
template <class R, class M> RWGT_HD void pair_terms(M& m, int t, cx<R> (&f)[24]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    load_fence();
    const LaneHel h = lane_hel(opq_index(t));
    const Spinor<R> chi = m.spin(kChi + single_slot(i, h.h[i], h.quark));
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      if (l == i) continue;
      const int lo = i < l ? i : l, hi = i < l ? l : i;
      const int j = lo > 0 ? 0 : hi > 1 ? 1 : 2, k = hi < 3 ? 3 : lo < 2 ? 2 : 1;
      load_fence();
      const Lc<R> w = pair_coeffs(chi, m.spin(kPsi + single_slot(l, h.h[l], h.anti)));
      const cx<R> t = apply(w, m.vec(pair_slot(j, k, h.h[j], h.h[k])));
      f[flow(i, j, k)] = f[flow(i, j, k)] + t;
      f[flow(i, k, j)] = f[flow(i, k, j)] - t;
      settle(f[flow(i, j, k)]);
      settle(f[flow(i, k, j)]);
    }
  }
}

// chi(ij) phi(kl) for the pair (a b) of the row, (c d) of the column, rows
// and columns of the current half tables
template <class R, class M>
RWGT_HD void half_terms(M& m, int t, int a, int b, int c, int d, int row0, int col0, cx<R> (&f)[24]) {
  load_fence();
  const LaneHel h = lane_hel(opq_index(t));
  Spinor<R> r[2], p[2];
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    r[o] = m.spin(row0 + half_index(a, b, o, h.h[a], h.h[b], h.quark));
    p[o] = m.spin(col0 + half_index(c, d, o, h.h[c], h.h[d], h.anti));
  }
  add_dot(f[flow(a, b, c)], r[0], p[0]);
  add_dot(f[flow(b, a, c)], r[1], p[0]);
  add_dot(f[flow(a, b, d)], r[0], p[1]);
  add_dot(f[flow(b, a, d)], r[1], p[1]);
  settle(f[flow(a, b, c)]);
  settle(f[flow(b, a, c)]);
  settle(f[flow(a, b, d)]);
  settle(f[flow(b, a, d)]);
}

// One lane's part of an event.  sync() separates the groups of tasks; CNUM
// columns are the caller's: COLOUR(f) is J^dagger C J of the 24 flows.
//   pt, ptb   momenta of the outgoing quark and antiquark (E px py pz)
// Returns |M_h|^2 summed over colours, without g^2 of the last vertices.
template <class R, class M, class Cd, class Sync, class Colour>
RWGT_HD R lane_me2(M& m, int t, const R* pt, const R* ptb, const Cd& cd, Sync sync, Colour colour) {
  const LaneHel h = lane_hel(t);
  const Quarks<R> q = {lc_momentum(pt, R(1)), lc_momentum(ptb, R(1)), cd.mt};
  auto clamp = [&](int n) { const int x = opq_index(t); return x < n ? x : n - 1; };   // idle lanes repeat the last task
  const Spinor<R> ubar = oxx<R>(pt, q.m, h.quark ? 1 : -1, 1), v = ixx<R>(ptb, q.m, h.anti ? 1 : -1, -1);
  m.set_spin(kUbar + h.quark, ubar);
  m.set_spin(kV + h.anti, v);
  pol_task<R>(m, clamp(kPolTasks));
  sync();
  pair_task(m, clamp(kPairTasks), cd.g3);
  sync();
  triple_task(m, clamp(kTripleTasks), cd.g3, cd.g4);
  sync();
  cx<R> f[24];
  {
    const Lc<R> w = pair_coeffs(ubar, v) * quot(R(1), square(q.pt + q.ptb));
    const int cfg = t & 7;
    cx<R> b[6];
    m.set_vec(kFour + t, four_task(m, t >> 3, cfg, cd.g3, cd.g4));
    sync();
#pragma unroll
    for (int n = 0; n < 4; ++n) b[n] = apply(w, m.vec(kFour + 8 * n + cfg));
    sync();
    m.set_vec(kFour + (t & 15), four_task(m, 4 + ((t >> 3) & 1), cfg, cd.g3, cd.g4));
    sync();
#pragma unroll
    for (int n = 0; n < 2; ++n) b[4 + n] = apply(w, m.vec(kFour + 8 * n + cfg));
    sync();
    spread_four(f, b);
  }
  single_task(m, clamp(kSingleTasks), q, cd.gqq);
  sync();
  triple_terms(m, t, ubar, v, f);
  pair_terms(m, t, f);
  sync();
  // rows of the pairs with gluon 0, columns of the others
  int n = clamp(kHalfSmall);
  m.set_spin(kHalf + n, chi2_task(m, half_task(n), q, cd.gqq));
  m.set_spin(kHalf + kHalfSmall + t, phi2_task<R>(m, half_task(kHalfSmall + t)));
  n = kLanes + (t & 15);
  m.set_spin(kHalf + kHalfSmall + n, phi2_task<R>(m, half_task(kHalfSmall + n)));
  sync();
  half_terms(m, t, 0, 1, 2, 3, kHalf, kHalf, f);
  half_terms(m, t, 0, 2, 1, 3, kHalf, kHalf, f);
  half_terms(m, t, 0, 3, 1, 2, kHalf, kHalf, f);
  sync();
  // and the other way round
  n = clamp(kHalfSmall);
  m.set_spin(kHalf + n, phi2_task<R>(m, half_task(n)));
  m.set_spin(kHalf + kHalfSmall + t, chi2_task(m, half_task(kHalfSmall + t), q, cd.gqq));
  n = kLanes + (t & 15);
  m.set_spin(kHalf + kHalfSmall + n, chi2_task(m, half_task(kHalfSmall + n), q, cd.gqq));
  sync();
  half_terms(m, t, 1, 2, 0, 3, kHalf, kHalf, f);
  half_terms(m, t, 1, 3, 0, 2, kHalf, kHalf, f);
  half_terms(m, t, 2, 3, 0, 1, kHalf, kHalf, f);
  load_fence();
  return colour(f);
}

}  // namespace ordered
}  // namespace rwgt
