// Generated by paper_2510_05100_amd.procgen for 'ee_mumu'. Do not edit.
// 2 Feynman diagrams, 2 amplitude terms, 1 colour flows.
// Colour basis (gluon leg ids on the main line, row end first): ()
#pragma once
#include "helas.h"
#include "card.h"
namespace rwgt {
namespace gen_ee_mumu {
constexpr int NPART = 4;
constexpr int NCOL = 1;
constexpr int NHEL = 16;
constexpr int NGOOD = 4;
constexpr int NDIAG = 2;
constexpr int NAMP = 2;
constexpr double AVERAGE = 0.25;
constexpr int NSUM = 4;
constexpr double HELW = 1.0;
constexpr int CDEN = 1;
static __constant__ int GOOD[NGOOD] = {5, 6, 9, 10};
constexpr int GOOD_HOST[NGOOD] = {5, 6, 9, 10};
constexpr int CNUM[NCOL][NCOL] = {
  {1},
};
// Routine counts per helicity: ixx 2, oxx 2, vxx 0, ffv_in 0, ffv_out 0, ffv_vec0 1, ffv_vecm 1, vvv_vec 0, vvvv_vec 0, ffv_amp 2, pair_w 0
constexpr int N_IXX = 2;
constexpr int N_OXX = 2;
constexpr int N_VXX = 0;
constexpr int N_FFV_IN = 0;
constexpr int N_FFV_OUT = 0;
constexpr int N_FFV_VEC0 = 1;
constexpr int N_FFV_VECM = 1;
constexpr int N_VVV_VEC = 0;
constexpr int N_VVVV_VEC = 0;
constexpr int N_FFV_AMP = 2;
constexpr int N_PAIR_W = 0;

// D is the momentum type: double on the device; an operation-counting
// type when the host instantiates this to count arithmetic.
// J indexes like cx<R>[NCOL]: a register array, or an accessor into LDS.
template <class R, class D, class J>
__host__ __device__ __forceinline__ void jamps(const D (&P)[4][4], int hel, const Card<R, D>& cd, J& jamp) {
  const int h0 = ((hel >> 3) & 1) ? 1 : -1;
  const int h1 = ((hel >> 2) & 1) ? 1 : -1;
  const int h2 = ((hel >> 1) & 1) ? 1 : -1;
  const int h3 = ((hel >> 0) & 1) ? 1 : -1;
  for (int c = 0; c < NCOL; ++c) jamp[c] = cx<R>{R(0), R(0)};
  note_reset(jamp);
  cx<R> amp;
  const D pw3[4] = {opq(P[3][0]), opq(P[3][1]), opq(P[3][2]), opq(P[3][3])};
  const Spinor<R> w3 = oxx<R>(pw3, Massless{}, h3, 1);
  const D pw2[4] = {opq(P[2][0]), opq(P[2][1]), opq(P[2][2]), opq(P[2][3])};
  const Spinor<R> w2 = ixx<R>(pw2, Massless{}, h2, -1);
  const D q1[4] = {-opq(P[2][0]) - opq(P[3][0]), -opq(P[2][1]) - opq(P[3][1]), -opq(P[2][2]) - opq(P[3][2]), -opq(P[2][3]) - opq(P[3][3])};
  const Vec<R> v2 = ffv_vec0_v<R>(w3, w2, cd.a[1], q1);
  const D pw0[4] = {opq(P[0][0]), opq(P[0][1]), opq(P[0][2]), opq(P[0][3])};
  const Spinor<R> w0 = oxx<R>(pw0, Massless{}, h0, -1);
  const D pw1[4] = {opq(P[1][0]), opq(P[1][1]), opq(P[1][2]), opq(P[1][3])};
  const Spinor<R> w1 = ixx<R>(pw1, Massless{}, h1, 1);
  amp = ffv_amp_v<R>(w0, w1, v2, cd.a[0]);
  jamp[0] = jamp[0] + amp;
  note_amp(jamp, amp, 1);
  term_fence();
  const D q3[4] = {-opq(P[2][0]) - opq(P[3][0]), -opq(P[2][1]) - opq(P[3][1]), -opq(P[2][2]) - opq(P[3][2]), -opq(P[2][3]) - opq(P[3][3])};
  const Vec<R> v4 = ffv_vecm_c<R>(w3, w2, cd.zL[1], cd.zR[1], q3, cd.mz, cd.wz);
  amp = ffv_amp_c<R>(w0, w1, v4, cd.zL[0], cd.zR[0]);
  jamp[0] = jamp[0] + amp;
  note_amp(jamp, amp, 1);
  term_fence();
}

template <class R, class J>
__host__ __device__ __forceinline__ R colour_sum(const J& jamp) {
  R me = R(0);
  { const R zr = R(1) * jamp[0].re;
    const R zi = R(1) * jamp[0].im;
    me += jamp[0].re * zr + jamp[0].im * zi; }
  return me * R(1.0 / 1.0);
}
}  // namespace gen_ee_mumu
}  // namespace rwgt
