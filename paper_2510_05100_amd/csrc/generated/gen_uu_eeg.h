// Generated by paper_2510_05100_amd.procgen for 'uu_eeg'. Do not edit.
// 4 Feynman diagrams, 4 amplitude terms, 1 colour flows.
// Colour basis (gluon leg ids on the main line, row end first): (4)
#pragma once
#include "helas.h"
#include "card.h"
namespace rwgt {
namespace gen_uu_eeg {
constexpr int NPART = 5;
constexpr int NCOL = 1;
constexpr int NHEL = 32;
constexpr int NGOOD = 8;
constexpr int NDIAG = 4;
constexpr int NAMP = 4;
constexpr double AVERAGE = 0.027777777777777776;
constexpr int NSUM = 8;
constexpr double HELW = 1.0;
constexpr int CDEN = 1;
static __constant__ int GOOD[NGOOD] = {10, 11, 12, 13, 18, 19, 20, 21};
constexpr int GOOD_HOST[NGOOD] = {10, 11, 12, 13, 18, 19, 20, 21};
constexpr int CNUM[NCOL][NCOL] = {
  {4},
};
// Routine counts per helicity: ixx 2, oxx 2, vxx 1, ffv_in 3, ffv_out 0, ffv_vec0 1, ffv_vecm 1, vvv_vec 0, vvvv_vec 0, ffv_amp 4, pair_w 0
constexpr int N_IXX = 2;
constexpr int N_OXX = 2;
constexpr int N_VXX = 1;
constexpr int N_FFV_IN = 3;
constexpr int N_FFV_OUT = 0;
constexpr int N_FFV_VEC0 = 1;
constexpr int N_FFV_VECM = 1;
constexpr int N_VVV_VEC = 0;
constexpr int N_VVVV_VEC = 0;
constexpr int N_FFV_AMP = 4;
constexpr int N_PAIR_W = 0;

// D is the momentum type: double on the device; an operation-counting
// type when the host instantiates this to count arithmetic.
// J indexes like cx<R>[NCOL]: a register array, or an accessor into LDS.
template <class R, class D, class J>
__host__ __device__ __forceinline__ void jamps(const D (&P)[5][4], int hel, const Card<R, D>& cd, J& jamp) {
  const int h0 = ((hel >> 4) & 1) ? 1 : -1;
  const int h1 = ((hel >> 3) & 1) ? 1 : -1;
  const int h2 = ((hel >> 2) & 1) ? 1 : -1;
  const int h3 = ((hel >> 1) & 1) ? 1 : -1;
  const int h4 = ((hel >> 0) & 1) ? 1 : -1;
  for (int c = 0; c < NCOL; ++c) jamp[c] = cx<R>{R(0), R(0)};
  note_reset(jamp);
  cx<R> amp;
  const D pw4[4] = {opq(P[4][0]), opq(P[4][1]), opq(P[4][2]), opq(P[4][3])};
  const Vec<R> w4 = vxx<R>(pw4, h4, -1);
  const D pw1[4] = {opq(P[1][0]), opq(P[1][1]), opq(P[1][2]), opq(P[1][3])};
  const Spinor<R> w1 = oxx<R>(pw1, Massless{}, h1, -1);
  const D pw0[4] = {opq(P[0][0]), opq(P[0][1]), opq(P[0][2]), opq(P[0][3])};
  const Spinor<R> w0 = ixx<R>(pw0, Massless{}, h0, 1);
  const D pw3[4] = {opq(P[3][0]), opq(P[3][1]), opq(P[3][2]), opq(P[3][3])};
  const Spinor<R> w3 = oxx<R>(pw3, Massless{}, h3, 1);
  const D pw2[4] = {opq(P[2][0]), opq(P[2][1]), opq(P[2][2]), opq(P[2][3])};
  const Spinor<R> w2 = ixx<R>(pw2, Massless{}, h2, -1);
  const D q1[4] = {-opq(P[2][0]) - opq(P[3][0]), -opq(P[2][1]) - opq(P[3][1]), -opq(P[2][2]) - opq(P[3][2]), -opq(P[2][3]) - opq(P[3][3])};
  const Vec<R> v2 = ffv_vec0_v<R>(w3, w2, cd.a[0], q1);
  const D q3[4] = {opq(P[0][0]) - opq(P[2][0]) - opq(P[3][0]), opq(P[0][1]) - opq(P[2][1]) - opq(P[3][1]), opq(P[0][2]) - opq(P[2][2]) - opq(P[3][2]), opq(P[0][3]) - opq(P[2][3]) - opq(P[3][3])};
  const Spinor<R> f4 = ffv_in_v<R>(w0, v2, cd.a[2], q3, Massless{});
  amp = ffv_amp_v<R>(w1, f4, w4, cd.gqq);
  jamp[0] = jamp[0] + amp;
  note_amp(jamp, amp, 1);
  term_fence();
  const D q5[4] = {opq(P[0][0]) - opq(P[4][0]), opq(P[0][1]) - opq(P[4][1]), opq(P[0][2]) - opq(P[4][2]), opq(P[0][3]) - opq(P[4][3])};
  const Spinor<R> f6 = ffv_in_v<R>(w0, w4, cd.gqq, q5, Massless{});
  amp = ffv_amp_v<R>(w1, f6, v2, cd.a[2]);
  jamp[0] = jamp[0] + amp;
  note_amp(jamp, amp, 1);
  term_fence();
  const D q7[4] = {-opq(P[2][0]) - opq(P[3][0]), -opq(P[2][1]) - opq(P[3][1]), -opq(P[2][2]) - opq(P[3][2]), -opq(P[2][3]) - opq(P[3][3])};
  const Vec<R> v8 = ffv_vecm_c<R>(w3, w2, cd.zL[0], cd.zR[0], q7, cd.mz, cd.wz);
  amp = ffv_amp_c<R>(w1, f6, v8, cd.zL[2], cd.zR[2]);
  jamp[0] = jamp[0] + amp;
  note_amp(jamp, amp, 1);
  term_fence();
  const D q9[4] = {opq(P[0][0]) - opq(P[2][0]) - opq(P[3][0]), opq(P[0][1]) - opq(P[2][1]) - opq(P[3][1]), opq(P[0][2]) - opq(P[2][2]) - opq(P[3][2]), opq(P[0][3]) - opq(P[2][3]) - opq(P[3][3])};
  const Spinor<R> f10 = ffv_in_c<R>(w0, v8, cd.zL[2], cd.zR[2], q9, Massless{});
  amp = ffv_amp_v<R>(w1, f10, w4, cd.gqq);
  jamp[0] = jamp[0] + amp;
  note_amp(jamp, amp, 1);
  term_fence();
}

template <class R, class J>
__host__ __device__ __forceinline__ R colour_sum(const J& jamp) {
  R me = R(0);
  { const R zr = R(4) * jamp[0].re;
    const R zi = R(4) * jamp[0].im;
    me += jamp[0].re * zr + jamp[0].im * zi; }
  return me * R(1.0 / 1.0);
}
}  // namespace gen_uu_eeg
}  // namespace rwgt
