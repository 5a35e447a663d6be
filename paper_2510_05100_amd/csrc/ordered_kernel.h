// Device side of the colour-ordered recursions (ordered.h, ordered_pairs.h):
// half a wave per event.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "card_source.h"
#include "check.h"
#include "helas.h"
#include "kernels.h"
#include "ordered.h"
#include "ordered_pairs.h"

namespace rwgt {
namespace ordered {

// The shared currents of one event in LDS, component by component: eight
// lanes that read eight neighbouring slots (or the same one) touch the 128
// bytes of one LDS cycle.
template <int SLOTS, int POLS, int MOMENTA>
struct LdsMemory {
  typedef double v2 __attribute__((ext_vector_type(2)));
  struct Event {
    v2 vec[4][SLOTS];
    v2 pol[2][POLS];
    v2 mom[2][MOMENTA];
    double pol_u[(POLS + 1) / 2 * 2];
  };
  Event* s;
  static __device__ __forceinline__ cx<double> c(v2 a) { return {a.x, a.y}; }
  static __device__ __forceinline__ v2 r(cx<double> a) { return v2{a.re, a.im}; }
  __device__ __forceinline__ LcK<double> mom(int g) const {
    const v2 a = s->mom[0][g];
    return {a.x, a.y, c(s->mom[1][g])};
  }
  __device__ __forceinline__ void set_mom(int g, const LcK<double>& k) {
    s->mom[0][g] = v2{k.u, k.d};
    s->mom[1][g] = r(k.p);
  }
  __device__ __forceinline__ Lc<double> pol(int i) const {      // u real, d = -u
    const double u = s->pol_u[i];
    return {{u, 0.0}, {-u, 0.0}, c(s->pol[0][i]), c(s->pol[1][i])};
  }
  __device__ __forceinline__ void set_pol(int i, const Lc<double>& v) {
    s->pol_u[i] = v.u.re;
    s->pol[0][i] = r(v.p);
    s->pol[1][i] = r(v.m);
  }
  __device__ __forceinline__ Lc<double> vec(int i) const {
    return {c(s->vec[0][i]), c(s->vec[1][i]), c(s->vec[2][i]), c(s->vec[3][i])};
  }
  __device__ __forceinline__ void set_vec(int i, const Lc<double>& v) {
    s->vec[0][i] = r(v.u);
    s->vec[1][i] = r(v.d);
    s->vec[2][i] = r(v.p);
    s->vec[3][i] = r(v.m);
  }
  __device__ __forceinline__ Spinor<double> spin(int i) const {
    return {{c(s->vec[0][i]), c(s->vec[1][i]), c(s->vec[2][i]), c(s->vec[3][i])}};
  }
  __device__ __forceinline__ void set_spin(int i, const Spinor<double>& v) {
#pragma unroll
    for (int n = 0; n < 4; ++n) s->vec[n][i] = r(v.c[n]);
  }
};

// Momentum of particle a of event i, in the caller's layout.
__device__ __forceinline__ void load_momentum(const double* mom, int64_t nevt, int npart, int a, int64_t i,
                                              double (&p)[4]) {
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) p[mu] = RWGT_AT(mom, (i * npart + a) * 4 + mu, nevt * npart * 4);
}

// The recursions: their memory, the momenta it starts with, and a lane's part.
struct QuarkLine {                               // g g -> Q Q~ g g
  typedef LdsMemory<kSlots, kPols, 4> Memory;
  static __device__ __forceinline__ void fill(Memory& m, int t, const double* mom, int64_t nevt, int64_t i) {
    const int g = t & 3;                         // gluons: particles 0, 1 in, 4, 5 out
    double p[4];
    load_momentum(mom, nevt, 6, g < 2 ? g : g + 2, i, p);
    m.set_mom(g, lc_momentum(p, g < 2 ? 1.0 : -1.0));
  }
  template <class Cd, class Colour>
  static __device__ __forceinline__ double lane(Memory& m, int t, const double* mom, int64_t nevt, int64_t i,
                                                const Cd& cd, Colour colour) {
    double pt[4], ptb[4];
    load_momentum(mom, nevt, 6, 2, i, pt);
    load_momentum(mom, nevt, 6, 3, i, ptb);
    return lane_me2(m, t, pt, ptb, cd, [] { wave_sync(); }, colour);
  }
};
struct QuarkPairs {                              // g g -> Q Q~ Q Q~
  typedef LdsMemory<pairs::kSlots, pairs::kPols, 6> Memory;
  static __device__ __forceinline__ void fill(Memory& m, int t, const double* mom, int64_t nevt, int64_t i) {
    const int a = t < 6 ? t : 5;
    double p[4];
    load_momentum(mom, nevt, 6, a, i, p);
    m.set_mom(a, lc_momentum(p, 1.0));
  }
  template <class Cd, class Colour>
  static __device__ __forceinline__ double lane(Memory& m, int t, const double* mom, int64_t nevt, int64_t i,
                                                const Cd& cd, Colour colour) {
    auto load = [&](int a, double (&p)[4]) { load_momentum(mom, nevt, 6, a, i, p); };
    return pairs::lane_me2<double>(m, t, load, cd, [] { wave_sync(); }, colour);
  }
};

// Half a wave per event, one lane per evaluated helicity, under every card in
// turn.  LISTED: the events rows[0 .. *nrows), workgroups striding over the
// list; otherwise the events from first0 on, one workgroup per pair (no loop
// around the recursion: the listed form spills 46 registers where this one
// spills 28).
//
// Bound by the vector ALUs: they issue in 89 % of the cycles, 85 % of it FP64.
// A wave evaluates a card of its two events in 5850 vector instructions, where
// evaluating every diagram for every helicity takes about 5 times that
// (g g -> t t~ g g; g g -> t t~ t t~ 4 times); the colour sum is 260 of them,
// 650 without the flows' sums and differences.  Two waves per SIMD (LDS 17 KB
// per wave, 256 registers, 28 spilled; 166, none) hide the LDS latency; the
// fences (load_fence, settle) hold the compiler to the order of the source,
// without them it loads everything first and spills 1000 registers.  1e6
// events, one new card: 11.9 ms (75 ms diagram by diagram, one lane per event
// and two waves splitting its helicities; 12.9 with the plain colour sum, which
// other cards of the type ran in 12.5 to 14.4 as their clock allows), 777
// events: 0.034 (2.4) ms; g g -> t t~ t t~, 250001 events: 2.45 (9.36) ms.  A
// first form for g g -> t t~ g g with two waves per 64 events and one lane per
// event shared the gluon currents only and needed 512 registers with 310
// spilled, waiting in half of its cycles: 29.7 ms.
template <class PROC, class REC, bool LISTED, class CARDS>
__global__ __launch_bounds__(64, 2) void ordered_kernel(const double* __restrict__ mom, int64_t nevt,
                                                        const CARDS cards, int ncards,
                                                        const double* __restrict__ w_in, double* __restrict__ w_out,
                                                        double* __restrict__ me_out, const int32_t* __restrict__ rows,
                                                        const unsigned int* __restrict__ nrows,
                                                        unsigned long long* __restrict__ nonfinite, int64_t first0) {
  __shared__ typename REC::Memory::Event mem[2];
  const int t = int(threadIdx.x) & (kLanes - 1), half = int(threadIdx.x) / kLanes;
  typename REC::Memory m{&mem[half]};
  const int64_t n = LISTED ? int64_t(*nrows) : nevt;
  int64_t first = first0 + int64_t(blockIdx.x) * 2;
  int bad = 0;                                   // non-finite outputs of this half's events
  if (LISTED && first >= n) return;
  do {
    const bool valid = first + half < n;
    const int64_t r = valid ? first + half : n - 1;   // a missing second event repeats the last one
    const int64_t i = LISTED ? int64_t(RWGT_AT(rows, r, nevt)) : r;
    if (LISTED) wave_sync();
    REC::fill(m, t, mom, nevt, i);
    double norm = 0.0;
#pragma unroll 1
    for (int k = 0; k < ncards; ++k) {
      const auto& cd = cards(k);                 // read where it is used: held, it would cost registers
      wave_sync();
      double me = REC::lane(m, opq_index(t), mom, nevt, i, cd, [](cx<double>(&f)[PROC::NCOL]) {
        return PROC::template colour_sum_paired<double>(f);
      });
#pragma unroll
      for (int d = 1; d < kLanes; d <<= 1) me += __shfl_xor(me, d);
      me *= cd.gqq * cd.gqq * PROC::SCALE;
      if (t != 0 || !valid) continue;
      if (me_out) RWGT_AT(me_out, int64_t(k) * nevt + i, int64_t(ncards) * nevt) = me;
      if (w_out) {
        if (k == 0) {
          norm = (me == 0.0 ? 0.0 : 1.0 / me) * RWGT_AT(w_in, i, nevt);
        } else {
          const double w = norm * me;
          RWGT_AT(w_out, int64_t(k - 1) * nevt + i, int64_t(ncards - 1) * nevt) = w;
          if (!LISTED) bad += isfinite(w) ? 0 : 1;
        }
      } else if (!LISTED) {
        bad += isfinite(me) ? 0 : 1;
      }
    }
    first += int64_t(gridDim.x) * 2;
  } while (LISTED && first < n);
  if (!LISTED && nonfinite) {
    bad += __shfl_xor(bad, kLanes);
    if (threadIdx.x == 0) RWGT_AT(nonfinite, blockIdx.x, gridDim.x) = static_cast<unsigned long long>(bad);
  }
}

// Workgroups of the launch that starts at event first0 of nevt: one per pair of
// those left, up to 2^25 (2^31 work-items; a launch holds fewer than 2^32, and
// the pairs of 1.3e8 events, 26 GB of momenta, have as many).
constexpr int64_t kLaunchGroups = int64_t(1) << 25;
inline int64_t launch_groups(int64_t nevt, int64_t first0) {
  const int64_t pairs = (nevt - first0 + 1) / 2;
  return pairs < kLaunchGroups ? pairs : kLaunchGroups;
}

// The workgroups count their non-finite outputs as long as there are few
// enough of them for the caller to add up (8192 events; beyond, the separate
// pass is under 2 % of the call).
template <class PROC, class REC>
inline hipError_t launch(const Fp64Call& a, hipStream_t s) {
  const int64_t all = launch_groups(a.nevt, 0);
  const bool count = a.nonfinite && all <= kNonfiniteBlocks;
  if (a.counts) *a.counts = count ? int(all) : 0;
  return with_cards<QcdCard>(a, qcd_card, [&](const auto& cards) {
    typedef std::remove_cv_t<std::remove_reference_t<decltype(cards)>> Cards;
    hipError_t e = hipSuccess;
    int64_t groups = 0;
    for (int64_t first0 = 0; first0 < a.nevt && e == hipSuccess; first0 += 2 * groups) {
      groups = launch_groups(a.nevt, first0);
      hipLaunchKernelGGL((ordered_kernel<PROC, REC, false, Cards>), dim3(unsigned(groups)), dim3(64), 0, s, a.mom,
                         a.nevt, cards, a.ncards, a.w_in, a.w_out, a.me_out, static_cast<const int32_t*>(nullptr),
                         static_cast<const unsigned int*>(nullptr), count ? a.nonfinite : nullptr, first0);
      e = hipGetLastError();
    }
    return e;
  });
}

struct PairCards {                               // the mixed path's cards
  const CardPair* p;
  int n;
  __device__ __forceinline__ const Card<double>& operator()(int k) const { return RWGT_AT(p, k, n).d; }
};

// rows: at most nevt of them, counted on the device; 4096 workgroups keep
// every SIMD at its two waves twice over.
template <class PROC, class REC>
inline hipError_t launch_rows(const double* mom, int64_t nevt, const CardPair* cards, int ncards, const double* w_in,
                              double* w_out, double* me_out, const int32_t* rows, const unsigned int* nrows,
                              hipStream_t s) {
  const int64_t pairs = (nevt + 1) / 2;
  hipLaunchKernelGGL((ordered_kernel<PROC, REC, true, PairCards>), dim3(unsigned(pairs < 4096 ? pairs : 4096)),
                     dim3(64), 0, s, mom, nevt, PairCards{cards, ncards}, ncards, w_in, w_out, me_out, rows, nrows,
                     static_cast<unsigned long long*>(nullptr), int64_t(0));
  return hipGetLastError();
}

}  // namespace ordered
}  // namespace rwgt
