// One-event-per-lane matrix-element kernel, shared by the per-process
// translation units (each instantiates it for its generated process).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include <type_traits>

#include "card.h"
#include "check.h"
#include "colour_mfma.h"
#include "kernels.h"

namespace rwgt {

// ...: more members (RWGT_PAIRED_COLOUR for a process of several flows).
#define RWGT_PROCESS_TRAITS(NAME, ...)                                                         \
  struct Proc_##NAME {                                                                         \
    static constexpr int NPART = gen_##NAME::NPART;                                            \
    static constexpr int NCOL = gen_##NAME::NCOL;                                              \
    static constexpr int NGOOD = gen_##NAME::NGOOD;                                            \
    static constexpr double AVERAGE = gen_##NAME::AVERAGE;                                     \
    static constexpr int NSUM = gen_##NAME::NSUM;                                              \
    static constexpr double SCALE = gen_##NAME::AVERAGE * gen_##NAME::HELW;                    \
    static constexpr int CDEN = gen_##NAME::CDEN;                                              \
    static __device__ __forceinline__ const int (&cnum())[NCOL][NCOL] { return gen_##NAME::CNUM; } \
    static __device__ __forceinline__ int good(int i) { return gen_##NAME::GOOD[i]; }         \
    template <class R, class J>                                                                \
    static __device__ __forceinline__ void jamps(const double (&P)[NPART][4], int hel,         \
                                                 const Card<R>& cd, J& j) {                    \
      gen_##NAME::jamps<R, double>(P, hel, cd, j);                                             \
    }                                                                                          \
    template <class R, class J>                                                                \
    static __device__ __forceinline__ R colour_sum(const J& j) {                               \
      return gen_##NAME::colour_sum<R>(j);                                                     \
    }                                                                                          \
    __VA_ARGS__                                                                                \
  };
#define RWGT_PAIRED_COLOUR(NAME)                                                               \
  template <class R, class J>                                                                  \
  static __device__ __forceinline__ R colour_sum_paired(J& j) {                                \
    return gen_##NAME::colour_sum_paired<R>(j);                                                \
  }

template <class R> __device__ __forceinline__ const Card<R>& pick(const CardPair& c);
template <> __device__ __forceinline__ const Card<double>& pick<double>(const CardPair& c) { return c.d; }
template <> __device__ __forceinline__ const Card<float>& pick<float>(const CardPair& c) { return c.f; }

// Colour-flow amplitudes of the guarded mixed path: the flows and the
// incoherent sum of the amplitude terms, sum_t m_t |amp_t|^2 (m_t: the number
// of flows term t enters).  Its ratio to the coherent sum_c |J_c|^2 measures
// how much the terms cancel in the flows, which is what amplifies their
// single-precision rounding.
template <class R, int NCOL>
struct GuardJamp {
  cx<R> j[NCOL];
  R inco;
  __device__ __forceinline__ cx<R>& operator[](int c) { return j[c]; }
  __device__ __forceinline__ const cx<R>& operator[](int c) const { return j[c]; }
};
template <class R, int NCOL>
__device__ __forceinline__ void note_reset(GuardJamp<R, NCOL>& g) { g.inco = R(0); }
template <class R, int NCOL>
__device__ __forceinline__ void note_amp(GuardJamp<R, NCOL>& g, const cx<R>& a, int m) {
  g.inco += R(m) * (a.re * a.re + a.im * a.im);
}
template <class R, int NCOL>
__device__ __forceinline__ cx<R> (&flows(GuardJamp<R, NCOL>& g))[NCOL] { return g.j; }
template <class R, int NCOL>
__device__ __forceinline__ cx<R> (&flows(cx<R> (&j)[NCOL]))[NCOL] { return j; }

// |M|^2 of one event under one card with the colour flows in registers and
// the colour sum on the VALU (the form of few-flow processes).
template <class PROC, class R>
__device__ __forceinline__ double me2_event(const double (&P)[PROC::NPART][4], const Card<R>& cd) {
  double me = 0.0;
  for (int ih = 0; ih < PROC::NSUM; ++ih) {
    cx<R> jamp[PROC::NCOL];
    PROC::template jamps<R>(P, PROC::good(ih), cd, jamp);
    me += double(PROC::template colour_sum<R>(jamp));
  }
  return me * PROC::SCALE;
}

// LDS of the matrix-core colour sum (one region per wave), or nothing.
template <class CT> struct ColourLdsOf { typedef ColourLds<CT> type; };
template <> struct ColourLdsOf<void> { typedef char type; };

// Helicities: the first NSUM of the kept ones, weighted by HELW (for pure QCD
// one of each pair with every helicity reversed, whose |M_h|^2 are equal,
// weight 2; otherwise all of them, weight 1); SCALE = AVERAGE * HELW.
// Waves per event group: the helicity sum of a many-flow process is split
// between the HS waves of a 64 HS-lane workgroup (consecutive blocks of
// helicities, each wave-uniform, added through LDS per card): HS times the
// waves, each HS times shorter, so the last round of waves leaves fewer
// SIMDs idle, and with wave-uniform loop bounds fewer registers spill.
// Few-flow processes keep one lane per event in 256-lane workgroups and the
// one-lane summation order, which their card-per-event and batched kernels
// reproduce bit for bit.  Measured on g g -> t t~ g g with double amplitudes
// and all 64 helicities, 1e6 events: 161.4 ms with one wave, 152.9 ms with two
// (24 spilled registers instead of 54), 155.6 ms with four (56 spilled).
constexpr int kHelSplit = 2;
template <class PROC>
constexpr int hel_split() { return PROC::NCOL >= 8 ? kHelSplit : 1; }
template <class PROC>
constexpr int me_block() { return hel_split<PROC>() > 1 ? 64 * hel_split<PROC>() : kMeBlock; }

// One event per lane (of each wave of the helicity split).  R: amplitude
// precision (float: double precision has kernels of its own).  CT: 16-bit type
// of the matrix-core colour sum (_Float16 or __bf16), or void for the VALU
// form.  GUARD: also the cancellation measure kappa of each event, the largest
// over its cards of sum_hel sum_t m_t |amp_t|^2 / sum_hel sum_c |J_c|^2; events
// with kappa above g.kmax are appended to g.flagged.
template <class PROC, class R, class CT, bool GUARD = false>
__global__ __launch_bounds__(kMeBlock) void me_kernel(const double* __restrict__ soa, int64_t nevt,
                                                      const CardPair* __restrict__ cards, int ncards,
                                                      const double* __restrict__ w_in, double* __restrict__ w_out,
                                                      double* __restrict__ me_out, const GuardArgs g) {
  constexpr bool kMfma = !std::is_void<CT>::value;
  constexpr int HS = hel_split<PROC>(), B = me_block<PROC>();
  constexpr int EPB = HS > 1 ? 64 : B;                        // events per workgroup
  constexpr int NH = PROC::NSUM / HS;                         // helicities per wave
  static_assert(PROC::NSUM % HS == 0 && EPB % 64 == 0, "helicity split");
  static_assert(!GUARD || sizeof(R) == 4, "the guard watches single-precision amplitudes");
  // which helicities: wave-uniform, kept in a scalar register so that the
  // helicity of each loop trip stays uniform too
  const int half = HS > 1 ? __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)) : 0;
  const int64_t r = int64_t(blockIdx.x) * EPB + (HS > 1 ? int(threadIdx.x & 63) : int(threadIdx.x));
  // whole waves (split: whole workgroups) past the end leave together; inside
  // the last wave the lanes past the end recompute the last event (the
  // matrix-core colour sum needs every lane) and write nothing
  if constexpr (HS > 1) {
    if (int64_t(blockIdx.x) * EPB >= nevt) return;
  } else {
    if (int64_t(blockIdx.x) * B + (threadIdx.x & ~63) >= nevt) return;
  }
  const bool valid = r < nevt;
  const int64_t i = valid ? r : nevt - 1;                     // the event of this lane
  double P[PROC::NPART][4];
#pragma unroll
  for (int a = 0; a < PROC::NPART; ++a)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) P[a][mu] = RWGT_AT(soa, int64_t(a * 4 + mu) * nevt + i, PROC::NPART * 4 * nevt);

  [[maybe_unused]] __shared__ typename ColourLdsOf<CT>::type lds_colour[kMfma ? B / 64 : 1];
  [[maybe_unused]] __shared__ double lds_half[HS > 1 ? 64 * (HS - 1) : 1];   // the other waves' partial sums
  [[maybe_unused]] __shared__ double lds_guard[GUARD && HS > 1 ? 2 * 64 * (HS - 1) : 1];
  [[maybe_unused]] std::conditional_t<kMfma, ColourMfma<PROC::NCOL, std::conditional_t<kMfma, CT, _Float16>>, char> cm;
  if constexpr (kMfma) cm.init(PROC::cnum(), lds_colour[threadIdx.x >> 6]);

  double norm = 0.0;
  [[maybe_unused]] double kappa = 0.0;
  for (int k = 0; k < ncards; ++k) {
    const Card<R>& cd = pick<R>(RWGT_AT(cards, k, ncards));
    double me = 0.0;
    [[maybe_unused]] double inco = 0.0, coh = 0.0;
    for (int ih = half * NH; ih < (half + 1) * NH; ++ih) {
      // The generated code reads the momenta through opq() at every use, so
      // none of the helicity-independent algebra is hoisted out of this loop.
      std::conditional_t<GUARD, GuardJamp<R, PROC::NCOL>, cx<R>[PROC::NCOL]> jamp;
      PROC::template jamps<R>(P, PROC::good(ih), cd, jamp);
      if constexpr (kMfma) {
        me += cm.sum(flows(jamp), lds_colour[threadIdx.x >> 6]) * (1.0 / PROC::CDEN);
      } else {
        me += double(PROC::template colour_sum<R>(jamp));
      }
      if constexpr (GUARD) {
        R c2 = R(0);
#pragma unroll
        for (int c = 0; c < PROC::NCOL; ++c) c2 += jamp[c].re * jamp[c].re + jamp[c].im * jamp[c].im;
        coh += double(c2);
        inco += double(jamp.inco);
      }
    }
    if constexpr (HS > 1) {                      // the waves' partial sums in order, on the first wave
      if (half > 0) lds_half[(half - 1) * 64 + (threadIdx.x & 63)] = me;
      if constexpr (GUARD) {
        if (half > 0) {
          lds_guard[(half - 1) * 128 + (threadIdx.x & 63)] = inco;
          lds_guard[(half - 1) * 128 + 64 + (threadIdx.x & 63)] = coh;
        }
      }
      __syncthreads();
      if (half == 0)
        for (int w = 1; w < HS; ++w) me += lds_half[(w - 1) * 64 + threadIdx.x];
      if constexpr (GUARD) {
        if (half == 0)
          for (int w = 1; w < HS; ++w) {
            inco += lds_guard[(w - 1) * 128 + threadIdx.x];
            coh += lds_guard[(w - 1) * 128 + 64 + threadIdx.x];
          }
      }
      __syncthreads();                           // before the next card's partial sums
    }
    if constexpr (GUARD) {
      const double kk = coh > 0.0 ? inco / coh : (inco > 0.0 ? __builtin_inf() : 0.0);
      kappa = kk > kappa || !(kk == kk) ? kk : kappa;
    }
    me *= PROC::SCALE;                           // average (and the reversed helicities)
    if (!valid || half != 0) continue;
    if (me_out) RWGT_AT(me_out, int64_t(k) * nevt + i, int64_t(ncards) * nevt) = me;
    if (w_out) {
      if (k == 0) {
        norm = (me == 0.0 ? 0.0 : 1.0 / me) * RWGT_AT(w_in, i, nevt);
      } else {
        RWGT_AT(w_out, int64_t(k - 1) * nevt + i, int64_t(ncards - 1) * nevt) = norm * me;
      }
    }
  }
  if constexpr (GUARD) {
    if (valid && half == 0) {
      if (g.kappa) RWGT_AT(g.kappa, i, nevt) = kappa;
      if (g.flagged && !(kappa <= g.kmax)) RWGT_AT(g.flagged, atomicAdd(g.nflagged, 1u), nevt) = int32_t(i);
    }
  }
}

static __global__ void zero_count_kernel(unsigned int* c) { *c = 0u; }

// The same with a wave per 64 events and helicity, for launches that one wave
// per half of the helicities leaves unbalanced: at one wave per SIMD 1e5
// g g -> t t~ g g events are 3.05 rounds of 16 helicities, the last nearly
// empty, and 777 events are 26 of 1024 SIMDs.  A wave writes what its helicity
// adds under each card (and, for few waves, a wave per card too); the join
// below adds the helicities up as me_kernel does, so the results are the same
// to the bit.  g g -> t t~ g g, one new card: 777 events 1.57 -> 0.10 ms, 20,011
// 1.73 -> 1.09, 1e5 6.3 -> 5.0, 2e5 11.0 -> 9.9 (1e6 events: 48 ms, nothing to
// gain); u u~ -> e+ e- g, 77,777 events, 3 new cards: 0.27 -> 0.14 ms.
struct MePart { double me; float inco, coh; };    // of one helicity, card and event; all three as evaluated
constexpr int kPartWaves = 4;                     // per workgroup
template <class PROC, class R, class CT, bool GUARD>
__global__ __launch_bounds__(64 * kPartWaves) void me_part_kernel(const double* __restrict__ soa, int64_t nevt,
                                                                  const CardPair* __restrict__ cards, int ncards,
                                                                  int nper, MePart* __restrict__ parts) {
  constexpr bool kMfma = !std::is_void<CT>::value;
  static_assert(sizeof(R) == 4, "the parts hold single-precision sums");
  static_assert(PROC::NSUM % kPartWaves == 0, "whole workgroups");
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int ih0 = (int(blockIdx.y) * kPartWaves + wave) * nper;   // wave-uniform
  const int64_t r = int64_t(blockIdx.x) * 64 + (threadIdx.x & 63);
  const bool valid = r < nevt;                                // lanes past the end: the last event (see me_kernel)
  const int64_t i = valid ? r : nevt - 1;
  double P[PROC::NPART][4];
#pragma unroll
  for (int a = 0; a < PROC::NPART; ++a)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) P[a][mu] = RWGT_AT(soa, int64_t(a * 4 + mu) * nevt + i, PROC::NPART * 4 * nevt);
  [[maybe_unused]] __shared__ typename ColourLdsOf<CT>::type lds_colour[kMfma ? kPartWaves : 1];
  [[maybe_unused]] std::conditional_t<kMfma, ColourMfma<PROC::NCOL, std::conditional_t<kMfma, CT, _Float16>>, char> cm;
  if constexpr (kMfma) cm.init(PROC::cnum(), lds_colour[wave]);
  for (int k = int(blockIdx.z); k < ncards; k += int(gridDim.z)) {
    const Card<R>& cd = pick<R>(RWGT_AT(cards, k, ncards));
    MePart out = {0.0, 0.0f, 0.0f};
    // one trip, as a loop of sums: without it the compiler spills 140 registers
    // (the loop's end keeps what the store needs out of the amplitude code)
    for (int ih = ih0; ih < ih0 + nper; ++ih) {
      std::conditional_t<GUARD, GuardJamp<R, PROC::NCOL>, cx<R>[PROC::NCOL]> jamp;
      PROC::template jamps<R>(P, PROC::good(ih), cd, jamp);
      if constexpr (kMfma) {
        out.me += cm.sum(flows(jamp), lds_colour[wave]);
      } else {
        out.me += double(PROC::template colour_sum<R>(jamp));
      }
      if constexpr (GUARD) {
        R c2 = R(0);
#pragma unroll
        for (int c = 0; c < PROC::NCOL; ++c) c2 += jamp[c].re * jamp[c].re + jamp[c].im * jamp[c].im;
        out.coh += c2;
        out.inco += jamp.inco;
      }
    }
    if (valid)
      RWGT_AT(parts, (int64_t(k) * PROC::NSUM + ih0) * nevt + i, int64_t(ncards) * PROC::NSUM * nevt) = out;
  }
}

// The parts of each event in me_kernel's order: the helicities of each of its
// waves in sequence, then the waves.
template <class PROC, bool MFMA, bool GUARD>
__global__ __launch_bounds__(256) void me_join_kernel(const MePart* __restrict__ parts, int64_t nevt, int ncards,
                                                      const double* __restrict__ w_in, double* __restrict__ w_out,
                                                      double* __restrict__ me_out, const GuardArgs g) {
  constexpr int HS = hel_split<PROC>(), NH = PROC::NSUM / HS;
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= nevt) return;
  double norm = 0.0;
  [[maybe_unused]] double kappa = 0.0;
  for (int k = 0; k < ncards; ++k) {
    double me = 0.0, inco = 0.0, coh = 0.0;
#pragma unroll
    for (int w = 0; w < HS; ++w) {
      double m = 0.0, a = 0.0, c = 0.0;
#pragma unroll 8
      for (int h = w * NH; h < (w + 1) * NH; ++h) {
        const MePart p = RWGT_AT(parts, (int64_t(k) * PROC::NSUM + h) * nevt + i, int64_t(ncards) * PROC::NSUM * nevt);
        m = MFMA ? __builtin_fma(p.me, 1.0 / PROC::CDEN, m) : m + p.me;
        a += double(p.inco);
        c += double(p.coh);
      }
      me = w ? me + m : m;
      inco = w ? inco + a : a;
      coh = w ? coh + c : c;
    }
    if constexpr (GUARD) {
      const double kk = coh > 0.0 ? inco / coh : (inco > 0.0 ? __builtin_inf() : 0.0);
      kappa = kk > kappa || !(kk == kk) ? kk : kappa;
    }
    me *= PROC::SCALE;
    if (me_out) RWGT_AT(me_out, int64_t(k) * nevt + i, int64_t(ncards) * nevt) = me;
    if (w_out) {
      if (k == 0) {
        norm = (me == 0.0 ? 0.0 : 1.0 / me) * RWGT_AT(w_in, i, nevt);
      } else {
        RWGT_AT(w_out, int64_t(k - 1) * nevt + i, int64_t(ncards - 1) * nevt) = norm * me;
      }
    }
  }
  if constexpr (GUARD) {
    if (g.kappa) RWGT_AT(g.kappa, i, nevt) = kappa;
    if (g.flagged && !(kappa <= g.kmax)) RWGT_AT(g.flagged, atomicAdd(g.nflagged, 1u), nevt) = int32_t(i);
  }
}

// Bytes of the parts, 0: me_kernel itself (also where the caller has no such
// workspace).  me_kernel's time goes in rounds of 1024 waves, one per SIMD; the
// parts' with the events, but 4 % (g g -> t t~ g g) to 5.5 % (g g -> t t~ t t~,
// BF16) above full rounds.  So many-flow processes take them while the last
// round leaves more than that idle, up to 10 rounds: one new card, ms with and
// without, 91,750 events (2.8 rounds) 4.60 and 4.73 (g g -> t t~ t t~: 3.02 and
// 3.08), 98,304 (3) 4.90 and 4.74 (3.22 and 3.09), 188,000 to 196,608 events
// (5.7 to 6) 1.00 to 1.04 times as long.
// Few-flow kernels fit several waves on a SIMD: a round adds to the time of one
// (u u~ -> e+ e- g, one new card: 68 us and 34 for each further one), and the
// parts are 10 % above full rounds from the third on: 180,224 events (2.75
// rounds) 133 and 135 us, 196,608 (3) 144 and 135, 229,376 (3.5) 165 and 169,
// 262,144 (4) 188 and 171.  The join is one launch more (6 us), which fewer than
// 16 amplitudes in sequence do not repay (e+ e- -> mu+ mu- under two cards has 8:
// 51 us as it is, 57 split; u u~ -> e+ e- g has 16: 84 and 53).
template <class PROC>
inline size_t me_parts_t(int64_t nevt, int ncards) {
  constexpr bool many = hel_split<PROC>() > 1;
  const int64_t waves = (nevt + 63) / 64 * hel_split<PROC>(), full = (waves + 1023) / 1024 * 1024;
  if (waves > (many ? 10240 : 4096) || (!many && int64_t(PROC::NSUM) * ncards < 16)) return 0;
  if (many ? 19 * waves >= 18 * full : full > 2048 && 11 * waves >= 10 * full) return 0;
  const int64_t each = int64_t(sizeof(MePart)) * PROC::NSUM * nevt;
  return ncards <= kPartBytes / each ? size_t(each * ncards) : 0;
}

template <class PROC, class R, class CT, bool GUARD = false>
inline hipError_t launch_me_t(const double* soa, int64_t nevt, const CardPair* cards, int ncards,
                              const double* w_in, double* w_out, double* me_out, void* parts, hipStream_t s,
                              const GuardArgs& g = GuardArgs{}) {
  if (parts) {
    const int64_t groups = (nevt + 63) / 64;
    const bool by_card = groups * PROC::NSUM < 2048 && ncards <= 65535;   // two waves per SIMD
    hipLaunchKernelGGL((me_part_kernel<PROC, R, CT, GUARD>),
                       dim3(unsigned(groups), unsigned(PROC::NSUM / kPartWaves), unsigned(by_card ? ncards : 1)),
                       dim3(64 * kPartWaves), 0, s, soa,
                       nevt, cards, ncards, 1, static_cast<MePart*>(parts));
    hipLaunchKernelGGL((me_join_kernel<PROC, !std::is_void<CT>::value, GUARD>), dim3(unsigned((nevt + 255) / 256)),
                       dim3(256), 0, s, static_cast<const MePart*>(parts), nevt, ncards, w_in, w_out, me_out, g);
    return hipGetLastError();
  }
  constexpr int B = me_block<PROC>(), EPB = hel_split<PROC>() > 1 ? 64 : B;
  const int64_t blocks = (nevt + EPB - 1) / EPB;
  hipLaunchKernelGGL((me_kernel<PROC, R, CT, GUARD>), dim3(unsigned(blocks)), dim3(B), 0, s, soa, nevt,
                     cards, ncards, w_in, w_out, me_out, g);
  return hipGetLastError();
}

// Mixed precision with the cancellation guard: the float-amplitude kernel
// flags the events whose kappa exceeds g.kmax (g.kmax < 0: none, kappa only).
template <class PROC>
inline hipError_t launch_me_flag_t(int precision, const double* soa, int64_t nevt, const CardPair* cards, int ncards,
                                   const double* w_in, double* w_out, double* me_out, GuardArgs g, void* parts,
                                   hipStream_t s) {
  constexpr bool many = PROC::NCOL >= 8;
  if (g.nflagged) hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(1), 0, s, g.nflagged);
  return precision == kPrecMixedBF16
      ? launch_me_t<PROC, float, std::conditional_t<many, __bf16, void>, true>(soa, nevt, cards, ncards, w_in, w_out,
                                                                               me_out, parts, s, g)
      : launch_me_t<PROC, float, std::conditional_t<many, _Float16, void>, true>(soa, nevt, cards, ncards, w_in,
                                                                                 w_out, me_out, parts, s, g);
}
inline bool reevaluates(const GuardArgs& g) { return !(g.kmax < 0.0) && g.flagged && g.nflagged; }

// Mixed precision: float amplitudes with the colour sum on the matrix cores
// (FP16 or BF16 split) for many-flow processes, on the VALU otherwise.
template <class PROC>
inline hipError_t launch_me_prec(int precision, const double* soa, int64_t nevt, const CardPair* cards, int ncards,
                                 const double* w_in, double* w_out, double* me_out, void* parts, hipStream_t s) {
  constexpr bool many = PROC::NCOL >= 8;
  if (precision == kPrecMixedBF16)
    return launch_me_t<PROC, float, std::conditional_t<many, __bf16, void>>(soa, nevt, cards, ncards, w_in, w_out,
                                                                             me_out, parts, s);
  return launch_me_t<PROC, float, std::conditional_t<many, _Float16, void>>(soa, nevt, cards, ncards, w_in, w_out,
                                                                             me_out, parts, s);
}

}  // namespace rwgt
