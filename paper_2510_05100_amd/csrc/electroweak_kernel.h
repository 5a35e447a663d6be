// Kernels of the electroweak weights (electroweak.h), one event per lane.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "card_source.h"
#include "check.h"
#include "electroweak.h"
#include "kernels.h"

namespace rwgt {
namespace ew {

// LDS tile of a wave: 64 events of the caller's layout [event][NPART][4].  The
// rows are read 16 bytes at a time, eight lanes to an LDS cycle: rows of 160
// bytes start in different quarters of the banks by themselves, rows of 128
// bytes are padded to 144.
template <int NPART> struct Tile {
  static constexpr int W = NPART * 4, kRow = W % 16 == 0 ? W + 2 : W;
  alignas(16) double p[64 * kRow];
};

// The words of a tile of nloc events starting at e0, lane by lane: 512
// consecutive bytes per wave and load.  (A lane reading its own 128 - 160
// byte row directly touches 64 lines per load and leans on the L1 to keep
// them.)
template <int NPART>
__device__ __forceinline__ void fetch(const double* __restrict__ mom, int64_t e0, int nloc, int64_t nevt,
                                      double (&raw)[NPART * 4]) {
  constexpr int W = NPART * 4;
  const unsigned lane = threadIdx.x & 63, last = unsigned(nloc * W - 1);
  const double* base = mom + e0 * W;             // uniform: the lanes' addresses are 32-bit offsets
  const int64_t left = (nevt - e0) * W;
  if (nloc == 64) {
#pragma unroll
    for (int j = 0; j < W; ++j) raw[j] = RWGT_AT(base, lane + 64 * j, left);
  } else {                                       // past the last event: its last word again
#pragma unroll
    for (int j = 0; j < W; ++j) raw[j] = RWGT_AT(base, lane + 64 * j < last ? lane + 64 * j : last, left);
  }
}
// Hands the words to the lanes: the momenta of this lane's event (past the
// last event: of the last).
template <int NPART>
__device__ __forceinline__ void spread(Tile<NPART>& tile, const double (&raw)[NPART * 4], int nloc,
                                       double (&P)[NPART][4]) {
  constexpr int W = NPART * 4;
  const int lane = int(threadIdx.x) & 63;
  constexpr int R = Tile<NPART>::kRow;
  typedef double v2 __attribute__((ext_vector_type(2)));
  wave_sync();                                   // the tile's previous rows have been read
  const int at = R == W ? lane : lane + (R - W) * (lane / W);
  static_assert(R == W || 64 % W == 0, "64 words are whole rows where rows are padded");
#pragma unroll
  for (int j = 0; j < W; ++j) tile.p[at + j * (R == W ? 64 : 64 / W * R)] = raw[j];
  wave_sync();
  const v2* row = reinterpret_cast<const v2*>(&tile.p[(lane < nloc ? lane : nloc - 1) * R]);
#pragma unroll
  for (int k = 0; k < W / 2; ++k) {
    const v2 x = row[k];
    P[k / 2][k % 2 * 2] = x.x;
    P[k / 2][k % 2 * 2 + 1] = x.y;
  }
}

template <int NPART>
__device__ __forceinline__ void load_event(const double* __restrict__ mom, int64_t e, int64_t nevt,
                                           double (&P)[NPART][4]) {
#pragma unroll
  for (int a = 0; a < NPART; ++a)
#pragma unroll
    for (int m = 0; m < 4; ++m) P[a][m] = RWGT_AT(mom, (e * NPART + a) * 4 + m, nevt * NPART * 4);
}

// Every card of event i: |M|^2 and / or w' (card 0 is then the original).
// Returns the number of non-finite w' (without w_out: |M|^2).
template <class CARDS>
__device__ __forceinline__ int all_cards(const Weights& w, const CARDS& cards, int ncards, int64_t i, int64_t nevt,
                                         double w_in, double* __restrict__ w_out, double* __restrict__ me_out) {
  double norm = 0.0;
  int bad = 0;
  for (int k = 0; k < ncards; ++k) {
    const double me = me2(w, cards(k));
    if (me_out) RWGT_AT(me_out, int64_t(k) * nevt + i, int64_t(ncards) * nevt) = me;
    if (w_out) {
      if (k == 0) {
        norm = (me == 0.0 ? 0.0 : 1.0 / me) * w_in;
      } else {
        const double wk = norm * me;
        RWGT_AT(w_out, int64_t(k - 1) * nevt + i, int64_t(ncards - 1) * nevt) = wk;
        bad += isfinite(wk) ? 0 : 1;
      }
    } else {
      bad += isfinite(me) ? 0 : 1;
    }
  }
  return bad;
}

// All events, straight from the caller's momenta (no ingest pass), one wave
// per workgroup striding over tiles of 64.  The next tile's words are on
// their way while a tile is evaluated.  Bound by the vector ALUs (833
// instructions per tile and card pair, issuing in 73 % of the cycles) about
// as much as by memory (10.8 KB per tile).  1e6 u u~ -> e+ e- g events, one new
// card: 45 us, 3.9 TB/s (ingest 52 us and the diagrams of 8 helicities under
// both cards 640 us before; 65 us without the prefetch).
// PRODUCT: see pair_mass.
template <int NPART, bool PRODUCT, class CARDS>
__global__ __launch_bounds__(64) void event_kernel(const double* __restrict__ mom, int64_t nevt, const CARDS cards,
                                                   int ncards, const double* __restrict__ w_in,
                                                   double* __restrict__ w_out, double* __restrict__ me_out,
                                                   unsigned long long* __restrict__ nonfinite) {
  __shared__ Tile<NPART> tile;
  const int lane = int(threadIdx.x);
  const int64_t stride = int64_t(gridDim.x) * 64;
  int64_t e0 = int64_t(blockIdx.x) * 64;
  if (e0 >= nevt) return;
  double raw[NPART * 4], w_next;
  auto fetch_tile = [&](int64_t first) {
    const int n = nevt - first < 64 ? int(nevt - first) : 64;
    w_next = w_out ? RWGT_AT(w_in, first + (lane < n ? lane : n - 1), nevt) : 0.0;
    fetch<NPART>(mom, first, n, nevt, raw);
  };
  int bad = 0;
  fetch_tile(e0);
  for (;;) {
    const int nloc = nevt - e0 < 64 ? int(nevt - e0) : 64;
    const int64_t next = e0 + stride;
    double P[NPART][4];
    spread<NPART>(tile, raw, nloc, P);
    const double weight = w_next;
    if (next < nevt) fetch_tile(next);
    const Weights w = Process<NPART>::template weights<PRODUCT>(P);
    if (lane < nloc) bad += all_cards(w, cards, ncards, e0 + lane, nevt, weight, w_out, me_out);
    if (next >= nevt) break;
    e0 = next;
  }
  if (nonfinite) {
    for (int d = 32; d > 0; d >>= 1) bad += __shfl_xor(bad, d);
    if (lane == 0) RWGT_AT(nonfinite, blockIdx.x, gridDim.x) = static_cast<unsigned long long>(bad);
  }
}

template <int NPART> struct PairCards {          // the mixed path's cards
  const CardPair* p;
  int n;
  double average;
  __device__ __forceinline__ Couplings operator()(int k) const { return couplings<NPART>(RWGT_AT(p, k, n).d, average); }
};

// The events rows[0 .. *nrows) (the mixed path's flagged ones).
template <int NPART>
__global__ __launch_bounds__(64) void listed_kernel(const double* __restrict__ mom, int64_t nevt,
                                                    const CardPair* __restrict__ cards, int ncards, double average,
                                                    const double* __restrict__ w_in, double* __restrict__ w_out,
                                                    double* __restrict__ me_out, const int32_t* __restrict__ rows,
                                                    const unsigned int* __restrict__ nrows) {
  const int64_t n = int64_t(*nrows);
  for (int64_t r = int64_t(blockIdx.x) * 64 + threadIdx.x; r < n; r += int64_t(gridDim.x) * 64) {
    const int64_t i = int64_t(RWGT_AT(rows, r, nevt));
    double P[NPART][4];
    load_event<NPART>(mom, i, nevt, P);
    all_cards(Process<NPART>::template weights<false>(P), PairCards<NPART>{cards, ncards, average}, ncards, i, nevt,
              w_out ? RWGT_AT(w_in, i, nevt) : 0.0, w_out, me_out);
  }
}

template <int NPART>
inline size_t table(const CardPair* cards, int n, double average, void* out) {
  return card_table<Couplings>(cards, n, out, [=](const Card<double>& c) { return couplings<NPART>(c, average); });
}

// A compute unit's LDS holds 14 (five particles) or 18 of event_kernel's
// waves; with 12 per unit the tiles are dealt evenly.
template <int NPART>
inline hipError_t launch(const Fp64Call& a, double average, hipStream_t s) {
  constexpr int64_t kWaves = 12 * 256;
  static_assert(kWaves <= kNonfiniteBlocks, "every workgroup has a count");
  const int64_t tiles = (a.nevt + 63) / 64, rounds = (tiles + kWaves - 1) / kWaves;
  const int64_t blocks = (tiles + rounds - 1) / rounds;
  if (a.counts) *a.counts = a.nonfinite ? int(blocks) : 0;
  auto of = [=](const Card<double>& c) { return couplings<NPART>(c, average); };
  return with_cards<Couplings>(a, of, [&](const auto& cards) {
    typedef std::remove_cv_t<std::remove_reference_t<decltype(cards)>> Cards;
    const auto kernel = a.scan ? event_kernel<NPART, true, Cards> : event_kernel<NPART, false, Cards>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(64), 0, s, a.mom, a.nevt, cards, a.ncards, a.w_in, a.w_out,
                       a.me_out, a.nonfinite);
    return hipGetLastError();
  });
}

template <int NPART>
inline hipError_t launch_rows(const double* mom, int64_t nevt, const CardPair* cards, int ncards, double average,
                              const double* w_in, double* w_out, double* me_out, const int32_t* rows,
                              const unsigned int* nrows, hipStream_t s) {
  const int64_t tiles = (nevt + 63) / 64;
  hipLaunchKernelGGL(listed_kernel<NPART>, dim3(unsigned(tiles < 1024 ? tiles : 1024)), dim3(64), 0, s, mom, nevt,
                     cards, ncards, average, w_in, w_out, me_out, rows, nrows);
  return hipGetLastError();
}

}  // namespace ew
}  // namespace rwgt
