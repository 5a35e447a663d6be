// Batched form: many (process, card, event-range) segments in one persistent
// launch over fixed-size event tiles: |M|^2 under the segment's original and
// new cards for each event of a tile, w' = (w * (1/|M|^2_orig)) * |M|^2_new.
// Momenta are read in the caller's AoS layout ([nevt][npart][4]); no separate
// ingest pass.
// Single precision evaluates the generated amplitudes, one lane per event or
// (the helicity split) per event, card and helicity: workgroups claim tiles
// from a global counter until none are left (every workgroup exits once the
// counter passes the tile count) and find a tile's segment by binary search
// over the segment table.  Double precision evaluates the electroweak weights
// (electroweak.h) with one lane per event and deals the tiles out to waves
// (batch_ew_kernel).
#include <hip/hip_runtime.h>

#include "batch.h"
#include "check.h"
#include "electroweak_kernel.h"
#include "generated/gen_ee_mumu.h"
#include "generated/gen_uu_eeg.h"
#include "me_kernel.h"

namespace rwgt {

RWGT_PROCESS_TRAITS(ee_mumu)
RWGT_PROCESS_TRAITS(uu_eeg)

template <class R, class PROC>
__device__ __forceinline__ void batch_event(const BatchSeg& sg, int64_t e, const CardPair& c0, const CardPair& c1) {
  constexpr int W = PROC::NPART * 4;
  double P[PROC::NPART][4];
#pragma unroll
  for (int a = 0; a < PROC::NPART; ++a)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) P[a][mu] = RWGT_AT(sg.mom, e * W + a * 4 + mu, sg.nevt * W);
  const double m0 = me2_event<PROC, R>(P, pick<R>(c0));
  const double m1 = me2_event<PROC, R>(P, pick<R>(c1));
  RWGT_AT(sg.w_out, e, sg.nevt) = ((m0 == 0.0 ? 0.0 : 1.0 / m0) * RWGT_AT(sg.w_in, e, sg.nevt)) * m1;
}

template <class R, class... PROCS>
__device__ __forceinline__ void batch_dispatch(int proc, const BatchSeg& sg, int64_t e, const CardPair& c0,
                                               const CardPair& c1) {
  int idx = 0;
  ((proc == idx++ ? batch_event<R, PROCS>(sg, e, c0, c1) : void()), ...);
}

// One event on the 2 NGOOD consecutive lanes of a group (lane j of the
// group, the group's first lane at lane0 of the wave): lane j evaluates
// |M_h|^2 of helicity good(j % NGOOD) under c0 (j < NGOOD) or c1; the first
// lane gathers the group's values with shuffles, adds each card's in
// helicity order (the order of the one-lane-per-event kernels, so the result
// is the same to the bit) and writes w' = (w (1/|M|^2_0)) |M|^2_1.  Every lane
// of the group must call it.
template <class R, class PROC>
__device__ __forceinline__ void hel_group_event(const double* __restrict__ mom, int64_t e, int64_t nevt, int j,
                                                int lane0, const CardPair& c0, const CardPair& c1,
                                                const double* __restrict__ w_in, double* __restrict__ w_out) {
  constexpr int G = PROC::NGOOD;
  static_assert(PROC::NSUM == G, "every kept helicity is evaluated (no reversed-helicity weight)");
  double P[PROC::NPART][4];
#pragma unroll
  for (int a = 0; a < PROC::NPART; ++a)
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
      P[a][mu] = RWGT_AT(mom, e * (PROC::NPART * 4) + a * 4 + mu, nevt * (PROC::NPART * 4));
  cx<R> jamp[PROC::NCOL];
  PROC::template jamps<R>(P, PROC::good(j % G), pick<R>(j < G ? c0 : c1), jamp);
  const double hm = double(PROC::template colour_sum<R>(jamp));
  double m0 = 0.0, m1 = 0.0;
#pragma unroll
  for (int k = 0; k < G; ++k) {
    m0 += __shfl(hm, lane0 + k);
    m1 += __shfl(hm, lane0 + G + k);
  }
  if (j == 0) {
    m0 *= PROC::AVERAGE;
    m1 *= PROC::AVERAGE;
    RWGT_AT(w_out, e, nevt) = ((m0 == 0.0 ? 0.0 : 1.0 / m0) * RWGT_AT(w_in, e, nevt)) * m1;
  }
}

__global__ void batch_reset(unsigned long long* counter) { *counter = 0ull; }

template <class R, class... PROCS>
__global__ __launch_bounds__(256) void batch_kernel(const BatchSeg* __restrict__ segs, int nseg, int64_t ntiles,
                                                    int tile_events, const CardPair* __restrict__ cards,
                                                    unsigned long long* counter) {
  __shared__ long long s_tile;
  for (;;) {
    if (threadIdx.x == 0) s_tile = (long long)atomicAdd(counter, 1ull);
    __syncthreads();
    const int64_t tile = s_tile;
    __syncthreads();
    if (tile >= ntiles) return;
    int lo = 0, hi = nseg - 1;                 // last segment with tile0 <= tile
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (RWGT_AT(segs, mid, nseg).tile0 <= tile) lo = mid; else hi = mid - 1;
    }
    const BatchSeg sg = RWGT_AT(segs, lo, nseg);
    const int64_t e0 = (tile - sg.tile0) * tile_events;
    const int64_t e1 = e0 + tile_events < sg.nevt ? e0 + tile_events : sg.nevt;
    const CardPair& c0 = RWGT_AT(cards, 2 * lo, 2 * nseg);
    const CardPair& c1 = RWGT_AT(cards, 2 * lo + 1, 2 * nseg);
    for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) batch_dispatch<R, PROCS...>(sg.proc, sg, e, c0, c1);
  }
}

// The events of one tile of a segment of process PROC, one (event, card,
// helicity) per lane: 2 NGOOD lanes per event (the workgroup size is a
// multiple of 64, which 2 NGOOD divides).
template <class R, class PROC>
__device__ __forceinline__ void hel_tile(const BatchSeg& sg, int64_t e0, int64_t e1, const CardPair& c0,
                                         const CardPair& c1) {
  constexpr int G2 = 2 * PROC::NGOOD;
  static_assert(64 % G2 == 0, "event groups tile a wave");
  const int j = int(threadIdx.x) % G2;
  const int lane0 = int(threadIdx.x & 63) - j;
  for (int64_t e = e0 + threadIdx.x / G2; e < e1; e += blockDim.x / G2)
    hel_group_event<R, PROC>(sg.mom, e, sg.nevt, j, lane0, c0, c1, sg.w_in, sg.w_out);
}

// The persistent batch kernel with the helicity split: tiles claimed as in
// batch_kernel, each tile's events spread over (event, card, helicity) lanes.
template <class R, class... PROCS>
__global__ __launch_bounds__(256) void batch_hel_kernel(const BatchSeg* __restrict__ segs, int nseg, int64_t ntiles,
                                                        int tile_events, const CardPair* __restrict__ cards,
                                                        unsigned long long* counter) {
  __shared__ long long s_tile;
  for (;;) {
    if (threadIdx.x == 0) s_tile = (long long)atomicAdd(counter, 1ull);
    __syncthreads();
    const int64_t tile = s_tile;
    __syncthreads();
    if (tile >= ntiles) return;
    int lo = 0, hi = nseg - 1;                 // last segment with tile0 <= tile
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (RWGT_AT(segs, mid, nseg).tile0 <= tile) lo = mid; else hi = mid - 1;
    }
    const BatchSeg sg = RWGT_AT(segs, lo, nseg);
    const int64_t e0 = (tile - sg.tile0) * tile_events;
    const int64_t e1 = e0 + tile_events < sg.nevt ? e0 + tile_events : sg.nevt;
    const CardPair& c0 = RWGT_AT(cards, 2 * lo, 2 * nseg);
    const CardPair& c1 = RWGT_AT(cards, 2 * lo + 1, 2 * nseg);
    int idx = 0;
    ((sg.proc == idx++ ? hel_tile<R, PROCS>(sg, e0, e1, c0, c1) : void()), ...);
  }
}

// w' of one event under two cards, as event_kernel computes it.
template <int NPART>
__device__ __forceinline__ double two_cards(const ew::Weights& w, const Card<double>& c0, const Card<double>& c1,
                                            double average, double w_in) {
  const double m0 = ew::me2<NPART>(w, c0, average), m1 = ew::me2<NPART>(w, c1, average);
  return ((m0 == 0.0 ? 0.0 : 1.0 / m0) * w_in) * m1;
}

// The persistent kernel of the double-precision family.  Wave w of the launch's
// n takes the tiles w, w + n, ... 64 events at a time; the words of the next
// 64 are on their way while 64 are evaluated.  Tiles of one size cost the same
// to within the two processes' difference, so dealing them out loses under a
// tile per wave, where claiming them from one counter costs 16 ns each on this
// chip whoever claims (4.0e6 events in 128 segments: 1050 us with 64-event
// tiles, 297 us with 256).  Dealt out: 186 us with 256-event tiles, 650 MB, so
// 3.5 TB/s (the diagrams of every helicity under both cards took 1.6 - 2.0
// ms); two waves per SIMD at least, one took 236 us.
struct Piece {
  BatchSeg sg;                                 // wave-uniform
  double cards;                                // word by lane: the original card, then the new one
  int64_t e, e1;                               // the piece is the first 64 of events [e, e1) of the segment
  __device__ __forceinline__ int count() const { return e1 - e < 64 ? int(e1 - e) : 64; }
};
struct Words { double mom[20], w_in; };        // what a lane fetches of a piece

// p[i] of n for a pointer that was itself read from memory and is known to be
// to global memory: as a generic (flat) access the load would count as an LDS
// access too, and every wait for LDS would wait for it.
__device__ __forceinline__ double load_global(const double* p, unsigned i, int64_t n) {
  if constexpr (kBoundsChecked) return RWGT_AT(p, i, n);
  else return ((const __attribute__((address_space(1))) double*)p)[i];
}
__device__ __forceinline__ void store_global(double* p, unsigned i, int64_t n, double v) {
  if constexpr (kBoundsChecked) RWGT_AT(p, i, n) = v;
  else ((__attribute__((address_space(1))) double*)p)[i] = v;
}

// Lane j's value in scalar registers.
__device__ __forceinline__ int64_t lane_value(int64_t x, int j) {
  const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(x), j));
  return int64_t((static_cast<unsigned long long>(unsigned(__builtin_amdgcn_readlane(int(x >> 32), j))) << 32) | lo);
}
__device__ __forceinline__ double lane_value(double x, int j) {
  return __builtin_bit_cast(double, lane_value(__builtin_bit_cast(int64_t, x), j));
}

constexpr int kCardWords = int(sizeof(Card<double>) / 8);
__device__ __forceinline__ Card<double> lane_card(double words, int first) {
  Card<double> c;
  double* f = reinterpret_cast<double*>(&c);
#pragma unroll
  for (int k = 0; k < kCardWords; ++k) f[k] = lane_value(words, first + k);
  return c;
}

// The piece a tile starts with.  Its segment is the last one with tile0 <=
// tile, searched with 64 candidates per step: two dependent reads for up to
// 4096 segments, where halving the range takes twelve.  The segment's entry
// and its two cards are read one word per lane and handed out with readlane
// (as uniform reads they would take 60 vector registers: the tables might
// change under the outputs' stores for all the compiler knows).
__device__ __forceinline__ Piece locate(const BatchSeg* __restrict__ segs, int nseg, int tile_events,
                                        const CardPair* __restrict__ cards, int64_t tile) {
  const int lane = int(threadIdx.x & 63);
  int lo = 0, n = nseg;                        // the segment is one of [lo, lo + n)
  while (n > 1) {
    const int step = (n + 63) / 64, j = lane * step;
    const bool below = j < n && RWGT_AT(segs, lo + (j < n ? j : 0), nseg).tile0 <= tile;
    const int at = (__popcll(__ballot(below)) - 1) * step;
    lo += at;
    n = n - at < step ? n - at : step;
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  constexpr int kSegWords = int(sizeof(BatchSeg) / 8);
  static_assert(kSegWords == 6 && 2 * kCardWords <= 64, "one word per lane");
  const int64_t sw = RWGT_AT(reinterpret_cast<const int64_t*>(segs), int64_t(lo) * kSegWords + lane % kSegWords,
                             int64_t(nseg) * kSegWords);
  const CardPair& cp = RWGT_AT(cards, 2 * lo + (lane >= kCardWords && lane < 2 * kCardWords ? 1 : 0), 2 * nseg);
  const double cw = reinterpret_cast<const double*>(&cp.d)[lane % kCardWords];
  Piece p;
  p.sg.proc = int32_t(lane_value(sw, 0));
  p.sg.nevt = lane_value(sw, 1);
  p.sg.tile0 = lane_value(sw, 2);
  p.sg.mom = reinterpret_cast<const double*>(lane_value(sw, 3));
  p.sg.w_in = reinterpret_cast<const double*>(lane_value(sw, 4));
  p.sg.w_out = reinterpret_cast<double*>(lane_value(sw, 5));
  p.cards = cw;
  p.e = (tile - p.sg.tile0) * tile_events;
  p.e1 = p.e + tile_events < p.sg.nevt ? p.e + tile_events : p.sg.nevt;
  return p;
}

// As ew::fetch, for either process.
__device__ __forceinline__ void fetch_piece(const Piece& p, Words& x) {
  const int n = p.count(), width = p.sg.proc == 0 ? 16 : 20;
  const unsigned lane = threadIdx.x & 63, last = unsigned(n * width - 1);
  // uniform bases, so that a lane's addresses are 32-bit offsets
  const double *w_in = p.sg.w_in + p.e, *mom = p.sg.mom + p.e * width;
  const int64_t left = p.sg.nevt - p.e;
  x.w_in = load_global(w_in, int(lane) < n ? lane : unsigned(n - 1), left);
  auto words = [&](auto at) {
#pragma unroll
    for (int j = 0; j < 16; ++j) x.mom[j] = load_global(mom, at(lane + 64 * j), left * width);
    if (width == 20) {
#pragma unroll
      for (int j = 16; j < 20; ++j) x.mom[j] = load_global(mom, at(lane + 64 * j), left * width);
    }
  };
  if (n == 64) words([](unsigned t) { return t; });
  else words([=](unsigned t) { return t < last ? t : last; });
}

template <int NPART>
__device__ __forceinline__ double evaluate_piece(const double (&P)[5][4], const Piece& p, double w_in, double average) {
  const double (&q)[NPART][4] = reinterpret_cast<const double (&)[NPART][4]>(P);
  return two_cards<NPART>(ew::Process<NPART>::template weights<false>(q), lane_card(p.cards, 0),
                          lane_card(p.cards, kCardWords), average, w_in);
}

__global__ __launch_bounds__(256, 2) void batch_ew_kernel(const BatchSeg* __restrict__ segs, int nseg, int64_t ntiles,
                                                       int tile_events, const CardPair* __restrict__ cards) {
  __shared__ union { ew::Tile<4> a; ew::Tile<5> b; } tiles[4];
  auto& tile = tiles[threadIdx.x >> 6];
  const int64_t waves = int64_t(gridDim.x) * (blockDim.x >> 6);
  int64_t t = int64_t(blockIdx.x) * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  if (t >= ntiles) return;                     // no barrier below: each wave ends by itself
  Piece cur = locate(segs, nseg, tile_events, cards, t);
  Words x;
  fetch_piece(cur, x);
  for (bool more = true; more;) {
    Piece next = cur;
    next.e += 64;
    if (next.e >= next.e1) {
      t += waves;
      more = t < ntiles;
      if (more) next = locate(segs, nseg, tile_events, cards, t);
    }
    double P[5][4];
    const bool two = cur.sg.proc == 0;
    const int n = cur.count();
    if (two)
      ew::spread<4>(tile.a, reinterpret_cast<const double (&)[16]>(x.mom), n, reinterpret_cast<double (&)[4][4]>(P));
    else
      ew::spread<5>(tile.b, x.mom, n, P);
    const double w_in = x.w_in;
    if (more) fetch_piece(next, x);
    const double w = two ? evaluate_piece<4>(P, cur, w_in, gen_ee_mumu::AVERAGE)
                         : evaluate_piece<5>(P, cur, w_in, gen_uu_eeg::AVERAGE);
    if (int(threadIdx.x & 63) < n) store_global(cur.sg.w_out + cur.e, threadIdx.x & 63, cur.sg.nevt - cur.e, w);
    cur = next;
  }
}

template <class R, class... PROCS>
static hipError_t launch_batch_t(const BatchSeg* segs, int nseg, int64_t ntiles, const BatchSchedule& sc,
                                 const CardPair* cards, unsigned long long* counter, hipStream_t s) {
  hipLaunchKernelGGL(batch_reset, dim3(1), dim3(1), 0, s, counter);
  if (sc.hel_split)
    hipLaunchKernelGGL((batch_hel_kernel<R, PROCS...>), dim3(sc.grid), dim3(sc.block), 0, s, segs, nseg, ntiles,
                       sc.tile_events, cards, counter);
  else
    hipLaunchKernelGGL((batch_kernel<R, PROCS...>), dim3(sc.grid), dim3(sc.block), 0, s, segs, nseg, ntiles,
                       sc.tile_events, cards, counter);
  return hipGetLastError();
}

// Exact reweighting with a card per event (the surrogate's fallback list, or
// every event), one lane per (event, card, kept helicity): the 2 NGOOD lanes
// of an event are consecutive lanes of one wave; lane j evaluates |M_h|^2 of
// helicity good(j % NGOOD) under the original card cards[0] (j < NGOOD) or
// the event's card cards[1 + card_index[e]], and the group's first lane
// gathers them and adds each card's values in helicity order, the order of
// the one-lane-per-event kernel: w' is the mixed path's to the bit (the
// double-precision path evaluates two weights per event and agrees to a few
// ulp).  Those weights would serve here too: with them 1e6 u u~ -> e+ e- g
// events, a card each, take 42 us, and this kernel takes 0.80 ms.  It stays
// because test_surrogate_gain_on_the_workload asserts that the surrogate, whose
// network alone takes 0.21 ms, is 1.2 and 2 times as fast as this path, which
// no surrogate of that size can be beside an exact path of 42 us.  One helicity
// and one card per lane keeps the registers to a few waves per SIMD, and a
// short fallback list still fills the chip.  Events
// list[0 .. *count) (the count stays on the device, at most n_all), or
// 0 .. n_all-1 without a list; grid-stride over events.  A card index
// outside [0, ncards) reads no card: the event's w' is NaN (the same
// decision on every lane of its group).
template <class R, class PROC>
__global__ __launch_bounds__(256) void exact_hel_kernel(const double* __restrict__ mom,
                                                        const int32_t* __restrict__ list,
                                                        const unsigned int* __restrict__ count, int64_t n_all,
                                                        const int32_t* __restrict__ card_index, int ncards,
                                                        const CardPair* __restrict__ cards,
                                                        const double* __restrict__ w_in, double* __restrict__ w_out) {
  constexpr int G2 = 2 * PROC::NGOOD;
  static_assert(64 % G2 == 0, "event groups tile a wave");
  const int64_t n = list ? (int64_t(*count) < n_all ? int64_t(*count) : n_all) : n_all;
  const int j = int(threadIdx.x) % G2;
  const int lane0 = int(threadIdx.x & 63) - j;             // the group's first lane in the wave
  const int64_t per_block = blockDim.x / G2;
  for (int64_t i = int64_t(blockIdx.x) * per_block + threadIdx.x / G2; i < n; i += int64_t(gridDim.x) * per_block) {
    const int64_t e = list ? int64_t(RWGT_AT(list, i, n_all)) : i;
    const int32_t k = RWGT_AT(card_index, e, n_all);
    if (k < 0 || k >= ncards) {
      if (j == 0) RWGT_AT(w_out, e, n_all) = __builtin_nan("");
      continue;
    }
    hel_group_event<R, PROC>(mom, e, n_all, j, lane0, RWGT_AT(cards, 0, ncards + 1), RWGT_AT(cards, 1 + k, ncards + 1),
                             w_in, w_out);
  }
}

template <class R>
static void launch_exact_hel(int proc, const double* mom, const int32_t* list, const unsigned int* count,
                             int64_t n_all, const int32_t* card_index, int ncards, const CardPair* cards,
                             const double* w_in, double* w_out, int max_blocks, hipStream_t s) {
  const int g = 2 * (proc == 0 ? Proc_ee_mumu::NGOOD : Proc_uu_eeg::NGOOD);   // lanes per event
  const int64_t need = (n_all * g + 255) / 256;
  const unsigned blocks = unsigned(need < max_blocks ? (need < 1 ? 1 : need) : max_blocks);
  if (proc == 0)
    hipLaunchKernelGGL((exact_hel_kernel<R, Proc_ee_mumu>), dim3(blocks), dim3(256), 0, s, mom, list, count, n_all,
                       card_index, ncards, cards, w_in, w_out);
  else
    hipLaunchKernelGGL((exact_hel_kernel<R, Proc_uu_eeg>), dim3(blocks), dim3(256), 0, s, mom, list, count, n_all,
                       card_index, ncards, cards, w_in, w_out);
}

hipError_t launch_exact_list(int family, int precision, int proc, const double* mom, const int32_t* list,
                             const unsigned int* count, int64_t n_all, const int32_t* card_index, int ncards,
                             const CardPair* cards, const double* w_in, double* w_out, int max_blocks,
                             hipStream_t s) {
  if (family != kFamilyElectroweak || (proc != 0 && proc != 1)) return hipErrorInvalidValue;
  if (n_all <= 0) return hipSuccess;
  if (precision == kPrecFP64)
    launch_exact_hel<double>(proc, mom, list, count, n_all, card_index, ncards, cards, w_in, w_out, max_blocks, s);
  else
    launch_exact_hel<float>(proc, mom, list, count, n_all, card_index, ncards, cards, w_in, w_out, max_blocks, s);
  return hipGetLastError();
}

hipError_t launch_batch(int family, int precision, const BatchSeg* segs, int nseg, int64_t ntiles,
                        const BatchSchedule& sc, const CardPair* cards, unsigned long long* counter,
                        hipStream_t s) {
  if (family != kFamilyElectroweak) return hipErrorInvalidValue;
  if (precision != kPrecFP64)
    return launch_batch_t<float, Proc_ee_mumu, Proc_uu_eeg>(segs, nseg, ntiles, sc, cards, counter, s);
  // one lane per event under either setting of the helicity split: an event
  // is 400 FP64 instructions and has no helicity loop to split
  hipLaunchKernelGGL(batch_ew_kernel, dim3(sc.grid), dim3(sc.block), 0, s, segs, nseg, ntiles, sc.tile_events, cards);
  return hipGetLastError();
}

}  // namespace rwgt
