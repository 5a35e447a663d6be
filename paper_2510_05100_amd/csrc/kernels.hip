// Device kernels of the reweighting path (gfx950, wave64):
//   ingest_kernel  AoS [nevt][npart][4] -> SoA [npart*4][nevt] through LDS
//   launch_fp64,   dispatch to the per-process matrix-element kernels
//   launch_me      (electroweak_kernel.h, ordered_kernel.h; me_kernel.h)
//   xsec_*         reweighted cross sections and errors per card
//   factored       coupling-factored reweighting of many cards
#include <hip/hip_runtime.h>

#include <cstdint>

#include "card_source.h"
#include "check.h"
#include "kernels.h"

namespace rwgt {

constexpr int kIngestEvents = 64;

// One block moves kIngestEvents events: a coalesced read of their contiguous
// AoS rows into LDS, then one coalesced row write per SoA component.
template <int NPART>
__global__ __launch_bounds__(256) void ingest_kernel(const double* __restrict__ aos, double* __restrict__ soa,
                                                     int64_t nevt) {
  constexpr int W = NPART * 4;
  __shared__ double tile[kIngestEvents][W + 1];
  const int64_t e0 = int64_t(blockIdx.x) * kIngestEvents;
  const int64_t nloc = (nevt - e0) < kIngestEvents ? (nevt - e0) : kIngestEvents;
  for (int t = threadIdx.x; t < nloc * W; t += blockDim.x) tile[t / W][t % W] = RWGT_AT(aos, e0 * W + t, nevt * W);
  __syncthreads();
  for (int t = threadIdx.x; t < kIngestEvents * W; t += blockDim.x) {
    const int c = t / kIngestEvents, e = t % kIngestEvents;
    if (e < nloc) RWGT_AT(soa, int64_t(c) * nevt + e0 + e, nevt * W) = tile[e][c];
  }
}

// Reweighted cross sections (teaRex section): per card
//   sigma' = C S1,  dsigma' = dsigma R/N + sigma std(w'),  std = sqrt(S2/N),
// S1 = sum w', R = sum w'/w (terms with w = 0 count 0), S2 = sum (w' - S1/N)^2,
// and, when dsigma' is infinite, NaN or not positive, dsigma' = dsigma max(sigma'/sigma, sigma/sigma').
// One pass over w': a block takes 2048 weights of a card into registers, sums
// them, sums the squares about their own mean, and merges such pieces with
// their means' distance (Chan, Golub, LeVeque, Am. Stat. 37 (1983) 242), which
// keeps the variance of near-constant w' (a pure alpha_s change) where
// S2/N - m^2 would cancel to noise of order 1e-16 m^2.  Every order is fixed,
// so results are deterministic.  Bound by reading w': 64 cards x 200,003
// weights (102 MB) in 29 us, where a pass for the sums and one about the mean,
// each with one lane per card adding the block partials, took 175 us.
constexpr int kXsecBlock = 256, kXsecEach = 8, kXsecChunk = kXsecBlock * kXsecEach;

// The sum over the workgroup, on every lane: each wave by a butterfly, then the
// waves in order.
__device__ __forceinline__ double block_sum(double v, double (&sh)[kXsecBlock / 64]) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
  __syncthreads();                               // sh has been read
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = sh[0];
#pragma unroll
  for (int w = 1; w < kXsecBlock / 64; ++w) s += sh[w];
  return s;
}

// Block b of a card's nb takes its chunks b, b + nb, ...: part[k][b] = {S1, R, S2 about their mean}.
__global__ __launch_bounds__(kXsecBlock) void xsec_sums(const double* __restrict__ w_in,
                                                        const double* __restrict__ w_out, int64_t nevt,
                                                        double* __restrict__ part) {
  __shared__ double sh[kXsecBlock / 64];
  const int k = blockIdx.y;
  const int64_t nw = int64_t(gridDim.y) * nevt;            // w_out: [nsets][nevt], nsets = gridDim.y
  double s1 = 0.0, s2 = 0.0, r = 0.0, n = 0.0;
  for (int64_t c = int64_t(blockIdx.x) * kXsecChunk; c < nevt; c += int64_t(gridDim.x) * kXsecChunk) {
    double x[kXsecEach], wi[kXsecEach], s = 0.0, q = 0.0;
#pragma unroll
    for (int j = 0; j < kXsecEach; ++j) {
      const int64_t i = c + j * kXsecBlock + threadIdx.x;
      x[j] = i < nevt ? RWGT_AT(w_out, int64_t(k) * nevt + i, nw) : 0.0;
      wi[j] = i < nevt ? RWGT_AT(w_in, i, nevt) : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kXsecEach; ++j) {
      s += x[j];
      r += wi[j] != 0.0 ? x[j] / wi[j] : 0.0;
    }
    s = block_sum(s, sh);
    const double nc = double(nevt - c < kXsecChunk ? nevt - c : kXsecChunk), mean = s / nc;
#pragma unroll
    for (int j = 0; j < kXsecEach; ++j) {
      const double d = c + j * kXsecBlock + threadIdx.x < nevt ? x[j] - mean : 0.0;
      q += d * d;
    }
    q = block_sum(q, sh);
    if (n > 0.0) {
      const double d = mean - s1 / n;
      q += d * d * (n * nc / (n + nc));
    }
    s1 += s;
    s2 += q;
    n += nc;
  }
  r = block_sum(r, sh);
  if (threadIdx.x == 0) {
    const int64_t at = (int64_t(k) * gridDim.x + blockIdx.x) * 3, np = int64_t(gridDim.y) * gridDim.x * 3;
    RWGT_AT(part, at, np) = s1;
    RWGT_AT(part, at + 1, np) = r;
    RWGT_AT(part, at + 2, np) = s2;
  }
}

// One workgroup per card merges its nb blocks.
__global__ __launch_bounds__(kXsecBlock) void xsec_final(const double* __restrict__ part, int nb, int64_t nevt,
                                                         int nsets, double sigma, double dsigma, double norm,
                                                         double* __restrict__ out) {
  __shared__ double sh[kXsecBlock / 64];
  const int k = blockIdx.x;
  const int64_t chunks = (nevt + kXsecChunk - 1) / kXsecChunk, np = int64_t(nsets) * nb * 3;
  double s1 = 0.0, r = 0.0, s2 = 0.0;
  for (int b = threadIdx.x; b < nb; b += kXsecBlock) {
    s1 += RWGT_AT(part, (int64_t(k) * nb + b) * 3, np);
    r += RWGT_AT(part, (int64_t(k) * nb + b) * 3 + 1, np);
  }
  s1 = block_sum(s1, sh);
  r = block_sum(r, sh);
  const double n = double(nevt), mean = s1 / n;
  for (int b = threadIdx.x; b < nb; b += kXsecBlock) {     // the block's weights: whole chunks, the last one cut
    const int64_t mine = (chunks - b + nb - 1) / nb, cut = (chunks - 1) % nb == b ? chunks * kXsecChunk - nevt : 0;
    const double m = double(mine * kXsecChunk - cut), d = RWGT_AT(part, (int64_t(k) * nb + b) * 3, np) / m - mean;
    s2 += RWGT_AT(part, (int64_t(k) * nb + b) * 3 + 2, np) + d * d * m;
  }
  s2 = block_sum(s2, sh);
  if (threadIdx.x != 0) return;
  const double xs = norm * s1;
  double err = dsigma * (r / n) + sigma * sqrt(s2 / n);
  double fallback = 0.0;
  if (!(err > 0.0) || isinf(err)) {
    const double a = xs / sigma, b = sigma / xs;
    err = dsigma * (a > b ? a : b);
    fallback = 1.0;
  }
  RWGT_AT(out, k * 3 + 0, nsets * 3) = xs;
  RWGT_AT(out, k * 3 + 1, nsets * 3) = err;
  RWGT_AT(out, k * 3 + 2, nsets * 3) = fallback;
}

// Blocks per card: one per chunk, up to nblocks.
int xsec_blocks(int64_t nevt, int nblocks) {
  const int64_t chunks = (nevt + kXsecChunk - 1) / kXsecChunk;
  return int(chunks < nblocks ? chunks : nblocks);
}

hipError_t launch_xsec(const double* w_in, const double* w_out, int64_t nevt, int nsets, double sigma, double dsigma,
                       double norm, double* part, int nblocks, double* out, hipStream_t s) {
  const int nb = xsec_blocks(nevt, nblocks);
  hipLaunchKernelGGL(xsec_sums, dim3(nb, nsets), dim3(kXsecBlock), 0, s, w_in, w_out, nevt, part);
  hipLaunchKernelGGL(xsec_final, dim3(nsets), dim3(kXsecBlock), 0, s, part, nb, nevt, nsets, sigma, dsigma, norm, out);
  return hipGetLastError();
}

// Coupling-factored reweighting.  Electroweak family: every kept helicity
// amplitude is K_h(p) F_chi(card, s), chi the chirality class (LL, LR, RL, RR)
// of the two fermion lines, s the invariant mass of the resonant pair and
//   F_chi = A / s + B_chi / (s - M_Z^2 + i M_Z Gamma_Z)
// (A: product of the lines' photon couplings, B_chi: of their Z couplings),
// so |M|^2 = g sum_chi W_chi |F_chi|^2.  The class weights W_chi of an event
// come from four probe cards (Z couplings 1 on one class, all others 0):
// W_chi = |M|^2_probe,chi |s - M_p^2 + i M_p Gamma_p|^2.  QCD family (cards
// change alpha_s only): |M|^2 = g |M|^2_probe with g = (g_s / g_s,0)^8.
// Card 0 is the original card; w_out[k-1][i] = (w_in[i] / |M|^2_0) |M|^2_k.
template <bool EW>
__global__ __launch_bounds__(256) void factored_kernel(const double* __restrict__ soa, int64_t nsoa, int64_t nevt,
                                                       int ia, int ib,
                                                       const double* __restrict__ probe, double mzp, double wzp,
                                                       const FactorCard* __restrict__ fc, int ncards,
                                                       const double* __restrict__ w_in, double* __restrict__ w_out) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nevt) return;
  double W[4] = {0.0, 0.0, 0.0, 0.0};
  double s = 0.0;
  if constexpr (EW) {
    double pa[4], pb[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      pa[mu] = RWGT_AT(soa, int64_t(ia * 4 + mu) * nevt + i, nsoa);
      pb[mu] = RWGT_AT(soa, int64_t(ib * 4 + mu) * nevt + i, nsoa);
    }
    s = 2.0 * (pa[0] * pb[0] - pa[1] * pb[1] - pa[2] * pb[2] - pa[3] * pb[3]);
    const double xp = s - mzp * mzp, yp = mzp * wzp;
    const double dp = xp * xp + yp * yp;
#pragma unroll
    for (int c = 0; c < 4; ++c) W[c] = RWGT_AT(probe, int64_t(c) * nevt + i, 4 * nevt) * dp;
  } else {
    W[0] = RWGT_AT(probe, i, nevt);
  }
  auto me2 = [&](const FactorCard& k) {
    if constexpr (EW) {
      const double x = s - k.mz * k.mz, y = k.mz * k.wz;
      const double d = x * x + y * y;
      const double ga = k.A / s, gr = x / d, gi = -y / d;
      double sum = 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double re = ga + k.B[c] * gr, im = k.B[c] * gi;
        sum += W[c] * (re * re + im * im);
      }
      return k.g * sum;
    } else {
      return k.g * W[0];
    }
  };
  const double m0 = me2(RWGT_AT(fc, 0, ncards));
  const double norm = m0 != 0.0 ? RWGT_AT(w_in, i, nevt) * (1.0 / m0) : 0.0;
  for (int k = 1; k < ncards; ++k)
    RWGT_AT(w_out, int64_t(k - 1) * nevt + i, int64_t(ncards - 1) * nevt) = norm * me2(RWGT_AT(fc, k, ncards));
}

hipError_t launch_factored(bool ew, const double* soa, int npart, int64_t nevt, int ia, int ib, const double* probe,
                           double mzp, double wzp, const FactorCard* fc, int ncards, const double* w_in,
                           double* w_out, hipStream_t s) {
  if (nevt <= 0) return hipSuccess;
  const unsigned blocks = unsigned((nevt + 255) / 256);
  const int64_t nsoa = int64_t(npart) * 4 * nevt;
  if (ew)
    hipLaunchKernelGGL(factored_kernel<true>, dim3(blocks), dim3(256), 0, s, soa, nsoa, nevt, ia, ib, probe, mzp, wzp,
                       fc, ncards, w_in, w_out);
  else
    hipLaunchKernelGGL(factored_kernel<false>, dim3(blocks), dim3(256), 0, s, soa, nsoa, nevt, ia, ib, probe, mzp, wzp,
                       fc, ncards, w_in, w_out);
  return hipGetLastError();
}

// Per-event strong coupling on top of the fixed-coupling weights: every
// diagram of these processes carries the same power p of g_s, so |M|^2 under
// alpha_s(event) is |M|^2 under the card's alpha_s times (alpha_s(event) /
// alpha_s(card))^p.  The original uses the event's own alpha_s (or the
// original card's run to the event scale); card k its alpha_s run to the
// event scale at one loop: a(mu) = a / (1 + a b0 ln(mu^2 / m_ref^2)).
__device__ __forceinline__ double run_alphas(double a, double mu, double b0, double mref2) {
  return a / (1.0 + a * b0 * log(mu * mu / mref2));
}

__global__ __launch_bounds__(256) void alphas_kernel(double* __restrict__ w_out, int64_t nevt, int nsets,
                                                     const double* __restrict__ alphas_orig,
                                                     const double* __restrict__ scales, double as0,
                                                     const double* __restrict__ as_cards, int p, double b0,
                                                     double mref2) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nevt) return;
  const double mu = RWGT_AT(scales, i, nevt);
  const double a0 = alphas_orig ? RWGT_AT(alphas_orig, i, nevt) : run_alphas(as0, mu, b0, mref2);
  const bool zero = a0 == 0.0;             // |M|^2 of the original is 0: w' = 0
  const double r0 = zero ? 0.0 : as0 / a0;
  for (int k = 0; k < nsets; ++k) {
    const double ak = RWGT_AT(as_cards, k, nsets);
    const double rk = ak != 0.0 ? run_alphas(ak, mu, b0, mref2) / ak : 1.0;
    double f = 1.0, x = rk * r0;
    for (int q = 0; q < p; ++q) f *= x;
    double& w = RWGT_AT(w_out, int64_t(k) * nevt + i, int64_t(nsets) * nevt);
    w = zero ? 0.0 : w * f;
  }
}

hipError_t launch_alphas(double* w_out, int64_t nevt, int nsets, const double* alphas_orig, const double* scales,
                         double as0, const double* as_cards, int p, double b0, double mref2, hipStream_t s) {
  if (nevt <= 0) return hipSuccess;
  hipLaunchKernelGGL(alphas_kernel, dim3(unsigned((nevt + 255) / 256)), dim3(256), 0, s, w_out, nevt, nsets,
                     alphas_orig, scales, as0, as_cards, p, b0, mref2);
  return hipGetLastError();
}

// Count of the non-finite outputs of a call: a grid-stride pass, each wave
// sums its lanes' counts with shuffles, the block's four wave sums meet in
// LDS and thread 0 writes the block total (no atomics, nothing to clear).
__global__ __launch_bounds__(256) void nonfinite_kernel(const double* __restrict__ x, int64_t n,
                                                        unsigned long long* __restrict__ part) {
  __shared__ unsigned long long wsum[4];
  unsigned long long c = 0;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    c += isfinite(RWGT_AT(x, i, n)) ? 0 : 1;
  for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) RWGT_AT(part, blockIdx.x, gridDim.x) = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

int nonfinite_blocks(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return int(b < kNonfiniteBlocks ? (b < 1 ? 1 : b) : kNonfiniteBlocks);
}

hipError_t launch_nonfinite(const double* x, int64_t n, unsigned long long* part, hipStream_t s) {
  hipLaunchKernelGGL(nonfinite_kernel, dim3(unsigned(nonfinite_blocks(n))), dim3(256), 0, s, x, n, part);
  return hipGetLastError();
}

hipError_t launch_ingest(int npart, const double* aos, double* soa, int64_t nevt, hipStream_t s) {
  const int64_t blocks = (nevt + kIngestEvents - 1) / kIngestEvents;
  switch (npart) {
    case 4: hipLaunchKernelGGL(ingest_kernel<4>, dim3(unsigned(blocks)), dim3(256), 0, s, aos, soa, nevt); break;
    case 5: hipLaunchKernelGGL(ingest_kernel<5>, dim3(unsigned(blocks)), dim3(256), 0, s, aos, soa, nevt); break;
    case 6: hipLaunchKernelGGL(ingest_kernel<6>, dim3(unsigned(blocks)), dim3(256), 0, s, aos, soa, nevt); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fp64(int proc, const Fp64Call& a, hipStream_t s) {
  if (a.nevt < 1 || a.ncards < 1 || !a.cards || (a.ncards > kArgCards && !a.table) || !a.mom ||
      (a.w_out ? !a.w_in : !a.me_out))
    return hipErrorInvalidValue;
  switch (proc) {
    case kProcEeMumu: return launch_fp64_ee_mumu(a, s);
    case kProcUuEeg: return launch_fp64_uu_eeg(a, s);
    case kProcGgTtgg: return launch_fp64_gg_ttgg(a, s);
    case kProcGgTttt: return launch_fp64_gg_tttt(a, s);
  }
  return hipErrorInvalidValue;
}

size_t qcd_table(const CardPair* cards, int n, void* out) { return card_table<QcdCard>(cards, n, out, qcd_card); }

size_t fp64_table(int proc, const CardPair* cards, int n, void* out) {
  switch (proc) {
    case kProcEeMumu: return fp64_table_ee_mumu(cards, n, out);
    case kProcUuEeg: return fp64_table_uu_eeg(cards, n, out);
    case kProcGgTtgg: return fp64_table_gg_ttgg(cards, n, out);
    case kProcGgTttt: return fp64_table_gg_tttt(cards, n, out);
  }
  return 0;
}

hipError_t launch_me(int proc, int precision, const double* soa, int64_t nevt, const CardPair* cards, int ncards,
                     const double* w_in, double* w_out, double* me_out, void* parts, hipStream_t s) {
  switch (proc) {
    case kProcEeMumu: return launch_me_ee_mumu(precision, soa, nevt, cards, ncards, w_in, w_out, me_out, parts, s);
    case kProcUuEeg: return launch_me_uu_eeg(precision, soa, nevt, cards, ncards, w_in, w_out, me_out, parts, s);
    case kProcGgTtgg: return launch_me_gg_ttgg(precision, soa, nevt, cards, ncards, w_in, w_out, me_out, parts, s);
    case kProcGgTttt: return launch_me_gg_tttt(precision, soa, nevt, cards, ncards, w_in, w_out, me_out, parts, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_me_guarded(int proc, int precision, const double* soa, const double* mom, int64_t nevt,
                             const CardPair* cards, int ncards, const double* w_in, double* w_out, double* me_out, const GuardArgs& g,
                             void* parts, hipStream_t s) {
  switch (proc) {
    case kProcEeMumu:
      return launch_me_guarded_ee_mumu(precision, soa, mom, nevt, cards, ncards, w_in, w_out, me_out, g, parts, s);
    case kProcUuEeg:
      return launch_me_guarded_uu_eeg(precision, soa, mom, nevt, cards, ncards, w_in, w_out, me_out, g, parts, s);
    case kProcGgTtgg:
      return launch_me_guarded_gg_ttgg(precision, soa, mom, nevt, cards, ncards, w_in, w_out, me_out, g, parts, s);
    case kProcGgTttt:
      return launch_me_guarded_gg_tttt(precision, soa, mom, nevt, cards, ncards, w_in, w_out, me_out, g, parts, s);
  }
  return hipErrorInvalidValue;
}

size_t me_parts_bytes(int proc, int64_t nevt, int ncards) {
  switch (proc) {
    case kProcEeMumu: return me_parts_ee_mumu(nevt, ncards);
    case kProcUuEeg: return me_parts_uu_eeg(nevt, ncards);
    case kProcGgTtgg: return me_parts_gg_ttgg(nevt, ncards);
    case kProcGgTttt: return me_parts_gg_tttt(nevt, ncards);
  }
  return 0;
}

void process_constants(int proc, int* npart, int* ngood, int* ncol, int* ndiag) {
  switch (proc) {
    case kProcEeMumu: constants_ee_mumu(npart, ngood, ncol, ndiag); break;
    case kProcUuEeg: constants_uu_eeg(npart, ngood, ncol, ndiag); break;
    case kProcGgTtgg: constants_gg_ttgg(npart, ngood, ncol, ndiag); break;
    case kProcGgTttt: constants_gg_tttt(npart, ngood, ncol, ndiag); break;
    default: *npart = *ngood = *ncol = *ndiag = 0;
  }
}

double process_flops(int proc, bool executed) {
  switch (proc) {
    case kProcEeMumu: return flops_ee_mumu(executed);
    case kProcUuEeg: return flops_uu_eeg(executed);
    case kProcGgTtgg: return flops_gg_ttgg(executed);
    case kProcGgTttt: return flops_gg_tttt(executed);
  }
  return 0.0;
}

}  // namespace rwgt
