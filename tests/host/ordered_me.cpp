// The colour-ordered recursions of g g -> t t~ g g (ordered.h) and, built with
// -DPAIRS, of g g -> t t~ t t~ (ordered_pairs.h) on the host in double
// precision, one thread per lane: |M|^2 per event.
//   stdin:  n alpha_s m_t, then n lines of 6 x 4 momenta (E px py pz)
//   stdout: n values of |M|^2
#include <hip/hip_runtime.h>

#include <pthread.h>

#include <cmath>
#include <cstdio>
#include <thread>
#include <vector>

#ifdef PAIRS
#include "generated/gen_gg_tttt.h"
#include "ordered_pairs.h"
namespace gen = rwgt::gen_gg_tttt;
using namespace rwgt::ordered::pairs;
#else
#include "generated/gen_gg_ttgg.h"
#include "ordered.h"
namespace gen = rwgt::gen_gg_ttgg;
#endif

using namespace rwgt;
using namespace rwgt::ordered;

struct Memory {
  LcK<double> k[6];
  Lc<double> p[kPols];
  cx<double> v[kSlots][4];
  LcK<double> mom(int g) const { return k[g]; }
  Lc<double> pol(int s) const { return p[s]; }
  void set_pol(int s, const Lc<double>& q) { p[s] = q; }
  Lc<double> vec(int s) const { return {v[s][0], v[s][1], v[s][2], v[s][3]}; }
  void set_vec(int s, const Lc<double>& q) { v[s][0] = q.u; v[s][1] = q.d; v[s][2] = q.p; v[s][3] = q.m; }
  Spinor<double> spin(int s) const { return {{v[s][0], v[s][1], v[s][2], v[s][3]}}; }
  void set_spin(int s, const Spinor<double>& q) { for (int n = 0; n < 4; ++n) v[s][n] = q.c[n]; }
};

int main() {
  int n = 0;
  double as = 0.0, mt = 0.0;
  if (std::scanf("%d %lf %lf", &n, &as, &mt) != 3) return 1;
  std::vector<double> P(size_t(n) * 24);
  for (double& x : P)
    if (std::scanf("%lf", &x) != 1) return 2;
  Card<double, double> cd{};
  cd.gqq = cd.g3 = std::sqrt(4.0 * M_PI * as);
  cd.g4 = cd.g3 * cd.g3;
  cd.mt = mt;
  std::vector<Memory> mem(static_cast<size_t>(n));
  for (int e = 0; e < n; ++e) {
    const double* p = &P[size_t(e * 24)];
#ifdef PAIRS
    for (int a = 0; a < 6; ++a) mem[size_t(e)].k[a] = lc_momentum(p + 4 * a, 1.0);
#else
    static const int particle[4] = {0, 1, 4, 5};
    for (int g = 0; g < 4; ++g) mem[size_t(e)].k[g] = lc_momentum(p + 4 * particle[g], g < 2 ? 1.0 : -1.0);
#endif
  }
  pthread_barrier_t bar;
  pthread_barrier_init(&bar, nullptr, 32);
  std::vector<double> part(size_t(n) * 32);
  std::vector<std::thread> lanes;
  for (int t = 0; t < 32; ++t)
    lanes.emplace_back([&, t] {
      auto sync = [&] { pthread_barrier_wait(&bar); };
      auto colour = [](cx<double>(&f)[gen::NCOL]) { return gen::colour_sum_paired<double>(f); };
      for (int e = 0; e < n; ++e) {
        const double* p = &P[size_t(e * 24)];
#ifdef PAIRS
        auto load = [&](int a, double (&q)[4]) { for (int m = 0; m < 4; ++m) q[m] = p[4 * a + m]; };
        part[size_t(e * 32 + t)] = pairs::lane_me2<double>(mem[size_t(e)], t, load, cd, sync, colour);
#else
        part[size_t(e * 32 + t)] = lane_me2(mem[size_t(e)], t, p + 8, p + 12, cd, sync, colour);
#endif
      }
    });
  for (auto& l : lanes) l.join();
  for (int e = 0; e < n; ++e) {
    double me = 0.0;
    for (int t = 0; t < 32; ++t) me += part[size_t(e * 32 + t)];
    std::printf("%.17g\n", me * cd.gqq * cd.gqq * gen::AVERAGE * gen::HELW);
  }
  return 0;
}
