// The colour-ordered recursion of g g -> t t~ g g (ordered.h) on the host in
// double precision, one thread per lane: |M|^2 per event.
//   stdin:  n alpha_s m_t, then n lines of 6 x 4 momenta (E px py pz)
//   stdout: n values of |M|^2
#include <hip/hip_runtime.h>

#include <pthread.h>

#include <cmath>
#include <cstdio>
#include <thread>
#include <vector>

#include "generated/gen_gg_ttgg.h"
#include "ordered.h"

using namespace rwgt;
using namespace rwgt::ordered;

struct Memory {
  LcK<double> k[4];
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
  static const int particle[4] = {0, 1, 4, 5};
  for (int e = 0; e < n; ++e)
    for (int g = 0; g < 4; ++g) mem[size_t(e)].k[g] = lc_momentum(&P[size_t(e * 24 + particle[g] * 4)], g < 2 ? 1.0 : -1.0);
  pthread_barrier_t bar;
  pthread_barrier_init(&bar, nullptr, kLanes);
  std::vector<double> part(size_t(n) * kLanes);
  std::vector<std::thread> lanes;
  for (int t = 0; t < kLanes; ++t)
    lanes.emplace_back([&, t] {
      for (int e = 0; e < n; ++e)
        part[size_t(e * kLanes + t)] =
            lane_me2(mem[size_t(e)], t, &P[size_t(e * 24 + 8)], &P[size_t(e * 24 + 12)], cd,
                     [&] { pthread_barrier_wait(&bar); },
                     [](const cx<double>(&f)[24]) { return gen_gg_ttgg::colour_sum<double>(f); });
    });
  for (auto& l : lanes) l.join();
  for (int e = 0; e < n; ++e) {
    double me = 0.0;
    for (int t = 0; t < kLanes; ++t) me += part[size_t(e * kLanes + t)];
    std::printf("%.17g\n", me * cd.gqq * cd.gqq * gen_gg_ttgg::AVERAGE * gen_gg_ttgg::HELW);
  }
  return 0;
}
