// The electroweak weights (electroweak.h) on the host: |M|^2 per event.
//   stdin:  npart n average, one card (g_s; photon couplings, left and right Z
//           couplings of 4 species; M_Z, Gamma_Z), then n lines of momenta
//   stdout: n values of |M|^2
#include <hip/hip_runtime.h>

#include <cstdio>

#include "electroweak.h"

using namespace rwgt;

template <int NPART>
static int run(int n, const Card<double>& cd, double average) {
  for (int e = 0; e < n; ++e) {
    double P[NPART][4];
    for (auto& p : P)
      for (double& x : p)
        if (std::scanf("%lf", &x) != 1) return 2;
    std::printf("%.17g\n", ew::me2<NPART>(ew::Process<NPART>::template weights<false>(P), cd, average));
  }
  return 0;
}

int main() {
  int npart = 0, n = 0;
  double average = 0.0;
  Card<double> cd{};
  if (std::scanf("%d %d %lf %lf", &npart, &n, &average, &cd.gqq) != 4) return 1;
  for (double* c : {cd.a, cd.zL, cd.zR})
    for (int f = 0; f < 4; ++f)
      if (std::scanf("%lf", &c[f]) != 1) return 1;
  if (std::scanf("%lf %lf", &cd.mz, &cd.wz) != 2) return 1;
  return npart == 4 ? run<4>(n, cd, average) : run<5>(n, cd, average);
}
