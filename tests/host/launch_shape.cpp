// The event ranges that a double-precision QCD call is launched in
// (ordered_kernel.h).
//   argv[1]: number of events
//   stdout:  per launch "first event, workgroups"
#include "ordered_kernel.h"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
  if (argc != 2) return 1;
  const int64_t nevt = std::atoll(argv[1]);
  int64_t groups = 0;
  for (int64_t first = 0; first < nevt; first += 2 * groups) {
    groups = rwgt::ordered::launch_groups(nevt, first);
    std::printf("%lld %lld\n", static_cast<long long>(first), static_cast<long long>(groups));
    if (groups < 1) return 2;
  }
  return 0;
}
