// The generated FP64 amplitude code of g g -> t t~ g g, compiled for the host by
// test_amplitudes_host.py.  Reads the couplings and events of six momenta from
// standard input; prints per event |M|^2 summed over colours of the 64
// helicities, from the body for any momenta and from the one for beams.
#include <hip/hip_runtime.h>

#include "common.h"

namespace mg {
#include "generated/ggttgg.inc"
}
using namespace mg;

template <bool BEAM>
static void helicities(const double (&p)[6][4], const Couplings<double>& c) {
  for (unsigned h = 0; h < 64; ++h) {
    double q[6][4];
    for (int l = 0; l < 6; ++l)
      for (int m = 0; m < 4; ++m) q[l][m] = p[l][m];
    if constexpr (BEAM) set_beams(q);
    cx<double> J[gen_ggttgg::NCOL];
    gen_ggttgg::jamps<double, false, BEAM>(q, h, c, J);
    std::printf("%.17g ", gen_ggttgg::colour_sum<double>(J));
  }
}

int main() {
  Couplings<double> c{};
  if (std::scanf("%lf %lf %lf", &c.gs, &c.mt, &c.wt) != 3) return 1;
  c.gs2 = c.gs * c.gs;
  c.wtt = c.wt;
  for (;;) {
    double p[6][4];
    for (auto& k : p)
      for (double& x : k)
        if (std::scanf("%lf", &x) != 1) return 0;
    helicities<false>(p, c);
    if (beams_on_axis(p)) helicities<true>(p, c);
    std::printf("\n");
  }
}
