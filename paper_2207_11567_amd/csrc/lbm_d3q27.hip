// D3Q27 dispatch over precisions and scalar counts (the instances are generated units, one per
// precision and number of scalars).
#include "lbm_launch.hpp"

namespace lbm {
hipError_t launch_d3q27(int prec, int ns, int kind, const StepArgs &a, int nblocks, hipStream_t st,
                        const double *Ph, const double *u, const double *scal) {
  switch (prec) {
    case 0: return launch_ns<27, 0>(ns, kind, a, nblocks, st, Ph, u, scal);
    case 1: return launch_ns<27, 1>(ns, kind, a, nblocks, st, Ph, u, scal);
    case 2: return launch_ns<27, 2>(ns, kind, a, nblocks, st, Ph, u, scal);
  }
  return hipErrorInvalidValue;
}
}  // namespace lbm
