// Whole-step kernels of the homogeneous mixed-quadrature system (App. A) for
// equilibrium orders up to 20.
#include "launch.hpp"
#include "multi_steps.hpp"

namespace hhlb {

bool launch_multi_n20(const MultiArgs &a, const MultiShape &m, hipStream_t s) { return launch_multi_nm<20>(a, m, s); }

}  // namespace hhlb
