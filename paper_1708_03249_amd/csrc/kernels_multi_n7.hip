// Whole-step kernels of the homogeneous mixed-quadrature system (App. A) for
// equilibrium orders up to 7.
#include "launch.hpp"
#include "multi_steps.hpp"

namespace hhlb {

bool launch_multi_n7(const MultiArgs &a, const MultiShape &m, hipStream_t s) { return launch_multi_nm<7>(a, m, s); }

}  // namespace hhlb
