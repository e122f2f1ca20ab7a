// Whole-step kernels of the homogeneous mixed-quadrature system (App. A) for
// equilibrium orders up to 3.
#include "launch.hpp"
#include "multi_steps.hpp"

namespace hhlb {

bool launch_multi_n3(const MultiArgs &a, const MultiShape &m, hipStream_t s) { return launch_multi_nm<3>(a, m, s); }

}  // namespace hhlb
