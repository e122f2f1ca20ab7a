// Mixed-precision half-range step kernels, force block in F32 form.
#include "launch.hpp"
#include "mixed_kernels.hpp"

namespace hhlb {
namespace {

template <int Q, int NF, int ADV, int SLOTS>
void launch_step(const StageArgs &a, hipStream_t s) {
  hipLaunchKernelGGL((step_kernel_mixed<Q, NF, ADV, kPrecF32, SLOTS>), dim3(a.nwin), dim3(128 * NF), 0, s, a, a.tb,
                     a.chans, reinterpret_cast<const DevFusedWindow *>(a.wins), a.inv_dx, a.gw, (const float *)a.in_f,
                     (const float *)a.in_c);
}

template <int Q, int SLOTS>
void add(LaunchMap &m) {
  m[{0, Q, 1, 0, kPrecF32, SLOTS}] = launch_step<Q, 1, 0, SLOTS>;
  m[{0, Q, 1, 1, kPrecF32, SLOTS}] = launch_step<Q, 1, 1, SLOTS>;
  m[{0, Q, 2, 0, kPrecF32, SLOTS}] = launch_step<Q, 2, 0, SLOTS>;
  m[{0, Q, 2, 1, kPrecF32, SLOTS}] = launch_step<Q, 2, 1, SLOTS>;
}

}  // namespace

void register_mixed_f32(LaunchMap &m) {
  add<1, 1>(m); add<2, 1>(m); add<3, 1>(m); add<4, 1>(m); add<6, 1>(m); add<8, 1>(m); add<12, 1>(m); add<16, 1>(m);
  add<1, 2>(m); add<2, 2>(m); add<3, 2>(m); add<4, 2>(m); add<6, 2>(m); add<8, 2>(m); add<12, 2>(m); add<16, 2>(m);
}

}  // namespace hhlb
