// FP64 step kernels (up to 16 nodes per half): half-range and full-range models.
#include "fused_kernels.hpp"
#include "launch.hpp"

namespace hhlb {
namespace {

constexpr int kSimds = 1024;   // 256 CUs

template <int QUAD, int Q, int NF, int ADV, bool FEW>
void launch(const StageArgs &a, hipStream_t s) {
  hipLaunchKernelGGL((step_kernel<QUAD, Q, NF, ADV, FEW>), dim3(a.nwin), dim3(128 * NF), 0, s, a, a.tb, a.chans,
                     reinterpret_cast<const DevFusedWindow *>(a.wins), a.inv_dx, a.gw, (const double *)a.in_f,
                     (const double *)a.in_c);
}

template <int QUAD, int Q, int NF, int ADV>
void launch_step(const StageArgs &a, hipStream_t s) {
  // FEW where its waves all fit the GPU at once: beyond that the many-window
  // form's third or fourth wave per SIMD is worth more.  Up to four nodes per
  // half it gains nothing (607 against 613 us for 64 steps of a 64-cell channel).
  constexpr int H = QUAD == 0 ? Q : Q / 2;
  if constexpr (H > 4) {
    if ((int64_t)a.nwin * 2 * NF <= (int64_t)kSimds * few_waves(H)) {
      launch<QUAD, Q, NF, ADV, true>(a, s);
      return;
    }
  }
  launch<QUAD, Q, NF, ADV, false>(a, s);
}

template <int QUAD, int Q>
void add(LaunchMap &m) {
  m[{QUAD, Q, 1, 0, 0, 1}] = launch_step<QUAD, Q, 1, 0>;
  m[{QUAD, Q, 1, 1, 0, 1}] = launch_step<QUAD, Q, 1, 1>;
  m[{QUAD, Q, 2, 0, 0, 1}] = launch_step<QUAD, Q, 2, 0>;
  m[{QUAD, Q, 2, 1, 0, 1}] = launch_step<QUAD, Q, 2, 1>;
}

}  // namespace

void register_fp64(LaunchMap &m) {
  add<0, 1>(m); add<0, 2>(m); add<0, 3>(m); add<0, 4>(m);
  add<0, 6>(m); add<0, 8>(m); add<0, 12>(m); add<0, 16>(m);
  add<1, 2>(m); add<1, 4>(m); add<1, 8>(m); add<1, 16>(m);
}

}  // namespace hhlb
