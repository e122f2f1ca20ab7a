// FP64 step kernels (up to 16 nodes per half): half-range and full-range models.
#include "fused_kernels.hpp"
#include "launch.hpp"

namespace hhlb {
namespace {

constexpr int kSimds = 1024;   // 256 CUs

template <int QUAD, int Q, int NF, int ADV, bool FEW, int SLOTS>
void launch(const StageArgs &a, hipStream_t s) {
  hipLaunchKernelGGL((step_kernel<QUAD, Q, NF, ADV, FEW, SLOTS>), dim3(a.nwin), dim3(128 * NF), 0, s, a, a.tb, a.chans,
                     reinterpret_cast<const DevFusedWindow *>(a.wins), a.inv_dx, a.gw, (const double *)a.in_f,
                     (const double *)a.in_c);
}

template <int QUAD, int Q, int NF, int ADV, int SLOTS>
void launch_step(const StageArgs &a, hipStream_t s) {
  // FEW where its waves all fit the GPU at once: beyond that the many-window
  // form's third or fourth wave per SIMD is worth more.  Up to four nodes per
  // half it gains next to nothing (576 against 579 us for 64 steps of a 64-cell
  // channel).
  constexpr int H = QUAD == 0 ? Q : Q / 2;
  if constexpr (H > 4) {
    if ((int64_t)a.nwin * 2 * NF <= (int64_t)kSimds * few_waves(H, SLOTS, NF)) {
      launch<QUAD, Q, NF, ADV, true, SLOTS>(a, s);
      return;
    }
  }
  launch<QUAD, Q, NF, ADV, false, SLOTS>(a, s);
}

template <int QUAD, int Q, int SLOTS>
void add(LaunchMap &m) {
  m[{QUAD, Q, 1, 0, 0, SLOTS}] = launch_step<QUAD, Q, 1, 0, SLOTS>;
  m[{QUAD, Q, 1, 1, 0, SLOTS}] = launch_step<QUAD, Q, 1, 1, SLOTS>;
  m[{QUAD, Q, 2, 0, 0, SLOTS}] = launch_step<QUAD, Q, 2, 0, SLOTS>;
  m[{QUAD, Q, 2, 1, 0, SLOTS}] = launch_step<QUAD, Q, 2, 1, SLOTS>;
}

}  // namespace

void register_fp64(LaunchMap &m) {
#define HHLB_ADD(slots)                                                              \
  add<0, 1, slots>(m); add<0, 2, slots>(m); add<0, 3, slots>(m); add<0, 4, slots>(m); \
  add<0, 6, slots>(m); add<0, 8, slots>(m); add<0, 12, slots>(m); add<0, 16, slots>(m); \
  add<1, 2, slots>(m); add<1, 4, slots>(m); add<1, 8, slots>(m); add<1, 16, slots>(m);
  HHLB_ADD(1)
  HHLB_ADD(2)
#undef HHLB_ADD
}

}  // namespace hhlb
