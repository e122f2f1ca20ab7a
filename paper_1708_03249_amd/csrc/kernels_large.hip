// Launchers of the node-parallel FP64 stage for large velocity sets.
#include "large_kernels.hpp"
#include "launch.hpp"

namespace hhlb {
namespace {

dim3 grid(const LargeArgs &a, int H) { return dim3(a.nwin * 2 * ((H + kTileNodes - 1) / kTileNodes)); }

template <int ADV, int NFUN>
void stage(const LargeArgs &a, int H, int max_out, hipStream_t s) {
  // the window's cells and their halo in 16-cell blocks of the contraction
  if (max_out + 2 * kHalo <= 32)
    hipLaunchKernelGGL((large_stage_kernel<ADV, 2, NFUN>), grid(a, H), dim3(64 * kNodeWaves), 0, s, a);
  else
    hipLaunchKernelGGL((large_stage_kernel<ADV, 4, NFUN>), grid(a, H), dim3(64 * kNodeWaves), 0, s, a);
}

template <int ADV, int NFUN>
void sums(const LargeArgs &a, int H, hipStream_t s) {
  hipLaunchKernelGGL((large_sums_kernel<ADV, NFUN>), grid(a, H), dim3(64 * kNodeWaves), 0, s, a);
}

}  // namespace

void launch_large(const LargeArgs &a, int adv, int nfun, int H, int max_out, hipStream_t s) {
  if (adv == 0) nfun > 1 ? stage<0, 2>(a, H, max_out, s) : stage<0, 1>(a, H, max_out, s);
  else nfun > 1 ? stage<1, 2>(a, H, max_out, s) : stage<1, 1>(a, H, max_out, s);
}

void launch_large_sums(const LargeArgs &a, int adv, int nfun, int H, hipStream_t s) {
  if (adv == 0) nfun > 1 ? sums<0, 2>(a, H, s) : sums<0, 1>(a, H, s);
  else nfun > 1 ? sums<1, 2>(a, H, s) : sums<1, 1>(a, H, s);
}

}  // namespace hhlb
