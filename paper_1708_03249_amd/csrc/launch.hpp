// Registry of the step-kernel launchers, keyed by model shape and arithmetic
// form.  Each kernel family is instantiated in its own translation unit.
#pragma once
#include <hip/hip_runtime.h>

#include <map>
#include <tuple>

#include "step_kernels.hpp"

namespace hhlb {

using Launcher = void (*)(const StageArgs &, hipStream_t);
// (quadrature kind, Q, functions (1 = f, 2 = f and chi), advection, precision,
//  shape: 1 and 2 = one class, windows of one or two cells per lane; 3 = across
//  classes (FP64), keyed by the largest order it holds)
using LaunchKey = std::tuple<int, int, int, int, int, int>;
using LaunchMap = std::map<LaunchKey, Launcher>;

void register_fp64(LaunchMap &m);
void register_mixed_f32(LaunchMap &m);
void register_mixed_bf16(LaunchMap &m);
void register_mixed_f16(LaunchMap &m);
void register_classes(LaunchMap &m);

// The node-parallel FP64 stage of large half-range classes (Q > 16):
// kernels_large.hip.
struct LargeArgs;
void launch_large(const LargeArgs &a, int adv, int nfun, int H, int max_out, hipStream_t s);
// The partial sums of the state (in_f, in_c), which the first stage of a call reads.
void launch_large_sums(const LargeArgs &a, int adv, int nfun, int H, hipStream_t s);

// The mixed-quadrature (App. A) velocity-space stage: kernels_multi.hip.
struct MultiArgs;
struct MultiShape;
// Whole-step kernels by the largest equilibrium order of the axes: false if
// there is no instance for the set's V_x.
bool launch_multi_n3(const MultiArgs &a, const MultiShape &m, hipStream_t s);
bool launch_multi_n7(const MultiArgs &a, const MultiShape &m, hipStream_t s);
bool launch_multi_n20(const MultiArgs &a, const MultiShape &m, hipStream_t s);
void launch_multi(const MultiArgs &a, hipStream_t s, int V, int k_doubles, int n_max);

}  // namespace hhlb
