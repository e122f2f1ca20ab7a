// gfx950 kernel for whole TVD RK-3 steps of the half-range model in mixed
// precision.  The populations are kept as phi_k = f_k / w_k (and
// chi_k / w_k), which keeps every stored value of order one whatever the
// node weight.  Advection (WENO-5 / upwind-3), collision, the force
// contraction and the RK-3 combination run in FP32 arithmetic; the moment
// sums, the wall-density flux balance of Eq. (nplus_def) and the
// equilibrium coefficients stay in FP64.
//
// Storage.  A state rounded to FP32 at every step would lose the part of
// each step's increment below half an ulp, the same part every step once the
// flow is nearly steady: the slow modes then settle off the FP64 solution by
// about eps / (dt lambda) and the conserved mass drifts linearly.  So
//  * y^n is stored as an FP32 value hi plus a 16-bit correction word lo,
//    a fixed-point fraction of hi's ulp (y = hi + lo 2^(e-39) for
//    hi = m 2^e, m in [1/2, 1)), which carries y^n to about 2^-39;
//  * the stages advance the increments d1 = y1 - y^n and d2 = y2 - y^n, in
//    FP32, so their rounding is relative to the increment;
//  * the last stage adds (2/3)(d2 + dt L[y2]) to (hi, lo) with an exact
//    two-sum.
// With the increments, stage s computes d_out = (1 - a_s)(d_in + dt L[y_s]),
// y_s = hi + d_in, a_s = 0, 3/4, 1/3 the weights of y^n in Eq. (rk3).  The
// force block -F (K y) is contracted on the matrix cores: FP32 MFMA (16 x 16 x 4) for the FP32 form
// at Q = 16, BF16 or FP16 MFMA (16 x 16 x 16, FP32 accumulation) for those
// forms above Q = 4 (zero-padded to 16), and FP32 VALU otherwise.
//
// Mapping, window geometry (two cells or one per lane) and the split of the
// equilibrium between the waves are those of the FP64 step kernel: (hi, lo) and
// the increment of a window stay in registers through the three stages, and a step reads and
// writes 6 bytes per population where a stage per launch moved 52 per step.
#pragma once
#include "fused_kernels.hpp"

namespace hhlb {

enum { kPrecF32 = 1, kPrecBF16 = 2, kPrecF16 = 3 };

__device__ __forceinline__ float dpp_shr1f(float x) {  // lane l <- lane l-1
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float dpp_shl1f(float x) {  // lane l <- lane l+1
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ float readlane_f(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// WENO-5 faces of a lane's two cells (wind positions 2 l and 2 l + 1) in FP32,
// as deviations fa, fb of the downwind face's value from the cell's own: the
// construction of faces_down2, every term formed from neighbour differences,
// which are exact in FP32 for neighbours within a factor two of each other, so
// the rounding scales with the differences rather than with y, and the flux
// difference a stage forms from the deviations inherits that accuracy.  dm and
// da are the differences of each cell to its upwind neighbour.
//
// The sigmas are always rescaled by an exact power of two (in smooth flow the
// unscaled product of four of them underflows FP32).  Then the largest q lies
// in [1/4, 1); a q below 1e-17 counts as vanishing, and the products are
// regular above 1e-37, which the pairs of non-vanishing q always exceed;
// below it the limits of Table (weno) apply.
struct WenoWeightsF {
  float qL, qC, qR, pL, pC, pR, dd;
  __device__ __forceinline__ WenoWeightsF(float dm, float dp, float DL, float D, float DR, float sqL, float sqC,
                                          float sqR) {
    constexpr float h = (float)(0.5 / kSq1312);
    const float tL = fmaf(h, DL, dm), tC = fmaf(h, D, dm), tR = fmaf(-h, DR, dp);
    const float sL = fmaf(tL, tL, sqL), sC = fmaf(tC, tC, sqC), sR = fmaf(tR, tR, sqR);
    const int ex = -__builtin_amdgcn_frexp_expf(fmaxf(sL, fmaxf(sC, sR)));
    const float rL = ldexpf(sL, ex), rC = ldexpf(sC, ex), rR = ldexpf(sR, ex);
    qL = rL * rL; qC = rC * rC; qR = rR * rR;
    pL = qC * qR; pC = qL * qR; pR = qL * qC;
    dd = fmaf(0.5f, pR, fmaf(1.0f / 6.0f, pL, pC));
  }
  __device__ __forceinline__ bool regular() const { return dd > 1e-37f; }
  __device__ __forceinline__ void limit() {
    if (!regular()) {
      const float tiny = 1e-17f;
      pL = qL < tiny ? 1.0f : 0.0f;
      pC = qC < tiny ? 1.0f : 0.0f;
      pR = qR < tiny ? 1.0f : 0.0f;
      dd = fmaf(0.5f, pR, fmaf(1.0f / 6.0f, pL, pC));
    }
  }
  __device__ __forceinline__ float dev(float dm, float dp, float dLD, float dDR) const {
    const float m = fmaf(1.5f, pR * dDR, pL * dLD) * __builtin_amdgcn_rcpf(dd);
    return fmaf((float)(1.0 / (18.0 * kSq1312)), m, fmaf(1.0f / 3.0f, dp, (1.0f / 6.0f) * dm));
  }
};

template <int ADV>
__device__ __forceinline__ void devs_down2(float ya, float yb, bool usedA, bool usedB, float &dm, float &da, float &fa,
                                           float &fb) {
  da = yb - ya;
  const float db = dpp_shl1f(ya) - yb;
  dm = dpp_shr1f(db);
  if constexpr (ADV == 0) {
    constexpr float k = (float)kSq1312;
    const float Da = k * (da - dm), Db = k * (db - da);
    const float Dl = dpp_shr1f(Db), Dr = dpp_shl1f(Da);
    const float qa = Da * Da, qb = Db * Db, dab = Da - Db;
    WenoWeightsF wa(dm, da, Dl, Da, Db, Dl * Dl, qa, qb), wb(da, db, Da, Db, Dr, qa, qb, Dr * Dr);
    if ((!wa.regular() && usedA) || (!wb.regular() && usedB)) {
      wa.limit();
      wb.limit();
    }
    fa = wa.dev(dm, da, Dl - Da, dab);
    fb = wb.dev(da, db, dab, Db - Dr);
  } else {
    fa = fmaf(1.0f / 3.0f, da, (1.0f / 6.0f) * dm);
    fb = fmaf(1.0f / 3.0f, db, (1.0f / 6.0f) * da);
  }
}

// The same for one cell per lane.
template <int ADV>
__device__ __forceinline__ void dev_down1(float y, bool used, float &dm, float &f) {
  const float dp = dpp_shl1f(y) - y;
  dm = dpp_shr1f(dp);
  if constexpr (ADV == 0) {
    const float D = (float)kSq1312 * (dp - dm), Dl = dpp_shr1f(D), Dr = dpp_shl1f(D);
    WenoWeightsF w(dm, dp, Dl, D, Dr, Dl * Dl, D * D, Dr * Dr);
    if (!w.regular() && used) w.limit();
    f = w.dev(dm, dp, Dl - D, D - Dr);
  } else {
    f = fmaf(1.0f / 3.0f, dp, (1.0f / 6.0f) * dm);
  }
}

// Correction word of y = hi + lo: lo counts 2^-15 ulps of hi (|lo| <= 2^14).
__device__ __forceinline__ float lo_value(float hi, int16_t lo) {
  return ldexpf((float)lo, __builtin_amdgcn_frexp_expf(hi) - 39);
}
// y^n + delta -> (hi', lo'): the FP32 sum, and its exact rounding error
// (two-sum) stored as the correction word.
__device__ __forceinline__ void add_to_state(float hi, int16_t lo, float delta, float &hi_out, int16_t &lo_out) {
  const float t = lo_value(hi, lo) + delta;
  const float s = hi + t;
  const float bb = s - hi;
  const float e = (hi - (s - bb)) + (t - bb);
  hi_out = s;
  // |e| <= ulp(s)/2 gives |lo| <= 2^14 for normal s; the clamp only guards
  // denormal sums
  const float q = __builtin_rintf(ldexpf(e, 39 - __builtin_amdgcn_frexp_expf(s)));
  lo_out = (int16_t)fminf(fmaxf(q, -32767.0f), 32767.0f);
}

typedef float flt4 __attribute__((ext_vector_type(4)));
typedef short bfx4 __attribute__((ext_vector_type(4)));
typedef _Float16 hfx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short to_bf16(float x) { return __builtin_bit_cast(short, (__bf16)x); }
__device__ __forceinline__ float bf16_value(short h) { return __uint_as_float((uint32_t)(uint16_t)h << 16); }
// FP16 low parts are formed 2^11 times larger than the remainder they stand
// for: the remainder of an entry below FP16's normal range (2^-14) would
// otherwise fall into its subnormals, which keep only an absolute 2^-24.
// The products of the low parts are scaled back in FP32 before the product
// of the high parts is added.  BF16 has the FP32 exponent range: no scale.
constexpr float kF16LoScale = 2048.0f, kF16LoUnscale = 1.0f / 2048.0f;

// A operand of the force block for the matrix cores, built from the FP32
// table Ks (H x H, row-major), zero outside the H x H block.  Lane i + 16 g
// holds M[i][4 g + t], t = 0..3.  Register layouts (checked on the GPU):
//   16x16x4 f32:        A[i][k] in lane i + 16 k; instruction t takes the
//                       columns k = 4 g + t, so operand t serves it
//   16x16x16 bf16/f16:  A[i][k] in lane i + 16 (k / 4), element k % 4
//   both:               B[k][j] like A with j for i; D[i][j] in lane
//                       j + 16 (i / 4), accumulator register i % 4
template <int PREC>
struct ForceA;
template <int H>
__device__ __forceinline__ float force_entry(const float *Ks, int i, int k) {
  return (i < H && k < H) ? Ks[(i < H ? i : 0) * H + (k < H ? k : 0)] : 0.0f;
}
template <>
struct ForceA<kPrecF32> {
  float v[4];
  template <int H>
  __device__ __forceinline__ void load(const float *Ks, int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = force_entry<H>(Ks, lane & 15, 4 * (lane >> 4) + t);
  }
};
// BF16: three operands hold an FP32 entry exactly (the entry rounded to the
// operand format, the remainder rounded again, and what is left).
template <>
struct ForceA<kPrecBF16> {
  bfx4 v, lo, rest;
  template <int H>
  __device__ __forceinline__ void load(const float *Ks, int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float x = force_entry<H>(Ks, lane & 15, 4 * (lane >> 4) + t);
      v[t] = to_bf16(x);
      const float r = x - bf16_value(v[t]);
      lo[t] = to_bf16(r);
      rest[t] = to_bf16(r - bf16_value(lo[t]));
    }
  }
};
// FP16: the table as a high part v (the entry rounded to the operand format)
// plus a low part lo (the remainder, exact in FP32, rounded again), so that
// the products carry about twice the operand precision.
template <>
struct ForceA<kPrecF16> {   // loaded from the row-scaled table Ks16
  hfx4 v, lo;
  template <int H>
  __device__ __forceinline__ void load(const float *Ks, int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float x = force_entry<H>(Ks, lane & 15, 4 * (lane >> 4) + t);
      v[t] = (_Float16)x;
      lo[t] = (_Float16)((x - (float)v[t]) * kF16LoScale);
    }
  }
};

// Mass defect of the FP16 form's split product Kh (yh + yl) + Kl yh:
// sum_j crs_j (yh_j + yl_j) + crs_lo_j yh_j, spread over the half by iwh.
// Lane i + 16 g holds the entries of the columns 4 g + t of its B operands and
// the row scales of the rows 4 g + t of its results.
template <int PREC>
struct ForceDefect {
  template <int H>
  __device__ __forceinline__ void load(const DevTables *, int) {}
};
template <>
struct ForceDefect<kPrecF16> {
  float c[4], cl[4], rs[4], iwh;
  template <int H>
  __device__ __forceinline__ void load(const DevTables *tb, int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = 4 * (lane >> 4) + t, kk = k < H ? k : 0;
      c[t] = k < H ? tb->crs[kk] : 0.0f;
      cl[t] = k < H ? tb->crs_lo[kk] : 0.0f;
      rs[t] = tb->irsc[kk];
    }
    iwh = tb->iwh;
  }
};

// OUT[i] = sum_k M[i][k] X[k] (i, k < H) for the 64 cells of the wave (one
// per lane), as four 16-cell products on the matrix cores, less the mass
// defect of the FP16 form.  The values go through the wave's
// LDS tile into the B layout and back, four nodes to an access: row `cell`
// holds its 16 nodes as four quads, quad g in place g ^ ((cell >> 2) & 3),
// so that the 16 lanes of a group touch all 64 banks once.
template <int PREC, int H>
__device__ __forceinline__ void mfma_force(const ForceA<PREC> &aM, const ForceDefect<PREC> &fd, const float X[H],
                                           float OUT[H], float *T, int lane) {
  constexpr int NG = (H + 3) / 4;
  flt4 *const Q4 = reinterpret_cast<flt4 *>(T);
  const int own = 4 * lane, sw = (lane >> 2) & 3;
  // FP16: scale the cell by a power of two so that max |y| < 1
  float sc = 1.0f, isc = 1.0f;
  if constexpr (PREC == kPrecF16) {
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < H; ++j) m = fmaxf(m, fabsf(X[j]));
    const int e = __builtin_amdgcn_frexp_expf(m);
    sc = ldexpf(1.0f, -e);
    isc = ldexpf(1.0f, e);
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    flt4 q;
#pragma unroll
    for (int t = 0; t < 4; ++t) q[t] = 4 * g + t < H ? (PREC == kPrecF16 ? X[4 * g + t] * sc : X[4 * g + t]) : 0.0f;
    Q4[own + (g ^ sw)] = q;
  }
  __builtin_amdgcn_wave_barrier();
  const int g = lane >> 4, r = 4 * (lane & 15) + (g ^ ((lane >> 2) & 3));
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    flt4 b = Q4[64 * cb + r];
    if constexpr (NG < 4) {
      if (g >= NG) b = flt4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    flt4 acc = flt4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (PREC == kPrecF32) {
#pragma unroll
      for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(aM.v[t], b[t], acc, 0, 0, 0);
    } else if constexpr (PREC == kPrecBF16) {
      // y as the exact sum of three BF16 operands too; six of the nine
      // products, the smallest first (the dropped ones are below 2^-26 of
      // |K||y|), so the result is as good as an FP32 contraction and needs
      // no correction.  (Two operands each and three products left 2^-17,
      // 1e-7 to 7e-7 in the moments of batched channels after 1000 steps.)
      bfx4 bh, bl, br;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        bh[t] = to_bf16(b[t]);
        const float r = b[t] - bf16_value(bh[t]);
        bl[t] = to_bf16(r);
        br[t] = to_bf16(r - bf16_value(bl[t]));
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aM.rest, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aM.v, br, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aM.lo, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aM.lo, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aM.v, bl, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(aM.v, bh, acc, 0, 0, 0);
    } else {
      // hi/lo split of both operands: Kh yh + Kh yl + Kl yh, the small
      // products first (the dropped Kl yl is below 2^-22 of |K||y|; the low
      // parts come scaled by kF16LoScale)
      float df = 0.0f;
      hfx4 bh, bl;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        bh[t] = (_Float16)b[t];
        const float yh = (float)bh[t];
        bl[t] = (_Float16)((b[t] - yh) * kF16LoScale);
        df = fmaf(fd.c[t], fmaf((float)bl[t], kF16LoUnscale, yh), fmaf(fd.cl[t], yh, df));
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x16f16(aM.lo, bh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x16f16(aM.v, bl, acc, 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] *= kF16LoUnscale;   // exact: a power of two
      acc = __builtin_amdgcn_mfma_f32_16x16x16f16(aM.v, bh, acc, 0, 0, 0);
      // the cell's defect over the four lanes that hold its nodes
      df += __shfl_xor(df, 16, 64);
      df += __shfl_xor(df, 32, 64);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = fmaf(-df, fd.iwh, acc[t] * fd.rs[t]);
    }
    // results of these 16 cells take the place of their values
    if (NG == 4 || g < NG) Q4[64 * cb + r] = acc;
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const flt4 q = Q4[own + (g ^ sw)];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (4 * g + t < H) OUT[4 * g + t] = PREC == kPrecF16 ? q[t] * isc : q[t];
  }
  __builtin_amdgcn_wave_barrier();
}

// waves per SIMD the registers are fitted to: y^n, its correction word, the
// increment and the sources take 7 H registers per lane with two slots, 4 H
// with one
constexpr int mixed_waves(int H, int slots) { return H <= 8 ? 4 : 3; }

// The force block on the matrix cores: FP32 at Q = 16 (below, the vector ALU does
// without the padding to 16), the other forms above four nodes: a block of 2 x 2
// or 4 x 4 is 16 to 64 times padding there, and takes FP32 vector arithmetic in
// every form (64 channels of 16384 cells, BF16: Q = 2 193 -> 105, Q = 4 245 -> 166
// us a step).
template <int Q, int PREC>
constexpr bool mixed_mfma() { return PREC == kPrecF32 ? Q == 16 : Q > 4; }

// LDS of a window (bytes): the moment partials, the equilibrium populations,
// a tile per wave for the force block.  At H = 16, and for f alone, the tiles
// lie in the memory of the partials (two slots): 48 KB, three blocks per CU, where 60 KB
// would leave two (f alone, Q = 6: 20 KB, seven blocks of two waves, not five).
template <int Q, int NFUN, int PREC, int SLOTS>
struct MixedLds {
  static constexpr bool kMfma = mixed_mfma<Q, PREC>();
  static constexpr bool kAlias = kMfma && (Q > 12 || NFUN == 1);
  static constexpr int kTile = 64 * 16 * 4;
  static constexpr int part = 2 * step_sums(NFUN) * 64 * SLOTS * 8;
  static constexpr int tiles = kMfma ? 2 * NFUN * kTile : 0;
  static constexpr int tile_at = kAlias ? 0 : part;
  static constexpr int geq_at = kAlias ? (tiles > part ? tiles : part) : part + tiles;
  static constexpr int nw_at = geq_at + 2 * SLOTS * Q * 64 * 8;
  static constexpr int bytes = nw_at + 2 * 8;
};

// nsteps steps of nst stages of one window, run by a block of 2 NFUN waves
// (3; or 1: one forward-Euler stage, whose increment goes to the output, for
// the residual).
template <int Q, int NFUN, int ADV, int PREC, int SLOTS>
__global__ __launch_bounds__(128 * NFUN) __attribute__((amdgpu_waves_per_eu(mixed_waves(Q, SLOTS)))) void
step_kernel_mixed(StageArgs A, const DevTables *__restrict__ tb, const DevChannel *__restrict__ chans,
                  const DevFusedWindow *__restrict__ wins, const double *__restrict__ inv_dx,
                  const double *__restrict__ gw, const float *__restrict__ in_f, const float *__restrict__ in_c) {
  using L = MixedLds<Q, NFUN, PREC, SLOTS>;
  constexpr int H = Q, P = step_cells(SLOTS);
  constexpr bool kMfmaEq = step_mfma<0, Q>();
  constexpr bool kMfmaK = L::kMfma, kAlias = L::kAlias;
  __shared__ __align__(16) char s_lds[L::bytes];
  const DevFusedWindow win = wins[A.xcd_map ? xcd_window(blockIdx.x, A.nwin) : (int)blockIdx.x];
  ConstTables tp = (ConstTables)tb;
  ConstChannel cp = (ConstChannel)(chans + win.ch);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hw = wv & 1, fn = NFUN > 1 ? wv >> 1 : 0;
  const int lane = threadIdx.x & 63;
  const int pl = hw ? 63 - lane : lane;                 // index of the lane's cells in the shared arrays
  const int Nx = cp->Nx, c0 = win.c0;
  const double sg = hw ? -1.0 : 1.0;
  double *s_part = (double *)s_lds;
  float *s_tile = (float *)(s_lds + L::tile_at + wv * L::kTile);
  double *s_geq = (double *)(s_lds + L::geq_at), *s_nw = (double *)(s_lds + L::nw_at);
  // plane (position modulo the slots) and cell of each slot (the first, of one)
  const int plane[2] = {SLOTS == 1 ? 0 : hw, 1 - hw};
  const int i[2] = {hw ? c0 + (P - 1) - SLOTS * lane : c0 + SLOTS * lane,
                    hw ? c0 + (P - 2) - SLOTS * lane : c0 + SLOTS * lane + 1};
  const int first = win.i0 - c0, last = first + win.nout - 1;   // output positions
  const bool needL = c0 < 0, needR = Nx - 1 - c0 <= P - 1 - kStepGhosts;
  const bool down = hw ? needL : needR, up = hw ? needR : needL;

  const int w0 = c0 < 0 ? 0 : c0, w1 = c0 + P < Nx ? c0 + P : Nx;
  const uint32_t wcells = (uint32_t)(w1 - w0);
  uint32_t cell[SLOTS];   // index in the window's rows; huge where the position has no cell
  bool inside[SLOTS];
  double dxi[SLOTS];
  const int64_t obase = cp->off + (int64_t)(hw * H) * Nx + w0;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    inside[s] = i[s] >= 0 && i[s] < Nx;
    cell[s] = inside[s] ? (uint32_t)(i[s] - w0) : 0x0fffffffu;
    dxi[s] = row_load(row_rsrc(inv_dx + cp->cell_off + w0, wcells * 8u), cell[s] * 8u);
  }
  // reach of the correction rule `lane`
  const double lad = tb->lad_y[lane < kLadderAll ? lane : kLadderAll - 1];

  // y^n as hi + lo (two correction words to a register) and the increment
  // d = y_s - y^n of the stage.  Where a position has no cell hi and lo are
  // zero, and a ghost's value stands in d.
  float hi[H][SLOTS], d[H][SLOTS];
  unsigned lo[H];
  {
    RowWalk w(fn == 0 ? in_f : in_c, obase, 4), wl(fn == 0 ? A.lo_in_f : A.lo_in_c, obase, 2);
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const __amdgpu_buffer_rsrc_t r = w.take((int64_t)Nx * 4, wcells * 4u);
      // the one stage for the residual reads no correction words
      const __amdgpu_buffer_rsrc_t rl = wl.take((int64_t)Nx * 2, A.nst == 1 ? 0u : wcells * 2u);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        hi[j][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, cell[s] * 4u, 0, 0));
        d[j][s] = 0.0f;
      }
      lo[j] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rl, cell[0] * 2u, 0, 0);
      if constexpr (SLOTS == 2)
        lo[j] |= (unsigned)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rl, cell[1] * 2u, 0, 0) << 16;
    }
  }

  int wide = 0;   // evaluations whose correction lay beyond the calibrated ladder
#pragma unroll 1
  for (int it = 0; it < A.nsteps * A.nst; ++it) {
    const int st = A.nst == 1 ? 0 : it % 3;
    const double b_s = st == 0 ? 1.0 : (st == 1 ? 0.25 : 2.0 / 3.0);   // 1 - a_s
    // positions whose result is still exact after this stage
    const int left = 3 * (A.nst - 1 - st);
    const int lo_q = needL ? 0 : first - left, hi_q = needR ? P - 1 : last + left;

    // ---- closure, part 1: ghosts of the nodes flowing into a wall are
    // extrapolated quadratically from the three nearest cells (Sec. IV.C.3);
    // the wall density from the incoming wall-face fluxes, balanced in FP64 ----
    double nw_mine = 0.0;
    if (down) {
      int ln = lane;   // what the closure needs of the lane is formed anew, not kept through the steps
      asm volatile("" : "+v"(ln));
      const int pd = hw ? P - 1 + c0 : Nx - 1 - c0;   // wind position of the wall cell
      const int lp = SLOTS == 2 ? pd >> 1 : pd;
      const bool odd = pd & 1;
      float c_[3][SLOTS];
      bool ghost[SLOTS];
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        const int gi = SLOTS * ln + s - pd;   // ghost order 1, 2 (else <= 0)
        ghost[s] = gi == 1 || gi == 2;
        c_[0][s] = gi == 1 ? 3.0f : 6.0f;
        c_[1][s] = gi == 1 ? -3.0f : -8.0f;
        c_[2][s] = gi == 1 ? 1.0f : 3.0f;
      }
      float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        float y0, y1, y2;
        const float ye = hi[j][0] + d[j][0];
        if constexpr (SLOTS == 1) {
          y0 = readlane_f(ye, lp);
          y1 = readlane_f(ye, lp - 1);
          y2 = readlane_f(ye, lp - 2);
        } else {
          const float yo = hi[j][1] + d[j][1];
          const float e0 = readlane_f(ye, lp), o0 = readlane_f(yo, odd ? lp : lp - 1), e1 = readlane_f(ye, lp - 1),
                      o1 = readlane_f(yo, lp - 1);
          y0 = odd ? o0 : e0;
          y1 = odd ? e0 : o0;
          y2 = odd ? o1 : e1;
        }
        if (ln == j) { a0 = y0; a1 = y1; a2 = y2; }
        // taken here: sunk to where the f wave uses them, every node's values
        // would stay in scalar registers (Q = 16: 100 of them spilled)
        if constexpr (H > 12) asm volatile("" : "+v"(a0), "+v"(a1), "+v"(a2));
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
          if (ghost[s]) d[j][s] = fmaf(c_[2][s], y2, fmaf(c_[1][s], y1, c_[0][s] * y0));
      }
      if (fn == 0) {
        const double d0 = a0, d1 = a1, d2 = a2;
        const double g1 = fma(3.0, d0 - d1, d2), g2 = fma(6.0, d0, fma(-8.0, d1, 3.0 * d2));
        const double fv = face_value<ADV>(d2, d1, d0, g1, g2);
        // flux p_k f_k = (w_k p_k) phi_k, with the FP32 velocities of the
        // advection so that the balance holds for the fluxes the stage applies
        const double acc = row_sum16(ln < H ? tb->wpfq[ln < H ? ln : 0] * fv : 0.0);
        nw_mine = -sg * acc * (hw ? cp->inv_DL : cp->inv_DR);
      }
    }

    // ---- partial moments of this half (FP64) and the rank-1 force projections ----
    asm volatile("" : "+s"(tp), "+s"(cp));
    auto part = [&](int h, int q, int s) -> double & {
      return s_part[((h * step_sums(NFUN) + q) * SLOTS + plane[s]) * 64 + pl];
    };
    {
      double m0[SLOTS] = {}, mb[SLOTS] = {};
      if (fn == 0) {   // uniform over the wave
        double m1[SLOTS] = {}, m2[SLOTS] = {};
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) {
            const double y = hi[j][s] + d[j][s];
            m0[s] = fma(tp->wq[j], y, m0[s]);
            m1[s] = fma(tp->wpq[j], y, m1[s]);
            m2[s] = fma(tp->wp2q[j], y, m2[s]);
            mb[s] = fma(tp->kbs[j], y, mb[s]);
          }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          part(hw, 0, s) = m0[s];
          part(hw, 1, s) = sg * m1[s];
          part(hw, 2, s) = m2[s];
          part(hw, 3, s) = mb[s];
        }
      } else {
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) {
            const double y = hi[j][s] + d[j][s];
            m0[s] = fma(tp->wq[j], y, m0[s]);
            mb[s] = fma(tp->kbs[j], y, mb[s]);
          }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          part(hw, 4, s) = m0[s];
          part(hw, 5, s) = mb[s];
        }
      }
    }
    if (fn == 0 && lane == 0) s_nw[hw] = nw_mine;
    __syncthreads();

    // ---- closure, part 2: emergent ghosts phi = n_w g^w_k / w_k ----
    if (up) {
      const double nw = s_nw[1 - hw];
      const double sc = fn == 0 ? nw : nw * (cp->half_Dt * (hw ? cp->TR : cp->TL));
      typedef const __attribute__((address_space(4))) double *ConstDoubles;
      ConstDoubles gww = (ConstDoubles)gw + cp->gw_off + (hw ? 3 * H : 0);
      asm volatile("" : "+s"(gww));
      bool gh[SLOTS];
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) gh[s] = hw ? i[s] >= Nx : i[s] < 0;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const float ghost = (float)(sc * gww[j] * tp->iwq[j]);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) d[j][s] = gh[s] ? ghost : d[j][s];
      }
    }
    if (A.nwall && it == A.nsteps * A.nst - 1 && A.nst == 3 && fn == 0 && lane == 0) {
      if (hw == 1 && needL) A.nwall[2 * win.ch] = nw_mine;
      if (hw == 0 && needR) A.nwall[2 * win.ch + 1] = nw_mine;
    }

    // ---- moments (Eq. fmoms), FP64 ----
    double n[SLOTS], u[SLOTS], T[SLOTS];
    float bp[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const double ns = part(0, 0, s) + part(1, 0, s), mom = part(0, 1, s) + part(1, 1, s);
      const double s2 = part(0, 2, s) + part(1, 2, s);
      double ech = 0.0;
      if constexpr (NFUN > 1) ech = part(0, 4, s) + part(1, 4, s);
      bp[s] = (float)(part(0, fn ? 5 : 3, s) + part(1, fn ? 5 : 3, s));
      const double rn = recip(ns);
      n[s] = inside[s] ? ns : 1.0;
      u[s] = inside[s] ? mom * rn : 0.0;
      T[s] = inside[s] ? fma(2.0, ech, fma(-u[s], mom, s2)) * (cp->inv_1pDt * rn) : 1.0;
    }

    // ---- equilibrium populations phi^eq_k / n of this half (FP64): with f
    // and chi, each of the half's two waves takes one slot (of one slot, the f
    // wave) ----
    asm volatile("" : "+s"(tp), "+s"(cp));
    const bool collide = cp->inv_Kn != 0.0;
    if (collide) {
#pragma unroll 1
      for (int e = NFUN > 1 ? fn : 0; e < (NFUN > 1 && (SLOTS == 2 || fn == 0) ? fn + 1 : SLOTS); ++e) {
        double G[Q];
        const int qp = (e == 0 ? plane[0] : plane[SLOTS - 1]) + SLOTS * pl;   // position
        half_range_coeffs<Q>(tp, e == 0 ? u[0] : u[SLOTS - 1], e == 0 ? T[0] : T[SLOTS - 1], sg, lane, lad,
                             (e == 0 ? inside[0] : inside[SLOTS - 1]) && qp >= lo_q && qp <= hi_q, wide, G);
        asm volatile("" : "+s"(tp));
        double *ge = s_geq + (hw * SLOTS + e) * H * 64;
        if constexpr (kMfmaEq) {
          double aH[H / 4];
          mfma_operand<H>(tb->HWss, lane, aH);
#pragma unroll
          for (int l = 0; l < Q; ++l) ge[l * 64 + lane] = G[l];
          mfma_tile<H>(aH, ge, lane);
        } else {
#pragma unroll
          for (int k = 0; k < H; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l < Q; ++l) acc = fma(tp->HWss[k * Q + l], G[l], acc);
            ge[k * 64 + lane] = acc;
          }
        }
      }
    }
    __syncthreads();

    // ---- pass 1: b (d + dt (-F (K y)_k - (y_k - y^eq_k)/tau)) ----
    asm volatile("" : "+s"(tp), "+s"(cp));
    const double bdt = b_s * cp->dt;
    const float b_f = (float)b_s, cF = (float)(-cp->g * sg * bdt);
    float src[H][SLOTS];
    if constexpr (kMfmaK) {
      ForceA<PREC> aK;
      aK.template load<H>(PREC == kPrecF16 ? tb->Ks16 : tb->Ks, lane);
      ForceDefect<PREC> fd;
      fd.template load<H>(tb, lane);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        float y[H], ky[H];
#pragma unroll
        for (int j = 0; j < H; ++j) y[j] = hi[j][s] + d[j][s];
        mfma_force<PREC, H>(aK, fd, y, ky, s_tile, lane);
#pragma unroll
        for (int j = 0; j < H; ++j) src[j][s] = cF * fmaf(tp->kas[j], bp[s], ky[j]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) src[j][s] = 0.0f;
#pragma unroll
      for (int jj = 0; jj < H; ++jj) {
        const float y0 = hi[jj][0] + d[jj][0], y1 = hi[jj][SLOTS - 1] + d[jj][SLOTS - 1];
#pragma unroll
        for (int j = 0; j < H; ++j) {
          src[j][0] = fmaf(tp->Ks[j * H + jj], y0, src[j][0]);
          if constexpr (SLOTS == 2) src[j][1] = fmaf(tp->Ks[j * H + jj], y1, src[j][1]);
        }
      }
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) src[j][s] = cF * fmaf(tp->kas[j], bp[s], src[j][s]);
    }
    if (collide) {
      // BGK term formed in FP64 and rounded once: a rounded y^eq would bias
      // the collision's mass, momentum and energy by one rounding of the
      // equilibrium per step, the same each step in a steady state, while
      // this keeps the error relative to y - y^eq
      double cT[SLOTS], nT[SLOTS];
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        cT[s] = n[s] * cp->inv_Kn * bdt;
        nT[s] = n[s] * cT[s];
        if (fn == 1) nT[s] *= cp->half_Dt * T[s];
      }
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          const double y = hi[j][s] + d[j][s];
          const float v = (float)fma(nT[s], s_geq[((hw * SLOTS + s) * H + j) * 64 + lane], -(cT[s] * y));
          src[j][s] = fmaf(b_f, d[j][s], src[j][s] + v);
        }
    } else {
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) src[j][s] = fmaf(b_f, d[j][s], src[j][s]);
    }
    // keep the finished sources in registers
#pragma unroll
    for (int j = 0; j < H; ++j)
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) asm volatile("" : "+v"(src[j][s]));

    // ---- pass 2: advection (Sec. IV.C.2): the flux difference of a cell from
    // its faces' deviations, v (y_i - y_{i-1}) + (v dev_i - v dev_{i-1}) with
    // i - 1 upwind; a wall's emergent face is the ghost itself (deviation 0) ----
    bool use[SLOTS], wf[SLOTS];
    float sdx[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const int q = plane[s] + SLOTS * pl;
      use[s] = inside[s] && q >= lo_q - 1 && q <= hi_q + 1;
      wf[s] = hw ? i[s] == Nx : i[s] == -1;
      sdx[s] = (float)(-dxi[s] * bdt);
    }
    asm volatile("" : "+s"(tp));
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const float v = fabsf(tp->pf[j]);
      float dm, da, fa, fb;
      if constexpr (SLOTS == 2)
        devs_down2<ADV>(hi[j][0] + d[j][0], hi[j][1] + d[j][1], use[0], use[1], dm, da, fa, fb);
      else
        dev_down1<ADV>(hi[j][0] + d[j][0], use[0], dm, fa);
      if (up) {
        asm volatile("");
        if (wf[0]) fa = 0.0f;
        if constexpr (SLOTS == 2)
          if (wf[1]) fb = 0.0f;
      }
      fa *= v;
      if constexpr (SLOTS == 2) fb *= v;
      const float fu = dpp_shr1f(SLOTS == 2 ? fb : fa);
      d[j][0] = fmaf(sdx[0], fmaf(v, dm, fa - fu), src[j][0]);
      if constexpr (SLOTS == 2) d[j][1] = fmaf(sdx[1], fmaf(v, da, fb - fa), src[j][1]);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) asm volatile("" : "+v"(d[j][s]));
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kAlias) __syncthreads();   // the next partials overwrite the tiles
    if (st == 2) {
#pragma unroll
      for (int j = 0; j < H; ++j) {
        unsigned l2 = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          float hn;
          int16_t ln;
          add_to_state(hi[j][s], (int16_t)(lo[j] >> (16 * s)), d[j][s], hn, ln);
          hi[j][s] = inside[s] ? hn : 0.0f;
          d[j][s] = 0.0f;
          l2 |= (unsigned)(uint16_t)ln << (16 * s);
        }
        lo[j] = l2;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) asm volatile("" : "+v"(hi[j][s]), "+v"(lo[j]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- the window's output cells ----
  bool o[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    o[s] = i[s] >= win.i0 && i[s] < win.i0 + win.nout;
    cell[s] = o[s] ? cell[s] : 0x0fffffffu;
  }
  RowWalk w(fn == 0 ? A.out_f : A.out_c, obase, 4);
  if (A.nst == 1) {
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const __amdgpu_buffer_rsrc_t r = w.take((int64_t)Nx * 4, wcells * 4u);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d[j][s]), r, cell[s] * 4u, 0, 0);
    }
  } else {
    RowWalk wl(fn == 0 ? A.lo_out_f : A.lo_out_c, obase, 2);
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const __amdgpu_buffer_rsrc_t r = w.take((int64_t)Nx * 4, wcells * 4u);
      const __amdgpu_buffer_rsrc_t rl = wl.take((int64_t)Nx * 2, wcells * 2u);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(hi[j][s]), r, cell[s] * 4u, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16((short)(lo[j] >> (16 * s)), rl, cell[s] * 2u, 0, 0);
      }
    }
  }
  if (wide && lane == 0 && A.wide) atomicAdd(A.wide, (unsigned long long)wide);
}

}  // namespace hhlb
