// gfx950 kernel for whole TVD RK-3 steps (the three stages of Eq. rk3) of one
// model class per launch, FP64, half-range (HHLB) and full-range (HLB) models
// with at most 16 nodes per half.
//
// A stage per launch moves 8 array passes per function and step and ran at
// 88 % of a device copy's rate on 256 channels of 16384 cells (Q = 16, 1.57 ms
// a launch): nothing but fewer bytes could speed it up.  Here a window keeps
// y^n and the stage state in registers through the three stages and touches
// memory twice per function and step: y^n in, y^{n+1} out.
//
// Mapping: a block of one wave per momentum half and function (f, chi) holds
// 128 consecutive cells, two neighbouring cells (slots) per lane.  Two cells per
// lane halve the lane shifts of the WENO-5 stencil (10 moves per two faces
// instead of 20) and the share of halo lanes (110 of 128 cells are written,
// where a window of 64 would write 46 of 64), and give every wave two
// independent chains.  The waves of a half share the equilibrium: each evaluates
// it for one of the two cells of its lanes.  The halves meet in LDS: moment
// sums, wall densities, the equilibrium populations (and, full range, the
// populations the dense force matrix couples): two barriers per stage, a third
// for the full range's energy or where tiles share the partials' memory.
//
// Classes of short channels take windows of 64 cells instead, one slot per lane
// (the host weighs the two, see slots_of): most positions of a 128-cell window
// would hold no cell of a 48-cell channel, and the lanes work on them all the
// same.
//
// Window geometry.  Position q holds cell c0 + q.  Each stage's stencil reaches
// 3 cells, so the cells next to a window edge that is not a wall go stale at 3
// per stage: a window writes the cells at least 9 from such an edge.  At a
// wall the closure (Sec. IV.C.3) rebuilds the ghosts from the current stage
// every stage, so nothing is lost there; the faces read the first two ghosts
// only, and a wall sits where those two fit (cell 0 at position 2, cell Nx-1
// at the third position from the end or below).  The host builds each channel's
// windows (step_windows).  A channel that fits one window (Nx <= 124, or 60)
// needs no neighbour at all: such classes take many steps in one launch.
//
// Lanes run down the wind of their half (see weno5_down): wind position
// S l + s of slot s of lane l (S slots) is position S l + s for p > 0 and
// 64 S - 1 - (S l + s) for p < 0.
#pragma once
#include "step_kernels.hpp"

namespace hhlb {

constexpr int kStepHalo = 3 * kHalo;    // stale cells at an edge that is not a wall
constexpr int kStepGhosts = 2;          // ghosts kept beyond a wall
// cells a window of `slots` cells per lane holds, and its output cells: both
// walls in the window, one, none
constexpr int step_cells(int slots) { return 64 * slots; }
constexpr int step_single(int slots) { return step_cells(slots) - 2 * kStepGhosts; }
constexpr int step_wall(int slots) { return step_cells(slots) - kStepGhosts - kStepHalo; }
constexpr int step_inner(int slots) { return step_cells(slots) - 2 * kStepHalo; }

// waves per SIMD the registers are fitted to: y^n, the stage state and the
// sources take 3 H doubles per lane and slot
constexpr int step_waves(int H, int slots) {
  return slots == 1 ? (H <= 12 ? 4 : 3) : (H <= 4 ? 4 : (H <= 8 ? 3 : 2));
}

// One window: channel, first output cell, cell of position 0 and the number
// of output cells.
struct DevFusedWindow {
  int32_t ch, i0, c0, nout;
};
struct DevFusedClassWindow {
  int32_t ch, i0, c0, nout;
  int32_t cls, Q;   // model class (index of its tables) and its order
  int32_t slots;    // cells per lane of the window
  int32_t pad;
};

// Orders whose H x H contractions (equilibrium table, force block) run on the
// matrix cores.
#ifndef HHLB_STEP_MFMA
#define HHLB_STEP_MFMA 16
#endif
template <int QUAD, int Q>
constexpr bool step_mfma() { return QUAD == 0 && Q >= HHLB_STEP_MFMA && Q % 4 == 0; }

// Partial sums of a half and cell: n, momentum, energy and the projection of f;
// with chi its sum and projection.
constexpr int step_sums(int nfun) { return nfun > 1 ? 6 : 4; }

// LDS of a window (doubles): the moment partials of the halves; a tile of H x 64
// per wave for the matrix cores, in the partials' memory; the equilibrium
// populations; every node's population for the dense force matrix.  f alone with
// one slot (kOwnEq): the wave takes the equilibrium from its tile into its
// sources at once, so the tile serves both products (20 KB a block at Q = 16).
template <int QUAD, int Q, int NFUN, int SLOTS>
struct StepLds {
  static constexpr int H = QUAD == 0 ? Q : Q / 2;
  static constexpr bool kMfma = step_mfma<QUAD, Q>();
  static constexpr bool kOwnEq = kMfma && NFUN == 1 && SLOTS == 1;
  static constexpr bool kAlias = kMfma && !kOwnEq;
  static constexpr int part = 2 * step_sums(NFUN) * 64 * SLOTS;
  static constexpr int tiles = kMfma ? 2 * NFUN * H * 64 : 0;
  static constexpr int tile_at = kAlias ? 0 : part;
  static constexpr int geq_at = kAlias ? (tiles > part ? tiles : part) : part + tiles;
  static constexpr int y_at = geq_at + (kOwnEq ? 0 : 2 * SLOTS * H * 64);
  static constexpr int nw_at = y_at + (QUAD == 0 ? 0 : NFUN * 2 * H * 64 * SLOTS);
  static constexpr int doubles = nw_at + 2;
};

// Register layout of v_mfma_f64_16x16x4f64 (checked on the GPU):
//   A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
//   D[i][j] in lane j + 16 (i % 4), accumulator register i / 4.
// X[i][cell] <- sum_k M[i][k] X[k][cell] for the H x H table M (A operands
// aM[kc] = M[lane % 16][4 kc + lane / 16], zero outside) and the H rows of 64
// cells of a tile in LDS, in place.  Node-major rows serve all four accesses
// (a lane's own cell, B operand, D result, own cell again) without padding:
// every 16 lanes touch one run of 128 bytes.
template <int H>
__device__ __forceinline__ void mfma_tile(const double *aM, double *T, int lane) {
  constexpr int KC = H / 4;
  __builtin_amdgcn_wave_barrier();
  dbl4 acc[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    acc[cb] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(aM[kc], T[(4 * kc + (lane >> 4)) * 64 + 16 * cb + (lane & 15)],
                                                     acc[cb], 0, 0, 0);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int r = 0; r < KC; ++r) T[(4 * r + (lane >> 4)) * 64 + 16 * cb + (lane & 15)] = acc[cb][r];
  __builtin_amdgcn_wave_barrier();
}
template <int H>
__device__ __forceinline__ void mfma_operand(const double *M, int lane, double *aM) {
  const int i = lane & 15;
#pragma unroll
  for (int kc = 0; kc < H / 4; ++kc) aM[kc] = i < H ? M[(i < H ? i : 0) * H + 4 * kc + (lane >> 4)] : 0.0;
}

// exp(a) for -1/2 <= a <= 0 (the correction rule within its calibrated
// range): the Taylor polynomial of degree 14, remainder below 3e-17, as
// four interleaved polynomials in a^4 (a chain of 6 instead of 14).
__device__ __forceinline__ double exp_small(double a) {
  const double a2 = a * a, a4 = a2 * a2;
  const double p0 = fma(a4, fma(a4, fma(a4, 1.0 / 479001600, 1.0 / 40320), 1.0 / 24), 1.0);
  const double p1 = fma(a4, fma(a4, fma(a4, 1.0 / 6227020800.0, 1.0 / 362880), 1.0 / 120), 1.0);
  const double p2 = fma(a4, fma(a4, fma(a4, 1.0 / 87178291200.0, 1.0 / 3628800), 1.0 / 720), 0.5);
  const double p3 = fma(a4, fma(a4, 1.0 / 39916800, 1.0 / 5040), 1.0 / 6);
  return fma(a2, fma(a, p3, p2), fma(a, p1, p0));
}

// 1/sqrt(x) for normal, finite x > 0: the hardware estimate refined by two
// Newton-Raphson steps.
__device__ __forceinline__ double rsqrt_full(double x) {
  double r = __builtin_amdgcn_rsq(x);
  double e = fma(-x * r, r, 1.0);
  r = fma(0.5 * r, e, r);
  e = fma(-x * r, r, 1.0);
  return fma(0.5 * r, e, r);
}

// Sum over the first 16 lanes (lanes 16.. hold zero), returned as a scalar.
__device__ __forceinline__ double row_sum16(double x) {
#define HHLB_ROW_ADD(ctrl)                                                                              \
  x += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), ctrl, 0xf, 0xf, true),        \
                        __builtin_amdgcn_update_dpp(0, __double2loint(x), ctrl, 0xf, 0xf, true))
  HHLB_ROW_ADD(0x111);   // row_shr:1, 2, 4, 8
  HHLB_ROW_ADD(0x112);
  HHLB_ROW_ADD(0x114);
  HHLB_ROW_ADD(0x118);
#undef HHLB_ROW_ADD
  return readlane_d(x, 15);
}

// Largest of the wave's non-negative values, rounded up to FP32 (compared as
// integers: the bits of non-negative floats order like them).
__device__ __forceinline__ float wave_max_up(double x) {
  const float up = (float)x * 1.0000002f;
  unsigned m = up > 0.0f ? __float_as_uint(up) : 0u;   // NaN counts as zero
#define HHLB_ROW_MAX(ctrl, rows)                                                                  \
  {                                                                                               \
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, ctrl, rows, 0xf, false);  \
    m = o > m ? o : m;                                                                            \
  }
  HHLB_ROW_MAX(0x111, 0xf)
  HHLB_ROW_MAX(0x112, 0xf)
  HHLB_ROW_MAX(0x114, 0xf)
  HHLB_ROW_MAX(0x118, 0xf)
  HHLB_ROW_MAX(0x142, 0xa)   // row_bcast:15 into rows 1 and 3
  HHLB_ROW_MAX(0x143, 0xc)   // row_bcast:31 into rows 2 and 3
#undef HHLB_ROW_MAX
  return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)m, 63));
}

// Equilibrium coefficients G_l (l < Q) of one half at a lane's (u, T) by the
// exact change of variables (Sec. IV.B.3): main rule over [0, inf) and a
// correction over [y0, 0] (monic recurrence; the normalisation is folded into
// the table the coefficients meet).  sg is the half's sign, lad the reach of
// ladder entry `lane`, `used` marks the lanes whose result counts; an
// evaluation beyond the calibrated ladder is counted in `wide`.
template <int Q>
__device__ __forceinline__ void half_range_coeffs(ConstTables tp, double ue, double Te, double sg, int lane, double lad,
                                                  bool used, int &wide, double (&G)[Q]) {
#pragma unroll
  for (int l = 0; l < Q; ++l) G[l] = 0.0;
  const double rT = rsqrt_full(Te);
  const double ub = sg * ue * tp->inv_p0, sc = Te * rT * tp->inv_p0, y0 = -ue * rT;
  auto accum = [&](double x, double wt) {
    double qm = 1.0, q = x - tp->a[0];
    G[0] += wt;
    if (Q > 1) G[1] = fma(wt, q, G[1]);
#pragma unroll
    for (int l = 1; l + 1 < Q; ++l) {
      const double qn = fma(x - tp->a[l], q, -(tp->mb[l] * qm));
      qm = q; q = qn;
      G[l + 1] = fma(wt, q, G[l + 1]);
    }
  };
  const int nm = tp->nm;
#pragma unroll 2
  for (int j = 0; j < nm; ++j) accum(fma(sc, tp->zm[j], ub), tp->wm[j]);
  // correction: the smallest ladder entry that covers the wave's
  // largest |y0| (the last when none does, also for a non-finite one)
  const float ymax = wave_max_up(used ? fabs(y0) : 0.0);
  if (ymax == 0.0f) return;
  const unsigned long long reach =
      __ballot(lane >= 1 && (lane == kLadderAll - 1 || (lane < kLadderAll && lad >= (double)ymax)));
  const int li = __ffsll(reach) - 1;
  const int nc = tp->lad_n[li], o = tp->lad_off[li];
  if (nc > tp->lad_n[kLadder - 1]) ++wide;
  const double sy = -sg * y0, hy = -0.5 * y0 * y0;
  if (ymax <= 1.000001f) {
#pragma unroll 2
    for (int j = 0; j < nc; ++j) {
      const double t = tp->ltau[o + j];
      accum(fma(-ub, t, ub), sy * tp->llamw[o + j] * exp_small(hy * (t * t)));
    }
  } else {
#pragma unroll 1
    for (int j = 0; j < nc; ++j) {
      const double t = tp->ltau[o + j];
      accum(fma(-ub, t, ub), sy * tp->llamw[o + j] * exp(hy * (t * t)));
    }
  }
}

// WENO-5 values at the downwind faces of a lane's two cells (wind positions
// 2 l and 2 l + 1): weno5_down with the differences the two faces share
// formed once, and one branch for the rare rescaling of either.
struct WenoWeights {
  double sL, sC, sR, pL, pC, pR, dd;
  __device__ __forceinline__ void products(double a, double b, double c) {
    const double q1 = a * a, q2 = b * b, q3 = c * c;
    pL = q2 * q3; pC = q1 * q3; pR = q1 * q2;
    dd = fma(0.5, pR, fma(1.0 / 6.0, pL, pC));
  }
  __device__ __forceinline__ void form(double dm, double dp, double DL, double D, double DR, double qL, double qD,
                                       double qR) {
    constexpr double h = 0.5 / kSq1312;
    const double tL = fma(h, DL, dm), tC = fma(h, D, dm), tR = fma(-h, DR, dp);
    sL = fma(tL, tL, qL); sC = fma(tC, tC, qD); sR = fma(tR, tR, qR);
    products(sL, sC, sR);
  }
  __device__ __forceinline__ bool regular() const { return dd > 1e-260 && dd < 1e260; }
  __device__ __forceinline__ void rescale() {
    const int ex = __builtin_amdgcn_frexp_exp(fmax(sL, fmax(sC, sR)));
    const double rL = ldexp(sL, -ex), rC = ldexp(sC, -ex), rR = ldexp(sR, -ex);
    products(rL, rC, rR);
    if (!(dd > 1e-250)) {
      const double tiny = 1e-125;
      pL = rL * rL < tiny ? 1.0 : 0.0;
      pC = rC * rC < tiny ? 1.0 : 0.0;
      pR = rR * rR < tiny ? 1.0 : 0.0;
      dd = fma(0.5, pR, fma(1.0 / 6.0, pL, pC));
    }
  }
  __device__ __forceinline__ double face(double dm, double dp, double dLD, double dDR, double y) const {
    const double r = __builtin_amdgcn_rcp(dd), e = fma(-dd, r, 1.0), e2 = fma(e, e, e);
    double m = fma(1.5, pR * dDR, pL * dLD) * r;
    m = fma(m, e2, m);
    return fma(1.0 / (18.0 * kSq1312), m, fma(1.0 / 3.0, dp, fma(1.0 / 6.0, dm, y)));
  }
};

// The same for G nodes at once: one branch for all of them, so that their
// chains interleave.
template <int ADV, int G>
__device__ __forceinline__ void faces_down2(const double (&ya)[G], const double (&yb)[G], bool usedA, bool usedB,
                                            double (&fa)[G], double (&fb)[G]) {
  double da[G], db[G], dm[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    da[g] = yb[g] - ya[g];
    db[g] = dpp_shl1(ya[g]) - yb[g];
    dm[g] = dpp_shr1(db[g]);
  }
  if constexpr (ADV == 0) {
    WenoWeights wa[G], wb[G];
    double dl[G], dab[G], dr[G];
    bool odd = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double Da = kSq1312 * (da[g] - dm[g]), Db = kSq1312 * (db[g] - da[g]);
      const double Dl = dpp_shr1(Db), Dr = dpp_shl1(Da);
      const double qa = Da * Da, qb = Db * Db;
      wa[g].form(dm[g], da[g], Dl, Da, Db, Dl * Dl, qa, qb);
      wb[g].form(da[g], db[g], Da, Db, Dr, qa, qb, Dr * Dr);
      dl[g] = Dl - Da;
      dab[g] = Da - Db;
      dr[g] = Db - Dr;
      odd |= (!wa[g].regular() && usedA) || (!wb[g].regular() && usedB);
    }
    if (odd) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        wa[g].rescale();
        wb[g].rescale();
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      fa[g] = wa[g].face(dm[g], da[g], dl[g], dab[g], ya[g]);
      fb[g] = wb[g].face(da[g], db[g], dab[g], dr[g], yb[g]);
    }
  } else {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      fa[g] = fma(1.0 / 3.0, da[g], fma(1.0 / 6.0, dm[g], ya[g]));
      fb[g] = fma(1.0 / 3.0, db[g], fma(1.0 / 6.0, da[g], yb[g]));
    }
  }
}

// The faces of one cell per lane, of G nodes.
template <int ADV, int G>
__device__ __forceinline__ void faces_down1(const double (&y)[G], bool used, double (&f)[G]) {
  double dp[G], dm[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    dp[g] = dpp_shl1(y[g]) - y[g];
    dm[g] = dpp_shr1(dp[g]);
  }
  if constexpr (ADV == 0) {
    WenoWeights w[G];
    double dl[G], dr[G];
    bool odd = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double D = kSq1312 * (dp[g] - dm[g]), Dl = dpp_shr1(D), Dr = dpp_shl1(D);
      w[g].form(dm[g], dp[g], Dl, D, Dr, Dl * Dl, D * D, Dr * Dr);
      dl[g] = Dl - D;
      dr[g] = D - Dr;
      odd |= !w[g].regular() && used;
    }
    if (odd) {
#pragma unroll
      for (int g = 0; g < G; ++g) w[g].rescale();
    }
#pragma unroll
    for (int g = 0; g < G; ++g) f[g] = w[g].face(dm[g], dp[g], dl[g], dr[g], y[g]);
  } else {
#pragma unroll
    for (int g = 0; g < G; ++g) f[g] = fma(1.0 / 3.0, dp[g], fma(1.0 / 6.0, dm[g], y[g]));
  }
}

// nsteps steps of nst stages (3; or 1: one forward-Euler stage, whose increment
// dt L[y^n] goes to the output, for the residual) of one window, run by a block of 2 NFUN waves.
template <int QUAD, int Q, int NFUN, int ADV, int GROUP, int SLOTS>
__device__ __forceinline__ void step_window(const StageArgs &A, const DevTables *tb, const DevChannel *chans,
                                            const DevFusedWindow win, const double *__restrict__ inv_dx,
                                            const double *__restrict__ gw, const double *__restrict__ in_f,
                                            const double *__restrict__ in_c, double *s_lds) {
  using L = StepLds<QUAD, Q, NFUN, SLOTS>;
  constexpr int H = L::H, P = step_cells(SLOTS);
  constexpr bool kMfma = L::kMfma, kOwnEq = L::kOwnEq, kAlias = L::kAlias;
  ConstTables tp = (ConstTables)tb;
  ConstChannel cp = (ConstChannel)(chans + win.ch);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hw = wv & 1, fn = NFUN > 1 ? wv >> 1 : 0;
  const int lane = threadIdx.x & 63;
  const int pl = hw ? 63 - lane : lane;                 // index of the lane's cells in the shared arrays
  const int Nx = cp->Nx, c0 = win.c0;
  const double sg = hw ? -1.0 : 1.0;
  // Shared arrays: the partials, s_nw and (full range) the populations s_y are
  // written before the first barrier of a stage and read behind it, before the
  // last, so the next stage may write them; the energy's partial and its barrier
  // lie between (full range); s_geq is written before the last barrier and read
  // behind it.  Tiles in the partials' memory are written behind the last barrier
  // and read to the end of the stage, which then ends with a barrier.
  double *s_part = s_lds, *s_tile = s_lds + L::tile_at + wv * H * 64;   // the tile: matrix cores only
  double *s_geq = s_lds + L::geq_at, *s_y = s_lds + L::y_at, *s_nw = s_lds + L::nw_at;
  // plane (position modulo the slots) and cell of each slot (the first, of one)
  const int plane[2] = {SLOTS == 1 ? 0 : hw, 1 - hw};
  const int i[2] = {hw ? c0 + (P - 1) - SLOTS * lane : c0 + SLOTS * lane,
                    hw ? c0 + (P - 2) - SLOTS * lane : c0 + SLOTS * lane + 1};
  const int first = win.i0 - c0, last = first + win.nout - 1;   // output positions
  const bool needL = c0 < 0, needR = Nx - 1 - c0 <= P - 1 - kStepGhosts;
  const bool down = hw ? needL : needR, up = hw ? needR : needL;

  const int w0 = c0 < 0 ? 0 : c0, w1 = c0 + P < Nx ? c0 + P : Nx;
  const uint32_t wbytes = (uint32_t)(w1 - w0) * 8u;
  uint32_t off[SLOTS];
  bool inside[SLOTS];
  double dxi[SLOTS];
  const int64_t obase = cp->off + (int64_t)(hw * H) * Nx + w0;
  const int64_t stride = (int64_t)Nx * 8;
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    inside[s] = i[s] >= 0 && i[s] < Nx;
    off[s] = (uint32_t)(i[s] - w0) * 8u;
    dxi[s] = row_load(row_rsrc(inv_dx + cp->cell_off + w0, wbytes), off[s]);
  }
  double lad = 0.0;   // reach of the correction rule `lane`
  if constexpr (QUAD == 0) lad = tb->lad_y[lane < kLadderAll ? lane : kLadderAll - 1];

  double yn[H][SLOTS], y[H][SLOTS];
  {
    RowWalk w(fn == 0 ? in_f : in_c, obase);
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const __amdgpu_buffer_rsrc_t r = w.take(stride, wbytes);
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) y[j][s] = yn[j][s] = row_load(r, off[s]);
    }
  }

  int wide = 0;   // evaluations whose correction lay beyond the calibrated ladder
#pragma unroll 1
  for (int it = 0; it < A.nsteps * A.nst; ++it) {
    const int st = A.nst == 1 ? 0 : it % 3;
    // Eq. (rk3): y_{s+1} = a_s y^n + b_s (y_s + dt L[y_s])
    const double a_s = st == 0 ? 0.0 : (st == 1 ? 0.75 : 1.0 / 3.0);
    const double b_s = st == 0 ? 1.0 : (st == 1 ? 0.25 : 2.0 / 3.0);
    // positions whose result is still exact after this stage
    const int left = 3 * (A.nst - 1 - st);
    const int lo = needL ? 0 : first - left, hi = needR ? P - 1 : last + left;

    // ---- closure, part 1: ghosts of the nodes flowing into a wall are
    // extrapolated quadratically from the three nearest cells (Sec. IV.C.3)
    // and their wall-face fluxes give the wall density (Eq. nplus_def) ----
    double nw_mine = 0.0;
    if (down) {
      int ln = lane;   // what the closure needs of the lane is formed anew, not kept through the steps
      asm volatile("" : "+v"(ln));
      const int pd = hw ? P - 1 + c0 : Nx - 1 - c0;   // wind position of the wall cell
      const int lp = SLOTS == 2 ? pd >> 1 : pd;
      const bool odd = pd & 1;
      double c_[3][SLOTS];
      bool ghost[SLOTS];
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        const int gi = SLOTS * ln + s - pd;   // ghost order 1, 2 (else <= 0)
        ghost[s] = gi == 1 || gi == 2;
        c_[0][s] = gi == 1 ? 3.0 : 6.0;
        c_[1][s] = gi == 1 ? -3.0 : -8.0;
        c_[2][s] = gi == 1 ? 1.0 : 3.0;
      }
      // lane j gathers node j's three wall-adjacent values; ghost lanes
      // extrapolate every node of this half
      double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        double y0, y1, y2;
        if constexpr (SLOTS == 1) {
          y0 = readlane_d(y[j][0], lp);
          y1 = readlane_d(y[j][0], lp - 1);
          y2 = readlane_d(y[j][0], lp - 2);
        } else {
          const double e0 = readlane_d(y[j][0], lp), o0 = readlane_d(y[j][1], odd ? lp : lp - 1),
                       e1 = readlane_d(y[j][0], lp - 1), o1 = readlane_d(y[j][1], lp - 1);
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
          if (ghost[s]) y[j][s] = fma(c_[2][s], y2, fma(c_[1][s], y1, c_[0][s] * y0));
      }
      if (fn == 0) {
        // incoming wall-face flux of node `lane`, all nodes in parallel
        const double g1 = fma(3.0, a0 - a1, a2), g2 = fma(6.0, a0, fma(-8.0, a1, 3.0 * a2));
        const double fv = face_value<ADV>(a2, a1, a0, g1, g2);
        const double acc = row_sum16(ln < H ? tb->p[ln < H ? ln : 0] * fv : 0.0);
        nw_mine = -sg * acc * (hw ? cp->inv_DL : cp->inv_DR);
      }
    }

    // ---- partial moments of this half and the rank-1 force projections ----
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
            m0[s] += y[j][s];
            m1[s] = fma(tp->p[j], y[j][s], m1[s]);
            if constexpr (QUAD == 0) {
              m2[s] = fma(tp->vv[j], y[j][s], m2[s]);
              mb[s] = fma(tp->kb[j], y[j][s], mb[s]);
            }
          }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          part(hw, 0, s) = m0[s];
          part(hw, 1, s) = sg * m1[s];
          if constexpr (QUAD == 0) {
            part(hw, 2, s) = m2[s];
            part(hw, 3, s) = mb[s];
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) {
            m0[s] += y[j][s];
            if constexpr (QUAD == 0) mb[s] = fma(tp->kb[j], y[j][s], mb[s]);
          }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          part(hw, 4, s) = m0[s];
          if constexpr (QUAD == 0) part(hw, 5, s) = mb[s];
        }
      }
    }
    if constexpr (QUAD == 1) {
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) s_y[((fn * 2 * H + hw * H + j) * SLOTS + plane[s]) * 64 + pl] = y[j][s];
    }
    if (fn == 0 && lane == 0) s_nw[hw] = nw_mine;
    __syncthreads();

    // ---- closure, part 2: emergent ghosts n_w g^w_k ----
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
        const double ghost = sc * gww[j];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) y[j][s] = gh[s] ? ghost : y[j][s];
      }
    }
    if (A.nwall && it == A.nsteps * A.nst - 1 && A.nst == 3 && fn == 0 && lane == 0) {
      if (hw == 1 && needL) A.nwall[2 * win.ch] = nw_mine;
      if (hw == 0 && needR) A.nwall[2 * win.ch + 1] = nw_mine;
    }

    // ---- moments (Eq. fmoms).  Half range: the energy from raw sums.  Full
    // range: about u, its partials behind a barrier of their own (raw sums
    // cancel, 2 to 5 times the rounding of T at |u| near 1) ----
    const bool collide = cp->inv_Kn != 0.0;
    double n[SLOTS], u[SLOTS], T[SLOTS], bp[SLOTS], rn[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const double ns = part(0, 0, s) + part(1, 0, s), mom = part(0, 1, s) + part(1, 1, s);
      bp[s] = QUAD == 0 ? part(0, fn ? 5 : 3, s) + part(1, fn ? 5 : 3, s) : 0.0;
      rn[s] = recip(ns);
      n[s] = inside[s] ? ns : 1.0;
      u[s] = inside[s] ? mom * rn[s] : 0.0;
      T[s] = 1.0;
      if constexpr (QUAD == 0) {
        const double s2 = part(0, 2, s) + part(1, 2, s);
        double ech = 0.0;
        if constexpr (NFUN > 1) ech = part(0, 4, s) + part(1, 4, s);
        if (inside[s]) T[s] = fma(2.0, ech, fma(-u[s], mom, s2)) * (cp->inv_1pDt * rn[s]);
      }
    }
    if constexpr (QUAD == 1) {
      if (collide) {   // uniform over the block
        if (fn == 0) {
          double e2[SLOTS] = {};
#pragma unroll
          for (int j = 0; j < H; ++j)
#pragma unroll
            for (int s = 0; s < SLOTS; ++s) {
              const double c = fma(sg, tp->p[j], -u[s]);
              e2[s] = fma(c * c, y[j][s], e2[s]);
            }
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) part(hw, 2, s) = e2[s];
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          const double e2 = part(0, 2, s) + part(1, 2, s);
          double ech = 0.0;
          if constexpr (NFUN > 1) ech = part(0, 4, s) + part(1, 4, s);
          if (inside[s]) T[s] = fma(2.0, ech, e2) * (cp->inv_1pDt * rn[s]);
        }
      }
    }

    // matrix cores, two slots: the second slot's force block stays in the tile
    // until pass 2 reads it, which keeps H values out of the register file
    constexpr bool kDefer = kMfma && SLOTS == 2;
    constexpr int SREG = kDefer ? 1 : SLOTS;
    double src[H][SREG];

    // ---- equilibrium populations g_k of this half: with f and chi, each of
    // the half's two waves takes one slot (of one slot, the f wave) ----
    asm volatile("" : "+s"(tp), "+s"(cp));
    if (collide) {
#pragma unroll 1
      for (int e = NFUN > 1 ? fn : 0; e < (NFUN > 1 && (SLOTS == 2 || fn == 0) ? fn + 1 : SLOTS); ++e) {
        const double ue = e == 0 ? u[0] : u[SLOTS - 1], Te = e == 0 ? T[0] : T[SLOTS - 1];
        double G[Q];
        if constexpr (QUAD == 0) {
          const int qp = (e == 0 ? plane[0] : plane[SLOTS - 1]) + SLOTS * pl;   // position
          half_range_coeffs<Q>(tp, ue, Te, sg, lane, lad,
                               (e == 0 ? inside[0] : inside[SLOTS - 1]) && qp >= lo && qp <= hi, wide, G);
        } else {
          // closed form (Sec. IV.A.3): G_{l+1} = ub G_l + l a G_{l-1}
          const double aa = fma(Te * tp->inv_p0, tp->inv_p0, -1.0), bb = ue * tp->inv_p0;
          G[0] = 1.0;
          if (Q > 1) G[1] = bb;
#pragma unroll
          for (int l = 1; l + 1 < Q; ++l) G[l + 1] = fma(bb, G[l], ((double)l * aa) * G[l - 1]);
        }
        asm volatile("" : "+s"(tp));
        double *ge = kOwnEq ? s_tile : s_geq + (hw * SLOTS + e) * H * 64;
        if constexpr (kMfma) {
          double aH[H / 4];
          mfma_operand<H>(tb->HWs, lane, aH);
#pragma unroll
          for (int l = 0; l < Q; ++l) ge[l * 64 + lane] = G[l];
          mfma_tile<H>(aH, ge, lane);
        } else {
          const __attribute__((address_space(4))) double *hw_t = QUAD == 0 ? tp->HWs : tp->HW + hw * H * Q;
#pragma unroll
          for (int k = 0; k < H; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l < Q; ++l) acc = fma(hw_t[k * Q + l], G[l], acc);
            ge[k * 64 + lane] = acc;
          }
        }
      }
    }
    if constexpr (kOwnEq) {   // n g_k - y_k
#pragma unroll
      for (int j = 0; j < H; ++j) src[j][0] = collide ? fma(n[0], s_tile[j * 64 + lane], -y[j][0]) : 0.0;
      __builtin_amdgcn_wave_barrier();
    }
    // full range: the other half's populations, read while they are those of
    // this stage (its waves write the next ones behind the barrier)
    double yo[QUAD == 1 ? H : 1][SLOTS];
    if constexpr (QUAD == 1) {
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s)
          yo[j][s] = s_y[((fn * 2 * H + (1 - hw) * H + j) * SLOTS + plane[s]) * 64 + pl];
    }
    __syncthreads();

    // ---- pass 1: b dt (-F (K y)_k + (y^eq_k - y_k)/tau), the difference formed
    // first and b y added last, each rounded once at its own size ----
    asm volatile("" : "+s"(tp), "+s"(cp));
    const double bdt = b_s * cp->dt, b_y = A.nst == 1 ? 0.0 : b_s;   // the one stage for the residual: its increment
    const double cF = -cp->g * (QUAD == 0 ? sg : 1.0) * bdt;
    double cT[SLOTS], nq[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      cT[s] = n[s] * cp->inv_Kn * bdt;
      nq[s] = fn == 1 ? n[s] * (cp->half_Dt * T[s]) : n[s];
    }
    if constexpr (kMfma) {
      double aK[H / 4];
      mfma_operand<H>(tb->Kin, lane, aK);
#pragma unroll
      for (int j = 0; j < H; ++j) s_tile[j * 64 + lane] = y[j][0];
      mfma_tile<H>(aK, s_tile, lane);
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const double k0 = fma(tp->ka[j], bp[0], s_tile[j * 64 + lane]);
        src[j][0] = kOwnEq ? fma(cT[0], src[j][0], cF * k0) : k0;
      }
      if constexpr (kDefer) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < H; ++j) s_tile[j * 64 + lane] = y[j][1];
        mfma_tile<H>(aK, s_tile, lane);
      }
    } else if constexpr (QUAD == 0) {
#pragma unroll
      for (int j = 0; j < H; ++j) {
        double k_[SLOTS];
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) k_[s] = tp->ka[j] * bp[s];
#pragma unroll
        for (int jj = 0; jj < H; ++jj)
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) k_[s] = fma(tp->Kin[j * H + jj], y[jj][s], k_[s]);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) src[j][s] = k_[s];
      }
    } else {
      const __attribute__((address_space(4))) double *Kr = tp->Kin + hw * H * Q;
#pragma unroll
      for (int j = 0; j < H; ++j) {
        double k_[SLOTS] = {};
#pragma unroll
        for (int jj = 0; jj < H; ++jj) {
          const double ks = Kr[j * Q + hw * H + jj], ko = Kr[j * Q + (1 - hw) * H + jj];
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) k_[s] = fma(ko, yo[jj][s], fma(ks, y[jj][s], k_[s]));
        }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) src[j][s] = k_[s];
      }
    }
    if constexpr (!kOwnEq) {
      if (collide) {
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
          for (int s = 0; s < SREG; ++s) {
            const double geq = s_geq[((hw * SLOTS + s) * H + j) * 64 + lane];
            src[j][s] = fma(cT[s], fma(nq[s], geq, -y[j][s]), cF * src[j][s]);
          }
      } else {
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
          for (int s = 0; s < SREG; ++s) src[j][s] *= cF;
        if constexpr (kDefer) {   // pass 2 reads the second slot's equilibrium
#pragma unroll
          for (int j = 0; j < H; ++j) s_geq[((hw * SLOTS + 1) * H + j) * 64 + lane] = 0.0;
        }
      }
    }

    // ---- pass 2: advection (WENO-5 / upwind-3 face fluxes, Sec. IV.C.2) and
    // the RK-3 combination into the registers; the faces of node j read only
    // node j's values, so y[j] is replaced once its fluxes are formed ----
    // position, use and scale of each slot
    bool use[SLOTS], wf[SLOTS];
    double sdx[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const int q = plane[s] + SLOTS * pl;
      use[s] = inside[s] && q >= lo - 1 && q <= hi + 1;
      wf[s] = hw ? i[s] == Nx : i[s] == -1;
      sdx[s] = -dxi[s] * bdt;
    }
    asm volatile("" : "+s"(tp));
#pragma unroll
    for (int j0 = 0; j0 < H; j0 += GROUP) {
      constexpr int G = H % GROUP == 0 ? GROUP : 1;
      static_assert(G == GROUP || GROUP == 1, "whole groups");
      double ya[G], yb[G], fa[G], fb[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        ya[g] = y[j0 + g][0];
        yb[g] = y[j0 + g][SLOTS - 1];
      }
      if constexpr (SLOTS == 2) faces_down2<ADV, G>(ya, yb, use[0], use[1], fa, fb);
      else faces_down1<ADV, G>(ya, use[0], fa);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int j = j0 + g;
        const double v = tp->p[j];
        if (up) {   // the emergent flux at the wall is the wall's own
          asm volatile("");
          if (wf[0]) fa[g] = ya[g];
          if constexpr (SLOTS == 2)
            if (wf[1]) fb[g] = yb[g];
        }
        const double fu = dpp_shr1(SLOTS == 2 ? fb[g] : fa[g]);
        y[j][0] = fma(a_s, yn[j][0], fma(b_y, ya[g], fma(sdx[0] * v, fa[g] - fu, src[j][0])));
        if constexpr (SLOTS == 2) {
          double src1;
          if constexpr (kDefer) {
            const double k1 = fma(tp->ka[j], bp[1], s_tile[j * 64 + lane]);
            const double geq = s_geq[((hw * SLOTS + 1) * H + j) * 64 + lane];
            src1 = fma(cT[1], fma(nq[1], geq, -yb[g]), cF * k1);
          } else {
            src1 = src[j][1];
          }
          y[j][1] = fma(a_s, yn[j][1], fma(b_y, yb[g], fma(sdx[1] * v, fb[g] - fa[g], src1)));
        }
        // keep the update here: sunk below the later nodes it would hold their
        // faces and y^n at once
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) asm volatile("" : "+v"(y[j][s]));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kAlias) __syncthreads();   // the next partials overwrite the tiles
    if (st == 2 && it + 1 < A.nsteps * A.nst) {
#pragma unroll
      for (int j = 0; j < H; ++j)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) yn[j][s] = y[j][s];
    }
  }

  // ---- the window's output cells ----
  uint32_t oo[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) oo[s] = i[s] >= win.i0 && i[s] < win.i0 + win.nout ? off[s] : 0xffffffffu;
  RowWalk w(fn == 0 ? A.out_f : A.out_c, obase);
#pragma unroll
  for (int j = 0; j < H; ++j) {
    const __amdgpu_buffer_rsrc_t r = w.take(stride, wbytes);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) row_store(r, oo[s], y[j][s]);
  }
  if (wide && lane == 0 && A.wide) atomicAdd(A.wide, (unsigned long long)wide);
}

// Two forms.  With many windows the registers are fitted to step_waves and the
// faces formed a node at a time; with FEW the whole register file serves the
// one or two blocks a CU holds anyway and the faces of two nodes interleave
// (their chains bound a lone wave: at Q = 8 the advection takes 8900 of a
// stage's 17000 cycles, 1100 a node for some 100 instructions).  16 steps of one channel
// of 512 cells, Q = 8: 404 -> 372 us, 64 steps of HLB(15;16) 1535 -> 1493 us, 16
// steps of 64 channels, Q = 12: 854 -> 835 us.  Groups of four gained under 1 % on
// the first two and cost a quarter on the third (beyond 256 registers).
constexpr int few_group(int H) { return H % 2 == 0 ? 2 : 1; }
// waves per SIMD that fit with FEW: 4 H doubles per slot and the faces of two
// nodes (f alone at H = 16 holds both tables' operands besides)
constexpr int few_waves(int H, int slots, int nfun) { return H <= 12 || (slots == 1 && nfun > 1) ? 2 : 1; }
template <int QUAD, int Q, int NFUN, int ADV, bool FEW, int SLOTS>
__global__ __launch_bounds__(128 * NFUN)
__attribute__((amdgpu_waves_per_eu(FEW ? 1 : step_waves(QUAD == 0 ? Q : Q / 2, SLOTS)))) void
step_kernel(StageArgs A, const DevTables *__restrict__ tb, const DevChannel *__restrict__ chans,
            const DevFusedWindow *__restrict__ wins, const double *__restrict__ inv_dx,
            const double *__restrict__ gw, const double *__restrict__ in_f, const double *__restrict__ in_c) {
  __shared__ double s_lds[StepLds<QUAD, Q, NFUN, SLOTS>::doubles];
  const int w = A.xcd_map ? xcd_window(blockIdx.x, A.nwin) : (int)blockIdx.x;
  step_window<QUAD, Q, NFUN, ADV, FEW ? few_group(QUAD == 0 ? Q : Q / 2) : 1, SLOTS>(A, tb, chans, wins[w], inv_dx, gw,
                                                                                     in_f, in_c, s_lds);
}

// One launch for the windows of several half-range model classes that share
// the functions and the scheme.  Record b names the window, its class and slots;
// the class's order Q and slots, the same for the whole block, select the code
// (orders up to QTOP).  Persistent form: with fewer blocks than windows each
// block takes windows b, b + gridDim.x, .. in turn.
template <int QTOP, int NFUN, int ADV, bool PERSIST>
__global__ __launch_bounds__(128 * NFUN) __attribute__((amdgpu_waves_per_eu(step_waves(QTOP, 2)))) void
step_kernel_classes(StageArgs A, const DevTables *__restrict__ tbs, const DevChannel *__restrict__ chans,
                    const DevFusedClassWindow *__restrict__ wins, const double *__restrict__ inv_dx,
                    const double *__restrict__ gw, const double *__restrict__ in_f,
                    const double *__restrict__ in_c) {
  __shared__ double s_lds[StepLds<0, QTOP, NFUN, 2>::doubles];
  for (int b = blockIdx.x; b < A.nwin; b += gridDim.x) {
    if (PERSIST && b != (int)blockIdx.x) __syncthreads();   // the last window's LDS reads are done
    const int w = A.xcd_map ? xcd_window(b, A.nwin) : b;
    const DevFusedClassWindow cw = wins[w];
    const DevFusedWindow win{cw.ch, cw.i0, cw.c0, cw.nout};
    const DevTables *tb = tbs + __builtin_amdgcn_readfirstlane(cw.cls);
    switch (__builtin_amdgcn_readfirstlane(2 * cw.Q + cw.slots - 1)) {
#define HHLB_CLASS_CASE(q, slots)                                                              \
  case 2 * q + slots - 1:                                                                      \
    if constexpr (q <= QTOP) {                                                                 \
      static_assert(StepLds<0, q, NFUN, slots>::doubles <= StepLds<0, QTOP, NFUN, 2>::doubles); \
      step_window<0, q, NFUN, ADV, 1, slots>(A, tb, chans, win, inv_dx, gw, in_f, in_c, s_lds); \
    }                                                                                          \
    break;
#define HHLB_CLASS_CASES(slots)                                                                \
  HHLB_CLASS_CASE(1, slots) HHLB_CLASS_CASE(2, slots) HHLB_CLASS_CASE(3, slots) HHLB_CLASS_CASE(4, slots) \
  HHLB_CLASS_CASE(6, slots) HHLB_CLASS_CASE(8, slots) HHLB_CLASS_CASE(12, slots) HHLB_CLASS_CASE(16, slots)
      HHLB_CLASS_CASES(1)
      HHLB_CLASS_CASES(2)
#undef HHLB_CLASS_CASES
#undef HHLB_CLASS_CASE
      default: break;
    }
    if constexpr (!PERSIST) break;   // one window per block
  }
}

}  // namespace hhlb
