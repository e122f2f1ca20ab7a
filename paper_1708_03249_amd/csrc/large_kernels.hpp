// Node-parallel FP64 stage for large velocity sets, equilibrium order
// N <= 20: the half-range model with 17 <= Q <= 256 nodes per half and the
// full-range model with 18 <= Q <= 512 nodes, the paper's HHLB(20;Q) and
// HLB(20;Q) models of the ballistic study (Sec. V.E).  The nodes of a half
// do not fit a lane's registers, so a block takes a tile of 16 nodes of one
// half over a window of at most 58 cells: the force -F (K y)_k contracted on
// FP64 MFMA tiles (half range: the within-half block of Eq. hh_Kk_hh plus the
// rank-1 cross term; full range: the dense matrix of Eq. H_Kk), the wall
// ghosts (Sec. IV.C.3), BGK towards the synthesised equilibrium, WENO-5 /
// upwind-3 advection (faces as in weno5_down) and the RK-3 combination.
//
// What a cell needs of all its nodes (the moments of Eq. fmoms, the rank-1
// projections) and a wall of its incoming ones (Eq. nplus_def) comes as
// partial sums per tile from the stage that wrote the state: each block sums
// over its tile what it has just computed, and the blocks of the next stage
// add up the at most 32 partials of a cell while their operands load.  So a
// stage is one launch.  (As two, a cell phase that read every population
// again took 4.8 us and a launch gap of 1.3 us of a stage's 17.7 us on 8
// channels of 24 cells, Q = 200.)
#pragma once
#include "step_kernels.hpp"

namespace hhlb {

constexpr int kQmaxLarge = 256;   // nodes per half
constexpr int kNmaxLarge = 20;    // equilibrium order
constexpr int kSums = 6;          // partial sums of a cell: n, momentum, energy, chi, the projections of f and chi
constexpr int kTileNodes = 16;
constexpr int kTilesMax = 2 * kQmaxLarge / kTileNodes;

// Tables of one large model class.  Half range: the transposed within-half
// block KinT[j * H + k] = Kin[k][j]; full range (full = 1): the transposed
// dense matrix KT[j * V + k] = K[k][j].  Then HWs[k * (N+1) + l] for the H
// nodes with p > 0.
struct DevLarge {
  int32_t H, N, nm, full;
  double inv_p0;
  double sq[kNmaxLarge + 2];                       // sqrt(l), full range
  double ka[kQmaxLarge], kb[kQmaxLarge];
  double a[kNmaxLarge + 2], mb[kNmaxLarge + 2];   // monic recurrence
  double zm[kQmaxDev], wm[kQmaxDev];               // main rule (half-range Gauss-Hermite)
  int32_t lad_n[kLadderAll], lad_off[kLadderAll];   // calibrated entries, then composite ones
  double lad_y[kLadderAll];
  double ltau[kLadderPts], llamw[kLadderPts];
};

struct LargeArgs {
  const DevLarge *tl;
  const double *KinT, *HWs, *p;   // KinT: KT in the full range; p: V momenta
  const DevChannel *chans;
  const DevWindow *wins;
  int32_t nwin, stage;
  const double *inv_dx, *gw;
  const double *in_f, *in_c;      // stage state
  const double *base_f, *base_c;  // y^n
  double *out_f, *out_c;
  double a_base, b_stage;
  // partial sums of the state read and of the state written: per cell of the
  // class [tile][sum][cell], per wall [tile][channel]
  const double *sums_in, *wall_in;
  double *sums_out, *wall_out;
  int32_t ncells, nch;
  double *nwall;                  // diagnostics copy (written in stage 2)
  unsigned long long *wide;       // cells whose equilibrium needed several correction panels
  int32_t xcd_map;                // 1: the tiles of a window run on one XCD
  int32_t increment;              // 1: out = b dt L[in] (the residual), the sums of which nobody reads
};

// Sum over aligned segments of W lanes (W = 64: the whole wave).
template <int W>
__device__ __forceinline__ double seg_sum(double x) {
#pragma unroll
  for (int off = W / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Equilibrium coefficients of one axis at (u, T) for a segment of W lanes
// (every lane of the segment returns the same G^+_l and G^-_l, l <= N;
// lane = the lane's index within its segment): Sec. IV.B.3 by the change of
// variables, the main rule and the correction spread over the lanes and
// collected by segment sums; for the full range the closed-form recurrence
// of Sec. IV.A.3.  Called by every lane of the wave; W >= 16 holds the main
// rule (at most 11 points for N <= 20) and the largest correction (16).
// NM bounds the order N (the register arrays' size).  Returns whether the
// correction took a composite rule (|y0| beyond the ladder's calibrated
// range).
template <int W = 64, int NM = kNmaxLarge>
__device__ __forceinline__ bool axis_coeffs(const DevLarge *tl, double u, double T, int lane,
                                            double (&Gp)[NM + 1], double (&Gm)[NM + 1]) {
  const int N = tl->N;
#pragma unroll
  for (int l = 0; l <= NM; ++l) Gp[l] = Gm[l] = 0.0;
  if (tl->full) {
    // full range (Sec. IV.A.3): G_l = E[He_l(X)], X ~ N(m u/p0, m T/p0^2),
    // obeys G_{l+1} = ub G_l + l a G_{l-1} with a = m T/p0^2 - 1; kept as
    // G_l / sqrt(l!) against HWs = w_k h_l(z_k) (h_l = He_l / sqrt(l!)).
    // The mirrored half has h_l(-z) = (-1)^l h_l(z).
    const double ub = u * tl->inv_p0, aa = T * tl->inv_p0 * tl->inv_p0 - 1.0;
    Gp[0] = 1.0;
    if (N >= 1) Gp[1] = ub;
#pragma unroll
    for (int l = 1; l < NM; ++l)
      if (l + 1 <= N) Gp[l + 1] = (ub * Gp[l] + tl->sq[l] * aa * Gp[l - 1]) / tl->sq[l + 1];
#pragma unroll
    for (int l = 0; l <= NM; ++l) Gm[l] = (l & 1) ? -Gp[l] : Gp[l];
    return false;
  }
  const double sT = sqrt(T), s = sT * tl->inv_p0, y0 = -u / sT;
  auto accum = [&](double (&G)[NM + 1], double x, double wt) {
    double qm = 1.0, q = x - tl->a[0];
    G[0] += wt;
    if (N >= 1) G[1] += wt * q;
#pragma unroll
    for (int l = 1; l < NM; ++l) {
      if (l + 1 <= N) {
        const double qn = (x - tl->a[l]) * q - tl->mb[l] * qm;
        qm = q;
        q = qn;
        G[l + 1] += wt * q;
      }
    }
  };
  if (lane < tl->nm) {
    accum(Gp, u * tl->inv_p0 + s * tl->zm[lane], tl->wm[lane]);
    accum(Gm, -u * tl->inv_p0 + s * tl->zm[lane], tl->wm[lane]);
  }
  const double ymax = fabs(y0);
  bool wide = false;
  if (ymax > 0.0) {
    // the first entry, calibrated or composite, whose reach covers |y0|
    // (the last when none does, also for a non-finite |y0|)
    int li = kLadderAll - 1;
    for (int j = 1; j < kLadderAll; ++j)
      if (tl->lad_y[j] >= ymax) { li = j; break; }
    const int nc = tl->lad_n[li], o = tl->lad_off[li];
    wide = nc > tl->lad_n[kLadder - 1];
    // the segment's lanes take the entry's points W at a time: one pass
    // for a calibrated count (nc <= 16 <= W), more for a composite rule
    const int passes = (nc + W - 1) / W;
    for (int rr = 0; rr < passes; ++rr) {
      const int q = rr * W + lane;
      if (q < nc) {
        const double t = tl->ltau[o + q], yt = y0 * t;
        const double e = y0 * tl->llamw[o + q] * exp(-0.5 * yt * yt);
        accum(Gp, u * tl->inv_p0 * (1.0 - t), -e);
        accum(Gm, -u * tl->inv_p0 * (1.0 - t), e);
      }
    }
  }
#pragma unroll
  for (int l = 0; l <= NM; ++l) {
    if (l <= N) {
      Gp[l] = seg_sum<W>(Gp[l]);
      Gm[l] = seg_sum<W>(Gm[l]);
    }
  }
  return wide;
}

constexpr int kNodeWaves = 8;                          // waves of a block: they share the contraction's rows
constexpr int kWaveNodes = kTileNodes / kNodeWaves;    // and then the tile's nodes

// Tables and records through the constant address space: scalar loads, which
// do not queue behind the vector loads of the operands.
typedef const __attribute__((address_space(4))) double *ConstDoubles;
typedef const __attribute__((address_space(4))) DevLarge *ConstLarge;
typedef const __attribute__((address_space(4))) DevWindow *ConstWindow;

// A wave's place in the launch: window, tile, and the cells of its lanes.
// Block b maps to a window and a tile of 16 nodes of one half (tiles never
// straddle the halves); with xcd_map the tiles of a window run on one XCD,
// whose L2 then holds the window's rows, which all of them read.
struct LargePlace {
  DevWindow win;
  int ty, hw, kt0, wave, lane, pos, i, k0, ng;
  bool out;
  __device__ __forceinline__ LargePlace(const LargeArgs &A, int H) {
    const int gph = (H + kTileNodes - 1) / kTileNodes, ntile = 2 * gph;
    const int lb = A.xcd_map ? xcd_window(blockIdx.x, A.nwin * ntile) : (int)blockIdx.x;
    ty = lb % ntile;
    ConstWindow w = (ConstWindow)A.wins + lb / ntile;
    win = DevWindow{w->ch, w->i0, w->nout};
    hw = ty / gph;                               // 0: p > 0, 1: p < 0
    kt0 = (ty % gph) * kTileNodes;               // first node of the tile
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lane = threadIdx.x & 63;
    pos = hw ? 63 - lane : lane;                 // lanes run down the wind (see weno5_down)
    i = win.i0 - kHalo + pos;
    k0 = kt0 + wave * kWaveNodes;                // first node of this wave
    ng = H - k0 < 0 ? 0 : (H - k0 < kWaveNodes ? H - k0 : kWaveNodes);
    out = pos >= kHalo && pos < kHalo + win.nout;
  }
};

// What a wave needs of its nodes: velocity (of the half p > 0), projections.
struct LargeNodes {
  double p[kWaveNodes], ka[kWaveNodes], kb[kWaveNodes];
  __device__ __forceinline__ LargeNodes(const LargeArgs &A, const LargePlace &P) {
    ConstLarge tl = (ConstLarge)A.tl;
    ConstDoubles pp = (ConstDoubles)A.p;
#pragma unroll
    for (int q = 0; q < kWaveNodes; ++q) {
      const int k = q < P.ng ? P.k0 + q : 0;
      p[q] = pp[k];
      ka[q] = tl->ka[k];
      kb[q] = tl->kb[k];
    }
  }
};

// Partial sums over the tile of the populations y, x (f and chi) its waves
// hold, valid in the output lanes: through s_sum (kNodeWaves x kSums x 64) and
// s_wall (kNodeWaves) to memory.  Called by every wave of the block.
template <int ADV>
__device__ __forceinline__ void emit_sums(const LargeArgs &A, const LargePlace &P, const LargeNodes &K, int Nx,
                                          int sum_off, int nfun, bool collide, const double (&y)[kWaveNodes],
                                          const double (&x)[kWaveNodes], double *s_sum, double *s_wall) {
  const double sg = P.hw ? -1.0 : 1.0;
  double m[kSums] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < kWaveNodes; ++q) {
    if (q >= P.ng) break;
    const double v = sg * K.p[q], kb = K.kb[q];
    m[0] += y[q];
    m[1] = fma(v, y[q], m[1]);
    m[2] = fma(v * v, y[q], m[2]);
    m[3] += x[q];
    m[4] = fma(kb, y[q], m[4]);
    m[5] = fma(kb, x[q], m[5]);
  }
#pragma unroll
  for (int q = 0; q < kSums; ++q) s_sum[(P.wave * kSums + q) * 64 + P.pos] = m[q];
  // incoming wall-face fluxes of f where the window ends at the wall the half
  // flows into: lane q takes node q's three wall-adjacent values, ghosts
  // extrapolated quadratically from them
  const bool wall = P.hw ? P.win.i0 == 0 : P.win.i0 + P.win.nout == Nx;
  if (wall) {
    const int l0 = P.hw ? 63 - kHalo : kHalo + P.win.nout - 1;   // lane of the wall cell
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, v = 0.0;
#pragma unroll
    for (int q = 0; q < kWaveNodes; ++q) {
      const double y0 = readlane_d(y[q], l0), y1 = readlane_d(y[q], l0 - 1), y2 = readlane_d(y[q], l0 - 2);
      if (P.lane == q && q < P.ng) { a0 = y0; a1 = y1; a2 = y2; v = sg * K.p[q]; }
    }
    const double g1 = 3.0 * a0 - 3.0 * a1 + a2, g2 = 6.0 * a0 - 8.0 * a1 + 3.0 * a2;
    double acc = P.lane < P.ng ? v * face_value<ADV>(a2, a1, a0, g1, g2) : 0.0;
#pragma unroll
    for (int o = 1; o < kWaveNodes; o *= 2) acc += __shfl_xor(acc, o, 64);
    if (P.lane == 0) s_wall[P.wave] = acc;
  }
  __syncthreads();
  for (int q = P.wave; q < kSums; q += kNodeWaves) {
    const int r = P.lane;   // position
    if (((q == 3 || q == 5) && nfun < 2) || (!collide && q < 4)) continue;   // nobody reads these
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kNodeWaves; ++w) v += s_sum[(w * kSums + q) * 64 + r];
    if (r >= kHalo && r < kHalo + P.win.nout)
      A.sums_out[((int64_t)P.ty * kSums + q) * A.ncells + sum_off + P.win.i0 - kHalo + r] = v;
  }
  if (wall && threadIdx.x == 0) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kNodeWaves; ++w) v += s_wall[w];
    A.wall_out[P.ty * A.nch + P.win.ch] = v;
  }
}

// The partial sums of a state that no stage wrote (the first of a call).
template <int ADV, int NFUN>
__global__ __launch_bounds__(64 * kNodeWaves) void large_sums_kernel(LargeArgs A) {
  __shared__ double s_sum[kNodeWaves * kSums * 64], s_wall[kNodeWaves];
  const int H = ((ConstLarge)A.tl)->H;
  const LargePlace P(A, H);
  const LargeNodes K(A, P);
  ConstChannel C = (ConstChannel)A.chans + P.win.ch;
  const int Nx = C->Nx;
  double y[kWaveNodes], x[kWaveNodes];
#pragma unroll
  for (int q = 0; q < kWaveNodes; ++q) {
    const int64_t o = C->off + (int64_t)(P.hw * H + P.k0 + q) * Nx + P.i;
    const bool ok = P.out && q < P.ng;
    y[q] = ok ? A.in_f[o] : 0.0;
    x[q] = NFUN > 1 && ok ? A.in_c[o] : 0.0;
  }
  emit_sums<ADV>(A, P, K, Nx, C->sum_off, NFUN, C->inv_Kn != 0.0, y, x, s_sum, s_wall);
}

// One stage.  The rows of the contraction D[node][cell] = sum_j K[node][j]
// y_j[cell] are split over the block's eight waves in steps of 4, the A
// operand (the transposed table) and the B operand (the rows of f or chi for
// the window's cells) load straight from memory in the MFMA layout, and the
// partial tiles are summed through LDS.  After that wave w owns nodes
// kt0 + 2 w and + 1, its lanes the window's cells in the half's wind order.
//
// Small channels are bound by the chain of memory latencies, so everything a
// stage reads (operands, the waves' own rows, y^n, the partial sums) is
// requested before the first wait, eight waves a block halve the rows of each,
// and NCB counts the 16-cell blocks of the largest window (24 cells and their
// halo: 2, not 4).
template <int ADV, int NCB, int NFUN>
__global__ __launch_bounds__(64 * kNodeWaves) __attribute__((amdgpu_waves_per_eu(2))) void large_stage_kernel(LargeArgs A) {
  constexpr int NG = kWaveNodes, NW = kNodeWaves;
  constexpr int S = 16 * NCB + 1;               // padded LDS row
  constexpr int kSteps = 32 / (NCB * NFUN);               // steps of a chunk: loads issued together
  constexpr int kStepsMax = 2 * kQmaxLarge / 4 / NW;       // of a wave
  constexpr int kRed = NW * kTileNodes * S, kG = NW * (kNmaxLarge + 1) * 64;
  __shared__ double s_red[kRed > kG ? kRed : kG];
  __shared__ double s_sum[NW * kSums * 64], s_wall[NW];
  __shared__ double s_hw[kTileNodes * (kNmaxLarge + 1)];   // HWs rows of the tile
  ConstLarge tl = (ConstLarge)A.tl;
  const int H = tl->H, N = tl->N;
  const LargePlace P(A, H);
  const LargeNodes K(A, P);
  ConstChannel cp = (ConstChannel)A.chans + P.win.ch;
  struct { int64_t off; int32_t Nx, cell_off, sum_off, gw_off; double g, inv_Kn, dt, TL, TR, inv_DL, inv_DR, half_Dt, inv_1pDt; } C{
      cp->off, cp->Nx, cp->cell_off, cp->sum_off, cp->gw_off, cp->g, cp->inv_Kn, cp->dt, cp->TL, cp->TR, cp->inv_DL, cp->inv_DR,
      cp->half_Dt, cp->inv_1pDt};
  const int Nx = C.Nx, hw = P.hw, lane = P.lane, wave = P.wave, i = P.i, k0 = P.k0, ng = P.ng;
  const bool inside = i >= 0 && i < Nx;
  const int ic = inside ? i : (i < 0 ? 0 : Nx - 1);      // clamped: loads stay in bounds
  const bool full = tl->full != 0;
  const double sg = full ? 1.0 : (hw ? -1.0 : 1.0);      // K = blockdiag(Kin, -Kin) + cross (half)
  const int64_t rowh = C.off + (int64_t)hw * H * Nx;     // first row of this half
  // rows of the contraction: the half's H rows, or all V = 2H (full range)
  const int nrows = full ? 2 * H : H;
  const double *rf = A.in_f + (full ? C.off : rowh), *rc = NFUN > 1 ? A.in_c + (full ? C.off : rowh) : nullptr;
  const bool collide = C.inv_Kn != 0.0;
  const int ntile = 2 * ((H + kTileNodes - 1) / kTileNodes);

  // What the block reads, as unconditional loads from clamped addresses: a
  // value selected on arrival is a wait per load.  The waves' own rows and y^n
  // (a clamped node where the wave has none), the partial sums of this wave's
  // share of the tiles, the partial densities of the wall this half flows out
  // of (the other half's tiles).
  double yf[NG], yc[NG], bf0[NG], bc0[NG];
  const bool need_base = A.a_base != 0.0;
  const double *bf = need_base ? A.base_f : A.in_f, *bc = need_base ? A.base_c : A.in_c;
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    const int64_t o = rowh + (int64_t)(q < ng ? k0 + q : H - 1) * Nx + ic;
    yf[q] = A.in_f[o];
    bf0[q] = bf[o];
    yc[q] = bc0[q] = 0.0;
    if constexpr (NFUN > 1) {
      yc[q] = A.in_c[o];
      bc0[q] = bc[o];
    }
  }
  const bool needL = P.win.i0 < kHalo, needR = P.win.i0 - kHalo + 63 >= Nx;
  const bool up = hw ? needR : needL;
  double gwk[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) gwk[q] = ((ConstDoubles)A.gw)[C.gw_off + (hw ? 3 * H : 0) + (q < ng ? k0 + q : 0)];
  const int half = ntile / 2;
  double wsum = A.wall_in[((1 - hw) * half + (lane < half ? lane : 0)) * A.nch + P.win.ch];
  constexpr int NT = kTilesMax / NW;
  double pv[NT][kSums];
  auto tile_sums = [&](int t) {
    const int tile = wave + NW * t < ntile ? wave + NW * t : 0;
    return A.sums_in + (int64_t)tile * kSums * A.ncells + C.sum_off + ic;
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const double *pi = tile_sums(t);
    pv[t][4] = pi[(int64_t)4 * A.ncells];
    if constexpr (NFUN > 1) pv[t][5] = pi[(int64_t)5 * A.ncells];
  }
  if (collide) {   // uniform over the block
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (NFUN > 1 || q != 3) pv[t][q] = tile_sums(t)[(int64_t)q * A.ncells];
  }
  const double dx_inv = A.inv_dx[C.cell_off + ic];

  // the tile's equilibrium rows HWs[k][0..N] (read after the first barrier)
  if (collide)
    for (int t = threadIdx.x; t < kTileNodes * (kNmaxLarge + 1); t += 64 * NW) {
      const int q = t / (kNmaxLarge + 1), l = t % (kNmaxLarge + 1), k = P.kt0 + q;
      s_hw[t] = (k < H && l <= N) ? A.HWs[(int64_t)k * (N + 1) + l] : 0.0;
    }

  // force: MFMA contraction over this wave's share of the rows
  const int nsteps = (nrows + 3) / 4, spw = (nsteps + NW - 1) / NW;
  const int s0 = wave * spw;
  const int nsw = nsteps - s0 < 0 ? 0 : (nsteps - s0 < spw ? nsteps - s0 : spw);
  const int kr = lane >> 4, jl = lane & 15;
  const int an = P.kt0 + jl;                             // A row: node within the half
  const int acol = full ? hw * H + an : an;              // its column of the table
  int bcell[NCB];
#pragma unroll
  for (int c = 0; c < NCB; ++c) {
    const int il = P.win.i0 - kHalo + 16 * c + jl;
    bcell[c] = il < 0 ? 0 : (il >= Nx ? Nx - 1 : il);
  }
  const __amdgpu_buffer_rsrc_t rk = row_rsrc(A.KinT, (uint32_t)(nrows * nrows) * 8u);
  dbl4 acc[NFUN][NCB];
#pragma unroll
  for (int fn = 0; fn < NFUN; ++fn)
#pragma unroll
    for (int c = 0; c < NCB; ++c) acc[fn][c] = dbl4{0.0, 0.0, 0.0, 0.0};
  // Loads past a wave's steps are not used and stay in bounds: past the table
  // they read zero, past the rows they go to row 0.  Columns past H give rows
  // of D that nobody reads.
  const int r0 = 4 * s0 + kr;
  const int64_t ro = (int64_t)(r0 < nrows ? r0 : 0) * Nx, rstep = (int64_t)4 * Nx;
  const uint32_t ka0 = (uint32_t)(r0 * nrows + acol) * 8u, kstep = (uint32_t)nrows * 32u;
#pragma unroll
  for (int t0 = 0; t0 < kStepsMax; t0 += kSteps) {   // a loop would wait for all that is in flight on entry
    if (t0 < nsw) {   // wave-uniform: MFMA runs with every lane active
      double av[kSteps], bv[NFUN][kSteps][NCB];
#pragma unroll
      for (int t = 0; t < kSteps; ++t) {
        av[t] = row_load(rk, ka0 + (uint32_t)(t0 + t) * kstep);
        const int64_t o = r0 + 4 * (t0 + t) < nrows ? ro + (t0 + t) * rstep : 0;
#pragma unroll
        for (int c = 0; c < NCB; ++c) {
          bv[0][t][c] = rf[o + bcell[c]];
          if constexpr (NFUN > 1) bv[1][t][c] = rc[o + bcell[c]];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < kSteps; ++t)
        if (t0 + t < nsw) {
#pragma unroll
          for (int fn = 0; fn < NFUN; ++fn)
#pragma unroll
            for (int c = 0; c < NCB; ++c)
              acc[fn][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t], bv[fn][t][c], acc[fn][c], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int q = 0; q < kSums; ++q) {
    double m = 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if ((NFUN > 1 || (q != 3 && q != 5)) && (collide || q >= 4) && wave + NW * t < ntile) m += pv[t][q];
    s_sum[(wave * kSums + q) * 64 + lane] = m;
  }
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    yf[q] = inside ? yf[q] : 0.0;
    yc[q] = inside ? yc[q] : 0.0;
  }
  wsum = lane < half ? wsum : 0.0;
  // D[node 4r + kr][cell 16c + jl] sits in acc[c][r]; partial tiles to LDS,
  // then wave w sums its NG nodes over the partials
  double kk[NFUN][NG];
#pragma unroll
  for (int fn = 0; fn < NFUN; ++fn) {
    if (fn > 0) __syncthreads();
#pragma unroll
    for (int c = 0; c < NCB; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_red[(wave * kTileNodes + 4 * r + kr) * S + 16 * c + jl] = acc[fn][c][r];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      double v = 0.0;
      const int pc = P.pos < 16 * NCB ? P.pos : 16 * NCB - 1;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += s_red[(w * kTileNodes + wave * NG + q) * S + pc];
      kk[fn][q] = v;
    }
  }
  double mom[kSums];
#pragma unroll
  for (int q = 0; q < kSums; ++q) {
    mom[q] = 0.0;
    if (NFUN < 2 && (q == 3 || q == 5)) continue;
#pragma unroll
    for (int w = 0; w < NW; ++w) mom[q] += s_sum[(w * kSums + q) * 64 + lane];
  }
  __syncthreads();   // the sums below overwrite both

  // ---- moments (Eq. fmoms) and the equilibrium coefficients of this half
  // (half range: Sec. IV.B.3 by the change of variables of half_range_coeffs,
  // the points shared among the waves; full range: the closed form of
  // Sec. IV.A.3), lanes = cells ----
  double n = 1.0, T = 1.0, geq[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) geq[q] = 0.0;
  if (collide) {   // uniform over the block
    n = mom[0];
    const double u = mom[1] / n;
    T = (mom[2] - u * mom[1] + 2.0 * mom[3]) * C.inv_1pDt / n;
    double G[kNmaxLarge + 1];
#pragma unroll
    for (int l = 0; l <= kNmaxLarge; ++l) G[l] = 0.0;
    const double *hwr = s_hw + wave * NG * (kNmaxLarge + 1);
    if (full) {
      // G_l = E[He_l(X)], X ~ N(m u/p0, m T/p0^2), obeys G_{l+1} = ub G_l +
      // l a G_{l-1} with a = m T/p0^2 - 1; kept as G_l / sqrt(l!) against
      // HWs = w_k h_l(z_k) (h_l = He_l / sqrt(l!)).  The mirrored half has
      // h_l(-z) = (-1)^l h_l(z).
      const double ub = (hw ? -u : u) * tl->inv_p0, aa = T * tl->inv_p0 * tl->inv_p0 - 1.0;
      G[0] = 1.0;
      G[1] = ub;
#pragma unroll
      for (int l = 1; l < kNmaxLarge; ++l)
        if (l + 1 <= N) G[l + 1] = (ub * G[l] + tl->sq[l] * aa * G[l - 1]) / tl->sq[l + 1];
    } else {
      const double sT = sqrt(T), sc = sT * tl->inv_p0, y0 = -u / sT, ub = sg * u * tl->inv_p0;
      auto accum = [&](double x, double wt) {
        double qm = 1.0, q = x - tl->a[0];
        G[0] += wt;
        G[1] = fma(wt, q, G[1]);
#pragma unroll
        for (int l = 1; l < kNmaxLarge; ++l) {
          if (l + 1 > N) break;
          const double qn = fma(x - tl->a[l], q, -(tl->mb[l] * qm));
          qm = q;
          q = qn;
          G[l + 1] = fma(wt, q, G[l + 1]);
        }
      };
      for (int j = wave; j < tl->nm; j += NW) accum(fma(sc, tl->zm[j], ub), tl->wm[j]);
      // correction: the first entry, calibrated or composite, whose reach
      // covers the window's largest |y0| (the last when none does, also for a
      // non-finite one)
      double ymax = P.out ? fabs(y0) : 0.0;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) ymax = fmax(ymax, __shfl_xor(ymax, o, 64));
      ymax = readlane_d(ymax, 0);
      if (ymax > 0.0) {
        int li = kLadderAll - 1;
        for (int j = 1; j < kLadderAll; ++j)
          if (tl->lad_y[j] >= ymax) { li = j; break; }
        const int nc = tl->lad_n[li], o = tl->lad_off[li];
        for (int j = wave; j < nc; j += NW) {
          const double t = tl->ltau[o + j], yt = y0 * t;
          accum(fma(-ub, t, ub), -sg * y0 * tl->llamw[o + j] * exp(-0.5 * yt * yt));
        }
      }
      if (P.ty == 0 && wave == 0 && A.wide) {   // each cell once
        const bool wd = P.out && fabs(y0) > tl->lad_y[kLadder - 1] && tl->lad_n[kLadderAll - 1] > tl->lad_n[kLadder - 1];
        const unsigned long long cells = __ballot(wd);
        if (cells && lane == 0) atomicAdd(A.wide, (unsigned long long)__popcll(cells));
      }
#pragma unroll
      for (int l = 0; l <= kNmaxLarge; ++l) s_red[(wave * (kNmaxLarge + 1) + l) * 64 + lane] = G[l];
      __syncthreads();
#pragma unroll
      for (int l = 0; l <= kNmaxLarge; ++l) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += s_red[(w * (kNmaxLarge + 1) + l) * 64 + lane];
        G[l] = v;
      }
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
      for (int l = 0; l <= kNmaxLarge; ++l) geq[q] = fma(hwr[q * (kNmaxLarge + 1) + l], G[l], geq[q]);
  }

  // ---- wall ghosts (Sec. IV.C.3): incoming nodes extrapolated quadratically
  // from the three nearest cells, emergent nodes n_w g^w_k in all three ----
  if (hw ? needL : needR) {
    const int l0 = hw == 1 ? 63 - kHalo + P.win.i0 : Nx - 1 - (P.win.i0 - kHalo);   // lane of the wall cell
    const int gi = lane - l0;
    const double c0 = gi == 1 ? 3.0 : (gi == 2 ? 6.0 : 10.0);
    const double c1 = gi == 1 ? -3.0 : (gi == 2 ? -8.0 : -15.0);
    const double c2 = gi == 1 ? 1.0 : (gi == 2 ? 3.0 : 6.0);
    const bool ghost = gi >= 1 && gi <= 3;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const double y0 = readlane_d(yf[q], l0), y1 = readlane_d(yf[q], l0 - 1), y2 = readlane_d(yf[q], l0 - 2);
      if (ghost) yf[q] = c0 * y0 + c1 * y1 + c2 * y2;
      if constexpr (NFUN > 1) {
        const double x0 = readlane_d(yc[q], l0), x1 = readlane_d(yc[q], l0 - 1), x2 = readlane_d(yc[q], l0 - 2);
        if (ghost) yc[q] = c0 * x0 + c1 * x1 + c2 * x2;
      }
    }
  }
  if (up) {
    const double nw = -wave_sum(wsum) * (hw ? C.inv_DR : C.inv_DL);
    // for the diagnostics: the last stage's densities, once per wall
    if (A.stage == 2 && A.nwall && P.kt0 == 0 && threadIdx.x == 0 &&
        (hw ? P.win.i0 + P.win.nout == Nx : P.win.i0 == 0))
      A.nwall[2 * P.win.ch + hw] = nw;
    const bool ghost = hw ? i >= Nx && i <= Nx + 2 : i < 0;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const double g = nw * gwk[q];
      if (ghost) {
        yf[q] = g;
        if constexpr (NFUN > 1) yc[q] = C.half_Dt * (hw ? C.TR : C.TL) * g;
      }
    }
  }

  // ---- advection (lane-parallel face values) and the RK-3 combination ----
  const bool face_used = inside && P.lane >= kHalo - 1 && (hw ? P.pos >= kHalo && P.pos <= kHalo + P.win.nout
                                                              : P.pos < kHalo + P.win.nout);
  const bool wall_face = hw == 0 ? (i == -1) : (i == Nx);
  const bool out_lane = P.out && inside;
  const double inv_tau = collide ? n * C.inv_Kn : 0.0, eqc = C.half_Dt * T;
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    if (q >= ng) break;
    const int k = k0 + q;
    const double v = K.p[q], ka = K.ka[q];
    const int64_t o = rowh + (int64_t)k * Nx + ic;
#pragma unroll
    for (int fn = 0; fn < NFUN; ++fn) {
      const double y0v = fn == 0 ? yf[q] : yc[q];
      double src = -C.g * sg * fma(ka, mom[4 + fn], kk[fn][q]);
      if (collide) src -= (y0v - (fn == 0 ? n : eqc * n) * geq[q]) * inv_tau;
      double fv = face_value_down<ADV>(y0v, face_used);
      if (wall_face) fv = y0v;
      const double fo = dpp_shr1(fv);
      const double L = fma(-dx_inv * v, fv - fo, src);
      const double yn = A.a_base * (fn == 0 ? bf0[q] : bc0[q]) + A.b_stage * ((A.increment ? 0.0 : y0v) + C.dt * L);
      if (out_lane) (fn == 0 ? A.out_f : A.out_c)[o] = yn;
      (fn == 0 ? yf : yc)[q] = yn;
    }
  }
#pragma unroll
  for (int q = 0; q < NG; ++q)
    if (q >= ng) yf[q] = yc[q] = 0.0;
  emit_sums<ADV>(A, P, K, Nx, C.sum_off, NFUN, collide, yf, yc, s_sum, s_wall);
}

}  // namespace hhlb
