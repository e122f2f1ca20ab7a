// Records, lane moves and face values shared by the kernels of the half-range
// (HHLB) and full-range (HLB) lattice Boltzmann models with a force term: the
// tables of a model class, channels and windows, WENO-5 / upwind-3 faces of
// lanes that run down the wind, rows as buffer resources, the block map.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hhlb {

constexpr int kQmaxDev = 16;   // largest per-half order with a kernel
constexpr int kLadder = 8;     // calibrated correction point counts the half-range kernel chooses from
constexpr int kComposite = 6;  // beyond them: the top count on 2, 4, .., 64 panels
constexpr int kLadderAll = kLadder + kComposite;
constexpr int kLadderTop = 16; // the top calibrated count
constexpr int kLadderPts = 64 + kLadderTop * (2 + 4 + 8 + 16 + 32 + 64);   // points over all entries
constexpr int kWin = 58;       // most output cells of a window of the node-parallel stage (64 lanes)

constexpr int kHalo = 3;

// Per model class (quadrature, Q, N, p0): uploaded once.
struct DevTables {
  double p[2 * 256];                      // p_k / m (every node, also of the large-Q classes)
  double vv[kQmaxDev];                    // half: (p_k / m)^2
  double w[kQmaxDev];                     // weights of the positive nodes
  double a[kQmaxDev + 2];                 // recurrence: sqrt(b_{l+1}) h_{l+1} = (z-a_l) h_l - sqrt(b_l) h_{l-1}
  double Kin[kQmaxDev * kQmaxDev];        // half: + half within block (H x H); full: dense V x V
  double ka[kQmaxDev], kb[kQmaxDev];      // half: rank-1 cross term
  double HW[kQmaxDev * kQmaxDev];         // full: V x Q (zero beyond N)
  double inv_p0;
  // half-range kernel: monic recurrence q_{l+1} = (x - a_l) q_l - b_l q_{l-1}
  double mb[kQmaxDev + 2];                // b_l
  double HWs[kQmaxDev * kQmaxDev];        // H x Q: w_k h_l(z_k) / sqrt(b_0 .. b_l) (zero beyond N)
  // correction ladder: count lad_n[j] is exact enough up to |y0| <= lad_y[j];
  // entries kLadder.. are composite rules of the top count (2^(j-kLadder+1)
  // panels over [y0, 0], each panel within the top count's reach)
  int lad_n[kLadderAll], lad_off[kLadderAll];
  double lad_y[kLadderAll];
  double ltau[kLadderPts], llamw[kLadderPts];
  // main-part rule of the equilibrium: the M-point half-range Gauss rule,
  // M = ceil((N+1)/2), exact for the degree-N integrands
  int nm;
  double zm[kQmaxDev], wm[kQmaxDev];
  // mixed-precision form: the state is kept as phi_k = f_k / w_k, so the
  // half-range tables are rescaled by the node weights
  double wq[kQmaxDev], iwq[kQmaxDev];     // w_k, 1/w_k of a half
  double wpq[2 * kQmaxDev];               // w_k p_k/m (both halves)
  double wpfq[2 * kQmaxDev];              // w_k (p_k/m rounded to FP32): the wall-flux balance uses
                                          // the velocities the FP32 advection uses
  double wp2q[2 * kQmaxDev];              // w_k (p_k/m)^2
  double kbs[kQmaxDev];                   // kb_j w_j
  double HWss[kQmaxDev * kQmaxDev];       // HWs[k][l] / w_k
  float Ks[kQmaxDev * kQmaxDev];          // Kin[k][j] w_j / w_k
  float kas[kQmaxDev];                    // ka_k / w_k
  float pf[2 * kQmaxDev];                 // p_k/m
  // reduced-precision force operands (FP16 form): the FP16 table is
  // Ks with row k scaled by rsc_k (a power of two, |row| <= 1) and irsc_k =
  // 1/rsc_k.  The matrix cores see the table as a high part Kh (the operand
  // rounding of it) plus a low part Kl (the rounding of the remainder);
  // crs_j = sum_k w_k Kh_kj and crs_lo_j = sum_k w_k Kl_kj are their weighted
  // column sums exactly as rounded, whose mass defect the kernel removes;
  // iwh = 1 / sum over a half of w_k
  float Ks16[kQmaxDev * kQmaxDev];
  float irsc[kQmaxDev];
  float crs[kQmaxDev];
  float crs_lo[kQmaxDev];                 // the same sums for the table's low part (hi/lo split)
  float iwh;
};

// The tables through the constant address space: every entry a wave needs
// uniformly comes by a scalar load, also from a pointer the compiler has been
// kept from seeing through.
typedef const __attribute__((address_space(4))) DevTables *ConstTables;

// Per channel.
struct DevChannel {
  int64_t off;        // offset (doubles) of this channel in each state array
  int32_t Nx;
  int32_t cell_off;   // offset of this channel's cells in per-cell arrays
  int32_t gw_off;     // offset of the wall equilibria (2V doubles: left, right)
  int32_t sum_off;    // Q > 16: offset of its cells among those of its class
  double g;           // acceleration (F = m g)
  double inv_Kn;      // 1/Kn (0 when collisionless)
  double dt;
  double TL, TR;      // wall temperatures
  double inv_DL;      // 1 / sum_{p_k>0} (p_k/m) gwL_k  (mixed form: p_k/m rounded to FP32)
  double inv_DR;      // 1 / sum_{p_k<0} (p_k/m) gwR_k
  double half_Dt;     // Dt/2
  double inv_1pDt;    // 1/(1+Dt)
};

typedef const __attribute__((address_space(4))) DevChannel *ConstChannel;

// Window: channel id, first output cell and number of output cells.
struct DevWindow {
  int32_t ch, i0, nout;
};

struct StageArgs {
  const DevTables *tb;
  const DevChannel *chans;
  const DevWindow *wins;
  int32_t nwin;
  int32_t xcd_map;           // 1: XCD-aware block -> window mapping, 0: identity
  int32_t nblocks;           // launch across classes: blocks (0: one per window, -1: what the GPU holds at once)
  int32_t nsteps, nst;       // steps of the launch and stages per step (3; 1: one forward-Euler stage)
  const double *inv_dx;      // per cell
  const double *gw;          // wall equilibria
  // state arrays: double (FP64 form) or float (mixed form)
  const void *in_f, *in_c;   // y^n
  void *out_f, *out_c;
  double *nwall;             // 2 per channel (may be null)
  // count of waves whose equilibrium needed more than one correction panel
  // (|y0| beyond the calibrated range of the ladder; may be null)
  unsigned long long *wide;
  // mixed form only: 16-bit correction words of y^n and of y^{n+1}
  const int16_t *lo_in_f, *lo_in_c;
  int16_t *lo_out_f, *lo_out_c;
};

__device__ __forceinline__ double dpp_shr1(double x) {  // lane l <- lane l-1
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_update_dpp(0, lo, 0x138, 0xf, 0xf, true);
  hi = __builtin_amdgcn_update_dpp(0, hi, 0x138, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double dpp_shl1(double x) {  // lane l <- lane l+1
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_update_dpp(0, lo, 0x130, 0xf, 0xf, true);
  hi = __builtin_amdgcn_update_dpp(0, hi, 0x130, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double readlane_d(double x, int l) {
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_readlane(lo, l);
  hi = __builtin_amdgcn_readlane(hi, l);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// 1/x for normal, finite x > 0: the hardware estimate refined by two
// Newton-Raphson steps (within an ulp or so; the weights it scales are
// renormalised anyway).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// WENO-5 face value (Eqs. weno5_flux, weno5_omega, weno_sigma) for the
// upwind-ordered stencil (a..e) = (f_{i-2}, .., f_{i+2}), with the limits of
// Table (weno) when smoothness indicators vanish.  The weights are formed as
// delta_q prod_{r!=q} sigma_r^2 (mathematically delta_q/sigma_q^2 times the
// common factor prod_r sigma_r^2) after an exact power-of-two rescaling of
// the sigmas; when that product underflows the limit rule is applied.
__device__ __forceinline__ double weno5(double a, double b, double c, double d, double e) {
  const double k13 = 13.0 / 12.0;
  double t1 = a - 2.0 * b + c, t2 = a - 4.0 * b + 3.0 * c;
  const double s1 = k13 * t1 * t1 + 0.25 * t2 * t2;
  t1 = b - 2.0 * c + d; t2 = b - d;
  const double s2 = k13 * t1 * t1 + 0.25 * t2 * t2;
  t1 = c - 2.0 * d + e; t2 = 3.0 * c - 4.0 * d + e;
  const double s3 = k13 * t1 * t1 + 0.25 * t2 * t2;
  const double F1 = (2.0 * a - 7.0 * b + 11.0 * c) * (1.0 / 6.0);
  const double F2 = (-b + 5.0 * c + 2.0 * d) * (1.0 / 6.0);
  const double F3 = (2.0 * c + 5.0 * d - e) * (1.0 / 6.0);
  // exact power-of-two rescaling so that the largest sigma lies in [0.5, 1)
  // (all-zero sigmas stay zero and fall through to the limit rule)
  const int ex = __builtin_amdgcn_frexp_exp(fmax(s1, fmax(s2, s3)));
  const double r1 = ldexp(s1, -ex), r2 = ldexp(s2, -ex), r3 = ldexp(s3, -ex);
  const double q1s = r1 * r1, q2s = r2 * r2, q3s = r3 * r3;
  const double p1 = 0.1 * q2s * q3s, p2 = 0.6 * q1s * q3s, p3 = 0.3 * q1s * q2s;
  double n1 = p1, n2 = p2, n3 = p3, dd = p1 + p2 + p3;
  if (!(dd > 1e-250)) {
    // limit of Table (weno): ideal weights restricted to the vanishing
    // sigmas (a branch no lane takes in smooth flow, so the common path
    // carries no selects)
    const double tiny = 1e-125;
    n1 = q1s < tiny ? 0.1 : 0.0;
    n2 = q2s < tiny ? 0.6 : 0.0;
    n3 = q3s < tiny ? 0.3 : 0.0;
    dd = n1 + n2 + n3;
  }
  return (n1 * F1 + n2 * F2 + n3 * F3) * recip(dd);
}

// Lane-parallel WENO-5 of a half: lanes run down the wind (lane l - 1 is
// upwind of lane l), lane l forms the value at its downwind face.  Waves of
// the p > 0 half hold the cells in ascending order, waves of the p < 0 half in
// descending order, so both run this one form.
//
// Eqs. (weno5_flux), (weno5_omega) and (weno_sigma) in differences: with
// dp = y_{l+1} - y_l, dm = y_l - y_{l-1}, D = dp - dm and D_L, D_R the second
// differences of the neighbouring lanes,
//   sigma_1 = 13/12 D_L^2 + (dm + D_L/2)^2,  sigma_2 = 13/12 D^2 + (dm + D/2)^2,
//   sigma_3 = 13/12 D_R^2 + (dp - D_R/2)^2,
//   F^2 = y + dp/3 + dm/6,  F^1 - F^2 = (D_L - D)/3,  F^3 - F^2 = (D - D_R)/6,
// so a face is F^2 plus a weighted sum of third differences.  Only y, dp and
// D cross lanes (four shifts; 24 of the 61 instructions of a form that shifted
// sigmas and candidates went into such moves and into terms common to all
// candidates; this one has 49 with the flux difference and the RK-3 sum).  D
// is kept times sqrt(13/12); a common factor of the weights cancels, so
// they are divided by the ideal weight 0.6 of the centre.
// The weights delta_q prod_{r!=q} sigma_r^2 are formed directly; when their
// sum leaves [1e-260, 1e260] (where its product with a third difference could
// leave the exponent range) the sigmas are rescaled by an exact power of two
// and, if the sum still underflows, the limit of Table (weno) applies (as in
// weno5).  `used` marks lanes whose value is consumed: only they may send the
// wave into that branch.
constexpr double kSq1312 = 1.0408329997330663;        // sqrt(13/12)
__device__ __forceinline__ double weno5_down(double y, bool used) {
  const double dp = dpp_shl1(y) - y, dm = dpp_shr1(dp);
  const double D = kSq1312 * (dp - dm);
  const double DL = dpp_shr1(D), DR = dpp_shl1(D);
  constexpr double h = 0.5 / kSq1312;
  const double tL = fma(h, DL, dm), tC = fma(h, D, dm), tR = fma(-h, DR, dp);
  const double sL = fma(tL, tL, DL * DL), sC = fma(tC, tC, D * D), sR = fma(tR, tR, DR * DR);
  double qL = sL * sL, qC = sC * sC, qR = sR * sR;
  double pL = qC * qR, pC = qL * qR, pR = qL * qC;
  double dd = fma(0.5, pR, fma(1.0 / 6.0, pL, pC));
  if (!(dd > 1e-260 && dd < 1e260) && used) {
    const int ex = __builtin_amdgcn_frexp_exp(fmax(sL, fmax(sC, sR)));
    const double rL = ldexp(sL, -ex), rC = ldexp(sC, -ex), rR = ldexp(sR, -ex);
    qL = rL * rL; qC = rC * rC; qR = rR * rR;
    pL = qC * qR; pC = qL * qR; pR = qL * qC;
    dd = fma(0.5, pR, fma(1.0 / 6.0, pL, pC));
    if (!(dd > 1e-250)) {
      const double tiny = 1e-125;
      pL = qL < tiny ? 1.0 : 0.0;
      pC = qC < tiny ? 1.0 : 0.0;
      pR = qR < tiny ? 1.0 : 0.0;
      dd = fma(0.5, pR, fma(1.0 / 6.0, pL, pC));
    }
  }
  // 1/dd: the hardware estimate r, then r (1 + e + e^2), e = 1 - dd r
  const double r = __builtin_amdgcn_rcp(dd), e = fma(-dd, r, 1.0), e2 = fma(e, e, e);
  double m = fma(1.5, pR * (D - DR), pL * (DL - D)) * r;
  m = fma(m, e2, m);
  const double F2 = fma(1.0 / 3.0, dp, fma(1.0 / 6.0, dm, y));
  return fma(1.0 / (18.0 * kSq1312), m, F2);
}

// Third-order upwind value of the lane's downwind face, (-y_{l-1} + 5 y_l +
// 2 y_{l+1})/6: the central candidate F^2.
__device__ __forceinline__ double upwind3_down(double y) {
  const double dp = dpp_shl1(y) - y, dm = dpp_shr1(dp);
  return fma(1.0 / 3.0, dp, fma(1.0 / 6.0, dm, y));
}

template <int ADV>
__device__ __forceinline__ double face_value_down(double y, bool used) {
  if constexpr (ADV == 0) return weno5_down(y, used);
  else return upwind3_down(y);
}

// A stretch of `bytes` bytes of a row of the state as a buffer resource: the
// address stays in scalar registers, a lane's access is one 32-bit byte
// offset, and offsets outside [0, bytes) (among them negative ones) read zero
// and store nothing.  So an access costs no address arithmetic, no clamping
// and no branch (a global access under a lane mask took four vector
// instructions here).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double row_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  return __hiloint2double((int)v.y, (int)v.x);
}
__device__ __forceinline__ void row_store(__amdgpu_buffer_rsrc_t r, uint32_t off, double x) {
  const u32x2 v = {(unsigned)__double2loint(x), (unsigned)__double2hiint(x)};
  __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
}

// Walks down the rows of one array: the address of the current row in a
// scalar register pair.  The fence on each move keeps the compiler from
// forming the addresses of all rows ahead of the loads (they do not fit the
// scalar registers and spill into vector lanes).
struct RowWalk {
  const char *p;
  __device__ __forceinline__ RowWalk(const void *base, int64_t elem, int size = 8)
      : p((const char *)base + elem * size) {}
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t take(int64_t stride_bytes, uint32_t bytes) {
    const __amdgpu_buffer_rsrc_t r = row_rsrc(p, bytes);
    p += stride_bytes;
    asm volatile("" : "+s"(p));
    return r;
  }
};

// Third-order upwind-biased face value (-f_{i-1} + 5 f_i + 2 f_{i+1})/6.
__device__ __forceinline__ double upwind3(double b, double c, double d) {
  return (-b + 5.0 * c + 2.0 * d) * (1.0 / 6.0);
}

template <int ADV>
__device__ __forceinline__ double face_value(double a, double b, double c, double d, double e) {
  if constexpr (ADV == 0) return weno5(a, b, c, d, e);
  else return upwind3(b, c, d);
}

// Map a block index to a window so that consecutive windows (which share
// halo cells) are dispatched to the same XCD (blocks go round-robin over 8).
__device__ __forceinline__ int xcd_window(int b, int n) {
  const int q = n >> 3, r = n & 7;
  const int x = b & 7, pos = b >> 3;
  return x * q + (x < r ? x : r) + pos;
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

}  // namespace hhlb
