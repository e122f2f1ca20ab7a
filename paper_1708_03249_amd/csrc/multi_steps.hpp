// Whole RK-3 steps of the homogeneous mixed-quadrature system (App. A) in one
// launch.  Points do not couple, so a point's populations stay in registers
// from the first stage to the last: memory is touched once in and once out per
// launch of up to kMultiStepsPerLaunch steps, where one launch per stage moved
// two or three copies of f each and staged the tables anew (HH(4) x H(4) x
// H(4), 1e6 points: 1.44 ms per stage against 0.52 ms of memory time).
//
// Mapping: P = V / V_x lanes per point, floor(64 / P) points per wave.  A lane
// holds the V_x populations of one pair of y and z velocities, so the rows it
// loads are contiguous over the lanes and the x contraction is a V_x x V_x
// product in its own registers against scalar table entries.  The z
// contraction of four velocities is four lane permutations inside quads (QZ);
// other z axes and the y axis read the neighbours' populations from LDS, one
// read per term with the matrix entry held for all V_x rows.  Each lane
// evaluates the equilibrium factors of its own y and z velocity; the factors
// along x come from one evaluation per half, shared over pairs of lanes (and
// its quadrature points over quads).
#pragma once
#include "fused_kernels.hpp"
#include "multi_kernels.hpp"

namespace hhlb {

typedef const __attribute__((address_space(4))) DevMulti *ConstMulti;
typedef const __attribute__((address_space(4))) DevLarge *ConstLarge;
typedef const __attribute__((address_space(4))) double *ConstDoubles;

template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kQuadXor3 = 0x1B;   // quad_perm [1,0,3,2], [2,3,0,1], [3,2,1,0]
constexpr int kQuadEven = 0xA0, kQuadOdd = 0xF5;                       // quad_perm [0,0,2,2], [1,1,3,3]
constexpr int kHalfMirror = 0x141, kMirror = 0x140;                    // row_half_mirror, row_mirror

constexpr double kInvSqrt[kNmaxLarge + 1] = {   // 1/sqrt(l)
    0.0, 1, 0.70710678118654746, 0.57735026918962584, 0.5, 0.44721359549995793, 0.40824829046386307,
    0.3779644730092272, 0.35355339059327373, 0.33333333333333331, 0.31622776601683794, 0.30151134457776363,
    0.28867513459481292, 0.27735009811261457, 0.2672612419124244, 0.2581988897471611, 0.25, 0.24253562503633297,
    0.23570226039551587, 0.22941573387056174, 0.22360679774997896};

// Sum over the aligned groups of P lanes, P a power of two; every lane of a
// group returns it.
__device__ __forceinline__ double group_sum(double x, int P) {
  if (P > 1) x += dpp_d<kQuadXor1>(x);
  if (P > 2) x += dpp_d<kQuadXor2>(x);
  if (P > 4) x += dpp_d<kHalfMirror>(x);
  if (P > 8) x += dpp_d<kMirror>(x);
  if (P > 16) x += __shfl_xor(x, 16, 64);
  if (P > 32) x += __shfl_xor(x, 32, 64);
  return x;
}

// Equilibrium coefficients G_l, l <= NM, of the half sg of a half-range axis
// at (u, T): the main rule and the correction (Sec. IV.B.3 by the change of
// variables of the step kernel), the correction's point count one for the wave
// (the smallest that covers its largest |y0|).  SPLIT: the lane takes the even
// (second = false) or the odd quadrature points only.  `lad` is lane j's reach
// of entry j.
template <int NM, bool SPLIT>
__device__ __forceinline__ void half_coeffs(ConstLarge tl, double sg, double u, double T, double lad, int lane,
                                            bool second, double (&G)[NM + 1]) {
#pragma unroll
  for (int l = 0; l <= NM; ++l) G[l] = 0.0;
  const double rT = rsqrt_full(T), ub = sg * u * tl->inv_p0, sc = T * rT * tl->inv_p0, y0 = -u * rT;
  auto accum = [&](double x, double wt) {
    double qm = 1.0, q = x - tl->a[0];
    G[0] += wt;
    if (NM > 0) G[1] = fma(wt, q, G[1]);
#pragma unroll
    for (int l = 1; l < NM; ++l) {
      const double qn = fma(x - tl->a[l], q, -(tl->mb[l] * qm));
      qm = q; q = qn;
      G[l + 1] = fma(wt, q, G[l + 1]);
    }
  };
  // point j of a rule of cnt points, or with SPLIT the lane's of j and j + 1
  // (weight zero past the end)
  auto point = [&](ConstDoubles x, ConstDoubles w, int j, int cnt, double &xj, double &wj) {
    if constexpr (SPLIT) {
      const bool more = j + 1 < cnt;
      const int j1 = more ? j + 1 : j;
      const double x0 = x[j], x1 = x[j1], w0 = w[j], w1 = w[j1];
      xj = second ? x1 : x0;
      wj = second ? (more ? w1 : 0.0) : w0;
    } else {
      xj = x[j];
      wj = w[j];
    }
  };
  constexpr int dq = SPLIT ? 2 : 1;
  const float ymax = wave_max_up(fabs(y0));
  const unsigned long long reach =
      __ballot(lane >= 1 && (lane == kLadderAll - 1 || (lane < kLadderAll && lad >= (double)ymax)));
  const int li = __ffsll(reach) - 1;
  const int nm = tl->nm, nc = ymax != 0.0f ? tl->lad_n[li] : 0, o = tl->lad_off[li];
  double xj, wj;
#pragma unroll 1
  for (int j = 0; j < nm; j += dq) {
    point(tl->zm, tl->wm, j, nm, xj, wj);
    accum(fma(sc, xj, ub), wj);
  }
  const double sy = -sg * y0, hy = -0.5 * y0 * y0;
  if (!(ymax > 1.000001f)) {
#pragma unroll 1
    for (int j = 0; j < nc; j += dq) {
      point(tl->ltau + o, tl->llamw + o, j, nc, xj, wj);
      accum(fma(-ub, xj, ub), sy * wj * exp_small(hy * (xj * xj)));
    }
  } else {
#pragma unroll 1
    for (int j = 0; j < nc; j += dq) {
      point(tl->ltau + o, tl->llamw + o, j, nc, xj, wj);
      accum(fma(-ub, xj, ub), sy * wj * exp(hy * (xj * xj)));
    }
  }
}
// Full range: G_l / sqrt(l!) by the closed-form recurrence (Sec. IV.A.3); the
// mirrored half has ub -> -ub.
template <int NM>
__device__ __forceinline__ void full_coeffs(ConstLarge tl, double sg, double u, double T, double (&G)[NM + 1]) {
  const double ub = sg * u * tl->inv_p0, aa = fma(T * tl->inv_p0, tl->inv_p0, -1.0);
  G[0] = 1.0;
  if (NM > 0) G[1] = ub;
#pragma unroll
  for (int l = 1; l < NM; ++l) G[l + 1] = fma(ub, G[l], tl->sq[l] * (aa * G[l - 1])) * kInvSqrt[l + 1];
}

#ifndef HHLB_MULTI_STEPS_OCC
#define HHLB_MULTI_STEPS_OCC 3
#endif
template <int NX, int NM, bool QZ>
__global__ __launch_bounds__(64 * kMultiWaves)
__attribute__((amdgpu_waves_per_eu(NX <= 8 && NM <= 7 ? HHLB_MULTI_STEPS_OCC : 1))) void multi_steps_kernel(MultiArgs A) {
  extern __shared__ double s_mem[];
  const int wave = threadIdx.x >> 6, lane0 = threadIdx.x & 63;
  ConstMulti tm = (ConstMulti)A.tm;
  ConstDoubles tab = (ConstDoubles)A.tab;
  constexpr int H0 = NX / 2;
  const int d = tm->d, az = d - 1;
  const int Vy = d == 3 ? tm->Va[1] : 1, Vz = tm->Va[az], P = Vy * Vz, V = NX * P;
  const int ppw = 64 / P;
  const bool pow2 = (P & (P - 1)) == 0;
  // the lane's point and its y and z velocity; lanes past the last whole
  // point of the wave repeat the first one's, lanes past the last point of all
  // that one's, and store nothing
  int seg0 = lane0 / P;
  const int sub = lane0 - seg0 * P;
  const bool spare = seg0 >= ppw;
  if (spare) seg0 = 0;
  const int j0 = d == 3 ? sub / Vz : 0, k0 = sub - j0 * Vz;
  const int64_t pt_wave = ((int64_t)blockIdx.x * kMultiWaves + wave) * ppw;   // the wave's first point
  const int64_t pt0 = pt_wave + seg0;
  const bool valid = !spare && pt0 < A.npts;
  const int64_t pt = pt0 < A.npts ? pt0 : A.npts - 1;

  // block tables: F_a K_a of the lane axes, their equilibrium tables
  constexpr int NG = NM + 1;   // row of the equilibrium tables, zero beyond the axis' order
  double *s_Ky = s_mem, *s_Kz = s_Ky + Vy * Vy, *s_hx = s_Kz + Vz * Vz, *s_hy = s_hx + H0 * NG;
  double *s_hz = s_hy + (Vy / 2) * NG;
  double *s_f = s_hz + (Vz / 2) * NG + wave * NX * 64;
  {
    const double Fy = d == 3 ? A.F[1] : 0.0, Fz = d == 3 ? A.F[2] : A.F[1];
    auto stage_rows = [&](double *to, int a, int rows) {
      const int N = tm->ax[a].N, from = tm->hw_off[a];
      for (int t = threadIdx.x; t < rows * NG; t += 64 * kMultiWaves) {
        const int r = t / NG, l = t - r * NG;
        to[t] = l <= N ? A.tab[from + r * (N + 1) + (l <= N ? l : 0)] : 0.0;
      }
    };
    if (d == 3) {
      for (int t = threadIdx.x; t < Vy * Vy; t += 64 * kMultiWaves) s_Ky[t] = Fy * A.tab[tm->k_off[1] + t];
      stage_rows(s_hy, 1, Vy / 2);
    }
    for (int t = threadIdx.x; t < Vz * Vz; t += 64 * kMultiWaves) s_Kz[t] = Fz * A.tab[tm->k_off[az] + t];
    stage_rows(s_hz, az, Vz / 2);
    stage_rows(s_hx, 0, H0);
  }
  __syncthreads();
  // (in, out) may be the same array: a wave without a point would read the last
  // one while its own wave stores it
  if (pt_wave >= A.npts) return;
  const double py = d == 3 ? A.tab[tm->p_off[1] + j0] : 0.0, pz = A.tab[tm->p_off[az] + k0];
  double kq[4];   // z matrix entries of the quad's lanes
  if constexpr (QZ) {
#pragma unroll
    for (int m = 0; m < 4; ++m) kq[m] = s_Kz[k0 * 4 + (k0 ^ m)];
  }
  const int ll = lane0 < kLadderAll ? lane0 : kLadderAll - 1;
  const bool fx = tm->ax[0].full != 0, fy = d == 3 && tm->ax[1].full != 0, fz = tm->ax[az].full != 0;
  const double ladx = A.tm->ax[0].lad_y[ll], lady = A.tm->ax[1].lad_y[ll], ladz = A.tm->ax[az].lad_y[ll];
  const bool collide = A.inv_Kn != 0.0;

  double f[NX], fn[NX];
  const double *src = A.in + pt * V + sub;
#pragma unroll
  for (int x = 0; x < NX; ++x) f[x] = fn[x] = src[x * P];

  const int total = A.rhs_only ? 1 : 3 * A.nsteps;
#pragma unroll 1
  for (int it = 0; it < total; ++it) {
    const int st = it % 3;
    const double a_s = st == 0 ? 0.0 : (st == 1 ? 0.75 : 1.0 / 3.0);
    const double b_s = st == 0 ? 1.0 : (st == 1 ? 0.25 : 2.0 / 3.0);
    // addresses and lane selections are formed anew in each stage: kept
    // through the stages they would take the registers of the state
    int lane = lane0, seg = seg0, j = j0, k = k0;
    asm volatile("" : "+v"(lane), "+v"(seg), "+v"(j), "+v"(k));
    const double sgy = j < Vy / 2 || d == 2 ? 1.0 : -1.0, sgz = k < Vz / 2 ? 1.0 : -1.0;
    const int hy = d == 3 ? (j < Vy / 2 ? j : j - Vy / 2) : 0, hz = k < Vz / 2 ? k : k - Vz / 2;
    asm volatile("" : "+s"(tm), "+s"(tab));
    // ---- moments: n, u, then T from the spread about u ----
    ConstDoubles px = tab + tm->p_off[0];
    double n0 = 0.0, mx = 0.0;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      n0 += f[x];
      mx = fma(px[x], f[x], mx);
    }
    // sums over the point's lanes
    auto sum_lanes = [&](double (&q)[4], int nq) {
      if (pow2) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < nq) q[c] = group_sum(q[c], P);
        return;
      }
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {   // over z, then over y
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < nq) s_f[c * 64 + lane] = q[c];
        __builtin_amdgcn_wave_barrier();
        const int cnt = pass == 0 ? Vz : Vy, step = pass == 0 ? 1 : Vz, base = seg * P + (pass == 0 ? j * Vz : k);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < nq) {
            double acc = 0.0;
            for (int t = 0; t < cnt; ++t) acc += s_f[c * 64 + base + t * step];
            q[c] = acc;
          }
      }
      __builtin_amdgcn_wave_barrier();
    };
    double q4[4] = {n0, mx, py * n0, pz * n0};
    sum_lanes(q4, 4);
    const double n = q4[0], rn = recip(n);
    const double ux = q4[1] * rn, uy = d == 3 ? q4[2] * rn : 0.0, uz = q4[3] * rn;
    double c2 = fma(py - uy, py - uy, (pz - uz) * (pz - uz)) * n0;
    if (d == 2) c2 = (pz - uz) * (pz - uz) * n0;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      const double c = px[x] - ux;
      c2 = fma(c * c, f[x], c2);
    }
    double q1[4] = {c2, 0.0, 0.0, 0.0};
    sum_lanes(q1, 1);
    const double T = q1[0] * rn * (d == 3 ? 1.0 / 3.0 : 0.5);

    // ---- force: sum_a F_a (K_a f)_v ----
    double acc[NX];
    ConstDoubles Kx = tab + tm->k_off[0];
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      double t = 0.0;
#pragma unroll
      for (int y = 0; y < NX; ++y) t = fma(Kx[x * NX + y], f[y], t);
      acc[x] = A.F[0] * t;
    }
    if (d == 3 || !QZ) {
#pragma unroll
      for (int x = 0; x < NX; ++x) s_f[x * 64 + lane] = f[x];
      __builtin_amdgcn_wave_barrier();
    }
    if (d == 3) {
      const double *fr = s_f + seg * P + k, *Kr = s_Ky + j * Vy;
      for (int t = 0; t < Vy; ++t) {
        const double kv = Kr[t];
#pragma unroll
        for (int x = 0; x < NX; ++x) acc[x] = fma(kv, fr[x * 64 + t * Vz], acc[x]);
      }
    }
    if constexpr (QZ) {
#pragma unroll
      for (int x = 0; x < NX; ++x) {
        acc[x] = fma(kq[0], f[x], acc[x]);
        acc[x] = fma(kq[1], dpp_d<kQuadXor1>(f[x]), acc[x]);
        acc[x] = fma(kq[2], dpp_d<kQuadXor2>(f[x]), acc[x]);
        acc[x] = fma(kq[3], dpp_d<kQuadXor3>(f[x]), acc[x]);
      }
    } else {
      const double *fr = s_f + seg * P + j * Vz, *Kr = s_Kz + k * Vz;
      for (int t = 0; t < Vz; ++t) {
        const double kv = Kr[t];
#pragma unroll
        for (int x = 0; x < NX; ++x) acc[x] = fma(kv, fr[x * 64 + t], acc[x]);
      }
    }
    __builtin_amdgcn_wave_barrier();

    // ---- equilibrium factors and the relaxation: acc <- L ----
    if (collide) {
      const double rate = n * A.inv_Kn;
      double gyz = n * rate;
      {
        double G[NG];
        if (d == 3) {
          if (fy) full_coeffs<NM>(&tm->ax[1], sgy, uy, T, G);
          else half_coeffs<NM, false>(&tm->ax[1], sgy, uy, T, lady, lane, false, G);
          double g = 0.0;
#pragma unroll
          for (int l = 0; l <= NM; ++l) g = fma(s_hy[hy * NG + l], G[l], g);
          gyz *= g;
        }
        if (fz) full_coeffs<NM>(&tm->ax[az], sgz, uz, T, G);
        else half_coeffs<NM, false>(&tm->ax[az], sgz, uz, T, ladz, lane, false, G);
        double g = 0.0;
#pragma unroll
        for (int l = 0; l <= NM; ++l) g = fma(s_hz[hz * NG + l], G[l], g);
        gyz *= g;
      }
      // x: even lanes take the half p > 0, odd ones p < 0; in whole quads the
      // two pairs take every other quadrature point
      double Gp[NG], Gm[NG];
      asm volatile("" : "+s"(tm), "+s"(tab));
      if (fx) {
        full_coeffs<NM>(&tm->ax[0], 1.0, ux, T, Gp);
#pragma unroll
        for (int l = 0; l <= NM; ++l) Gm[l] = l & 1 ? -Gp[l] : Gp[l];
      } else {
        const double sx = lane & 1 ? -1.0 : 1.0;
        double G[NG];
        if (P % 4 == 0) {
          half_coeffs<NM, true>(&tm->ax[0], sx, ux, T, ladx, lane, (lane & 2) != 0, G);
#pragma unroll
          for (int l = 0; l <= NM; ++l) G[l] += dpp_d<kQuadXor2>(G[l]);
        } else {
          half_coeffs<NM, false>(&tm->ax[0], sx, ux, T, ladx, lane, false, G);
        }
#pragma unroll
        for (int l = 0; l <= NM; ++l) {
          Gp[l] = dpp_d<kQuadEven>(G[l]);
          Gm[l] = dpp_d<kQuadOdd>(G[l]);
        }
      }
#pragma unroll
      for (int x = 0; x < H0; ++x) {
        double gp = 0.0, gm = 0.0;
#pragma unroll
        for (int l = 0; l <= NM; ++l) {
          const double h = s_hx[x * NG + l];
          gp = fma(h, Gp[l], gp);
          gm = fma(h, Gm[l], gm);
        }
        acc[x] = fma(gyz, gp, -fma(rate, f[x], acc[x]));
        acc[H0 + x] = fma(gyz, gm, -fma(rate, f[H0 + x], acc[H0 + x]));
      }
    } else {
#pragma unroll
      for (int x = 0; x < NX; ++x) acc[x] = -acc[x];
    }

    // ---- Eq. (rk3) ----
    if (A.rhs_only) {
#pragma unroll
      for (int x = 0; x < NX; ++x) f[x] = acc[x];
    } else {
      const double bdt = b_s * A.dt;
#pragma unroll
      for (int x = 0; x < NX; ++x) {
        f[x] = fma(a_s, fn[x], fma(b_s, f[x], bdt * acc[x]));
        if (st == 2) fn[x] = f[x];
      }
    }
  }
  if (valid) {
    double *dst = A.out + pt * V + sub;
#pragma unroll
    for (int x = 0; x < NX; ++x) dst[x * P] = f[x];
  }
}

// Dynamic LDS of a block (doubles).
inline size_t multi_steps_lds(const MultiShape &m, int NM) {
  const int Vz = m.Va[m.d - 1], Vy = m.d == 3 ? m.Va[1] : 1;
  return (size_t)Vy * Vy + (size_t)Vz * Vz + (size_t)(m.Va[0] / 2 + Vy / 2 + Vz / 2) * (NM + 1) +
         (size_t)kMultiWaves * m.Va[0] * 64;
}

template <int NX, int NM>
void launch_multi_nx(const MultiArgs &a, const MultiShape &m, hipStream_t s) {
  const int P = (m.d == 3 ? m.Va[1] : 1) * m.Va[m.d - 1];
  const int64_t per_block = (int64_t)(64 / P) * kMultiWaves;
  const dim3 grid((unsigned)((a.npts + per_block - 1) / per_block));
  const size_t shm = sizeof(double) * multi_steps_lds(m, NM);
  if (m.Va[m.d - 1] == 4) hipLaunchKernelGGL((multi_steps_kernel<NX, NM, true>), grid, dim3(64 * kMultiWaves), shm, s, a);
  else hipLaunchKernelGGL((multi_steps_kernel<NX, NM, false>), grid, dim3(64 * kMultiWaves), shm, s, a);
}

// Runs it if there is an instance for the set's V_x whose LDS fits.
template <int NM>
bool launch_multi_nm(const MultiArgs &a, const MultiShape &m, hipStream_t s) {
  if (sizeof(double) * multi_steps_lds(m, NM) > 65536) return false;
  switch (m.Va[0]) {
    case 4: launch_multi_nx<4, NM>(a, m, s); return true;
    case 6: launch_multi_nx<6, NM>(a, m, s); return true;
    case 8: launch_multi_nx<8, NM>(a, m, s); return true;
    case 10: launch_multi_nx<10, NM>(a, m, s); return true;
    case 12: launch_multi_nx<12, NM>(a, m, s); return true;
    case 16: launch_multi_nx<16, NM>(a, m, s); return true;
    case 20: launch_multi_nx<20, NM>(a, m, s); return true;
    case 24: launch_multi_nx<24, NM>(a, m, s); return true;
    default: return false;
  }
}

}  // namespace hhlb
