// HIP kernels of the element steps on tetrahedra (d = 3) for gfx950.
//
// One thread per element; velocity-like vectors are SoA [3][P][T] (consecutive lanes,
// consecutive elements).  The reference tables of the residual (basis values and gradients
// at the volume and face points, the face-point permutations) are staged in LDS.  A face
// integral is evaluated by both neighbours at the same points of the fully symmetric face
// rule: the neighbour's point is found through the permutation of the face's vertices, so
// both sides carry out the same operations in mirrored order (no atomics).  The facet
// kernels (PCG) are shared with the triangle path (7 BSR blocks per face row).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>

#include "dfdg_device.h"
#include "dfdg_internal.h"
#include "dfdg_kernels.h"

namespace dfdg {

template <int K>
struct ResTabs3 {
  static constexpr int P = nP3(K), NQV = nQV3(K), NQF = nQF3(K);
  double Vv[NQV][P], Gv[NQV][3][P], Wv[NQV];
  double Vf[4][NQF][P], Gf[4][NQF][3][P], Wf[NQF];
  int pidx[6][NQF];
};
template <int K>
__device__ inline void stage_tabs3(ResTabs3<K>& s, const DevTabs& tb) {
  constexpr int P = nP3(K), NQV = nQV3(K), NQF = nQF3(K);
  double* d = &s.Vv[0][0];
  for (int i = threadIdx.x; i < NQV * P; i += blockDim.x) d[i] = tb.Vv[i];
  d = &s.Gv[0][0][0];
  for (int i = threadIdx.x; i < NQV * 3 * P; i += blockDim.x) d[i] = tb.Gv[i];
  for (int i = threadIdx.x; i < NQV; i += blockDim.x) s.Wv[i] = tb.Wv[i];
  d = &s.Vf[0][0][0];
  for (int i = threadIdx.x; i < 4 * NQF * P; i += blockDim.x) d[i] = tb.Vf[i];
  d = &s.Gf[0][0][0][0];
  for (int i = threadIdx.x; i < 4 * NQF * 3 * P; i += blockDim.x) d[i] = tb.Gf[i];
  for (int i = threadIdx.x; i < NQF; i += blockDim.x) s.Wf[i] = tb.Wf[i];
  int* p = &s.pidx[0][0];
  for (int i = threadIdx.x; i < 6 * NQF; i += blockDim.x) p[i] = tb.fpidx[i];
  __syncthreads();
}

// A new scalar pointer to the same table: what is read through it is loaded again.
__device__ inline const double* again(const double* p) {
  asm volatile("" : "+s"(p));
  return p;
}
// Ends a group of table reads, after N basis functions.
template <int N>
__device__ inline void table_group(int i) {
  if (i % N == N - 1) __builtin_amdgcn_sched_barrier(0);
}

__device__ inline void load_Jinv3(const DevGeo& g, int t, double (&Ji)[3][3]) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int j = 0; j < 3; ++j) Ji[r][j] = g.Jinv[(size_t)(3 * r + j) * g.T + t];
}

// ---------------------------------------------------------------------------------------
// a3: DG residual L(u)(v) = -C_h(u;u,v) - B_h(u,v) on the broken basis (eqs. (adv),
// (viscous)).  Per own face (outward normal n, neighbour values at the same points),
// un = {u}.n, u_up the outflow-side value, du = u_own - u_nbr; the face contributes to the
// own test function v
//     -(un u_up - nu {grad u} n + nu sigma du) . v  +  (nu/2) (du (x) n) : grad v.
// The volume term is int (u (x) u - nu grad u) : grad v.  VISC = false: nu = 0.
//
// Everything polynomial is carried by modes.  A trace is in P^K of the face (NF modes), a normal
// derivative in P^{K-1} (the first NM modes): the viscous face terms are products of modes,
// and only the upwind flux goes to the face points, from the modes and back into them, so
// that the basis (P functions) is applied once per face and side and not once per point.  A
// neighbour's modes are permuted to the own face parameters.  In the volume grad v is in
// P^{K-1}(T): the flux u (x) u is projected onto its NP modes point by point, the viscous flux
// is formed in modes.  At K = 2 with viscosity 10700 FP64 multiply-adds an element in the
// place of 24000 with values and gradients at every point.
//
// Bound: FP64 multiply-adds of two waves per SIMD (launch bounds: 256 registers, which the
// accumulators and modes fill; with one wave 138 us in the place of 94) and the wait for the
// neighbours' coefficients.  27^3 BDM_2 (118098 elements): 292 us before, 83-90 now; nu = 0:
// 94 -> 66; 32^3 BDM_1: 78 -> 45; 8^3 BDM_2: 137 -> 49.
template <int K, bool VISC>
__global__ __launch_bounds__(kEBlk, 2) void k_residual3(DevGeo g, DevTabs tb, const double* __restrict__ U,
                                                     double* __restrict__ Lout, double nu) {
  using RL = ResLayout3;
  constexpr int P = nP3(K), NP = nPp3(K), NF = nF3(K), NM = RL::nm(K), NQV = nQV3(K), NQF = nQF3(K);
  __shared__ __align__(16) double s[RL::lds(K)];  // the neighbour's tables differ from lane to lane
  for (int i = threadIdx.x; i < RL::lds(K); i += blockDim.x) s[i] = tb.res[i];
  __syncthreads();
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const double isq = g.isq[t];
  double acc[3][P];
  {
    double u[3][P];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) u[c][i] = U[(size_t)(c * P + i) * T + t];
    double Ji[3][3];
    load_Jinv3(g, t, Ji);
    // modes of u_c u_d (c <= d) of the reference coefficients
    double w[6][NP];
#pragma unroll
    for (int x = 0; x < 6; ++x)
#pragma unroll
      for (int j = 0; j < NP; ++j) w[x][j] = 0;
    const auto vo = cst(tb.res + RL::vol(K));
#pragma unroll 1
    for (int q = 0; q < NQV; ++q) {
      const auto row = vo + q * RL::volStride(K);
      double a[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        a[c] = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) a[c] += u[c][i] * row[i];
      }
      const double uu[6] = {a[0] * a[0], a[0] * a[1], a[0] * a[2], a[1] * a[1], a[1] * a[2], a[2] * a[2]};
#pragma unroll
      for (int x = 0; x < 6; ++x)
#pragma unroll
        for (int j = 0; j < NP; ++j) w[x][j] += uu[x] * row[P + j];
    }
    // flux modes fl[c][d] = isq w_cd - nu gr[c][e] Jinv[e][d], then their products with Jinv^T
    constexpr int kD = 4 * P * NF;
    double gr[3][3][NP];
    if constexpr (VISC) {
      const auto D = cst(again(tb.cond) + kD);
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int e = 0; e < 3; ++e)
#pragma unroll
          for (int j = 0; j < NP; ++j) gr[c][e][j] = 0;
#pragma unroll
      for (int i = 0; i < P; ++i) {
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
          for (int e = 0; e < 3; ++e)
#pragma unroll
            for (int c = 0; c < 3; ++c) gr[c][e][j] += D[(i * NP + j) * 3 + e] * u[c][i];
        table_group<3>(i);
      }
    }
    constexpr int kSym[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        double fl[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          fl[d] = isq * w[kSym[c][d]][j];
          if constexpr (VISC) fl[d] -= nu * (gr[c][0][j] * Ji[0][d] + gr[c][1][j] * Ji[1][d] + gr[c][2][j] * Ji[2][d]);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) gr[c][a][j] = fl[0] * Ji[a][0] + fl[1] * Ji[a][1] + fl[2] * Ji[a][2];
      }
    const auto D = cst(again(tb.cond) + kD);
#pragma unroll
    for (int i = 0; i < P; ++i) {
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[c][i] = 0;
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int e = 0; e < 3; ++e)
#pragma unroll
          for (int c = 0; c < 3; ++c) acc[c][i] += D[(i * NP + j) * 3 + e] * gr[c][e][j];
      table_group<3>(i);
    }
  }

  // faces
#pragma unroll 1
  for (int f = 0; f < 4; ++f) {
    const size_t idx = (size_t)f * T + t;
    const int nb = g.nbr[idx];
    const int code = g.code[idx];
    // a closed boundary face (wall or inflow, nbr = -1): no term (u.n = 0 on a wall; on an
    // inflow the term acts on v.n only, which the increments keep 0); no viscous face terms
    // on any boundary (interior faces only: free slip).  On an outflow face the own trace
    // stands on both sides: -int max(u.n, 0) (u . v), backflow sees zero.
    const bool open = nb < 0;
    if (open && !((code >> 6) & 1)) continue;
    const int tn = open ? t : nb, fn = open ? f : code & 3, pid = open ? 0 : (code >> 2) & 7;
    const double n[3] = {g.nx[idx], g.ny[idx], g.nz[idx]};
    const double li = g.flen[idx] * isq;
    double nJ[3] = {}, gn[3][NM] = {};
    if constexpr (VISC) {
      const double* J = again(g.Jinv);  // read again for every face rather than held, as U below
#pragma unroll
      for (int a = 0; a < 3; ++a)
        nJ[a] = n[0] * J[(size_t)(3 * a) * T + t] + n[1] * J[(size_t)(3 * a + 1) * T + t] +
                n[2] * J[(size_t)(3 * a + 2) * T + t];
    }
    // the neighbour's trace and (sum of both sides') normal derivative, in its face parameters
    double vn[3][NF], vo[3][NF];
    {
      const double isqn = g.isq[tn];
      const double* tr = s + RL::tr(K) + fn * P * NF;
      const double* dg = s + RL::dg(K) + fn * P * NM * 3;
      double nJn[3] = {};
      if constexpr (VISC) {
        double Jn[3][3];
        load_Jinv3(g, tn, Jn);
#pragma unroll
        for (int a = 0; a < 3; ++a) nJn[a] = n[0] * Jn[a][0] + n[1] * Jn[a][1] + n[2] * Jn[a][2];
      }
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < NF; ++m) vo[c][m] = 0;
      double gd[3][NM] = {};
      // two coefficients at a time: with all unrolled, 512 registers and scratch; one at a
      // time waits longer (94 us in the place of 83), five spill (90 us)
      double w[2][3];
#pragma unroll 1
      for (int i0 = 0; i0 < P; i0 += 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int c = 0; c < 3; ++c) w[j][c] = isqn * U[(size_t)(c * P + i0 + j) * T + tn];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int i = i0 + j;
#pragma unroll
          for (int m = 0; m < NF; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c) vo[c][m] += tr[i * NF + m] * w[j][c];
          if constexpr (VISC)
#pragma unroll
            for (int m = 0; m < NM; ++m) {
              const int o = (i * NM + m) * 3;
              const double b = nJn[0] * dg[o] + nJn[1] * dg[o + 1] + nJn[2] * dg[o + 2];
#pragma unroll
              for (int c = 0; c < 3; ++c) gd[c][m] += b * w[j][c];
            }
          table_group<1>(j);
        }
      }
      // to the own face parameters (the modes of P^{K-1} among themselves)
      const double* Q = s + RL::q(K) + pid * NF * NF;
#pragma unroll
      for (int m = 0; m < NF; ++m) {
#pragma unroll
        for (int c = 0; c < 3; ++c) vn[c][m] = 0;
#pragma unroll
        for (int k = 0; k < NF; ++k)
#pragma unroll
          for (int c = 0; c < 3; ++c) vn[c][m] += Q[m * NF + k] * vo[c][k];
        if constexpr (VISC)
          if (m < NM)
#pragma unroll
            for (int k = 0; k < NM; ++k)
#pragma unroll
              for (int c = 0; c < 3; ++c) gn[c][m < NM ? m : 0] += Q[m * NF + k] * gd[c][k];
      }
    }
    // the own ones (vo: own trace)
    {
      const auto tr = cst(again(tb.res) + RL::tr(K) + f * P * NF);
      const auto dg = cst(again(tb.res) + RL::dg(K) + f * P * NM * 3);
      const double* Uo = again(U);  // read again for every face rather than held
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < NF; ++m) vo[c][m] = 0;
      double w[2][3];
#pragma unroll 1
      for (int i0 = 0; i0 < P; i0 += 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int c = 0; c < 3; ++c) w[j][c] = isq * Uo[(size_t)(c * P + i0 + j) * T + t];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int i = i0 + j;
#pragma unroll
          for (int m = 0; m < NF; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c) vo[c][m] += tr[i * NF + m] * w[j][c];
          if constexpr (VISC)
#pragma unroll
            for (int m = 0; m < NM; ++m) {
              const int o = (i * NM + m) * 3;
              const double b = nJ[0] * dg[o] + nJ[1] * dg[o + 1] + nJ[2] * dg[o + 2];
#pragma unroll
              for (int c = 0; c < 3; ++c) gn[c][m] += b * w[j][c];
            }
          table_group<1>(j);
        }
      }
    }
    // upwind flux at the face points, back into modes
    double q[3][NF];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < NF; ++m) q[c][m] = 0;
    const auto pt = cst(tb.res + RL::pt(K));
#pragma unroll 1
    for (int r = 0; r < NQF; ++r) {
      const auto L = pt + r * RL::ptStride(K);
      double uo[3], un[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        uo[c] = un[c] = 0;
#pragma unroll
        for (int m = 0; m < NF; ++m) {
          uo[c] += L[m] * vo[c][m];
          un[c] += L[m] * vn[c][m];
        }
      }
      const double unrm = 0.5 * ((uo[0] + un[0]) * n[0] + (uo[1] + un[1]) * n[1] + (uo[2] + un[2]) * n[2]);
      const bool own_up = unrm >= 0.0;
      const double w = open && !own_up ? 0.0 : L[NF] * unrm;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double fc = w * (own_up ? uo[c] : un[c]);
#pragma unroll
        for (int m = 0; m < NF; ++m) q[c][m] += L[m] * fc;
      }
    }
    // plus the viscous flux; du in vo
    const double nuf = open ? 0.0 : nu, nsig = VISC ? nuf * g.sig[idx] : 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < NF; ++m) {
        if constexpr (VISC) {
          vo[c][m] -= vn[c][m];
          q[c][m] += nsig * vo[c][m];
          if (m < NM) {
            q[c][m] -= 0.5 * nuf * gn[c][m < NM ? m : 0];
            vo[c][m] *= 0.5 * nuf * li;
          }
        }
        q[c][m] *= -li;
      }
    {
      const auto tr = cst(again(tb.res) + RL::tr(K) + f * P * NF);
      const auto dg = cst(again(tb.res) + RL::dg(K) + f * P * NM * 3);
#pragma unroll
      for (int i = 0; i < P; ++i) {
#pragma unroll
        for (int m = 0; m < NF; ++m)
#pragma unroll
          for (int c = 0; c < 3; ++c) acc[c][i] += tr[i * NF + m] * q[c][m];
        if constexpr (VISC)
#pragma unroll
          for (int m = 0; m < NM; ++m) {
            const int o = (i * NM + m) * 3;
            const double b = nJ[0] * dg[o] + nJ[1] * dg[o + 1] + nJ[2] * dg[o + 2];
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[c][i] += b * vo[c][m];
          }
        table_group<2>(i);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) Lout[(size_t)(c * P + i) * T + t] = acc[c][i];
}

// ---------------------------------------------------------------------------------------
// adjoint form on tetrahedra: Ubar = J_L(U)^T Lbar, as on triangles (upwind side frozen):
// with y the broken field of coefficients Lbar, the own coefficients receive
//   volume  int phi . (grad y u + grad y^T u) - nu grad y : grad phi,
//   face    -int [1/2 (phi.n)(u_up . dy) + un (phi . dy) (own side upwind)]
//           + the viscous face terms of y (B_h symmetric), dy = y_own - y_nbr;
// an outflow face -int H(u.n) [(phi.n)(u.y) + (u.n)(phi.y)]; walls and inflows nothing.
// ---------------------------------------------------------------------------------------
template <int K>
__global__ __launch_bounds__(kEBlk) void k_residual_vjp3(DevGeo g, DevTabs tb, const double* __restrict__ U,
                                                         const double* __restrict__ Y, double* __restrict__ Ubar,
                                                         double nu) {
  constexpr int P = nP3(K), NQV = nQV3(K), NQF = nQF3(K);
  __shared__ ResTabs3<K> s;
  stage_tabs3<K>(s, tb);
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= T) return;
  double u[3][P], y[3][P], acc[3][P];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) {
      u[c][i] = U[(size_t)(c * P + i) * T + t];
      y[c][i] = Y[(size_t)(c * P + i) * T + t];
      acc[c][i] = 0;
    }
  double Ji[3][3];
  load_Jinv3(g, t, Ji);
  const double det = g.detJ[t], isq = g.isq[t], sq = det * isq;
  for (int q = 0; q < NQV; ++q) {
    double uq[3], gy[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double a = 0, b[3] = {0, 0, 0};
#pragma unroll
      for (int i = 0; i < P; ++i) {
        a += u[c][i] * s.Vv[q][i];
#pragma unroll
        for (int e = 0; e < 3; ++e) b[e] += y[c][i] * s.Gv[q][e][i];
      }
      uq[c] = a * isq;
#pragma unroll
      for (int j = 0; j < 3; ++j) gy[c][j] = isq * (b[0] * Ji[0][j] + b[1] * Ji[1][j] + b[2] * Ji[2][j]);
    }
    double av[3], Gt[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      av[c] = 0;
#pragma unroll
      for (int j = 0; j < 3; ++j) av[c] += gy[c][j] * uq[j] + gy[j][c] * uq[j];
#pragma unroll
      for (int a = 0; a < 3; ++a)
        Gt[c][a] = -nu * (gy[c][0] * Ji[a][0] + gy[c][1] * Ji[a][1] + gy[c][2] * Ji[a][2]);
    }
    const double w = s.Wv[q] * sq;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i)
        acc[c][i] += w * (av[c] * s.Vv[q][i] + Gt[c][0] * s.Gv[q][0][i] + Gt[c][1] * s.Gv[q][1][i] +
                          Gt[c][2] * s.Gv[q][2][i]);
  }
#pragma unroll 1
  for (int f = 0; f < 4; ++f) {
    const size_t idx = (size_t)f * T + t;
    const int nb = g.nbr[idx];
    const int code = g.code[idx];
    if (nb < 0 && !((code >> 6) & 1)) continue;  // closed boundary face: nothing
    const double n[3] = {g.nx[idx], g.ny[idx], g.nz[idx]};
    const double li = g.flen[idx] * isq;
    if (nb < 0) {  // outflow face
      for (int r = 0; r < NQF; ++r) {
        double uo[3], yo[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          double a = 0, ya = 0;
#pragma unroll
          for (int i = 0; i < P; ++i) {
            a += u[c][i] * s.Vf[f][r][i];
            ya += y[c][i] * s.Vf[f][r][i];
          }
          uo[c] = a * isq;
          yo[c] = ya * isq;
        }
        const double un = uo[0] * n[0] + uo[1] * n[1] + uo[2] * n[2];
        if (un > 0.0) {
          const double w = s.Wf[r] * li, uy = uo[0] * yo[0] + uo[1] * yo[1] + uo[2] * yo[2];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const double av = -(n[c] * uy + un * yo[c]);
#pragma unroll
            for (int i = 0; i < P; ++i) acc[c][i] += w * av * s.Vf[f][r][i];
          }
        }
      }
      continue;
    }
    const int fn = code & 3, pid = (code >> 2) & 7;
    const double sig = g.sig[idx], isqn = g.isq[nb];
    double Jn[3][3];
    load_Jinv3(g, nb, Jn);
    double nJ[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) nJ[a] = n[0] * Ji[a][0] + n[1] * Ji[a][1] + n[2] * Ji[a][2];
    for (int r = 0; r < NQF; ++r) {
      const int rn = s.pidx[pid][r];
      double uo[3], un[3], yo[3], ynb[3], go[3][3], gn[3][3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double a = 0, an = 0, ya = 0, yan = 0, b[3] = {0, 0, 0}, bn[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const double vn = U[(size_t)(c * P + i) * T + nb], wn = Y[(size_t)(c * P + i) * T + nb];
          a += u[c][i] * s.Vf[f][r][i];
          an += vn * s.Vf[fn][rn][i];
          ya += y[c][i] * s.Vf[f][r][i];
          yan += wn * s.Vf[fn][rn][i];
#pragma unroll
          for (int e = 0; e < 3; ++e) {
            b[e] += y[c][i] * s.Gf[f][r][e][i];
            bn[e] += wn * s.Gf[fn][rn][e][i];
          }
        }
        uo[c] = a * isq;
        un[c] = an * isqn;
        yo[c] = ya * isq;
        ynb[c] = yan * isqn;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          go[c][j] = isq * (b[0] * Ji[0][j] + b[1] * Ji[1][j] + b[2] * Ji[2][j]);
          gn[c][j] = isqn * (bn[0] * Jn[0][j] + bn[1] * Jn[1][j] + bn[2] * Jn[2][j]);
        }
      }
      const double unrm = 0.5 * ((uo[0] + un[0]) * n[0] + (uo[1] + un[1]) * n[1] + (uo[2] + un[2]) * n[2]);
      const bool own_up = unrm >= 0.0;
      double dy[3], updy = 0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        dy[c] = yo[c] - ynb[c];
        updy += (own_up ? uo[c] : un[c]) * dy[c];
      }
      double Av[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double avgn = 0.5 * ((go[c][0] + gn[c][0]) * n[0] + (go[c][1] + gn[c][1]) * n[1] +
                                   (go[c][2] + gn[c][2]) * n[2]);
        const double conv = -(0.5 * n[c] * updy + (own_up ? unrm * dy[c] : 0.0));
        Av[c] = conv + nu * avgn - nu * sig * dy[c];  // minus the viscous flux Q(y)
      }
      const double w = s.Wf[r] * li;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double h = 0.5 * nu * dy[c];
#pragma unroll
        for (int i = 0; i < P; ++i)
          acc[c][i] += w * (Av[c] * s.Vf[f][r][i] +
                            h * (nJ[0] * s.Gf[f][r][0][i] + nJ[1] * s.Gf[f][r][1][i] + nJ[2] * s.Gf[f][r][2][i]));
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) Ubar[(size_t)(c * P + i) * T + t] = acc[c][i];
}

// ---------------------------------------------------------------------------------------
// a4 / a6: element condensation and recovery (eq. (FE3), orthonormal basis: M_T = I)
// ---------------------------------------------------------------------------------------
// The reference matrices of the condensation, DevTabs::cond: the face moments [4][P][NF] and
// the divergence moments [P][NP][3], so that what one basis function i needs lies together.
// They are read as scalars, a group of a few i at a time.  Left to itself the compiler loads
// all 720 SGPRs' worth once (K = 2) and keeps them in the lanes of vector registers: 4200
// v_readlane of 6600 instructions and 50 KB of code in k_mf_apply3, which every launch fetches
// again.  From LDS the same values took as long, in more registers.  The face basis
// permutations Qf differ from lane to lane: LDS (as loads from memory they were 288 a thread).
template <int K>
struct CondTabs3 {
  static constexpr int P = nP3(K), NF = nF3(K), NP = nPp3(K);
  double Qf[6][NF][NF];
};
template <int K>
__device__ inline void stage_cond3(CondTabs3<K>& s, const double* __restrict__ Qf) {  // (the caller synchronises)
  double* d = &s.Qf[0][0][0];
  for (int i = threadIdx.x; i < 6 * nF3(K) * nF3(K); i += blockDim.x) d[i] = Qf[i];
}
// y <- W_T y = y - D_T^T (D_T D_T^T)^{-1} D_T y, D_T = sum_a Jinv[a][c] Dh[a]
template <int K>
__device__ inline void apply_W3(double (&y)[3][nP3(K)], const double (&Ji)[3][3], const double* __restrict__ G, int T,
                                int t, const double* cond) {
  constexpr int P = nP3(K), NP = nPp3(K), kD = 4 * P * nF3(K);
  auto D = cst(again(cond) + kD);
  double d[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) d[j] = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) {  // the reference components w = Jinv y serve every j
    double w[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) w[e] = Ji[e][0] * y[0][i] + Ji[e][1] * y[1][i] + Ji[e][2] * y[2][i];
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int e = 0; e < 3; ++e) d[j] += D[(i * NP + j) * 3 + e] * w[e];
    table_group<3>(i);
  }
  D = cst(again(cond) + kD);
  double x[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) x[j] = 0;
#pragma unroll
  for (int j = 0, p = 0; j < NP; ++j)
#pragma unroll
    for (int l = 0; l <= j; ++l, ++p) {
      const double gv = G[(size_t)p * T + t];
      x[j] += gv * d[l];
      if (l != j) x[l] += gv * d[j];
    }
#pragma unroll
  for (int i = 0; i < P; ++i) {
    double w[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      w[e] = 0;
#pragma unroll
      for (int j = 0; j < NP; ++j) w[e] += D[(i * NP + j) * 3 + e] * x[j];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) y[c][i] -= Ji[0][c] * w[0] + Ji[1][c] * w[1] + Ji[2][c] * w[2];
    table_group<3>(i);
  }
}

// m = the face moments of y (n: the normal times sqrt(2|F| / det J)), and y += their transpose.
template <int K>
__device__ inline void face_rows3(const double (&y)[3][nP3(K)], const double (&n)[3], const double* cond, int f,
                                  double (&m)[nF3(K)]) {
  constexpr int P = nP3(K), NF = nF3(K);
  const auto Ch = cst(again(cond) + f * P * NF);
#pragma unroll
  for (int a = 0; a < NF; ++a) m[a] = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const double yn = n[0] * y[0][i] + n[1] * y[1][i] + n[2] * y[2][i];
#pragma unroll
    for (int a = 0; a < NF; ++a) m[a] += Ch[i * NF + a] * yn;
    table_group<3>(i);
  }
}
template <int K>
__device__ inline void face_add3(double (&y)[3][nP3(K)], const double (&n)[3], const double* cond, int f,
                                 const double (&m)[nF3(K)]) {
  constexpr int P = nP3(K), NF = nF3(K);
  const auto Ch = cst(again(cond) + f * P * NF);
#pragma unroll
  for (int i = 0; i < P; ++i) {
    double s = 0;
#pragma unroll
    for (int a = 0; a < NF; ++a) s += m[a] * Ch[i * NF + a];
#pragma unroll
    for (int c = 0; c < 3; ++c) y[c][i] += n[c] * s;
    table_group<3>(i);
  }
}
// m <- Q m (R side to L side) or Q^T m.
template <int K, bool TR>
__device__ inline void face_map3(const double (&Q)[nF3(K)][nF3(K)], double (&m)[nF3(K)]) {
  constexpr int NF = nF3(K);
  double w[NF];
#pragma unroll
  for (int a = 0; a < NF; ++a) {
    w[a] = 0;
#pragma unroll
    for (int b = 0; b < NF; ++b) w[a] += (TR ? Q[b][a] : Q[a][b]) * m[b];
  }
#pragma unroll
  for (int a = 0; a < NF; ++a) m[a] = w[a];
}

// q[4][NF][T] = C_T W_T F_T per element and local face, in the L side's face basis (the
// R side maps its own face moments through the orthogonal matrix Qf of the permutation).
template <int K>
__global__ __launch_bounds__(kEBlk) void k_cond_rhs3(DevGeo g, DevTabs tb, const double* __restrict__ F,
                                                     double* __restrict__ q) {
  constexpr int P = nP3(K), NF = nF3(K);
  __shared__ __align__(16) CondTabs3<K> s;
  stage_cond3<K>(s, tb.Qf);
  __syncthreads();
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= T) return;
  double y[3][P];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) y[c][i] = F[(size_t)(c * P + i) * T + t];
  double Ji[3][3];
  load_Jinv3(g, t, Ji);
  apply_W3<K>(y, Ji, g.G, T, t, tb.cond);
#pragma unroll 1
  for (int f = 0; f < 4; ++f) {
    const size_t idx = (size_t)f * T + t;
    const double sc = g.sF[idx];
    const double n[3] = {sc * g.nx[idx], sc * g.ny[idx], sc * g.nz[idx]};
    const int code = g.code[idx];
    double m[NF];
    face_rows3<K>(y, n, tb.cond, f, m);
    if ((code >> 5) & 1) face_map3<K, false>(s.Qf[(code >> 2) & 7], m);
#pragma unroll
    for (int mm = 0; mm < NF; ++mm) q[(size_t)(f * NF + mm) * T + t] = m[mm];
  }
}

// u = W_T (F_T - C_T^T lambda_T); out = u (mode 0) or a Un + b (Us + dt u) (mode 1).
template <int K>
__global__ __launch_bounds__(kEBlk) void k_recover3(DevGeo g, DevTabs tb, const double* __restrict__ F,
                                                    const double* __restrict__ lam, double* __restrict__ out, int mode,
                                                    double ca, const double* __restrict__ Un, double cb,
                                                    const double* __restrict__ Us, double dt) {
  constexpr int P = nP3(K), NF = nF3(K);
  __shared__ __align__(16) CondTabs3<K> s;
  stage_cond3<K>(s, tb.Qf);
  __syncthreads();
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= T) return;
  double y[3][P];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) y[c][i] = F[(size_t)(c * P + i) * T + t];
#pragma unroll 1
  for (int f = 0; f < 4; ++f) {
    const size_t idx = (size_t)f * T + t;
    const int Fc = g.efacet[idx];
    const int code = g.code[idx];
    double lm[NF];
#pragma unroll
    for (int a = 0; a < NF; ++a) lm[a] = lam[(size_t)Fc * NF + a];
    if ((code >> 5) & 1) face_map3<K, true>(s.Qf[(code >> 2) & 7], lm);  // own face coefficients
    const double sc = -g.sF[idx];
    const double n[3] = {sc * g.nx[idx], sc * g.ny[idx], sc * g.nz[idx]};
    face_add3<K>(y, n, tb.cond, f, lm);
  }
  double Ji[3][3];
  load_Jinv3(g, t, Ji);
  apply_W3<K>(y, Ji, g.G, T, t, tb.cond);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const size_t o = (size_t)(c * P + i) * T + t;
      if (mode == 0) out[o] = y[c][i];
      else out[o] = ca * Un[o] + cb * (Us[o] + dt * y[c][i]);
    }
}

// ---------------------------------------------------------------------------------------
// a5: matrix-free product of the facet system, S p = sum_T C_T W_T C_T^T p (eq. (FE3)
// condensed), in the PCG iteration it (read from the scalars): beta and the stopping test
// from the partials of the previous updates, exactly as the BSR kernel forms them.
// ---------------------------------------------------------------------------------------
// Element pass: p = z + beta p_old at the element's four faces (the L side's face basis,
// mapped to the own one on R faces), y = W_T C_T^T p, and the face contributions C_T y
// (mapped back) into A.mfq [E][side][NF], where the two sides of a face lie together for the
// next kernel.  The L side writes p.  The element's share of (p, S p) is |y|^2 (W_T is an
// orthogonal projector), that of (z, S p) comes from its contributions; one partial of each
// per block, over a grid-stride loop on the facet kernels' grid.
//
// All indices, normals and face values are loaded ahead of the arithmetic, at two waves per
// SIMD (rolled over the faces, three waves: 70 us against 67 at 32^3, and 44 against 36 at
// K = 1).  Bound by the latency of that chain and by the 312 B of geometry and 576 B of face
// values an element; 1500 FP64 instructions are 8 us of it.  With the face pass 136 -> 67 us
// at 32^3 BDM_2 (16^3: 43 -> 26, 24^3: 41).
template <int K>
__global__ __launch_bounds__(kBlk) void k_mf_apply3(DevGeo g, DevBsr A, const double* __restrict__ z,
                                                    const double* __restrict__ p_old, double* __restrict__ p_new,
                                                    PcgScalars* sc, const double* __restrict__ rz_prev,
                                                    const double* __restrict__ rz_prev2, double* __restrict__ pq) {
  constexpr int P = nP3(K), NF = nF3(K);
  if (sc->done != PCG_RUNNING) return;
  __shared__ __align__(16) CondTabs3<K> s;
  const int G = gridDim.x, it = sc->it, T = g.T;
  PartLoad<2> q1, q2;
  partials_load<2>(rz_prev, G, true, q1);
  partials_load<2>(rz_prev2, G, it >= 2, q2);
  stage_cond3<K>(s, A.mfQf);  // visible after the sums' synchronisation
  // the grid is the facet kernels'; the blocks with elements are spread over all XCDs
  const int nb = min(G, (T + kBlk - 1) / kBlk);
  const int t0 = (int)blockIdx.x < nb ? xcd_block(nb) * kBlk + threadIdx.x : T;
  double t1[2], t2[2], beta = 0;
  partials_sum<2>(q1, G, t1);
  partials_sum<2>(q2, G, t2);
  if (it >= 2) beta = t1[0] / t2[0];
  int status = PCG_RUNNING;
  if (!isfinite(t1[0]) || !isfinite(t1[1]) || !isfinite(beta)) status = PCG_NONFINITE;
  else if (t1[1] <= sc->tol2) status = PCG_CONVERGED;
  else if (it - 1 >= sc->maxit) status = PCG_MAXIT;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->iters = it - 1;
    sc->rr = t1[1];
    sc->rz = t1[0];
    if (it == 1) sc->rr0 = t1[1];
    if (status != PCG_RUNNING) sc->done = status;
  }
  if (status != PCG_RUNNING) return;
  double v[2] = {0, 0};
  for (int t = t0; t < T; t += nb * kBlk) {
    // indices, normals and the kernel vector's values of all faces first: the face values
    // are one round trip behind them
    int code[4], Fc[4];
    double zd[4], n[4][3];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const size_t idx = (size_t)f * T + t;
      code[f] = g.code[idx];
      Fc[f] = g.efacet[idx];
    }
    double lz[4][NF];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const size_t idx = (size_t)f * T + t;
      const double sc2 = g.sF[idx];
      n[f][0] = sc2 * g.nx[idx];
      n[f][1] = sc2 * g.ny[idx];
      n[f][2] = sc2 * g.nz[idx];
      zd[f] = g.zdef[Fc[f]];
    }
    double y[3][P];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) y[c][i] = 0;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const size_t o = (size_t)Fc[f] * NF;
#pragma unroll
      for (int a = 0; a < NF; ++a) lz[f][a] = z[o + a] + beta * p_old[o + a];
    }
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const size_t o = (size_t)Fc[f] * NF;
      double (&lm)[NF] = lz[f];
      if ((code[f] >> 5) & 1) {
        face_map3<K, true>(s.Qf[(code[f] >> 2) & 7], lm);
      } else {
#pragma unroll
        for (int a = 0; a < NF; ++a) p_new[o + a] = lm[a];
        if ((code[f] >> 6) & 1)  // an outflow face: its row of S is the identity
#pragma unroll
          for (int a = 0; a < NF; ++a) v[0] += lm[a] * lm[a];
      }
      face_add3<K>(y, n[f], A.mfcond, f, lm);
    }
    double Ji[3][3];
    load_Jinv3(g, t, Ji);
    apply_W3<K>(y, Ji, g.G, T, t, A.mfcond);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) v[0] += y[c][i] * y[c][i];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const bool R = (code[f] >> 5) & 1;
      double m[NF];
      face_rows3<K>(y, n[f], A.mfcond, f, m);
      if (R) {
        face_map3<K, false>(s.Qf[(code[f] >> 2) & 7], m);
      } else if ((code[f] >> 6) & 1) {
        const size_t o = (size_t)Fc[f] * NF;
#pragma unroll
        for (int a = 0; a < NF; ++a) m[a] = z[o + a] + beta * p_old[o + a];
      }
      double* q = A.mfq + ((size_t)Fc[f] * 2 + (R ? 1 : 0)) * NF;
#pragma unroll
      for (int mm = 0; mm < NF; ++mm) q[mm] = m[mm];
      v[1] += zd[f] * m[0];
    }
  }
  block_write_partial<2>(v, pq);
}

// Sums of the two sides' contributions of entry i (mode i % NF of face i / NF), and of entries
// i and i + 1 (NF even, i even); a boundary face has one side, its other half stays zero.
template <int NF>
__device__ inline double mf_sp(const double* __restrict__ q, long i) {
  const long o = i + (i / NF) * NF;
  return q[o] + q[o + NF];
}
template <int NF>
__device__ inline double2 mf_sp2(const double* __restrict__ q, long i) {
  const long o = i + (i / NF) * NF;
  const double2 a = *(const double2*)(q + o), b = *(const double2*)(q + o + NF);
  return {a.x + b.x, a.y + b.y};
}

// Sp = S p for the multigrid iterations, whose next kernel gathers it.
template <int NF>
__global__ __launch_bounds__(kBlk) void k_mf_sum(long n, const double* __restrict__ q, double* __restrict__ Sp,
                                                 const PcgScalars* sc) {
  if (sc->done != PCG_RUNNING) return;
  for (long u = (long)xcd_block() * kBlk + threadIdx.x; NF * u < n; u += (long)gridDim.x * kBlk) {
    const long i = NF * u;
    if constexpr (NF % 2 == 0) {
#pragma unroll
      for (int a = 0; a < NF; a += 2) *(double2*)(Sp + i + a) = mf_sp2<NF>(q, i + a);
    } else {
#pragma unroll
      for (int a = 0; a < NF; ++a) Sp[i + a] = mf_sp<NF>(q, i + a);
    }
  }
}

// The PCG update of point- and facet-block-Jacobi iterations (k_pcg_update) with S p summed
// from the two sides on the way: it is neither written nor read as a vector.
template <int NF, bool BJ>
__global__ __launch_bounds__(kBlk) void k_mf_update(DevGeo g, DevBsr A, const double* __restrict__ p,
                                                    double* __restrict__ x, double* __restrict__ r,
                                                    double* __restrict__ z, PcgScalars* sc,
                                                    const double* __restrict__ rz_prev,
                                                    const double* __restrict__ pq, double* __restrict__ rz_out) {
  const int done = sc->done;  // tested after the sums (see PcgScalars)
  const int G = gridDim.x;
  double t1[2], t2[2];
  block_sum_partials<2>(rz_prev, G, t1);
  block_sum_partials<2>(pq, G, t2);
  if (done != PCG_RUNNING) return;
  int status = PCG_RUNNING;
  if (!isfinite(t2[0])) status = PCG_NONFINITE;
  else if (!(t2[0] > 0)) status = PCG_BREAKDOWN;
  if (status != PCG_RUNNING) {
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->done = status;
    return;
  }
  const double alpha = t1[0] / t2[0], dz = t2[1];
  const double* __restrict__ q = A.mfq;
  double v[2] = {0, 0};
  if constexpr (!BJ && NF % 2 == 0) {
    const long n2 = (long)g.E * NF / 2;
    for (long u = (long)xcd_block() * kBlk + threadIdx.x; u < n2; u += (long)G * kBlk) {
      const long i = 2 * u;
      const double2 s = mf_sp2<NF>(q, i), pv = ((const double2*)p)[u], dv = ((const double2*)A.dinv)[u];
      double2 xv = ((double2*)x)[u], rv = ((double2*)r)[u], zv;
      xv.x += alpha * pv.x;
      xv.y += alpha * pv.y;
      const double s0 = i % NF == 0 ? s.x - dz * g.zdef[i / NF] : s.x;
      rv.x -= alpha * s0;
      rv.y -= alpha * s.y;
      zv.x = dv.x * rv.x;
      zv.y = dv.y * rv.y;
      ((double2*)x)[u] = xv;
      ((double2*)r)[u] = rv;
      ((double2*)z)[u] = zv;
      v[0] += rv.x * zv.x + rv.y * zv.y;
      v[1] += rv.x * rv.x + rv.y * rv.y;
    }
  } else {
    for (int F = xcd_block() * kBlk + threadIdx.x; F < g.E; F += G * kBlk) {
      double rr[NF], zz[NF];
#pragma unroll
      for (int a = 0; a < NF; ++a) {
        const long o = (long)F * NF + a;
        double s = mf_sp<NF>(q, o);
        if (a == 0) s -= dz * g.zdef[F];
        x[o] += alpha * p[o];
        rr[a] = r[o] - alpha * s;
        r[o] = rr[a];
      }
#pragma unroll
      for (int a = 0; a < NF; ++a) {
        if constexpr (BJ) {
          zz[a] = 0;
#pragma unroll
          for (int b = 0; b < NF; ++b) zz[a] += A.binv[((size_t)F * NF + a) * NF + b] * rr[b];
        } else {
          zz[a] = A.dinv[(size_t)F * NF + a] * rr[a];
        }
        z[(size_t)F * NF + a] = zz[a];
        v[0] += rr[a] * zz[a];
        v[1] += rr[a] * rr[a];
      }
    }
  }
  block_write_partial<2>(v, rz_out);
  if (blockIdx.x == 0 && threadIdx.x == 0) sc->it = sc->it + 1;
}

// A launch that carries the start / stop events of the timing entry point where they are set.
#define DFDG_LAUNCH_EV(E0, E1, KER, GRID, S, ...)                                          \
  do {                                                                                    \
    if ((E0) || (E1)) hipExtLaunchKernelGGL(KER, GRID, dim3(kBlk), 0, S, E0, E1, 0, __VA_ARGS__); \
    else hipLaunchKernelGGL(KER, GRID, dim3(kBlk), 0, S, __VA_ARGS__);                    \
  } while (0)

hipError_t launch_mf_spmv3(int NF, const DevGeo& g, const DevBsr& A, const double* z, const double* p_old,
                           double* p_new, double* Sp, const PcgBufs& pb, int it, bool form_Sp, hipStream_t s) {
  const double* prev = pb.rz[(it - 1) & 1];
  const double* prev2 = pb.rz[it & 1];
  hipEvent_t e0, e1;  // kernel timing: start of the element pass to the end of the face pass
  get_dispatch_events(&e0, &e1);
  const dim3 gr(g.fgrid);
  const hipEvent_t last = form_Sp ? nullptr : e1;
  const long n = (long)g.E * NF;
  const double* q = A.mfq;
  const PcgScalars* csc = pb.sc;
  if (A.mfK == 1 && NF == 3) {
    DFDG_LAUNCH_EV(e0, last, (k_mf_apply3<1>), gr, s, g, A, z, p_old, p_new, pb.sc, prev, prev2, pb.pq);
    if (form_Sp) DFDG_LAUNCH_EV((hipEvent_t)nullptr, e1, (k_mf_sum<3>), gr, s, n, q, Sp, csc);
  } else if (A.mfK == 2 && NF == 6) {
    DFDG_LAUNCH_EV(e0, last, (k_mf_apply3<2>), gr, s, g, A, z, p_old, p_new, pb.sc, prev, prev2, pb.pq);
    if (form_Sp) DFDG_LAUNCH_EV((hipEvent_t)nullptr, e1, (k_mf_sum<6>), gr, s, n, q, Sp, csc);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_mf_update3(int NF, bool bj, const DevGeo& g, const DevBsr& A, const double* p, double* x, double* r,
                             double* z, const PcgBufs& pb, int it, hipStream_t s) {
  const dim3 gr(g.fgrid), bl(kBlk);
  const double *prev = pb.rz[(it - 1) & 1], *pq = pb.pq;
  double* out = pb.rz[it & 1];
  if (NF == 3 && bj) hipLaunchKernelGGL((k_mf_update<3, true>), gr, bl, 0, s, g, A, p, x, r, z, pb.sc, prev, pq, out);
  else if (NF == 3) hipLaunchKernelGGL((k_mf_update<3, false>), gr, bl, 0, s, g, A, p, x, r, z, pb.sc, prev, pq, out);
  else if (NF == 6 && bj) hipLaunchKernelGGL((k_mf_update<6, true>), gr, bl, 0, s, g, A, p, x, r, z, pb.sc, prev, pq, out);
  else if (NF == 6) hipLaunchKernelGGL((k_mf_update<6, false>), gr, bl, 0, s, g, A, p, x, r, z, pb.sc, prev, pq, out);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// a2 / a10: load vector, evaluation and diagnostics
// ---------------------------------------------------------------------------------------
template <int K>
__global__ __launch_bounds__(kEBlk) void k_load_vector3(DevGeo g, DevTabs tb, int nqp, const double* __restrict__ fq,
                                                        double* __restrict__ F) {
  constexpr int P = nP3(K);
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const double sq = sqrt(g.detJ[t]);
  double acc[3][P];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) acc[c][i] = 0;
  for (int q = 0; q < nqp; ++q) {
    const double w = tb.Wp[q] * sq;
    double f[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) f[c] = fq[(size_t)(c * nqp + q) * T + t] * w;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const double v = tb.Vp[q * P + i];
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[c][i] += f[c] * v;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) F[(size_t)(c * P + i) * T + t] = acc[c][i];
}

template <int K>
__global__ __launch_bounds__(kEBlk) void k_eval3(DevGeo g, int npts, const double* __restrict__ tab,
                                                 const double* __restrict__ U, double* __restrict__ out) {
  constexpr int P = nP3(K);
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const double isq = g.isq[t];
  double u[3][P];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int i = 0; i < P; ++i) u[c][i] = U[(size_t)(c * P + i) * T + t];
  for (int p = 0; p < npts; ++p)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double s = 0;
#pragma unroll
      for (int i = 0; i < P; ++i) s += u[c][i] * tab[p * P + i];
      out[(size_t)(c * npts + p) * T + t] = s * isq;
    }
}

// Per block: sum 0.5 U^2, sum |curl u|^2 (volume rule), max |div u| (volume points),
// max |[[u.n]]| (face points, faces this element owns as L side).
template <int K>
__global__ __launch_bounds__(kEBlk) void k_diag3(DevGeo g, DevTabs tb, const double* __restrict__ U,
                                                 double* __restrict__ partials) {
  constexpr int P = nP3(K), NQV = nQV3(K), NQF = nQF3(K);
  const int T = g.T;
  const int t = xcd_block() * blockDim.x + threadIdx.x;
  double en = 0, ens = 0, dmax = 0, jmax = 0;
  if (t < T) {
    double u[3][P];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) {
        u[c][i] = U[(size_t)(c * P + i) * T + t];
        en += 0.5 * u[c][i] * u[c][i];
      }
    double Ji[3][3];
    load_Jinv3(g, t, Ji);
    const double det = g.detJ[t], isq = g.isq[t];
    for (int q = 0; q < NQV; ++q) {
      double gr[3][3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double b[3] = {0, 0, 0};
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
          for (int e = 0; e < 3; ++e) b[e] += u[c][i] * tb.Gv[(q * 3 + e) * P + i];
#pragma unroll
        for (int j = 0; j < 3; ++j) gr[c][j] = isq * (b[0] * Ji[0][j] + b[1] * Ji[1][j] + b[2] * Ji[2][j]);
      }
      const double w0 = gr[2][1] - gr[1][2], w1 = gr[0][2] - gr[2][0], w2 = gr[1][0] - gr[0][1];
      ens += tb.Wv[q] * det * (w0 * w0 + w1 * w1 + w2 * w2);
      dmax = fmax(dmax, fabs(gr[0][0] + gr[1][1] + gr[2][2]));
    }
    for (int f = 0; f < 4; ++f) {
      const size_t idx = (size_t)f * T + t;
      const int code = g.code[idx];
      if ((code >> 5) & 1) continue;  // the L side measures the face
      if ((code >> 6) & 1) continue;  // outflow boundary: u.n is free there
      const int nb = g.nbr[idx], fn = code & 3, pid = (code >> 2) & 7;
      const bool wall = nb < 0;  // the jump across a wall is u.n itself
      const int nbs = wall ? t : nb;
      const double n0 = g.nx[idx], n1 = g.ny[idx], n2 = g.nz[idx], isqn = g.isq[nbs];
      for (int r = 0; r < NQF; ++r) {
        const int rn = tb.fpidx[pid * NQF + r];
        double jo = 0, jn = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const double vo = tb.Vf[(f * NQF + r) * P + i], vn = tb.Vf[(fn * NQF + rn) * P + i];
          jo += (u[0][i] * n0 + u[1][i] * n1 + u[2][i] * n2) * vo;
          if (!wall)
            jn += (U[(size_t)i * T + nbs] * n0 + U[(size_t)(P + i) * T + nbs] * n1 + U[(size_t)(2 * P + i) * T + nbs] * n2) * vn;
        }
        jmax = fmax(jmax, fabs(jo * isq - jn * isqn));
      }
    }
  }
  __shared__ double sh[4][kEBlk / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  en = wave_sum(en);
  ens = wave_sum(ens);
  dmax = wave_max(dmax);
  jmax = wave_max(jmax);
  if (lane == 0) { sh[0][wid] = en; sh[1][wid] = ens; sh[2][wid] = dmax; sh[3][wid] = jmax; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0, b = 0, c = 0, d = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      a += sh[0][w]; b += sh[1][w]; c = fmax(c, sh[2][w]); d = fmax(d, sh[3][w]);
    }
    partials[4 * blockIdx.x + 0] = a;
    partials[4 * blockIdx.x + 1] = b;
    partials[4 * blockIdx.x + 2] = c;
    partials[4 * blockIdx.x + 3] = d;
  }
}

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
#define DFDG_DISPATCH_K3(K, ...)                                  \
  switch (K) {                                                    \
    case 1: { constexpr int KK = 1; __VA_ARGS__; } break;         \
    case 2: { constexpr int KK = 2; __VA_ARGS__; } break;         \
    default: return hipErrorInvalidValue;                         \
  }

// A launch that carries the start/stop events set by set_dispatch_events (kernel timing).
#define DFDG_LAUNCH_TIMED3(KER, GRID, BLK, S, ...)                                       \
  do {                                                                                  \
    hipEvent_t e0_, e1_;                                                                \
    get_dispatch_events(&e0_, &e1_);                                                    \
    if (e0_) hipExtLaunchKernelGGL(KER, GRID, BLK, 0, S, e0_, e1_, 0, __VA_ARGS__);     \
    else hipLaunchKernelGGL(KER, GRID, BLK, 0, S, __VA_ARGS__);                         \
  } while (0)

hipError_t launch_residual3(int K, const DevGeo& g, const DevTabs& tb, const double* U, double* L, double nu,
                            hipStream_t s) {
  const dim3 grid(nblk(g.T, kEBlk)), blk(kEBlk);
  DFDG_DISPATCH_K3(K, {
    if (nu != 0.0) DFDG_LAUNCH_TIMED3((k_residual3<KK, true>), grid, blk, s, g, tb, U, L, nu);
    else DFDG_LAUNCH_TIMED3((k_residual3<KK, false>), grid, blk, s, g, tb, U, L, nu);
  });
  return hipGetLastError();
}

hipError_t launch_residual_vjp3(int K, const DevGeo& g, const DevTabs& tb, const double* U, const double* Lbar,
                                double* Ubar, double nu, hipStream_t s) {
  DFDG_DISPATCH_K3(K, hipLaunchKernelGGL((k_residual_vjp3<KK>), dim3(nblk(g.T, kEBlk)), dim3(kEBlk), 0, s, g, tb, U,
                                         Lbar, Ubar, nu));
  return hipGetLastError();
}

hipError_t launch_cond_rhs3(int K, const DevGeo& g, const DevTabs& tb, const double* F, double* q, hipStream_t s) {
  DFDG_DISPATCH_K3(K, hipLaunchKernelGGL((k_cond_rhs3<KK>), dim3(nblk(g.T, kEBlk)), dim3(kEBlk), 0, s, g, tb, F, q));
  return hipGetLastError();
}

hipError_t launch_recover3(int K, const DevGeo& g, const DevTabs& tb, const double* F, const double* lam, double* out,
                           int mode, double a, const double* Un, double b, const double* Us, double dt, hipStream_t s) {
  DFDG_DISPATCH_K3(K, hipLaunchKernelGGL((k_recover3<KK>), dim3(nblk(g.T, kEBlk)), dim3(kEBlk), 0, s, g, tb, F, lam,
                                         out, mode, a, Un, b, Us, dt));
  return hipGetLastError();
}

hipError_t launch_load_vector3(int K, int nqp, const DevGeo& g, const DevTabs& tb, const double* fq, double* F,
                               hipStream_t s) {
  DFDG_DISPATCH_K3(K, hipLaunchKernelGGL((k_load_vector3<KK>), dim3(nblk(g.T, kEBlk)), dim3(kEBlk), 0, s, g, tb, nqp,
                                         fq, F));
  return hipGetLastError();
}

hipError_t launch_eval3(int K, int npts, const DevGeo& g, const double* tab, const double* U, double* out,
                        hipStream_t s) {
  DFDG_DISPATCH_K3(K, hipLaunchKernelGGL((k_eval3<KK>), dim3(nblk(g.T, kEBlk)), dim3(kEBlk), 0, s, g, npts, tab, U,
                                         out));
  return hipGetLastError();
}

hipError_t launch_diagnostics3(int K, const DevGeo& g, const DevTabs& tb, const double* U, double* partials,
                               double* res, hipStream_t s) {
  const unsigned nb = nblk(g.T, kEBlk);
  DFDG_DISPATCH_K3(K, hipLaunchKernelGGL((k_diag3<KK>), dim3(nb), dim3(kEBlk), 0, s, g, tb, U, partials));
  return launch_diag_finish((int)nb, partials, res, s);
}

}  // namespace dfdg
