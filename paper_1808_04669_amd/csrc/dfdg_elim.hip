// Block elimination of the facet system on small meshes, the PCG's preconditioner there
// (gfx950): an exact solve in FP32 up to rounding, in three kernels and one for (r, z).
//
// Why.  On a small mesh every kernel of the multigrid cycle costs 2.4 to 8 us of serial memory
// round trips plus a kernel boundary, whatever its few rows; an iteration of 10 to 12 kernels
// takes about 50 us and a solve 9 to 30 of them.  The elimination reads more (up to 128 M
// values, against about 45 a row of S), at rates the chip has to spare there, in four kernels,
// and a solve needs two iterations: 16x16 BDM_1 projection 541 -> 135 us, 57x57 BDM_2 915 ->
// 179, 11^3 tetrahedra BDM_1 1217 -> 408.
//
// What bounds a kernel of the solve: its reads of the matrices, 57x57 BDM_2 (22 M values) at
// 2.5 to 4 TB/s from the Infinity Cache; below about 1 M values the memory latency.
//
// Set-up (FP64, once per context): cell fronts are assembled from the element matrices and
// swept over their interior unknowns 32 pivots at a time, which leaves the inverse of the
// interior block, G = S_BB^{-1} S_BN and the Schur complement in place; the interface matrix
// is the sum of the Schur complements, inverted by the same sweeps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "dfdg_device.h"
#include "dfdg_kernels.h"

namespace dfdg {

static constexpr int kPiv = 32;   // pivots per sweep step
static constexpr int kTile = 64;  // tile of the sweep's update

// ---- set-up ------------------------------------------------------------------------------

// Front of a cell (a workgroup each): the sum of its elements' matrices S_T [nr][nr], one
// element after the other.
__global__ __launch_bounds__(kBlk) void k_el_fronts(ElimDev D, int nfac, const double* __restrict__ ST) {
  const int c = blockIdx.x, NF = D.NF, nr = nfac * NF;
  const int nB = D.boff[c + 1] - D.boff[c], nN = D.noff[c + 1] - D.noff[c], V = (nB + nN) * NF;
  double* F = D.front + D.foff[c];
  for (long i = threadIdx.x; i < (long)V * V; i += kBlk) F[i] = 0;
  __syncthreads();
  for (int k = D.eoff[c]; k < D.eoff[c + 1]; ++k) {
    const int t = D.elem[k];
    for (int i = threadIdx.x; i < nr * nr; i += kBlk) {
      const int a = i / nr, b = i % nr;
      const int ra = D.elp[(size_t)t * nfac + a / NF] * NF + a % NF;
      const int rb = D.elp[(size_t)t * nfac + b / NF] * NF + b % NF;
      F[(size_t)ra * V + rb] += ST[(size_t)t * nr * nr + i];
    }
    __syncthreads();
  }
}

// Matrix `c` of a batch: the cell fronts (which = 0, pivots the interior unknowns) or the
// interface matrix (which = 1, all unknowns).
// Only the tiles on and above the diagonal are kept up to date by the sweeps.
struct SweepMat {
  double* A;
  int V, np;  // rows, pivots
  __device__ inline double at(int i, int j) const {
    return i / kTile <= j / kTile ? A[(size_t)i * V + j] : A[(size_t)j * V + i];
  }
};
__device__ inline SweepMat sweep_mat(const ElimDev& D, int which, int c) {
  if (which) return {D.top, D.ng * D.NF, D.ng * D.NF};
  const int nB = D.boff[c + 1] - D.boff[c], nN = D.noff[c + 1] - D.noff[c];
  return {D.front + D.foff[c], (nB + nN) * D.NF, nB * D.NF};
}

// Interface matrix, a workgroup per interface facet (its NF rows): the Schur complements of
// the facet's two cells, plus shift zhat zhat^T (zhat the normalised kernel vector on the
// interface; shift = 0 for a definite system).
__global__ __launch_bounds__(kBlk) void k_el_interface(ElimDev D, double shift) {
  const int gi = blockIdx.x, NF = D.NF, n = D.ng * NF;
  double* R = D.top + (size_t)gi * NF * n;
  const double zi = D.zhat[gi];
  for (int i = threadIdx.x; i < NF * n; i += kBlk) {
    const int m = i / n, j = i % n;
    R[i] = (m == 0 && j % NF == 0) ? shift * zi * D.zhat[j / NF] : 0.0;
  }
  __syncthreads();
  for (int side = 0; side < 2; ++side) {
    const int pos = D.gpos[2 * gi + side];
    if (pos >= 0) {
      const int c = D.gcell[2 * gi + side], n0 = D.noff[c];
      const int nB = D.boff[c + 1] - D.boff[c], nN = D.noff[c + 1] - n0, V = (nB + nN) * NF;
      const SweepMat F{D.front + D.foff[c], V, 0};
      const int r0 = (nB + pos - n0) * NF, q0 = nB * NF;
      for (int i = threadIdx.x; i < NF * nN * NF; i += kBlk) {
        const int m = i / (nN * NF), j = i % (nN * NF);
        R[(size_t)m * n + D.ngam[n0 + j / NF] * NF + j % NF] += F.at(r0 + m, q0 + j);
      }
    }
    __syncthreads();
  }
}

// Step over the pivots K = [k0, k0 + kw): for 64 columns j of matrix c, the old rows
// W = A_Kj and R = A_KK^{-1} A_Kj (R = -A_KK^{-1} for j in K).  Every workgroup inverts the
// pivot block itself (Gauss-Jordan in LDS; the blocks of a positive definite sweep need no
// pivoting).
__global__ __launch_bounds__(kBlk) void k_el_panel(ElimDev D, int which, int k0, int ldw) {
  const int c = blockIdx.y, j0 = blockIdx.x * kTile;
  const SweepMat M = sweep_mat(D, which, c);
  if (k0 >= M.np || j0 >= M.V) return;
  const int kw = min(kPiv, M.np - k0);
  __shared__ double P[kPiv][2 * kPiv + 1], W[kPiv][kTile + 1];
  for (int i = threadIdx.x; i < kPiv * 2 * kPiv; i += kBlk) {
    const int r = i / (2 * kPiv), q = i % (2 * kPiv);
    double v = (q - kPiv == r || (r >= kw && q == r)) ? 1.0 : 0.0;
    if (q < kPiv && r < kw && q < kw) v = M.at(k0 + r, k0 + q);
    P[r][q] = v;
  }
  const bool low = j0 / kTile < k0 / kTile;  // kept as columns: neighbouring threads along r
  for (int i = threadIdx.x; i < kPiv * kTile; i += kBlk) {
    const int r = low ? i % kPiv : i / kTile, q = low ? i / kPiv : i % kTile;
    W[r][q] = (r < kw && j0 + q < M.V) ? M.at(k0 + r, j0 + q) : 0.0;
  }
  __syncthreads();
  // thread: row tr of the pivot block, eight of its 64 columns
  const int tr = threadIdx.x >> 3, tq = threadIdx.x & 7;
  for (int p = 0; p < kw; ++p) {
    const double ip = 1.0 / P[p][p], f = P[tr][p];
    double row[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) row[u] = P[p][tq + 8 * u] * ip;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (tr == p) P[tr][tq + 8 * u] = row[u];
      else P[tr][tq + 8 * u] -= f * row[u];
    }
    __syncthreads();
  }
  double* Wb = D.panW + (size_t)c * kPiv * ldw;
  double* Rb = D.panR + (size_t)c * kPiv * ldw;
  for (int i = threadIdx.x; i < kPiv * kTile; i += kBlk) {
    const int r = i / kTile, jj = i % kTile, j = j0 + jj;
    if (j >= M.V || r >= kw) continue;
    double s = 0;
    for (int q = 0; q < kw; ++q) s += P[r][kPiv + q] * W[q][jj];
    if (j >= k0 && j < k0 + kw) s = -P[r][kPiv + j - k0];
    Wb[(size_t)r * ldw + j] = W[r][jj];
    Rb[(size_t)r * ldw + j] = s;
  }
}

// A -= W^T R outside the pivots, R and R^T in their rows and columns (a 64 x 64 tile on or
// above the diagonal a workgroup, 4 x 4 values a thread; W and R through LDS).
__global__ __launch_bounds__(kBlk) void k_el_update(ElimDev D, int which, int k0, int ldw) {
  const int c = blockIdx.z, i0 = blockIdx.y * kTile, j0 = blockIdx.x * kTile;
  const SweepMat M = sweep_mat(D, which, c);
  if (k0 >= M.np || i0 >= M.V || j0 >= M.V || i0 > j0) return;
  const int kw = min(kPiv, M.np - k0);
  __shared__ double W[kPiv][kTile], R[kPiv][kTile];
  const double* Wb = D.panW + (size_t)c * kPiv * ldw;
  const double* Rb = D.panR + (size_t)c * kPiv * ldw;
  for (int i = threadIdx.x; i < kPiv * kTile; i += kBlk) {
    const int r = i / kTile, q = i % kTile;
    W[r][q] = (r < kw && i0 + q < M.V) ? Wb[(size_t)r * ldw + i0 + q] : 0.0;
    R[r][q] = (r < kw && j0 + q < M.V) ? Rb[(size_t)r * ldw + j0 + q] : 0.0;
  }
  __syncthreads();
  const int ti = (threadIdx.x >> 4) * 4, tj = threadIdx.x & 15;
  double acc[4][4] = {};
  for (int k = 0; k < kw; ++k) {
    double w[4], r[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) w[a] = W[k][ti + a];
#pragma unroll
    for (int b = 0; b < 4; ++b) r[b] = R[k][tj + 16 * b];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] += w[a] * r[b];
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = i0 + ti + a, j = j0 + tj + 16 * b;
      if (i >= M.V || j >= M.V) continue;
      double& A = M.A[(size_t)i * M.V + j];
      if (i >= k0 && i < k0 + kw) A = Rb[(size_t)(i - k0) * ldw + j];
      else if (j >= k0 && j < k0 + kw) A = Rb[(size_t)(j - k0) * ldw + i];
      else A -= acc[a][b];
    }
}

// The solve matrices in FP32: per cell [S_BB^{-1} | -G], rows padded to four values.
__global__ __launch_bounds__(kBlk) void k_el_store_cells(ElimDev D) {
  const int c = blockIdx.y, NF = D.NF;
  const int nB = (D.boff[c + 1] - D.boff[c]) * NF, V = nB + (D.noff[c + 1] - D.noff[c]) * NF, ld = (V + 3) & ~3;
  const SweepMat F{D.front + D.foff[c], V, 0};
  float* M = D.mat + D.moff[c];
  for (long i = (long)blockIdx.x * kBlk + threadIdx.x; i < (long)nB * ld; i += (long)gridDim.x * kBlk) {
    const int r = (int)(i / ld), q = (int)(i % ld);
    M[i] = q < V ? (float)-F.at(r, q) : 0.0f;
  }
}
// The interface inverse in FP32 without its component along the kernel vector.
__global__ __launch_bounds__(kBlk) void k_el_store_top(ElimDev D, double ishift) {
  const int NF = D.NF, n = D.ng * NF, ld = (n + 3) & ~3;
  const SweepMat A{D.top, n, 0};
  for (long i = (long)blockIdx.x * kBlk + threadIdx.x; i < (long)n * ld; i += (long)gridDim.x * kBlk) {
    const int r = (int)(i / ld), q = (int)(i % ld);
    double v = 0;
    if (q < n) {
      v = -A.at(r, q);
      if (r % NF == 0 && q % NF == 0) v -= ishift * D.zhat[r / NF] * D.zhat[q / NF];
    }
    D.tmat[i] = (float)v;
  }
}

hipError_t launch_elim_factor(const ElimDev& D, int nfac, const double* ST, double shift, hipStream_t s) {
  hipLaunchKernelGGL(k_el_fronts, dim3(D.nc), dim3(kBlk), 0, s, D, nfac, ST);
  for (int which = 0; which < 2; ++which) {
    const int V = which ? D.ng * D.NF : D.maxV, np = which ? V : D.maxB, nm = which ? 1 : D.nc;
    const int t = (V + kTile - 1) / kTile, ldw = which ? V : D.maxV;
    if (which) hipLaunchKernelGGL(k_el_interface, dim3(D.ng), dim3(kBlk), 0, s, D, shift);
    for (int k0 = 0; k0 < np; k0 += kPiv) {
      hipLaunchKernelGGL(k_el_panel, dim3(t, nm), dim3(kBlk), 0, s, D, which, k0, ldw);
      hipLaunchKernelGGL(k_el_update, dim3(t, t, nm), dim3(kBlk), 0, s, D, which, k0, ldw);
    }
  }
  hipLaunchKernelGGL(k_el_store_cells, dim3(8, D.nc), dim3(kBlk), 0, s, D);
  hipLaunchKernelGGL(k_el_store_top, dim3(512), dim3(kBlk), 0, s, D, shift > 0 ? 1.0 / shift : 0.0);
  return hipGetLastError();
}

// ---- solve -------------------------------------------------------------------------------
// The residual r and the result z are the PCG's FP64 vectors; the elimination runs in FP32
// like the multigrid cycle (a preconditioner's rounding costs iterations, not accuracy).

// Interior values of cell c in LDS.
__device__ inline void load_interior(const ElimDev& D, int c, const double* __restrict__ r, float* v) {
  const int NF = D.NF, b0 = D.boff[c], nB = (D.boff[c + 1] - b0) * NF;
  for (int i = threadIdx.x; i < nB; i += blockDim.x) v[i] = (float)r[(size_t)D.bfac[b0 + i / NF] * NF + i % NF];
}

// contrib_N = -G^T r_B: 64 columns a workgroup, 16 threads of four columns by 16 row groups.
// First the iteration's stopping test, on the G (r, r) partials of its update: a solve that
// has converged skips its last application (the next kernels return at the flag).
__global__ __launch_bounds__(kBlk) void k_el_forward(ElimDev D, const double* __restrict__ r,
                                                     const double* __restrict__ rz, int G, PcgScalars* sc) {
  if (sc->done != PCG_RUNNING) return;
  double rr[2];
  block_sum_partials<2>(rz, G, rr);
  const bool stop = isfinite(rr[1]) && rr[1] <= sc->tol2;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    const int it = sc->it;  // already advanced by the update
    sc->iters = it - 1;
    sc->rr = rr[1];
    if (it == 1) sc->rr0 = rr[1];
    if (stop) sc->done = PCG_CONVERGED;
  }
  if (stop) return;
  const int c = blockIdx.x, NF = D.NF;
  const int nB = (D.boff[c + 1] - D.boff[c]) * NF, nN = (D.noff[c + 1] - D.noff[c]) * NF;
  const int j0 = blockIdx.y * 64;
  if (j0 >= nN) return;
  const int ld = (nB + nN + 3) & ~3;
  extern __shared__ __align__(16) float v[];
  __shared__ float part[16][64];
  load_interior(D, c, r, v);
  __syncthreads();
  const int q = threadIdx.x & 15, g = threadIdx.x >> 4;
  const float* __restrict__ M = D.mat + D.moff[c] + nB;
  float s[4] = {0, 0, 0, 0};
  int col[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) col[u] = min(j0 + q + 16 * u, nN - 1);
#pragma unroll 4
  for (int i = g; i < nB; i += 16) {
    const float vi = v[i];
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] += vi * M[(size_t)i * ld + col[u]];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) part[g][q + 16 * u] = s[u];
  __syncthreads();
  if (threadIdx.x < 64 && j0 + (int)threadIdx.x < nN) {
    float t = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) t += part[k][threadIdx.x];
    D.contrib[(size_t)D.noff[c] * NF + j0 + threadIdx.x] = t;
  }
}

// Dot products of `rows` rows (row0 on) of M with the vector v in LDS: L lanes a row, 16
// bytes a lane and load; out(row, value) by one lane each.
template <int L, typename OUT>
__device__ inline void rows_dot(const float* __restrict__ M, int ld, int row0, int rows, const float* v, OUT out) {
  const int l = threadIdx.x & (L - 1), n4 = ld >> 2;
  for (int i = threadIdx.x / L; i < rows; i += blockDim.x / L) {
    const float4* __restrict__ m = reinterpret_cast<const float4*>(M + (size_t)(row0 + i) * ld);
    const float4* x = reinterpret_cast<const float4*>(v);
    float s = 0;
#pragma unroll 8
    for (int k = l; k < n4; k += L) {
      const float4 a = m[k], b = x[k];
      s += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
    }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, L);
    if (l == 0) out(row0 + i, s);
  }
}

// The interface: right-hand side with both cells' contributions, dense product.  Every
// workgroup forms the whole right-hand side, so it takes kTopRows rows, a wave each: few
// enough workgroups that this stays a small part, and a CU still has 16 waves loading.
static constexpr int kTopRows = 16;
__global__ __launch_bounds__(64 * kTopRows) void k_el_top(ElimDev D, const double* __restrict__ r,
                                                          double* __restrict__ z, const PcgScalars* sc) {
  if (sc->done != PCG_RUNNING) return;
  const int NF = D.NF, n = D.ng * NF, ld = (n + 3) & ~3;
  extern __shared__ __align__(16) float v[];
  for (int i = threadIdx.x; i < ld; i += blockDim.x) {
    float t = 0;
    if (i < n) {
      const int gi = i / NF, m = i % NF, p0 = D.gpos[2 * gi], p1 = D.gpos[2 * gi + 1];
      t = (float)r[(size_t)D.gfac[gi] * NF + m] + D.contrib[(size_t)p0 * NF + m] + D.contrib[(size_t)p1 * NF + m];
    }
    v[i] = t;
  }
  __syncthreads();
  const int row0 = blockIdx.x * kTopRows;
  rows_dot<64>(D.tmat, ld, row0, min(kTopRows, n - row0), v, [&](int i, float s) {
    z[(size_t)D.gfac[i / NF] * NF + i % NF] = (double)s;
  });
}

// Interiors: x_B = [S_BB^{-1} | -G] (r_B, x_N).
__global__ __launch_bounds__(kBlk) void k_el_backward(ElimDev D, const double* __restrict__ r,
                                                      double* __restrict__ z, int rows, const PcgScalars* sc) {
  if (sc->done != PCG_RUNNING) return;
  const int c = blockIdx.x, NF = D.NF, n0 = D.noff[c];
  const int nB = (D.boff[c + 1] - D.boff[c]) * NF, V = nB + (D.noff[c + 1] - n0) * NF, ld = (V + 3) & ~3;
  const int row0 = blockIdx.y * rows;
  if (row0 >= nB) return;
  extern __shared__ __align__(16) float v[];
  load_interior(D, c, r, v);
  for (int i = nB + threadIdx.x; i < ld; i += blockDim.x)
    v[i] = i < V ? (float)z[(size_t)D.nfac[n0 + (i - nB) / NF] * NF + (i - nB) % NF] : 0.0f;
  __syncthreads();
  const int b0 = D.boff[c];
  rows_dot<16>(D.mat + D.moff[c], ld, row0, min(rows, nB - row0), v, [&](int i, float s) {
    z[(size_t)D.bfac[b0 + i / NF] * NF + i % NF] = (double)s;
  });
}

// (r, z) partials into rz[2*block].
__global__ __launch_bounds__(kBlk) void k_el_dot(long n, const double* __restrict__ r, const double* __restrict__ z,
                                                 double* __restrict__ rz, const PcgScalars* sc) {
  if (sc->done != PCG_RUNNING) return;
  double v[1] = {0}, t[1];
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) v[0] += r[i] * z[i];
  block_sum_values<1>(v, t);
  if (threadIdx.x == 0) rz[2 * blockIdx.x] = t[0];
}

hipError_t launch_elim_apply(const ElimDev& D, const DevGeo& g, const double* r, double* z, double* rz,
                             PcgScalars* sc, hipStream_t s) {
  const int NF = D.NF, n = D.ng * NF, rows = 32;
  const size_t front = sizeof(float) * ((D.maxV + 3) & ~3), top = sizeof(float) * ((n + 3) & ~3);
  if (std::max(D.maxV, n) > kElimMaxVec) return hipErrorInvalidValue;  // the vectors are held in LDS
  const PcgScalars* csc = sc;
  hipLaunchKernelGGL(k_el_forward, dim3(D.nc, (D.maxN + 63) / 64), dim3(kBlk), front, s, D, r, (const double*)rz,
                     g.fgrid, sc);
  hipLaunchKernelGGL(k_el_top, dim3((n + kTopRows - 1) / kTopRows), dim3(64 * kTopRows), top, s, D, r, z, csc);
  hipLaunchKernelGGL(k_el_backward, dim3(D.nc, (D.maxB + rows - 1) / rows), dim3(kBlk), front, s, D, r, z, rows, csc);
  hipLaunchKernelGGL(k_el_dot, dim3(g.fgrid), dim3(g.fblk), 0, s, (long)g.E * NF, r, (const double*)z, rz, csc);
  return hipGetLastError();
}

}  // namespace dfdg
