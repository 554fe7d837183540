// Partition of a small mesh for the block elimination: recursive coordinate bisection of the
// elements, cells at the depth whose matrices hold the fewest values.
#include "dfdg_elim.h"

#include <algorithm>
#include <numeric>

namespace dfdg {

namespace {

// order: elements in bisection order; bounds[d]: first element of every cell of depth d (and T).
void bisect(const std::vector<double>& mid, int dim, int T, int leaf, std::vector<int>& order,
            std::vector<std::vector<int>>& bounds) {
  order.resize(T);
  std::iota(order.begin(), order.end(), 0);
  bounds.assign(1, {0, T});
  for (;;) {
    const std::vector<int>& b = bounds.back();
    int largest = 0;
    for (size_t i = 0; i + 1 < b.size(); ++i) largest = std::max(largest, b[i + 1] - b[i]);
    if (largest <= leaf) return;
    std::vector<int> next;
    for (size_t i = 0; i + 1 < b.size(); ++i) {
      const int lo = b[i], hi = b[i + 1];
      next.push_back(lo);
      if (hi - lo < 2) continue;
      int axis = 0;
      double best = -1;
      for (int a = 0; a < dim; ++a) {
        double mn = mid[(size_t)order[lo] * dim + a], mx = mn;
        for (int k = lo; k < hi; ++k) {
          mn = std::min(mn, mid[(size_t)order[k] * dim + a]);
          mx = std::max(mx, mid[(size_t)order[k] * dim + a]);
        }
        if (mx - mn > best * (1 + 1e-9)) {
          best = mx - mn;
          axis = a;
        }
      }
      auto at = [&](int k, int a) { return mid[(size_t)order[k] * dim + (axis + a) % dim]; };
      std::sort(order.begin() + lo, order.begin() + hi, [&](int x, int y) {
        for (int a = 0; a < dim; ++a) {
          const int c = (axis + a) % dim;
          const double u = mid[(size_t)x * dim + c], v = mid[(size_t)y * dim + c];
          if (u != v) return u < v;
        }
        return x < y;
      });
      // cut at the widest gap near the median: on a mesh in layers the one between two
      // layers, which cuts the fewest facets; of gaps as wide, the nearest to the median
      const int n = hi - lo, mdn = lo + n / 2;
      int half = mdn;
      double gap = 0;
      for (int d = 0; d <= n / 6; ++d)
        for (int k : {mdn - d, mdn + d})
          if (k > lo && k < hi && at(k, 0) - at(k - 1, 0) > 1.01 * gap) {
            gap = at(k, 0) - at(k - 1, 0);
            half = k;
          }
      next.push_back(half);
    }
    next.push_back(T);
    bounds.push_back(std::move(next));
  }
}

}  // namespace

bool build_elim(const MeshHost& m, int NF, ElimHost& el) {
  const int T = m.T, E = m.E, dim = m.dim, nf = dim + 1;
  if ((long)E * NF > (dim == 2 ? kElimUnknowns2 : kElimUnknowns3)) return false;
  std::vector<double> mid((size_t)T * dim, 0.0);
  for (int t = 0; t < T; ++t)
    for (int v = 0; v < nf; ++v)
      for (int a = 0; a < dim; ++a) mid[(size_t)t * dim + a] += m.xyz[((size_t)t * nf + v) * dim + a] / nf;
  std::vector<int> order, cell(T), best;
  std::vector<std::vector<int>> bounds;
  bisect(mid, dim, T, 12, order, bounds);
  long least = (dim == 2 ? kElimValues2 : kElimValues3) + 1;
  for (const std::vector<int>& b : bounds) {
    const int nc = (int)b.size() - 1;
    for (int c = 0; c < nc; ++c)
      for (int k = b[c]; k < b[c + 1]; ++k) cell[order[k]] = c;
    std::vector<long> nB(nc, 0), nN(nc, 0);
    long ng = 0;
    for (int F = 0; F < E; ++F) {
      const int a = cell[m.fL[F]], c = m.fR[F] < 0 ? a : cell[m.fR[F]];
      if (a == c) ++nB[a];
      else {
        ++nN[a];
        ++nN[c];
        ++ng;
      }
    }
    long vals = ng * NF * ng * NF;
    bool fits = ng * NF <= kElimMaxVec;
    for (int c = 0; c < nc; ++c) {
      vals += nB[c] * NF * (nB[c] + 2 * nN[c]) * NF;
      fits = fits && nB[c] > 0 && (nB[c] + nN[c]) * NF <= kElimMaxVec;
    }
    if (fits && ng > 0 && vals < least) {
      least = vals;
      best = b;
    }
  }
  if (best.empty()) return false;

  el = ElimHost{};
  el.nc = (int)best.size() - 1;
  for (int c = 0; c < el.nc; ++c) {
    el.eoff.push_back(best[c]);
    for (int k = best[c]; k < best[c + 1]; ++k) {
      cell[order[k]] = c;
      el.elem.push_back(order[k]);
    }
  }
  el.eoff.push_back(T);
  std::vector<std::vector<int>> B(el.nc), N(el.nc);
  std::vector<int> gam(E, -1);
  for (int F = 0; F < E; ++F) {
    const int a = cell[m.fL[F]], c = m.fR[F] < 0 ? a : cell[m.fR[F]];
    if (a == c) {
      B[a].push_back(F);
      continue;
    }
    gam[F] = el.ng++;
    el.gfac.push_back(F);
    N[a].push_back(F);
    N[c].push_back(F);
  }
  el.gpos.assign(2 * (size_t)el.ng, -1);
  el.elp.assign((size_t)T * nf, 0);
  std::vector<int> place(E, 0);
  for (int c = 0; c < el.nc; ++c) {
    const int nB = (int)B[c].size(), nN = (int)N[c].size();
    el.boff.push_back((int)el.bfac.size());
    el.noff.push_back((int)el.ngam.size());
    for (int i = 0; i < nB; ++i) {
      place[B[c][i]] = i;
      el.bfac.push_back(B[c][i]);
    }
    for (int i = 0; i < nN; ++i) {
      const int F = N[c][i];
      place[F] = nB + i;
      int* g = &el.gpos[2 * (size_t)gam[F]];
      g[g[0] < 0 ? 0 : 1] = (int)el.ngam.size();
      el.ngam.push_back(gam[F]);
      el.nfac.push_back(F);
    }
    for (int k = el.eoff[c]; k < el.eoff[c + 1]; ++k)
      for (int f = 0; f < nf; ++f)
        el.elp[(size_t)el.elem[k] * nf + f] = place[m.efacet[(size_t)el.elem[k] * nf + f]];
    const long b = (long)nB * NF, v = (long)(nB + nN) * NF;
    el.moff.push_back(el.mvals);
    el.foff.push_back(el.fvals);
    el.mvals += b * ((v + 3) / 4 * 4);
    el.fvals += v * v;
    el.maxB = std::max(el.maxB, (int)b);
    el.maxV = std::max(el.maxV, (int)v);
  }
  el.boff.push_back((int)el.bfac.size());
  el.noff.push_back((int)el.ngam.size());
  return true;
}

}  // namespace dfdg
