// Partition of a small mesh for the block elimination: recursive coordinate bisection of the
// elements, cells at the depth whose matrices hold the fewest values.
#include "dfdg_elim.h"

#include <algorithm>
#include <cmath>
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

// Extreme eigenvalues of a symmetric tridiagonal matrix, by bisection on Sturm counts.
static void tridiagonal_extremes(const std::vector<double>& a, const std::vector<double>& b, double& lo, double& hi) {
  const int n = (int)a.size();
  auto below = [&](double x) {  // eigenvalues < x
    int c = 0;
    double q = 1;
    for (int i = 0; i < n; ++i) {
      q = a[i] - x - (i ? b[i - 1] * b[i - 1] / q : 0.0);
      if (q == 0) q = 1e-300;
      c += q < 0;
    }
    return c;
  };
  double g0 = a[0], g1 = a[0];
  for (int i = 0; i < n; ++i) {
    const double r = (i ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < n ? std::fabs(b[i]) : 0.0);
    g0 = std::min(g0, a[i] - r);
    g1 = std::max(g1, a[i] + r);
  }
  for (int k : {0, n - 1}) {
    double l = g0, u = g1;
    for (int it = 0; it < 100; ++it) {
      const double x = 0.5 * (l + u);
      (below(x) > k ? u : l) = x;
    }
    (k ? hi : lo) = u;
    if (n == 1) hi = lo;
  }
}

// The condition of D^{-1/2} S D^{-1/2} (off its kernel) from below: Lanczos steps from a wave
// along each axis in turn, near the lowest modes of a stretched mesh, projected onto the facets'
// modes (by the means alone its steps across thin elements would hide the low modes).
static double condition_estimate(const MeshHost& m, const HostSetup& h, int NF) {
  constexpr int kSteps = 16;
  const int E = h.E, dim = m.dim, nf = dim + 1, NS = (int)(h.cols.size() / E);
  const long n = (long)E * NF;
  std::vector<double> q(n), qo(n), w(n), y(n), sd(n), z;
  for (long i = 0; i < n; ++i) sd[i] = std::sqrt(h.dinv[i]);  // D^{-1/2}
  double lo[3], hi[3];
  for (int c = 0; c < dim; ++c) {
    lo[c] = hi[c] = m.xyz[c];
    for (size_t i = c; i < m.xyz.size(); i += dim) {
      lo[c] = std::min(lo[c], m.xyz[i]);
      hi[c] = std::max(hi[c], m.xyz[i]);
    }
  }
  // projection onto the facet's basis (edges: Legendre polynomials from vertex f + 1 to f + 2;
  // faces: Dubiner polynomials from the lowest local vertex)
  std::vector<double> pt, pw, mode;
  if (dim == 2) gauss_legendre01(NF + 1, pt, pw);
  else sym_face_rule(6, pt, pw);
  const int np = (int)pw.size();
  mode.resize((size_t)np * NF);
  for (int r = 0; r < np; ++r) {
    if (dim == 2) {
      for (int a = 0; a < NF; ++a) mode[r * NF + a] = pw[r] * legendre01_orthonormal(a, pt[r]);
    } else {
      dubiner(NF == 3 ? 1 : 2, pt[2 * r], pt[2 * r + 1], &mode[r * NF], nullptr);
      for (int a = 0; a < NF; ++a) mode[r * NF + a] *= pw[r] * std::sqrt(0.5);
    }
  }
  const double pi = std::acos(-1.0);
  if (h.singular) {
    z.assign(n, 0.0);
    double zz = 0;
    for (int F = 0; F < E; ++F) {
      z[(size_t)F * NF] = h.zdef[F] / sd[(size_t)F * NF];
      zz += z[(size_t)F * NF] * z[(size_t)F * NF];
    }
    for (double& x : z) x /= std::sqrt(zz);
  }
  auto deflate = [&](std::vector<double>& x) {
    double t = 0;
    for (size_t i = 0; i < z.size(); ++i) t += z[i] * x[i];
    for (size_t i = 0; i < z.size(); ++i) x[i] -= t * z[i];
  };
  auto norm = [&](const std::vector<double>& x) {
    double t = 0;
    for (double v : x) t += v * v;
    return std::sqrt(t);
  };
  double least = HUGE_VAL, most = 0;
  for (int c = 0; c < dim; ++c) {
    std::fill(q.begin(), q.end(), 0.0);
    for (int F = 0; F < E; ++F) {
      const double* v = &m.xyz[(size_t)m.fL[F] * nf * dim];
      const int f = m.fLloc[F];
      int vert[3], k = 0;
      if (dim == 2) {
        vert[0] = (f + 1) % 3;
        vert[1] = (f + 2) % 3;
      } else {
        for (int i = 0; i < 4; ++i)
          if (i != f) vert[k++] = i;
      }
      for (int r = 0; r < np; ++r) {
        const double* o = v + vert[0] * dim;
        double x = o[c];
        for (int i = 1; i < dim; ++i) x += pt[(dim - 1) * r + i - 1] * (v[vert[i] * dim + c] - o[c]);
        const double s = std::cos((m.period[c] > 0 ? 2 * pi / m.period[c] : pi / (hi[c] - lo[c])) * (x - lo[c]));
        for (int a = 0; a < NF; ++a) q[(size_t)F * NF + a] += s * mode[r * NF + a] * h.nearnull[F];
      }
    }
    for (long i = 0; i < n; ++i) q[i] /= sd[i];
    deflate(q);
    const double q0 = norm(q);
    if (!(q0 > 0)) continue;
    for (double& x : q) x /= q0;
    std::vector<double> al, be;
    for (int it = 0; it < kSteps; ++it) {
      for (long i = 0; i < n; ++i) {
        y[i] = sd[i] * q[i];
        w[i] = 0;
      }
      for (int s = 0; s < NS; ++s)
        for (int a = 0; a < NF; ++a)
          for (int b = 0; b < NF; ++b) {
            const double* v = &h.vals[(((size_t)s * NF + a) * NF + b) * E];
            const int* col = &h.cols[(size_t)s * E];
            for (int F = 0; F < E; ++F) w[(size_t)F * NF + a] += v[F] * y[(size_t)col[F] * NF + b];
          }
      double t = 0;
      for (long i = 0; i < n; ++i) {
        w[i] = sd[i] * w[i] - (it ? be.back() * qo[i] : 0.0);
        t += w[i] * q[i];
      }
      for (long i = 0; i < n; ++i) w[i] -= t * q[i];
      deflate(w);
      al.push_back(t);
      const double b = norm(w);
      if (!(b > 1e-14)) break;
      be.push_back(b);
      qo.swap(q);
      for (long i = 0; i < n; ++i) q[i] = w[i] / b;
    }
    double l = 0, u = 0;
    tridiagonal_extremes(al, be, l, u);
    least = std::min(least, l);
    most = std::max(most, u);
  }
  return least > 0 ? most / least : HUGE_VAL;
}

bool elim_conditioned(const MeshHost& m, const HostSetup& h, int NF) {
  // On elements without thin directions the scaled condition grows with the number of
  // facets across the mesh only: far below the line at the sizes of kElimUnknowns.
  const int T = m.T, dim = m.dim, nf = dim + 1;
  bool thin = false;
  for (int t = 0; t < T && !thin; ++t) {
    const double* v = &m.xyz[(size_t)t * nf * dim];
    double edge = 0, face = 0;
    for (int i = 0; i < nf; ++i) {
      face = std::max(face, h.flen[(size_t)i * T + t]);
      for (int k = 0; k < i; ++k) {
        double d = 0;
        for (int c = 0; c < dim; ++c) d += (v[i * dim + c] - v[k * dim + c]) * (v[i * dim + c] - v[k * dim + c]);
        edge = std::max(edge, std::sqrt(d));
      }
    }
    const double height = h.detJ[t] / (dim == 3 ? 2 * face : face);
    thin = !(edge <= 16 * height);
  }
  return !thin || condition_estimate(m, h, NF) <= kElimCondition;
}

}  // namespace dfdg
