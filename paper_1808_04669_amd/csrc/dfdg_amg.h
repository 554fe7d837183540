// Smoothed-aggregation algebraic multigrid hierarchy for the facet matrix S (host set-up).
#pragma once
#include <string>
#include <vector>

namespace dfdg {

struct Csr {
  int n = 0, m = 0;              // rows, columns
  std::vector<int> ptr, col;     // ptr[n+1]
  std::vector<double> val;
  long nnz() const { return (long)col.size(); }
};

// One level below the finest: its operator A (scalar CSR), the prolongator P from it to
// the finer level (rows: finer unknowns) and R = P^T.  Level 0 is S itself (BSR on the
// device, given as CSR here).
struct AmgLevel {
  Csr A;            // operator of this level
  std::vector<double> dinv;
  double lmax = 0;  // spectral radius estimate of D^{-1} A (Chebyshev upper bound)
  Csr P;            // prolongator from the next coarser level to this one (empty on the coarsest)
  // on levels >= 1 that have a coarser one, with one damped Jacobi step x1 = D^{-1} b / th around
  // the coarse correction e:
  Csr Rs;           // the restricted residual of x1 from b, P^T (I - A D^{-1} / th)
  Csr Ps;           // the result from [b; e]: (2 - D^{-1} A / th) D^{-1} / th, then Rs^T
};
// A P and P^T A of a level that has a coarser one (no solve reads them: debugging)
void amg_products(const AmgLevel& L, Csr& AP, Csr& RA);
inline double amg_smooth_lmax(double lmax) { return 1.05 * lmax; }
// th of the coarse levels: the centre of [lmax / 30, lmax]
inline double amg_coarse_theta(double lmax) { return 0.5 * amg_smooth_lmax(lmax) * (1.0 + 1.0 / 30.0); }

struct AmgHierarchy {
  std::vector<AmgLevel> lv;          // lv[0] = fine operator S
  std::vector<double> coarse_inv;    // dense pseudo-inverse (n_c x n_c) of the coarsest operator
  int n_coarse = 0;
  // finest prolongator by facets: the columns of facet F's rows, p0_ptr[F] .. p0_ptr[F + 1]
  std::vector<int> p0_ptr, p0_col;
  int p0_w = 0, p0_wr = 0;           // the most columns of a facet, and facets of a column
  // the last restriction is multiplied into the dense solve (on the device, from Ps): with three
  // levels or more, if coarse_inv Rs of the level above the coarsest is within kAmgFoldValues
  bool fold = false;
};
// 32 MB in FP32, read at the rate of the memory-side cache in about the time of the launch saved
constexpr long kAmgFoldValues = 8l << 20;

// Builds the hierarchy for the BSR facet matrix (cols [NS][E], vals [NS][NF][NF][E]) with the
// near-null vector z (the constant multiplier, scalar length E*NF); singular: z spans the
// kernel of S (the coarsest level is then inverted as a pseudo-inverse that leaves out the
// coarse image of z), else S is definite and so is every level.  fine_smooth: damped-Jacobi
// steps applied to the finest level's tentative prolongator (1 or more; one below it).
// theta: strength threshold;
// coarsening stops at max_coarse rows, or earlier (at most 4096 rows) when aggregation
// no longer halves the level.
int build_amg(int E, int NF, int NS, const std::vector<int>& cols, const std::vector<double>& vals,
              const std::vector<double>& z, bool singular, double theta, int max_coarse, int fine_smooth,
              AmgHierarchy& H, std::string& err);

// Whether build_amg would give more than one level (dinv: the inverse diagonal [E][NF]), without
// building any; false also where it would fail on the diagonal.
bool amg_coarsens(int E, int NF, int NS, const std::vector<int>& cols, const std::vector<double>& vals,
                  const std::vector<double>& dinv, double theta, int max_coarse);

}  // namespace dfdg
