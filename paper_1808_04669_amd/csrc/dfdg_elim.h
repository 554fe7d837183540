// Block elimination of the facet system on small meshes (host part: the partition).
#pragma once
#include <string>
#include <vector>

#include "dfdg_setup.h"

namespace dfdg {

// The elements are split into cells; a facet whose elements lie in one cell is interior to
// it, the others form the interface.  The interiors B of the cells are decoupled from each
// other, so that S x = r is solved exactly by
//   r_G -= sum_cells G^T r_B,  x_G = (Schur complement)^+ r_G,  x_B = S_BB^{-1} r_B - G x_N,
// G = S_BB^{-1} S_BN, N the interface facets on the cell's boundary.
struct ElimHost {
  int nc = 0, ng = 0;                // cells, interface facets
  std::vector<int> boff, bfac;       // [nc+1]; interior facets of the cells
  std::vector<int> noff, ngam, nfac; // [nc+1]; boundary facets: index in the interface, facet
  std::vector<int> gfac, gpos;       // [ng] facet; [ng][2] its places in ngam (-1: none)
  std::vector<int> eoff, elem, elp;  // [nc+1]; elements; [T][facets] place in the cell's front
  std::vector<long> moff, foff;      // per cell: first value of its solve matrix, of its front
  int maxB = 0, maxV = 0;            // unknowns: largest interior, largest front
  long mvals = 0, fvals = 0;         // values of all solve matrices, of all fronts
};

// Largest systems that take the elimination: unknowns, and values its matrices hold.  Measured
// (MI355X, 1e-12, RK3 step with the elimination against the multigrid cycle): 16x16 BDM_1
// 0.45 / 1.40 ms, 57x57 BDM_2 0.55 / 1.74, 60x60 BDM_2 0.56 / 1.71, 72x72 BDM_1 0.64 / 1.56,
// cubes 6^3 BDM_1 0.59 / 2.22, 11^3 BDM_1 1.34 / 2.84, 8^3 BDM_2 1.44 / 3.51.
// The lines are not where the two cost the same.  Triangles: from 64x64 BDM_2 (36864 unknowns)
// on, the iteration counts of the multigrid solves, their growth with the mesh and what better
// start values save of them are tested properties of a context, and the elimination stays below.
// Tetrahedra: the separators of a cube make the matrices grow much faster than the system; at
// the line (11^3 BDM_1) a context keeps 0.5 GB (0.1 GB with the cycle), its bind works in 1.1 GB
// more, and it is set up in 0.10 s (0.11 s).
constexpr long kElimUnknowns2 = 32768, kElimUnknowns3 = 65536;
constexpr long kElimValues2 = 48L << 20, kElimValues3 = 128L << 20;

// The partition with the fewest values in its matrices; false if none is within the limits.
bool build_elim(const MeshHost& m, int NF, ElimHost& el);

// Whether S is conditioned well enough for an inverse in FP32.  Rounding the inverse entry by
// entry perturbs the preconditioned system by some 6e-8 kappa, kappa the condition of S scaled
// by its diagonal: a square of 24^2 BDM_2 stretched by 30 (kappa 6e5), 100 (7e6), 300 (6e7),
// 1000 (7e8) takes 4, 5, 9, 53 iterations to 1e-12 and by 2000 (3e9) never ends, where the
// cycle takes 181, 282, 309, 278 and 630.  The line lies a factor of 100 below that; the
// estimate was within 1 % of the dense eigenvalues on stretched squares and cubes and low by
// 14 % at most on layers growing from one wall.
constexpr double kElimCondition = 3e7;
bool elim_conditioned(const MeshHost& m, const HostSetup& h, int NF);

}  // namespace dfdg
