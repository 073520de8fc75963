// Aggregation algebraic multigrid for the Poisson system of Sec. 2.2 (eqs.
// (7), (laplace)): the analogue of the paper's fastest solver configuration
// (PETSc GAMG, Sec. 3.4.2), built here as plain (unsmoothed) aggregation.
//
// Setup (host, amg.cpp), per level from the finest:
//   strength  j != i is a strong neighbour of row i when
//             |a_ij| >= theta * max_{k != i} |a_ik|;
//   aggregates three passes in row order: (1) a row whose strong neighbours
//             are all free seeds an aggregate with them; (2) a free row joins
//             the aggregate of its strongest aggregated strong neighbour
//             (smallest index on ties); (3) a row still free seeds an
//             aggregate with its free strong neighbours (or alone);
//   coarse    A_c = P^T A P with the piecewise-constant prolongator P
//             (row i of P is the unit vector of its aggregate);
// until a level has at most coarse_max rows, whose inverse is formed densely
// (LU with partial pivoting).
// The cycle (device, amg_kernels.hip) is a V(1,1) cycle with damped Jacobi
// smoothing from a zero initial guess:
//   x = w D^-1 b;  b_c = P^T (b - A x);  x += P V(b_c);  x += w D^-1 (b - A x),
// with the dense inverse on the coarsest level.
#pragma once
#include <cstdint>
#include <string>
#include <vector>

#include "chunks.h"
#include "mesh.h"

namespace mifvm {

constexpr int kAmgMaxLevels = 16;

struct AmgCsr {                          // square matrix, diagonal included
    int64_t n = 0;
    std::vector<int64_t> ptr;
    std::vector<int32_t> col;
    std::vector<double> val;
};

struct AmgLevel {
    AmgCsr A;
    std::vector<int32_t> agg;             // row -> aggregate (coarse row); empty on the coarsest level
    int64_t ncoarse = 0;
};

// A level as the device stores it.  The rows of the levels between the finest
// and the coarsest are renumbered so that the members of an aggregate are
// consecutive (ascending as before), the aggregates in the coarser level's new
// order: a block of rows then holds whole aggregates, so one kernel forms a
// residual and its restriction, and the owner of a coarse row prolongs to
// consecutive rows.  The finest level keeps the state's order and lists its
// members.
struct AmgPacked {
    std::vector<int32_t> mptr, midx;      // members of each next-level row (midx: finest level only)
    std::vector<double> diag;
    // off-diagonal entries: slice q holds rows [srow[q], srow[q+1]), at most
    // 64, entry k of its row j at off[q] + 64 k + j (pad: value 0)
    std::vector<int64_t> off;
    std::vector<int32_t> width, srow, idx;
    std::vector<double> val;
    // block b: slices [bslice[b], bslice[b+1]), aggregates [bagg[b], bagg[b+1])
    std::vector<int32_t> bslice, bagg;
};

struct AmgHierarchy {
    std::vector<AmgLevel> lv;             // lv[0] is the input matrix
    std::vector<double> cinv;             // dense inverse of the coarsest matrix, row-major
    double theta = 0.25, omega = 2.0 / 3.0;
    int gamma = 1;                        // cycle of the device (1 V, 2 W)
    int max_levels = 10;
    int64_t coarse_max = 1024;
    std::vector<AmgPacked> packed;        // device form, made when first asked for
};

// Builds the hierarchy of A (moved into lv[0]).  Returns 0 or a negative
// mifvm status; err receives a message.
int amg_build(AmgCsr&& A, double theta, int max_levels, int64_t coarse_max, double omega, AmgHierarchy& H,
              std::string& err);

// the device form of every level
void amg_pack(const AmgHierarchy& h, std::vector<AmgPacked>& out);

}  // namespace mifvm
