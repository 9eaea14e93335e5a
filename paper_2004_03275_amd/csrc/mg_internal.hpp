// mg_internal.hpp -- entry points of the uniform multigrid solver
// (multigrid.hip) for the library's own use.
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/amrv_mg.h"

namespace amrv {

// Split order of a grid of 2^lg cells per side: the cells of colour 0 = (x + y +
// z) & 1, then those of colour 1, each [z][y][x / 2].  The cells 2 xh, 2 xh + 1
// of a row are a pair, p = row * n / 2 + xh: each half holds one cell of the
// pair at p, so both colours of a pair share their addresses up to the half.
template <int ND>
__device__ __forceinline__ int split_idx(int x, int y, int z, int lg) {
  const int i = ND == 3 ? (((z << lg) + y) << lg) + x : (y << lg) + x;
  return (i >> 1) + (((x + y + z) & 1) << (ND * lg - 1));
}

// The solver's own finest-level right-hand side and solution arrays (field
// 0, n^d device doubles each, in split order where *split): a caller that fills
// *f and zeroes *e itself and passes them to mg_enqueue_correction saves its
// copies and its fill.
int mg_correction_grids(amrv_mg* m, double** f, double** e, bool* split);

// Enqueues, on the solver's stream and without any host synchronisation,
// `cycles` V-cycles for lap(e) - lambda e = f from e = 0, then copies e to
// out (f, out: n^d device doubles; no copy where f or out is the solver's own
// array, the only case for a solver whose arrays are in split order).  e_zeroed: the solver's solution array already holds zeros (else
// it is cleared here).  The parameter block is uploaded only when lambda
// differs from the last one set.  For a solver with one field and the
// constant coefficient; lambda >= 0.  Returns 0 or a negative AMRV_E* code.
int mg_enqueue_correction(amrv_mg* m, const double* f, double* out, double lambda, int cycles, bool e_zeroed);

}  // namespace amrv
