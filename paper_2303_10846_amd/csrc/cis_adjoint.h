// Launchers of the adjoint solve's block preconditioner (FP64); the kernels are in cis_adjoint.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cis_internal.h"
#include "cis_macro.h"

namespace cis {

// Per-cell scratch of the block preconditioner, 26 doubles per cell: gW [nc][6], gq [nc][6], u [nc][6],
// r [nc][6] (face spectral radii of Eq. 41), D [nc][2] (macro diagonals).
constexpr int kBlockPrecondCellDoubles = 26;  // gW, gq, u (6 each), r_f (up to 6 slots), 2 diagonals

// out = P in over the full adjoint vector [G | R | W | q]: the W and q rows are eliminated exactly (their
// diagonal block is taken as the identity) and the phi Schur complement is approximated by the transpose of
// the linearised implicit step, micro_pairs transposed micro sweep pairs (0: the diagonal) followed by the
// transposed macro system with macro_pairs PR-SGS pairs.  tmp: a second full-length vector; cell: the scratch
// above.  in and out must not overlap tmp.  sweeps, flag: the state's macro sweeps (NULL: a launch
// per colour) and its error flag.
void launch_adj_block_precond(const Dev& d, const Bufs& b, const double* in, double* out, double* tmp, double* cell,
                              const int64_t* color_off, int64_t n_colors, int micro_pairs, int macro_pairs,
                              MacroSweeps* sweeps, int32_t* flag, hipStream_t st);

// Its macro part: Mac^T u = t ([n_cells][6]) with `pairs` PR-SGS pairs from u = 0.  rc [n_cells][max_faces] and mD
// [n_cells][2]: scratch.
void launch_adj_macro(const Dev& d, const Bufs& b, const double* t, double* u, double* rc, double* mD,
                      const int64_t* color_off, int64_t n_colors, int pairs, MacroSweeps* sweeps, int32_t* flag,
                      hipStream_t st);

}  // namespace cis
