// team_host.h -- host interface of the team solves (team.hip).
#pragma once

#include <vector>

#include "internal.h"

namespace apcg {

// Single solves take the team schedule above this many rows.
constexpr int32_t kTeamMinRows = 8192;

// Whether every system can be solved by teams on ctx's device: rows of at
// most 7 entries, windows that fit the LDS, no system larger than the chip.
// *rows receives the 64-row slices per wavefront to use, 0 when it cannot.
// Reads the matrices' column ranges back once per matrix.
apcg_status team_eligible(apcg_ctx ctx, int32_t nsys, const apcg_mat *A, int *rows);

// Jacobi-PCG (or CG) of the systems, started in `order` (largest cost
// first), results in info[i]; hist as in pcg_solve_marked (one system).
// Returns once the launch has finished; *left holds the systems it did not
// solve (their x untouched), which the caller solves with another schedule.
apcg_status team_pcg_solve(apcg_ctx ctx, int32_t nsys, const apcg_mat *A, const apcg_vec *b, const apcg_vec *x,
                           const std::vector<int32_t> &order, double rtol, int32_t maxit, const apcg_solve_opts &opts,
                           int rows, apcg_solve_info *info, double *hist, int32_t hist_cap,
                           std::vector<int32_t> *left);

}  // namespace apcg
