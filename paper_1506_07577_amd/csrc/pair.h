// pair.h -- CG iterations of a single mesh in two kernels (pair.hip).
#pragma once

#include "cg.h"

namespace ebbx {

struct PairArgs {
    const double *z, *p_old, *mass;
    double *p_new;
    double *part, *part_k;   // chunk partials (4 per chunk; p.Mp at PQ), block partials of p.Kp
    CGState *st;
    SolveCtl *ctl;
    double tol;
    int maxit, nch, par;     // par: parity of this iteration, the r.z slot it writes
    int record;              // 1: this iteration's k_pair_kp records the end of the one before
    uint32_t wg0;            // first workgroup of the vertex chunks
    const uint8_t *pinned;
};

// Tet blocks of a mesh up to which an iteration runs in two kernels: 44^3 cells have 1997, where
// they are the faster by 3% (FP64), 48^3 cells 2592, where they are the slower by 4%.
constexpr int64_t PAIR_BLOCKS = 2048;

// Whether F's solves run so: one mesh, BLOCK strategy with 256 tets per block, one per thread,
// incidence-order sums, at most PAIR_BLOCKS blocks, FP64 elements.  Solves with FP32 elements keep the plain
// iteration, and so their bits: p.Kp summed over the tets differs from the vertices' sum in the last place,
// and where that turns an FP32 rounding of a tet's gradients two solves part by 4e-10 normwise and 1.5e-8
// in the largest entry at 16^3 cells (to 1e-8), 5e-8 at 43^3 (100 iterations).  Neither is further from
// 64-bit arithmetic, and the two kernels would be up to 1.4x the faster (27^3).
bool pair_ok(const ebbx_fem_s *F);
// The per-vertex halo places that the iterations read (pair_tab), whole on return; before they are
// captured.
void pair_prepare(ebbx_fem_s *F, hipStream_t s);
// `count` iterations (at most maxit) from an even iteration onto stream s; first: from the solve's
// first one.  part_k: one double per tet block.
void pair_iterations(ebbx_fem_s *F, const ebbx_step_params &p, const StepVec &w, CGState *st, SolveCtl *ctl,
                     double *part, double *part_k, int nch, int count, bool first, hipStream_t s);

}  // namespace ebbx
