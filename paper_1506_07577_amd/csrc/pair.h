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
};

// Tet blocks of a mesh up to which an iteration runs in two kernels: 44^3 cells have 1997, where
// they are the faster by 3% (FP64), 48^3 cells 2592, where they are the slower by 4%.
constexpr int64_t PAIR_BLOCKS = 2048;
// The same for FP32 elements.  p.Kp summed over the tets differs from the vertices' sum in the last
// bit, and an FP32 rounding of a tet's gradients that this turns is a 1e-7 step there; how many are
// turned grows with tets times iterations.  Solves of 100 iterations or to 1e-8 (E = 1e6, nu = 0.45)
// against the vertices' sum, normwise and the largest entry: up to 27^3 cells at most 1.4e-10 / 3e-9,
// 36^3 3e-10 / 2e-8, 43^3 6e-10 / 5e-8.  Both forms are equally far from 64-bit arithmetic (3e-7 to
// 6e-7), but a solve should not depend on its kernels by more than 1e-9 / 4e-8, so larger meshes (28^3
// cells have 515 blocks) keep the four kernels, slower by a third at 30^3 and by 2% at 43^3.
constexpr int64_t PAIR_BLOCKS_F32 = 512;

// Whether F's solves run so: one mesh, BLOCK strategy with 256 tets per block, one per thread,
// incidence-order sums, at most PAIR_BLOCKS blocks (FP32 elements: PAIR_BLOCKS_F32).
bool pair_ok(const ebbx_fem_s *F);
// The per-vertex halo places that the iterations read (pair_tab), whole on return; before they are
// captured.
void pair_prepare(ebbx_fem_s *F, hipStream_t s);
// `count` iterations (at most maxit) from an even iteration onto stream s; first: from the solve's
// first one.  part_k: one double per tet block.
void pair_iterations(ebbx_fem_s *F, const ebbx_step_params &p, const StepVec &w, CGState *st, SolveCtl *ctl,
                     double *part, double *part_k, int nch, int count, bool first, hipStream_t s);

}  // namespace ebbx
