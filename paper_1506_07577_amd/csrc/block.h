// block.h -- the pieces of the BLOCK strategies' kernels: corner slots, run sums and gradients of
// staged vertex fields.
#pragma once

#include "fem.h"
#include "tetmath.h"

namespace ebbx {

// Block b holds tets [b*BT, (b+1)*BT) of the tables' order, BT = blockDim.x * TPT.
// Its vertex list blk_verts[b*S .. (b+1)*S), S the largest block's count, is sorted
// and padded with -1; each corner carries its slot in that list (packed: 4 x 8 bits
// per word when every block has <= 256 vertices, else 2 x 16 bits in each of two
// words).

template <int W> __device__ __forceinline__ void unpack_slots(const ElemArgs &a, uint32_t t, uint32_t *s) {
    if (W != 2) {
        const uint32_t w = ldc<uint32_t>(a.slot[0], t);
        s[0] = w & 255u;
        s[1] = (w >> 8) & 255u;
        s[2] = (w >> 16) & 255u;
        s[3] = w >> 24;
    } else {
        const uint32_t w0 = ldc<uint32_t>(a.slot[0], t), w1 = ldc<uint32_t>(a.slot[1], t);
        s[0] = w0 & 65535u;
        s[1] = w0 >> 16;
        s[2] = w1 & 65535u;
        s[3] = w1 >> 16;
    }
}

// LDS layout: the block's vertex fields with one column per component (d, and
// u for the stiffness product), then the per-corner results, three columns
// (x, y, z) whose rows follow the block's incidence order (by vertex, then
// local tet, then corner): each tet writes its four corners to the rows the
// block tables give them, so every block vertex then sums one contiguous run
// of rows (fixed order, FP64) and either stores it (the block owns the vertex)
// or writes it to the halo.  Every global load that does not depend on another
// is issued at kernel start.
template <class T>
__device__ __forceinline__ void reduce_slot(const ElemArgs &a, const T *s_h, uint32_t LB, uint32_t gv, int32_t hp,
                                            int32_t j0, int32_t j1) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll 4
    for (int32_t j = j0; j < j1; ++j) {   // this vertex's rows, in (local tet, corner) order
        a0 += (double)s_h[j];
        a1 += (double)s_h[LB + j];
        a2 += (double)s_h[2 * LB + j];
    }
    if (hp < 0) {
        // every incident tet is in this block: sole writer
        if (a.accumulate) {
            a0 += ldc<double>(a.out[0], gv);
            a1 += ldc<double>(a.out[1], gv);
            a2 += ldc<double>(a.out[2], gv);
        }
        stc<double>(a.out[0], gv, a0);
        stc<double>(a.out[1], gv, a1);
        stc<double>(a.out[2], gv, a2);
    } else {
        double *hq = a.halo + 3 * (size_t)hp;
        hq[0] = a0;
        hq[1] = a1;
        hq[2] = a2;
    }
}

// Gradient dD B of a vertex field staged in LDS (3 columns of S block vertices) over the
// tet whose corners sit in slots sl.
template <class T>
__device__ __forceinline__ void staged_grad(const double *s, uint32_t S, const uint32_t *sl, const T *b, T *G) {
    double q[4][3];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int k = 0; k < 3; ++k) q[c][k] = s[k * S + sl[c]];
    grad_from(q, b, G);
}

}  // namespace ebbx
