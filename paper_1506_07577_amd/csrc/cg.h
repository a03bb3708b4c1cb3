// cg.h -- what the kernels of a conjugate-gradient solve share: its state on the device, the
// fixed-order sums of chunk partials, and the finishing of an element map's halo.
#pragma once

#include "fem.h"
#include "wave.h"

namespace ebbx {

// CG state of one mesh, kept on the device.
struct CGState {
    double rz, rr, pq, alpha, beta, bnorm;
    int iters, status, done, converged;
    unsigned long long n_inv;
};

// Solve-wide flags: meshes still iterating; all_done = 1 once none is, when the solve's number is
// also written to *host (pinned host memory), for a host that waits on the solve.  The per-mesh
// finished flags (nm ints) follow the struct in memory.
struct SolveCtl {
    int n_active, all_done;
    int solve, pad;
    int *host;
};

__device__ __forceinline__ int *mesh_done(SolveCtl *c) { return (int *)(c + 1); }

constexpr int VT = 256;   // threads of the vertex kernels = vertices per chunk

// Sum of one double over a 256-thread block (fixed order).
__device__ __forceinline__ double block_sum(double x, double *s4) {
    x = lanes_sum<64>(x);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s4[threadIdx.x >> 6] = x;
    __syncthreads();
    return (s4[0] + s4[1]) + (s4[2] + s4[3]);
}

// N block sums at once (s: 4 N doubles), each combined exactly as block_sum combines one.
template <int N>
__device__ __forceinline__ void block_sums(double (&x)[N], double *s) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = lanes_sum<64>(x[i]);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) s[4 * i + (threadIdx.x >> 6)] = x[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = (s[4 * i] + s[4 * i + 1]) + (s[4 * i + 2] + s[4 * i + 3]);
}

// Chunk partials, 4 doubles per chunk: [0] p.q, [1] r.r, [2 + parity] r.z of the
// iterations of that parity (the initial residual counts as parity 1).
constexpr int PQ = 0, RR = 1, RZ = 2;

// Each thread's share of a fixed-order sum over chunks [c0, c1): acc[s] += the partials at
// offset o[s] of chunks c0 + t, c0 + t + VT, c0 + t + 2 VT, ... in that order.  The loads of
// PART_BATCH strided chunks are issued before any of them is added, so a workgroup waits for
// one round trip per batch rather than one per chunk; the order of the additions is unchanged.
constexpr int PART_BATCH = 8;
template <int NS>
__device__ __forceinline__ void part_acc(const double *part, int c0, int c1, const int (&o)[NS], double (&acc)[NS]) {
    for (int cb = c0 + (int)threadIdx.x; cb < c1; cb += PART_BATCH * VT) {
        double l[PART_BATCH][NS];
#pragma unroll
        for (int j = 0; j < PART_BATCH; ++j) {
            const int c = cb + j * VT;
#pragma unroll
            for (int s = 0; s < NS; ++s) l[j][s] = c < c1 ? part[4 * c + o[s]] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < PART_BATCH; ++j)
            if (cb + j * VT < c1)
#pragma unroll
                for (int s = 0; s < NS; ++s) acc[s] += l[j][s];
    }
}

// Fixed-order sum of the partials at offset o of chunks [c0, c1).
__device__ __forceinline__ double sum_parts(const double *part, int c0, int c1, int o, double *s4) {
    double acc[1] = {0.0};
    part_acc<1>(part, c0, c1, {o}, acc);
    return block_sum(acc[0], s4);
}

// Three fixed-order sums at once (offsets o0, o1, o2), each with exactly the
// operation order of sum_parts, sharing the barriers.
__device__ __forceinline__ void sum_parts3(const double *part, int c0, int c1, int o0, int o1, int o2, double *s12,
                                           double &r0, double &r1, double &r2) {
    double acc[3] = {0.0, 0.0, 0.0};
    part_acc<3>(part, c0, c1, {o0, o1, o2}, acc);
    const double a0 = lanes_sum<64>(acc[0]), a1 = lanes_sum<64>(acc[1]), a2 = lanes_sum<64>(acc[2]);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s12[threadIdx.x >> 6] = a0;
        s12[4 + (threadIdx.x >> 6)] = a1;
        s12[8 + (threadIdx.x >> 6)] = a2;
    }
    __syncthreads();
    r0 = (s12[0] + s12[1]) + (s12[2] + s12[3]);
    r1 = (s12[4] + s12[5]) + (s12[6] + s12[7]);
    r2 = (s12[8] + s12[9]) + (s12[10] + s12[11]);
}

// Two fixed-order sums at once (offsets o0, o1), as sum_parts3.
__device__ __forceinline__ void sum_parts2(const double *part, int c0, int c1, int o0, int o1, double *s12, double &r0,
                                           double &r1) {
    double acc[2] = {0.0, 0.0};
    part_acc<2>(part, c0, c1, {o0, o1}, acc);
    const double a0 = lanes_sum<64>(acc[0]), a1 = lanes_sum<64>(acc[1]);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s12[threadIdx.x >> 6] = a0;
        s12[4 + (threadIdx.x >> 6)] = a1;
    }
    __syncthreads();
    r0 = (s12[0] + s12[1]) + (s12[2] + s12[3]);
    r1 = (s12[4] + s12[5]) + (s12[6] + s12[7]);
}

// One thread of the mesh's block marks mesh m finished.
__device__ __forceinline__ void mark_done(CGState &st, SolveCtl *ctl, int m) {
    st.done = 1;
    mesh_done(ctl)[m] = 1;
    if (atomicSub(&ctl->n_active, 1) == 1) {
        ctl->all_done = 1;
        __hip_atomic_store(ctl->host, ctl->solve, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

struct StepVec {
    double *dn, *vn, *f, *y, *r, *z, *p, *q, *x, *diag;
};

// Vertex v's value of an element-map output that may still have its shared
// vertices' sums in the halo (same summation order as the halo pass).
__device__ __forceinline__ void finished(const HaloView &h, const double *y, int64_t nv, int64_t v, double *o) {
    const int32_t r = h.row ? h.row[v] : -1;
    if (r < 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) o[k] = y[k * nv + v];
        return;
    }
    double a[3] = {0.0, 0.0, 0.0};
    if (h.nc > 0) {
        int n;
        const int4 *t = h.at(r, n);
        for (int c = 0; c < n; ++c) halo_add(h.halo, t[c], a);
    } else {
        for (int32_t j = h.ptr[r]; j < h.ptr[r + 1]; ++j) {
            const double *hq = h.halo + 3 * (size_t)h.pos[j];
            a[0] += hq[0];
            a[1] += hq[1];
            a[2] += hq[2];
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) o[k] = a[k];
}

}  // namespace ebbx
