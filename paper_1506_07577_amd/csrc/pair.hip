// pair.hip -- CG iterations of a single mesh in two kernels, under the BLOCK strategy.
//
// An iteration of a small or mid-size mesh is a chain of latencies: every kernel costs its
// launch and a few dependent round trips, whatever it computes.  The four kernels of the plain
// iteration (K p; q and p.q; x, r, z; p) become two:
//   k_pair_kp      beta from the chunk partials of the update before; tet blocks stage
//                  p = z + beta p themselves, evaluate K p and leave a partial of p.Kp (every
//                  tet's corner results against p); further workgroups form and store p for the
//                  vertex chunks, with a partial of p.Mp;
//   k_pair_update  p.Ap = cm p.Mp - ck p.Kp from the partials, alpha, then for every vertex
//                  y = K p from the blocks' sums, q = Pi (cm M p - ck y), x, r, z and the
//                  partials of r.z and r.r.
// p alternates between two buffers, since blocks read their neighbours' old p while new p is
// stored.  What bounds both kernels is that chain (launch, tables, gathered vectors, partial sums,
// FP64 evaluation), about 6 us each however small the mesh.  Measured per iteration, FP64 StVK, four
// kernels (two for at most 4,096 vertices) against these two: 8^3 cells 14.9 -> 11.4 us, 12^3
// 27.1 -> 12.0, 16^3 16.9 -> 12.3, 24^3 18.4 -> 14.3, 32^3 22.0 -> 18.3, 40^3 28.9 -> 27.1, 44^3
// 32.7 -> 31.7; 48^3 37.7 -> 39.2 and 64^3 65.8 -> 78.6, since every block reads z and p where it
// read p and every vertex workgroup sums all blocks' partials: hence PAIR_BLOCKS.
// Every sum has a fixed order.  The stopping test of an iteration is made by the next
// iteration's k_pair_kp, and by k_pair_check at the end of a captured chunk.
#include <algorithm>

#include "block.h"
#include "cg.h"
#include "pair.h"

namespace ebbx {

namespace {

// beta of the iteration after the one whose partials are in slot par ^ 1; false if that iteration
// converged.  FIRST: the solve's first iteration, p = z.
template <bool FIRST>
__device__ __forceinline__ bool pair_beta(const PairArgs &c, double *s12, double &rz, double &rr, double &beta) {
    beta = 0.0;
    if (FIRST) return true;
    double rz0;
    sum_parts3(c.part, 0, c.nch, RZ + (c.par ^ 1), RR, RZ + c.par, s12, rz, rr, rz0);
    beta = rz / rz0;
    return !(sqrt(rr) <= c.tol * c.st[0].bnorm || rz == 0.0);
}

// Record an iteration's end in the mesh's state (one thread).
__device__ __forceinline__ void pair_record(const PairArgs &c, double rz, double rr, double beta, bool conv) {
    CGState &s = c.st[0];
    const int it = s.iters + 1;
    s.iters = it;
    s.rr = rr;
    if (conv) {
        s.converged = 1;
        mark_done(s, c.ctl, 0);
    } else {
        s.beta = beta;
        s.rz = rz;
        if (it >= c.maxit) mark_done(s, c.ctl, 0);
    }
}

// Workgroups [0, nblk): tet blocks (XCD x one contiguous range); from wg0 (a multiple of 8, so the
// chunks keep the XCDs of their blocks): vertex chunks.
template <int MODEL, int W, bool FIRST>
__global__ __launch_bounds__(VT) void k_pair_kp(ElemArgs a, PairArgs c) {
    extern __shared__ uint4 s_dyn4[];
    __shared__ double s12[12];
    // read here, tested (uniformly) once the loads below are in flight: a test here would put one
    // more round trip before them
    const int done = c.st[0].done;
    const uint32_t tid = threadIdx.x;
    double rz = 0.0, rr = 0.0, beta = 0.0;
    if (blockIdx.x >= c.wg0) {
        const uint32_t ch = xcd_block(blockIdx.x - c.wg0, (uint32_t)c.nch), v = ch * VT + tid;
        const bool in = v < a.nv;
        double z[3], p[3], m = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            z[k] = in ? c.z[(size_t)k * a.nv + v] : 0.0;
            p[k] = in && !FIRST ? c.p_old[(size_t)k * a.nv + v] : 0.0;
        }
        if (in) m = c.mass[v];
        if (done) return;
        const bool on = pair_beta<FIRST>(c, s12, rz, rr, beta);
        if (!FIRST && c.record && ch == 0 && tid == 0) pair_record(c, rz, rr, beta, !on);
        if (!on) return;
        double pm = 0.0;
        if (in)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double x = z[k] + beta * p[k];
                c.p_new[(size_t)k * a.nv + v] = x;
                pm += x * m * x;
            }
        pm = block_sum(pm, s12);
        if (tid == 0) c.part[4 * ch + PQ] = pm;
        return;
    }
    if (blockIdx.x >= a.nblk) return;
    const uint32_t blk = xcd_block(blockIdx.x, a.nblk), S = a.blk_stride, t = blk * VT + tid;
    constexpr uint32_t LB = 4 * VT;
    const bool in = t < a.nt;
    const int32_t *bverts = a.blk_verts + (size_t)blk * S;
    const int32_t *bhpos = a.blk_hpos + (size_t)blk * S;
    const uint16_t *brow = a.blk_row + (size_t)blk * (S + 1);
    // the LDS layout of the stiffness product's block kernel
    constexpr bool XB = W == 1;
    double *s_d = (double *)s_dyn4, *s_p = s_d + 3 * S, *s_x = s_p + 3 * S, *s_h = s_d;

    const int32_t gvs0 = tid < S ? bverts[tid] : -1;
    int32_t hp0 = -1, j00 = 0, j10 = 0;
    if (tid < S) {   // as in block_body, before the vertex id is waited for
        hp0 = bhpos[tid];
        j00 = brow[tid];
        j10 = brow[tid + 1];
    }
    double b[9], V0 = 1.0, mu = 0.0, lam = 0.0;
    uint32_t sl[4] = {0, 0, 0, 0}, pw[2] = {0, 0};
    if (in) {
        if (!XB) {
#pragma unroll
            for (int k = 0; k < 9; ++k) b[k] = ldc<double>(a.B[k], t);
            V0 = tet_V0(b);
        }
        if (a.mu_t) {
            mu = ldc<double>(a.mu_t, t);
            lam = ldc<double>(a.lam_t, t);
        } else {
            mu = a.mu;
            lam = a.lam;
        }
        unpack_slots<W>(a, t, sl);
        pw[0] = ldc<uint32_t>(a.blk_pos[0], t);
        pw[1] = ldc<uint32_t>(a.blk_pos[1], t);
    }
    // the first block vertex's fields are in flight while the partials are summed
    const bool has = gvs0 >= 0;
    const uint32_t gv0 = has ? (uint32_t)gvs0 : 0u;
    double d0[3], x0[3], z0[3], p0[3];
    if (has)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            z0[k] = ldc<double>(a.u[k], gv0);
            p0[k] = FIRST ? 0.0 : ldc<double>(c.p_old + (size_t)k * a.nv, gv0);
            d0[k] = ldc<double>(a.d[k], gv0);
            if (XB) x0[k] = ldc<double>(a.X[k], gv0);
        }
    if (done || !pair_beta<FIRST>(c, s12, rz, rr, beta)) return;   // the same sums in every workgroup
    if (has)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s_d[k * S + tid] = d0[k];
            s_p[k * S + tid] = z0[k] + beta * p0[k];
            if (XB) s_x[k * S + tid] = x0[k];
        }
    for (uint32_t i = tid + VT; i < S; i += VT) {
        const int32_t gvs = bverts[i];
        if (gvs < 0) continue;
        const uint32_t gv = (uint32_t)gvs;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s_d[k * S + i] = ldc<double>(a.d[k], gv);
            s_p[k * S + i] = ldc<double>(a.u[k], gv) + (FIRST ? 0.0 : beta * ldc<double>(c.p_old + (size_t)k * a.nv, gv));
            if (XB) s_x[k * S + i] = ldc<double>(a.X[k], gv);
        }
    }
    __syncthreads();
    const uint32_t q[4] = {pw[0] & 0xffffu, pw[0] >> 16, pw[1] & 0xffffu, pw[1] >> 16};
    double pk = 0.0;   // this tet's share of p.Kp
    double h[12], G[9], dF[9];
    if (in) {
        if (XB) rest_B(s_x, S, sl, b, V0);
        staged_grad(s_d, S, sl, b, G);
        staged_grad(s_p, S, sl, b, dF);
    }
    __syncthreads();   // the rows overwrite the staging
    if (in) {
        double dP[9];
        dstress_scaled<double, MODEL>(mu, lam, V0, G, dF, dP);
        corner_out(dP, b, h);
#pragma unroll
        for (int k = 0; k < 9; ++k) pk += dF[k] * dP[k];   // = the corners' sum against p
    }
    if (in)
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4) {
            s_h[q[k4]] = h[3 * k4];
            s_h[LB + q[k4]] = h[3 * k4 + 1];
            s_h[2 * LB + q[k4]] = h[3 * k4 + 2];
        }
    __syncthreads();
    if (has) reduce_slot<double>(a, s_h, LB, gv0, hp0, j00, j10);
    for (uint32_t i = tid + VT; i < S; i += VT) {
        const int32_t gvs = bverts[i];
        if (gvs >= 0) reduce_slot<double>(a, s_h, LB, (uint32_t)gvs, bhpos[i], brow[i], brow[i + 1]);
    }
    if (!isfinite(pk)) {   // so it is in
        // p is zero on pinned vertices, and their rows are no part of the system: a tet of four has no
        // share, also where its stress is not finite (0 * inf)
        unpack_slots<W>(a, t, sl);
        bool pinned = true;
#pragma unroll
        for (int k = 0; k < 4; ++k) pinned = pinned && c.pinned[bverts[sl[k]]];
        if (pinned) pk = 0.0;
    }
    pk = block_sum(pk, s12);
    if (tid == 0) c.part_k[blk] = pk;
}

// The halo places of every vertex, W int4 per vertex in block order: -1 padded; all -1 where a
// block owns the vertex outright; first -2 where no tet touches it.
__global__ void k_pair_tab(HaloView h, int64_t nv, int4 *tab) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nv * h.nc) return;
    const int64_t v = i / h.nc;
    const int c = (int)(i - v * h.nc);
    const int32_t r = h.row[v];
    int4 q = make_int4(-1, -1, -1, -1);
    if (r >= 0) {
        int n;
        const int4 *t = h.at(r, n);
        if (c < n) q = t[c];
        if (c == 0 && q.x < 0) q.x = -2;
    }
    tab[i] = q;
}

// pq = cm p.Mp - ck p.Kp; breakdown as in the plain iteration.  One chunk per workgroup.  NC > 0:
// the halo places come from the vertex's row of tab, one dependent load fewer than through the
// shared-vertex rows; NC = 0: from those (a vertex shared by more than 16 blocks).
template <int NC>
__global__ __launch_bounds__(VT) void k_pair_update(StepVec w, const double *p_now, const double *mass,
                                                    const uint8_t *pinned, int64_t nv, int nblk, double cm, double ck,
                                                    HaloView hv, const int4 *tab, PairArgs c) {
    __shared__ double s12[12];
    const int done = c.st[0].done;   // tested below, with the loads in flight
    const int ch = (int)xcd_block(blockIdx.x, gridDim.x);
    const int64_t v = (int64_t)ch * VT + threadIdx.x;
    const bool in = v < nv;
    double x[3], p[3], r[3], y[3], dg[3], m = 0.0;
    bool pin = false;
    if (in) {
        int4 q[NC > 0 ? NC : 1];
        if (NC > 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) q[i] = tab[v * NC + i];
#pragma unroll
            for (int k = 0; k < 3; ++k) y[k] = w.y[k * nv + v];
        }
        m = mass[v];
        pin = pinned[v] != 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int64_t i = k * nv + v;
            x[k] = w.x[i];
            p[k] = p_now[i];
            r[k] = w.r[i];
            dg[k] = w.diag[i];
        }
        if (NC == 0) {
            finished(hv, w.y, nv, v, y);
        } else if (q[0].x != -1) {   // summed from the halo, in block order
            y[0] = y[1] = y[2] = 0.0;
#pragma unroll
            for (int i = 0; i < NC; ++i) halo_add4(hv.halo, q[i], y);
        }
    }
    if (done) return;   // uniform
    double acc[3] = {0.0, 0.0, 0.0};   // p.Mp, r.z before, p.Kp
    {
        double two[2] = {0.0, 0.0};
        part_acc<2>(c.part, 0, c.nch, {PQ, RZ + (c.par ^ 1)}, two);
        acc[0] = two[0];
        acc[1] = two[1];
        for (int i0 = (int)threadIdx.x; i0 < nblk; i0 += PART_BATCH * VT) {
            double l[PART_BATCH];
#pragma unroll
            for (int j = 0; j < PART_BATCH; ++j) l[j] = i0 + j * VT < nblk ? c.part_k[i0 + j * VT] : 0.0;
#pragma unroll
            for (int j = 0; j < PART_BATCH; ++j) acc[2] += l[j];
        }
    }
    block_sums<3>(acc, s12);
    const double pq = cm * acc[0] - ck * acc[2];
    const bool first = ch == 0 && threadIdx.x == 0;
    if (!(pq > 0.0)) {   // breakdown: every workgroup sees it and leaves x, r alone
        if (first) {
            c.st[0].pq = pq;
            c.st[0].status = EBBX_E_NOT_SPD;
            mark_done(c.st[0], c.ctl, 0);
        }
        return;
    }
    const double alpha = acc[1] / pq;
    if (first) {
        c.st[0].pq = pq;
        c.st[0].alpha = alpha;
    }
    double red[2] = {0.0, 0.0};
    if (in)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int64_t i = k * nv + v;
            const double q = pin ? 0.0 : cm * m * p[k] - ck * y[k];
            w.x[i] = x[k] + alpha * p[k];
            const double rn = r[k] - alpha * q;
            const double z = rn / dg[k];
            w.r[i] = rn;
            w.z[i] = z;
            red[0] += rn * z;
            red[1] += rn * rn;
        }
    __syncthreads();   // s12 is read above
    block_sums<2>(red, s12);
    if (threadIdx.x == 0) {
        c.part[4 * ch + RZ + c.par] = red[0];
        c.part[4 * ch + RR] = red[1];
    }
}

// The stopping test after the last iteration of a chunk (its partials in slot par).
__global__ __launch_bounds__(VT) void k_pair_check(PairArgs c) {
    __shared__ double s12[12];
    if (c.st[0].done) return;
    double rz, rr, rz0;
    sum_parts3(c.part, 0, c.nch, RZ + c.par, RR, RZ + (c.par ^ 1), s12, rz, rr, rz0);
    const bool conv = sqrt(rr) <= c.tol * c.st[0].bnorm || rz == 0.0;
    __syncthreads();   // the state is read above
    if (threadIdx.x == 0) pair_record(c, rz, rr, rz / rz0, conv);
}

template <int MODEL, int W>
void launch_kp(const ElemArgs &a, const PairArgs &c, bool first, unsigned grid, size_t shmem, hipStream_t s) {
    if (first) hipLaunchKernelGGL((k_pair_kp<MODEL, W, true>), dim3(grid), dim3(VT), shmem, s, a, c);
    else hipLaunchKernelGGL((k_pair_kp<MODEL, W, false>), dim3(grid), dim3(VT), shmem, s, a, c);
}

template <int MODEL>
void launch_kp(const ebbx_fem_s *F, const ElemArgs &a, const PairArgs &c, bool first, unsigned grid, size_t shmem,
               hipStream_t s) {
    if (F->blk_w == 1) launch_kp<MODEL, 1>(a, c, first, grid, shmem, s);
    else launch_kp<MODEL, 2>(a, c, first, grid, shmem, s);
}

}  // namespace

bool pair_ok(const ebbx_fem_s *F) {
    return F->nm == 1 && F->strategy == EBBX_STRAT_BLOCK && F->blk_red == 0 && F->blk_tpt == 1 &&
           F->blk_tets == VT && F->halo_level == 0 && F->nt > 0 &&
           F->nblk <= PAIR_BLOCKS && F->prec == EBBX_F64;
}

void pair_prepare(ebbx_fem_s *F, hipStream_t s) {
    if (F->pair_tab.get()) return;   // of the present tables; an earlier solve may still be reading it
    const size_t bytes = (size_t)F->nv * F->sh_nc * sizeof(int4);
    if (bytes == 0 || F->sh_n == 0) return;
    F->pair_tab.reset(bytes, s);
    const int64_t n = F->nv * F->sh_nc;
    hipLaunchKernelGGL(k_pair_tab, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, elem_halo_view(F), F->nv,
                       F->pair_tab.as<int4>());
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(s));   // the solve that reads it runs on another stream
}

void pair_iterations(ebbx_fem_s *F, const ebbx_step_params &p, const StepVec &w, CGState *st, SolveCtl *ctl,
                     double *part, double *part_k, int nch, int count, bool first, hipStream_t s) {
    const int64_t nv = F->nv;
    const double cm = 1.0 + p.dt * p.alpha, ck = p.dt * p.dt + p.dt * p.beta;
    const HaloView hv = elem_halo_view(F);
    double *buf[2] = {w.p, w.q};
    PairArgs c{};
    c.z = w.z;
    c.mass = F->mass.as<double>();
    c.pinned = F->pinned.as<uint8_t>();
    c.part = part;
    c.part_k = part_k;
    c.st = st;
    c.ctl = ctl;
    c.tol = p.tol;
    c.maxit = p.maxit;
    c.nch = nch;
    c.wg0 = (uint32_t)((F->nblk + 7) / 8 * 8);
    const unsigned grid = c.wg0 + (unsigned)nch;
    size_t shmem = 0;
    const ElemArgs a = elem_block_args(F, OP_KMUL, w.dn, w.z, w.y, &shmem);
    int it = 0;
    for (; it < count && it < p.maxit; ++it) {
        c.par = it & 1;
        c.record = it > 0;   // the last iteration of the chunk before was recorded by its check
        c.p_old = buf[it & 1];
        c.p_new = buf[(it & 1) ^ 1];
        if (F->model == EBBX_STVK) launch_kp<EBBX_STVK>(F, a, c, first && it == 0, grid, shmem, s);
        else launch_kp<EBBX_NH>(F, a, c, first && it == 0, grid, shmem, s);
        auto update = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((unsigned)nch), dim3(VT), 0, s, w, (const double *)c.p_new, c.mass,
                               F->pinned.as<uint8_t>(), nv, (int)F->nblk, cm, ck, hv, F->pair_tab.as<int4>(), c);
        };
        switch (F->pair_tab.get() ? F->sh_nc : 0) {
        case 1: update(k_pair_update<1>); break;
        case 2: update(k_pair_update<2>); break;
        case 3: update(k_pair_update<3>); break;
        case 4: update(k_pair_update<4>); break;
        default: update(k_pair_update<0>);
        }
    }
    if (it > 0) {
        c.par = (it - 1) & 1;
        hipLaunchKernelGGL(k_pair_check, dim3(1), dim3(VT), 0, s, c);
    }
    HIPCHK(hipGetLastError());
}

}  // namespace ebbx
