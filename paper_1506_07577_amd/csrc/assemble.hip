// assemble.hip -- the stiffness matrix stored on the mesh edges.
//
// The Vega workload keeps its stiffness on the edges of the tet mesh, one 3x3
// block per pair of vertices that share a tet (Developing Domain Libraries,
// "Example: FEM tetmesh"; Performance Evaluation).  Here the edges relation
// holds every ordered pair (i, j), i == j included, grouped by the tail i and
// sorted by the head j, so that the blocks form a block-CSR matrix and K u is
// a sparse product instead of the matrix-free element map.
//
//  - k_asm_block: a workgroup owns the edges leaving a range of 8 or 4 vertices.  It
//    evaluates every tet that touches them into a compact record in LDS (the
//    corner vectors and the symmetric corner products that every 3x3 corner
//    block of the tet is a short sum of), then one thread per edge sums the
//    corner blocks of the tets holding both of its vertices in ascending tet
//    order (deterministic).  No per-tet matrix goes through memory;
//  - k_elem_matrix and k_edge_gather: the same blocks through a 144-value record
//    per tet in memory, for meshes with a vertex of so many tets (some 400
//    neo-Hookean or 240 StVK) that those of four vertices do not fit in LDS;
//  - k_bsr_spmv: sixteen lanes per vertex row; each lane takes edges of the row
//    (consecutive lanes read consecutive entries of each column) and the row
//    sum is a fixed butterfly over the sixteen lanes.
#include <algorithm>

#include "fem.h"
#include "sort.h"
#include "tetmath.h"
#include "wave.h"

namespace ebbx {

namespace {

constexpr int SPMV_LANES = 16;

struct AsmArgs {
    uint32_t nt;
    const int32_t *key[4];
    const void *B[9];
    const void *mu_t, *lam_t;
    double mu, lam;
    const double *d[3];
    void *ke;                    // (nt, 16, 9) at the element precision: block (a, b) of tet t at
                                 // ke[(16 t + 4 b + a) * 9]
    unsigned long long *n_inv;
    const int32_t *tmesh;
};

constexpr int EM_THREADS = 128;   // tets per workgroup of the element-matrix kernel
constexpr int EM_STRIDE = 37;     // LDS doubles per tet for one block column (36, padded)

// Per-tet record: 144 values at the element precision, block (a, b) (rows of corner a, columns
// of corner b) at (4 b + a) * 9, row-major; so the four blocks of one column b are 36
// contiguous values.
template <class T, int MODEL>
__global__ __launch_bounds__(EM_THREADS) void k_elem_matrix(AsmArgs a) {
    __shared__ double s_col[EM_THREADS * EM_STRIDE];
    const uint32_t t0 = blockIdx.x * EM_THREADS, t = t0 + threadIdx.x;
    const bool in = t < a.nt;
    const uint32_t nloc = min((uint32_t)EM_THREADS, a.nt - t0);   // tets of this workgroup
    double b[9], G[9], gb[4][3], V0 = 1.0, mu = 0.0, lam = 0.0;
    if (in) {
#pragma unroll
        for (int k = 0; k < 9; ++k) b[k] = (double)ldc<T>(a.B[k], t);
        V0 = tet_V0(b);
        mu = a.mu_t ? (double)ldc<T>(a.mu_t, t) : a.mu;
        lam = a.lam_t ? (double)ldc<T>(a.lam_t, t) : a.lam;
        double qd[4][3];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t v = (uint32_t)a.key[c][t];
#pragma unroll
            for (int k = 0; k < 3; ++k) qd[c][k] = a.d[k][v];
        }
        grad_from(qd, b, G);
        // grad N_b: rows of B for corners 1..3, minus their sum for corner 0
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            gb[1][j] = b[j];
            gb[2][j] = b[3 + j];
            gb[3][j] = b[6 + j];
            gb[0][j] = -(b[j] + b[3 + j] + b[6 + j]);
        }
    }
    bool ok = true;
    // one block column at a time: every tet's 36 values go through LDS, then the workgroup
    // writes each tet's 288 contiguous bytes of that column together
    for (int cb = 0; cb < 4; ++cb) {
        if (in) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                double dF[9], dP[9], h[12];
#pragma unroll
                for (int q = 0; q < 9; ++q) dF[q] = 0.0;
                dF[3 * k] = gb[cb][0];
                dF[3 * k + 1] = gb[cb][1];
                dF[3 * k + 2] = gb[cb][2];
                ok = dstress_scaled<double, MODEL>(mu, lam, V0, G, dF, dP) && ok;
                corner_out(dP, b, h);   // h[3 a + r] = df_{a,r} / dd_{cb,k}
#pragma unroll
                for (int ca = 0; ca < 4; ++ca)
#pragma unroll
                    for (int r = 0; r < 3; ++r) s_col[threadIdx.x * EM_STRIDE + ca * 9 + 3 * r + k] = h[3 * ca + r];
            }
        }
        __syncthreads();
        for (uint32_t e = threadIdx.x; e < nloc * 36u; e += EM_THREADS) {
            const uint32_t i = e / 36u, o = e - 36u * i;
            ((T *)a.ke)[(size_t)(t0 + i) * 144 + 36u * cb + o] = (T)s_col[i * EM_STRIDE + o];
        }
        __syncthreads();
    }
    if (MODEL == EBBX_NH && in && !ok) atomicAdd(a.n_inv + (a.tmesh ? a.tmesh[t] : 0), 1ull);
}

// blocks[q][e] = sum over the edge's (tet, a, b) entries, in tet order, of ke block q
template <class T>
__global__ __launch_bounds__(256) void k_edge_gather(const T *ke, const int32_t *gptr, const uint32_t *gent,
                                                     uint32_t ne, T *blocks) {
    // XCD x sums one contiguous range of edges (tails in mesh order), so the records of a tet,
    // which its four corners' edges all read, come into one L2 rather than up to four
    const uint32_t e = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (e >= ne) return;
    double s[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) s[q] = 0.0;
    const int32_t j0 = gptr[e], j1 = gptr[e + 1];
    for (int32_t j = j0; j < j1; ++j) {
        const uint32_t c = gent[j];   // 16 t + 4 a + b: block (a, b) of tet t
        const T *blk = ke + (size_t)(c >> 4) * 144 + (4u * (c & 3u) + ((c >> 2) & 3u)) * 9;
#pragma unroll
        for (int q = 0; q < 9; ++q) s[q] += (double)blk[q];
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) blocks[(size_t)q * ne + e] = (T)s[q];
}


// ---- blocks straight from the element records, in LDS ------------------------------------------

// A tet's 3x3 corner block (a, b) is a short sum of products of vectors at its corners.  With
// dF = e_j (x) grad N_b in the models' dP (tetmath.h), and everything scaled by -V0:
//   neo-Hookean, c_a = F^-T grad N_a:
//     block[i][j] = s_ab d_ij + p c_b[i] c_a[j] + q c_a[i] c_b[j],
//     s_ab = mu grad N_a . grad N_b, p = mu - lam ln J, q = lam;
//   StVK, c_a = F grad N_a:
//     block[i][j] = s_ab d_ij + m_ab (F F^T)[i][j] + p c_b[i] c_a[j] + q c_a[i] c_b[j],
//     s_ab = grad N_a . S grad N_b, m_ab = mu grad N_a . grad N_b, p = mu, q = lam.
// The record holds c (4 x 3), s (10 of the symmetric 4 x 4), p and q, and for StVK m (10) and
// F F^T (6), all FP64; an odd number of 8-byte entries, so that neighbouring records start in
// different LDS banks.
template <int MODEL> struct Rec;
template <> struct Rec<EBBX_NH> {
    static constexpr int S = 12, P = 22, Q = 23, M = 0, FF = 0, N = 25;
};
template <> struct Rec<EBBX_STVK> {
    static constexpr int S = 12, P = 22, Q = 23, M = 24, FF = 34, N = 41;
};

// place of (a, b) among the 10 entries of a symmetric 4 x 4: the diagonal first, then (0, 1),
// (0, 2), (0, 3), (1, 2), (1, 3), (2, 3); the same from a table of 4-bit places
constexpr int sym4_at(int a, int b) {
    return a == b ? a : 4 + (a < b ? a * (7 - a) / 2 + b - a - 1 : b * (7 - b) / 2 + a - b - 1);
}
__device__ __forceinline__ uint32_t sym4(uint32_t a, uint32_t b) {
    return (uint32_t)(0x3986927587146540ull >> (16u * a + 4u * b)) & 15u;
}
// and of (i, j) among the 6 of a symmetric 3 x 3
__host__ __device__ constexpr int sym3(int i, int j) { return i <= j ? i * (5 - i) / 2 + j : j * (5 - j) / 2 + i; }

constexpr int AB_THREADS = 192;         // k_asm_block: AB_OFF threads on off-diagonal blocks, the others on diagonal ones
constexpr int AB_OFF = 128;
constexpr int TB_THREADS = 256;         // table construction
constexpr int AB_MAXINC = 4096;          // incidences of one workgroup's vertices (table construction)
constexpr size_t AB_LDS = 80 * 1024;     // most LDS of one workgroup: two workgroups per CU
// Fewest vertices of a workgroup: every workgroup reserves the LDS of the fullest, so one vertex of many
// tets takes the whole mesh to fewer vertices in fewer workgroups per CU, and few vertices share few
// evaluations.  384k tets and one such vertex, at two workgroups per CU, against the path through memory:
// 8 vertices 142 against 402 us, 4 214 to 220 against 373 to 402 (FP32 elements 282 to 313), 2 368 to 370
// against 373 to 402 (282 to 313), 1 698 to 708 against 373 to 418.
constexpr int32_t AB_MINVB = 4;

// LDS of a workgroup with at most `tets` records and the entries of `inc` incidences (4 each)
size_t asm_lds(int32_t model, int64_t tets, int64_t inc) {
    return (size_t)(model == EBBX_NH ? Rec<EBBX_NH>::N : Rec<EBBX_STVK>::N) * (size_t)tets * sizeof(double) +
           (size_t)(4 * inc) * sizeof(uint16_t);
}

struct AsmBlockArgs {
    AsmArgs m;
    uint32_t nv, ne, vb, most;           // vb: owned vertices per workgroup, most: tets of the largest
    const int32_t *row, *gptr;           // edges of vertex i: [row[i], row[i+1]); entries of edge e: [gptr[e], gptr[e+1])
    const uint16_t *ent;                 // 16 (tet's place in the workgroup's list) + 4 a + b
    const int32_t *tptr, *tets;          // workgroup's tets, ascending
    const int4 *keys;                    // their corners
    const int32_t *diag;                 // vertex's own edge (i, i), -1 if it has no tet
    void *blocks;
};

template <class T, int MODEL>
__device__ __forceinline__ bool tet_record(const AsmArgs &a, uint32_t t, int4 key, double *s) {
    using R = Rec<MODEL>;
    double b[9], G[9], gb[4][3];
#pragma unroll
    for (int k = 0; k < 9; ++k) b[k] = (double)ldc<T>(a.B[k], t);
    const double V0 = tet_V0(b);
    const double mu = a.mu_t ? (double)ldc<T>(a.mu_t, t) : a.mu;
    const double lam = a.lam_t ? (double)ldc<T>(a.lam_t, t) : a.lam;
    {
        const uint32_t v[4] = {(uint32_t)key.x, (uint32_t)key.y, (uint32_t)key.z, (uint32_t)key.w};
        double qd[4][3];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int k = 0; k < 3; ++k) qd[c][k] = ldc<double>(a.d[k], v[c]);
        grad_from(qd, b, G);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        gb[1][j] = b[j];
        gb[2][j] = b[3 + j];
        gb[3][j] = b[6 + j];
        gb[0][j] = -(b[j] + b[3 + j] + b[6 + j]);
    }
    bool ok = true;
    if (MODEL == EBBX_NH) {
        const double jm1 = jm1_of(G), J = 1.0 + jm1, iJ = t_rcp(J), lnJ = t_log1p(jm1);
        double C[9];
        cof_IpG(G, C);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                s[3 * c + i] = iJ * (C[3 * i] * gb[c][0] + C[3 * i + 1] * gb[c][1] + C[3 * i + 2] * gb[c][2]);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = x; y < 4; ++y)
                s[R::S + sym4_at(x, y)] =
                    -V0 * mu * (gb[x][0] * gb[y][0] + gb[x][1] * gb[y][1] + gb[x][2] * gb[y][2]);
        s[R::P] = -V0 * (mu - lam * lnJ);
        s[R::Q] = -V0 * lam;
        ok = J > 0.0;
    } else {
        double S[9];
        stvk_S(mu, lam, G, -V0, S);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                s[3 * c + i] =
                    gb[c][i] + (G[3 * i] * gb[c][0] + G[3 * i + 1] * gb[c][1] + G[3 * i + 2] * gb[c][2]);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            double Sx[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) Sx[i] = S[3 * i] * gb[x][0] + S[3 * i + 1] * gb[x][1] + S[3 * i + 2] * gb[x][2];
#pragma unroll
            for (int y = x; y < 4; ++y) {
                s[R::S + sym4_at(x, y)] = Sx[0] * gb[y][0] + Sx[1] * gb[y][1] + Sx[2] * gb[y][2];
                s[R::M + sym4_at(x, y)] =
                    -V0 * mu * (gb[x][0] * gb[y][0] + gb[x][1] * gb[y][1] + gb[x][2] * gb[y][2]);
            }
        }
        double F[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) F[k] = G[k] + (k % 4 == 0 ? 1.0 : 0.0);
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i; j < 3; ++j)
                s[R::FF + sym3(i, j)] = F[3 * i] * F[3 * j] + F[3 * i + 1] * F[3 * j + 1] + F[3 * i + 2] * F[3 * j + 2];
        s[R::P] = -V0 * mu;
        s[R::Q] = -V0 * lam;
    }
    return ok;
}

// Bound by FP64 issue and LDS reads at the two to five workgroups per CU that the records leave
// LDS for; the blocks' write alone takes 27 us where the kernel takes 178 to 283.  Each tet is
// evaluated by every workgroup that owns one of its vertices, about three times on these meshes.
// Vertices per workgroup, 890k Morton-ordered tets, FP64: neo-Hookean 249 / 178 / 205 us and StVK
// 459 / 302 / 283 us for 16 / 8 / 4: fewer evaluations against more workgroups in flight, and
// StVK's records are the larger.  The records alone take 85 (neo-Hookean) and 125 us (StVK) of
// that.  128 and 256 threads measured 291 and 278 us (StVK), 200 and 176 us (neo-Hookean).  The two
// kernels above, through 1 GB of per-tet matrices, took 777 us (StVK).
template <class T, int MODEL>
__global__ __launch_bounds__(AB_THREADS) void k_asm_block(AsmBlockArgs a) {
    extern __shared__ double s_rec[];
    using R = Rec<MODEL>;
    const uint32_t tid = threadIdx.x;
    uint16_t *s_ent = (uint16_t *)(s_rec + R::N * a.most);
    const uint32_t wg = xcd_block(blockIdx.x, gridDim.x);
    const uint32_t v0 = wg * a.vb, v1 = min(v0 + a.vb, a.nv);
    const int32_t t0 = a.tptr[wg], nt = a.tptr[wg + 1] - t0;
    const uint32_t e0 = (uint32_t)a.row[v0], e1 = (uint32_t)a.row[v1];
    const int32_t g0 = a.gptr[e0], g1 = a.gptr[e1];
    // AB_OFF threads sum off-diagonal blocks, one edge each, the others diagonal blocks, one of the
    // six entries each; the first one's place is loaded ahead of the records
    const bool off = tid < AB_OFF;
    const uint32_t lt = off ? tid : tid - AB_OFF;
    int32_t e = -1, j0 = 0, j1 = 0;
    if (off) {
        if (e0 + lt < e1) e = (int32_t)(e0 + lt);
    } else if (lt < 6 * (v1 - v0)) {
        e = a.diag[v0 + lt / 6];
    }
    if (e >= 0) {
        j0 = a.gptr[e];
        j1 = a.gptr[e + 1];
    }
    for (int32_t j = (int32_t)tid; j < g1 - g0; j += AB_THREADS) s_ent[j] = a.ent[g0 + j];
    for (int32_t i = (int32_t)tid; i < nt; i += AB_THREADS) {
        const int4 key = a.keys[t0 + i];
        const uint32_t t = (uint32_t)a.tets[t0 + i];
        const bool ok = tet_record<T, MODEL>(a.m, t, key, s_rec + R::N * i);
        // an inverted tet is counted once, by the workgroup that owns corner 0
        if (MODEL == EBBX_NH && !ok && (uint32_t)key.x >= v0 && (uint32_t)key.x < v1)
            atomicAdd(a.m.n_inv + (a.m.tmesh ? a.m.tmesh[t] : 0), 1ull);
    }
    __syncthreads();
    T *out = (T *)a.blocks;
    if (off) {
        for (uint32_t at = e0 + lt; at < e1; at += AB_OFF) {
            if (at != e0 + lt) {
                j0 = a.gptr[at];
                j1 = a.gptr[at + 1];
            }
            const uint32_t first = s_ent[j0 - g0];
            if (((first >> 2) & 3u) == (first & 3u)) continue;   // a diagonal block
            double acc[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) acc[k] = 0.0;
#pragma unroll 2
            for (int32_t j = j0 - g0; j < j1 - g0; ++j) {
                const uint32_t c = s_ent[j], ca = (c >> 2) & 3u, cb = c & 3u, ab = sym4(ca, cb);
                const double *r = s_rec + R::N * (c >> 4);
                const double p = r[R::P], q = r[R::Q], sab = r[R::S + ab];
                const double mab = MODEL == EBBX_STVK ? r[R::M + ab] : 0.0;
                double x[3], y[3], u[3], w[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    x[i] = r[3 * ca + i];
                    y[i] = r[3 * cb + i];
                    u[i] = p * y[i];
                    w[i] = q * x[i];
                }
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        // the tet's block entry, formed before it joins the sum (the sum is rounded
                        // once per tet); rounded to the element precision, summed in FP64
                        double v = 0.0;
                        if (i == k) v += sab;
                        if (MODEL == EBBX_STVK) v += mab * r[R::FF + sym3(i, k)];
                        v += u[i] * x[k];
                        v += w[i] * y[k];
                        acc[3 * i + k] += (double)(T)v;
                    }
            }
#pragma unroll
            for (int k = 0; k < 9; ++k) out[(size_t)k * a.ne + at] = (T)acc[k];
        }
    } else {
        for (uint32_t w = lt; w < 6 * (v1 - v0); w += AB_THREADS - AB_OFF) {
            if (w != lt) {
                e = a.diag[v0 + w / 6];
                if (e >= 0) {
                    j0 = a.gptr[e];
                    j1 = a.gptr[e + 1];
                }
            }
            if (e < 0) continue;   // a vertex with no tet
            const uint32_t kf = w % 6u, i = kf < 3 ? 0u : kf < 5 ? 1u : 2u, l = kf < 3 ? kf : kf < 5 ? kf - 2u : 2u;
            const uint32_t f = R::FF + kf;
            double acc = 0.0;
#pragma unroll 4
            for (int32_t j = j0 - g0; j < j1 - g0; ++j) {
                const uint32_t c = s_ent[j], ca = c & 3u;
                const double *r = s_rec + R::N * (c >> 4);
                double v = 0.0;
                if (i == l) v += r[R::S + ca];
                if (MODEL == EBBX_STVK) v += r[R::M + ca] * r[f];
                v += (r[R::P] + r[R::Q]) * r[3 * ca + i] * r[3 * ca + l];
                acc += (double)(T)v;
            }
            out[(size_t)(3 * i + l) * a.ne + e] = (T)acc;
            if (i != l) out[(size_t)(3 * l + i) * a.ne + e] = (T)acc;
        }
    }
}

template <class T> struct BsrArgs {
    const int32_t *row, *col;
    const T *k[9];
    const double *u[3];
    double *y[3];
    uint32_t nv;
    int accumulate;
};

template <class T>
__global__ __launch_bounds__(256) void k_bsr_spmv(BsrArgs<T> a) {
    // XCD x takes one contiguous range of rows, whose neighbours' u it shares in its L2
    const uint32_t g = (xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) / SPMV_LANES;
    const uint32_t lane = threadIdx.x % SPMV_LANES;
    const uint32_t i = g < a.nv ? g : a.nv - 1;   // whole groups stay in the shuffles
    const int32_t e0 = a.row[i], e1 = g < a.nv ? a.row[i + 1] : e0;
    double y0 = 0.0, y1 = 0.0, y2 = 0.0;
    for (int32_t e = e0 + (int32_t)lane; e < e1; e += SPMV_LANES) {
        const uint32_t j = (uint32_t)a.col[e];
        const double u0 = a.u[0][j], u1 = a.u[1][j], u2 = a.u[2][j];
        y0 += (double)a.k[0][e] * u0 + (double)a.k[1][e] * u1 + (double)a.k[2][e] * u2;
        y1 += (double)a.k[3][e] * u0 + (double)a.k[4][e] * u1 + (double)a.k[5][e] * u2;
        y2 += (double)a.k[6][e] * u0 + (double)a.k[7][e] * u1 + (double)a.k[8][e] * u2;
    }
    y0 = lanes_sum<SPMV_LANES>(y0);
    y1 = lanes_sum<SPMV_LANES>(y1);
    y2 = lanes_sum<SPMV_LANES>(y2);
    if (lane == 0 && g < a.nv) {
        if (a.accumulate) {
            y0 += a.y[0][i];
            y1 += a.y[1][i];
            y2 += a.y[2][i];
        }
        a.y[0][i] = y0;
        a.y[1][i] = y1;
        a.y[2][i] = y2;
    }
}

unsigned grid_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// ---- tables, on the device ---------------------------------------------------------------------

namespace {

// Entry 16 t + 4 a + b is corner block (a, b) of tet t; its key orders the edges (tail, head).
__global__ void k_edge_keys(const int32_t *keys, int64_t nt, int shift, uint64_t *key, uint32_t *val) {
    const int64_t n = 16 * nt;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t t = i >> 4;
        const int a = (int)(i >> 2) & 3, b = (int)i & 3;
        key[i] = ((uint64_t)(uint32_t)keys[a * nt + t] << shift) | (uint32_t)keys[b * nt + t];
        val[i] = (uint32_t)i;
    }
}

__global__ void k_edge_heads(const uint64_t *key, int64_t n, int64_t *flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += (int64_t)gridDim.x * blockDim.x)
        flag[i] = i < n && (i == 0 || key[i] != key[i - 1]);
}

// at[i]: edges before entry i.  The first entry of an edge writes its head and its entries' start.
__global__ void k_edge_fill(const uint64_t *key, const int64_t *at, int64_t n, int shift, int32_t *col, int32_t *gptr) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (at[i + 1] != at[i]) {
            col[at[i]] = (int32_t)(key[i] & ((1ull << shift) - 1ull));
            gptr[at[i]] = (int32_t)i;
        }
        if (i == n - 1) gptr[at[n]] = (int32_t)n;
    }
}

// row[v]: edges whose tail is below v.
__global__ void k_edge_rows(const uint64_t *key, const int64_t *at, int64_t n, int64_t nv, int shift, int32_t *row) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v <= nv; v += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)(key[mid] >> shift) < v) lo = mid + 1;
            else hi = mid;
        }
        row[v] = (int32_t)at[lo];
    }
}

// The distinct tets of vertices [v0, v1), sorted ascending into s[0, *nu); false if they have
// more than AB_MAXINC incidences.
__device__ __forceinline__ bool tets_of(const int64_t *rp, const int32_t *inc, int64_t v0, int64_t v1, uint32_t *s,
                                        int32_t *sw, int32_t *nu) {
    const int64_t p0 = rp[v0], ninc = rp[v1] - p0;
    if (ninc > AB_MAXINC) return false;
    int32_t n = 64;
    while (n < ninc) n <<= 1;
    for (int32_t i = threadIdx.x; i < n; i += TB_THREADS) s[i] = i < ninc ? (uint32_t)inc[p0 + i] >> 2 : ~0u;
    lds_sort<TB_THREADS>(s, n);
    *nu = lds_distinct<TB_THREADS, AB_MAXINC>(s, n, sw);
    return true;
}

// Tets per workgroup of vb vertices into count[wg], the most tets and incidences of any into most[0], most[1].
__global__ __launch_bounds__(TB_THREADS) void k_asm_count(const int64_t *rp, const int32_t *inc, int64_t nv, int32_t vb,
                                                          int64_t *count, Tally *most) {
    __shared__ uint32_t s[AB_MAXINC];
    __shared__ int32_t sw[TB_THREADS / 64];
    const int64_t v0 = (int64_t)blockIdx.x * vb, v1 = v0 + vb < nv ? v0 + vb : nv;
    int32_t nu = 0;
    const bool fits = tets_of(rp, inc, v0, v1, s, sw, &nu);   // uniform over the workgroup
    if (threadIdx.x == 0) {
        count[blockIdx.x] = fits ? nu : 0;
        most[0].add(fits ? nu : 1 << 30, 0);
        most[1].add(fits ? rp[v1] - rp[v0] : 0, 0);
    }
}

// The workgroups' tet lists, and each entry of their edges as a place in its workgroup's list.
__global__ __launch_bounds__(TB_THREADS) void k_asm_fill(const int64_t *rp, const int32_t *inc, int64_t nv, int32_t vb,
                                                         const int64_t *base, const int32_t *row, const int32_t *gptr,
                                                         const uint32_t *gent, const int32_t *keys, int64_t nt,
                                                         int32_t *tptr, int32_t *tets, int4 *tkeys, int32_t *diag,
                                                         uint16_t *ent) {
    __shared__ uint32_t s[AB_MAXINC];
    __shared__ int32_t sw[TB_THREADS / 64];
    const int64_t v0 = (int64_t)blockIdx.x * vb, v1 = v0 + vb < nv ? v0 + vb : nv;
    int32_t nu = 0;
    if (!tets_of(rp, inc, v0, v1, s, sw, &nu)) return;
    const int64_t t0 = base[blockIdx.x];
    if (threadIdx.x == 0) {
        tptr[blockIdx.x] = (int32_t)t0;
        if (v1 == nv) tptr[blockIdx.x + 1] = (int32_t)(t0 + nu);
    }
    for (int32_t i = threadIdx.x; i < nu; i += TB_THREADS) {
        const int64_t t = s[i];
        tets[t0 + i] = (int32_t)t;
        tkeys[t0 + i] = make_int4(keys[t], keys[nt + t], keys[2 * nt + t], keys[3 * nt + t]);
    }
    for (int64_t v = v0 + threadIdx.x; v < v1; v += TB_THREADS) {
        int32_t own = -1;   // the edge whose entries have equal corners
        for (int32_t e = row[v]; e < row[v + 1]; ++e) {
            const uint32_t c = gent[gptr[e]];
            if (((c >> 2) & 3u) == (c & 3u)) own = e;
        }
        diag[v] = own;
    }
    for (int32_t p = gptr[row[v0]] + (int32_t)threadIdx.x; p < gptr[row[v1]]; p += TB_THREADS) {
        const uint32_t c = gent[p], t = c >> 4;
        int32_t lo = 0, hi = nu - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (s[mid] < t) lo = mid + 1;
            else hi = mid;
        }
        ent[p] = (uint16_t)(((uint32_t)lo << 4) | (c & 15u));
    }
}

}  // namespace

// The edges relation and the entry lists from the grouping's keys: the 16 nt corner blocks sorted
// by (tail, head), stably, so that an edge's entries ascend in (tet, corner, corner); then the
// workgroups' tables of k_asm_block: 8 vertices per workgroup (neo-Hookean) or 4 (StVK), measured
// at the kernel, or 4 where the LDS does not take 8.  Once per domain, synchronous.
void build_edges(ebbx_fem_s *F, hipStream_t s) {
    if (F->n_edges >= 0) return;
    const int64_t nt = F->nt, nv = F->nv, n = 16 * nt;
    if (nt >= (int64_t(1) << 28)) fail(EBBX_E_ARG, "assembled stiffness: at most 2^28 tets");
    int shift = 1;
    while ((int64_t(1) << shift) < nv) ++shift;
    auto room = [](int64_t count, size_t each) { return std::max<size_t>((size_t)count * each, 16); };
    auto grid = [](int64_t m) { return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((m + 255) / 256, 65536))); };
    F->e_row.reset(room(nv + 1, 4), s);
    F->e_gent.reset(room(n, 4), s);
    int64_t ne = 0;
    if (nt > 0) {
        DevBuf key(room(n, 8), s), at(room(n + 1, 8), s);
        hipLaunchKernelGGL(k_edge_keys, grid(n), dim3(256), 0, s, F->keys, nt, shift, key.as<uint64_t>(),
                           F->e_gent.as<uint32_t>());
        HIPCHK(hipGetLastError());
        radix_sort_pairs_u64(key.as<uint64_t>(), F->e_gent.as<uint32_t>(), n, 2 * shift, s);
        hipLaunchKernelGGL(k_edge_heads, grid(n + 1), dim3(256), 0, s, key.as<uint64_t>(), n, at.as<int64_t>());
        HIPCHK(hipGetLastError());
        exclusive_scan_i64(at.as<int64_t>(), n + 1, s);
        HIPCHK(hipMemcpyAsync(&ne, at.as<int64_t>() + n, sizeof ne, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        F->e_col.reset(room(ne, 4), s);
        F->e_gptr.reset(room(ne + 1, 4), s);
        hipLaunchKernelGGL(k_edge_fill, grid(n), dim3(256), 0, s, key.as<uint64_t>(), at.as<int64_t>(), n, shift,
                           F->e_col.as<int32_t>(), F->e_gptr.as<int32_t>());
        HIPCHK(hipGetLastError());
        hipLaunchKernelGGL(k_edge_rows, grid(nv + 1), dim3(256), 0, s, key.as<uint64_t>(), at.as<int64_t>(), n, nv,
                           shift, F->e_row.as<int32_t>());
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(s));
    } else {
        F->e_col.reset(room(0, 4), s);
        F->e_gptr.reset(room(1, 4), s);
        HIPCHK(hipMemsetAsync(F->e_row.get(), 0, F->e_row.bytes(), s));
        HIPCHK(hipMemsetAsync(F->e_gptr.get(), 0, F->e_gptr.bytes(), s));
    }
    F->a_vb = 0;
    const int64_t *rp = F->group->row_ptr.as<int64_t>();
    const int32_t *inc = F->group->inc.as<int32_t>();
    for (int32_t vb = F->model == EBBX_NH ? 8 : 4; vb >= AB_MINVB && ne > 0 && n < (int64_t(1) << 31) && !F->a_vb; vb /= 2) {
        const int64_t nwg = (nv + vb - 1) / vb;
        DevBuf base(room(nwg + 1, 8), s), mx(2 * sizeof(Tally), s);
        HIPCHK(hipMemsetAsync(mx.get(), 0, mx.bytes(), s));
        HIPCHK(hipMemsetAsync(base.get(), 0, base.bytes(), s));
        hipLaunchKernelGGL(k_asm_count, dim3((unsigned)nwg), dim3(TB_THREADS), 0, s, rp, inc, nv, vb,
                           base.as<int64_t>(), mx.as<Tally>());
        HIPCHK(hipGetLastError());
        exclusive_scan_i64(base.as<int64_t>(), nwg + 1, s);
        Tally found[2] = {};
        int64_t total = 0;
        HIPCHK(hipMemcpyAsync(found, mx.get(), sizeof found, hipMemcpyDeviceToHost, s));
        HIPCHK(hipMemcpyAsync(&total, base.as<int64_t>() + nwg, sizeof total, hipMemcpyDeviceToHost, s));
        HIPCHK(hipStreamSynchronize(s));
        const int64_t most[2] = {found[0].largest(), found[1].largest()};
        if (asm_lds(F->model, most[0], most[1]) > AB_LDS || total >= (int64_t(1) << 31)) continue;
        F->a_tptr.reset(room(nwg + 1, 4), s);
        F->a_tets.reset(room(total, 4), s);
        F->a_keys.reset(room(total, 16), s);
        F->a_diag.reset(room(nv, 4), s);
        F->a_ent.reset(room(n, 2), s);
        hipLaunchKernelGGL(k_asm_fill, dim3((unsigned)nwg), dim3(TB_THREADS), 0, s, rp, inc, nv, vb,
                           base.as<int64_t>(), F->e_row.as<int32_t>(), F->e_gptr.as<int32_t>(),
                           F->e_gent.as<uint32_t>(), F->keys, nt, F->a_tptr.as<int32_t>(),
                           F->a_tets.as<int32_t>(), F->a_keys.as<int4>(), F->a_diag.as<int32_t>(),
                           F->a_ent.as<uint16_t>());
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(s));
        F->e_gent.release();
        F->a_most = (int32_t)most[0];
        F->a_inc = (int32_t)most[1];
        F->a_vb = vb;
    }
    HIPCHK(hipStreamSynchronize(s));
    F->n_edges = ne;
}

namespace {

template <class T> void launch_assemble(ebbx_fem_s *F, const double *d, hipStream_t s) {
    const int64_t nt = F->nt, nv = F->nv, ne = F->n_edges;
    const size_t es = sizeof(T);
    if (ne == 0) return;
    AsmArgs a{};
    a.nt = (uint32_t)nt;
    for (int c = 0; c < 4; ++c) a.key[c] = F->keys + (size_t)c * nt;
    for (int k = 0; k < 9; ++k) a.B[k] = (const char *)F->B.get() + (size_t)k * nt * es;
    if (F->per_tet) {
        a.mu_t = F->mat.get();
        a.lam_t = (const char *)F->mat.get() + (size_t)nt * es;
    }
    a.mu = F->mu;
    a.lam = F->lam;
    for (int k = 0; k < 3; ++k) a.d[k] = d + (size_t)k * nv;
    a.ke = F->e_ke.get();
    a.n_inv = F->status.as<unsigned long long>();
    a.tmesh = F->tmesh;
    if (F->a_vb) {
        AsmBlockArgs b{};
        b.m = a;
        b.nv = (uint32_t)nv;
        b.ne = (uint32_t)ne;
        b.vb = (uint32_t)F->a_vb;
        b.most = (uint32_t)F->a_most;
        b.row = F->e_row.as<int32_t>();
        b.gptr = F->e_gptr.as<int32_t>();
        b.ent = F->a_ent.as<uint16_t>();
        b.tptr = F->a_tptr.as<int32_t>();
        b.tets = F->a_tets.as<int32_t>();
        b.keys = F->a_keys.as<int4>();
        b.diag = F->a_diag.as<int32_t>();
        b.blocks = F->e_blocks.get();
        const dim3 g(grid_of(nv, F->a_vb));
        if (F->model == EBBX_STVK)
            hipLaunchKernelGGL((k_asm_block<T, EBBX_STVK>), g, dim3(AB_THREADS),
                               asm_lds(F->model, F->a_most, F->a_inc), s, b);
        else
            hipLaunchKernelGGL((k_asm_block<T, EBBX_NH>), g, dim3(AB_THREADS),
                               asm_lds(F->model, F->a_most, F->a_inc), s, b);
        HIPCHK(hipGetLastError());
        return;
    }
    if (F->model == EBBX_STVK)
        hipLaunchKernelGGL((k_elem_matrix<T, EBBX_STVK>), dim3(grid_of(nt, EM_THREADS)), dim3(EM_THREADS), 0, s, a);
    else
        hipLaunchKernelGGL((k_elem_matrix<T, EBBX_NH>), dim3(grid_of(nt, EM_THREADS)), dim3(EM_THREADS), 0, s, a);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL((k_edge_gather<T>), dim3(grid_of(ne, 256)), dim3(256), 0, s, (const T *)F->e_ke.get(),
                       F->e_gptr.as<int32_t>(), F->e_gent.as<uint32_t>(), (uint32_t)ne, F->e_blocks.as<T>());
    HIPCHK(hipGetLastError());
}

template <class T> void launch_spmv(ebbx_fem_s *F, const double *u, double *y, int accumulate, hipStream_t s) {
    const int64_t nv = F->nv, ne = F->n_edges;
    BsrArgs<T> a{};
    a.row = F->e_row.as<int32_t>();
    a.col = F->e_col.as<int32_t>();
    for (int q = 0; q < 9; ++q) a.k[q] = F->e_blocks.as<T>() + (size_t)q * ne;
    for (int k = 0; k < 3; ++k) {
        a.u[k] = u + (size_t)k * nv;
        a.y[k] = y + (size_t)k * nv;
    }
    a.nv = (uint32_t)nv;
    a.accumulate = accumulate;
    hipLaunchKernelGGL((k_bsr_spmv<T>), dim3(grid_of(nv * SPMV_LANES, 256)), dim3(256), 0, s, a);
    HIPCHK(hipGetLastError());
}

}  // namespace

void assemble_stiffness(ebbx_fem_s *F, const double *d, hipStream_t s) {
    if (F->nt >= (int64_t(1) << 27)) fail(EBBX_E_ARG, "assembled stiffness: at most 2^27 tets");   // 32-bit entry lists
    build_edges(F, s);
    // the blocks, and where the LDS does not take the records the per-tet scratch, on the first assembly
    const size_t blk_bytes = std::max<size_t>((size_t)9 * F->n_edges * F->esize, 8);
    const size_t ke_bytes = F->a_vb ? 0 : std::max<size_t>((size_t)F->nt * 144 * F->esize, 8);
    if (F->e_blocks.bytes() != blk_bytes) F->e_blocks.reset(blk_bytes, s);
    if (F->e_ke.bytes() != ke_bytes) F->e_ke.reset(ke_bytes, s);
    if (F->prec == EBBX_F32) launch_assemble<float>(F, d, s);
    else launch_assemble<double>(F, d, s);
    F->assembled = true;
}

void assembled_spmv(ebbx_fem_s *F, const double *u, double *y, int accumulate, hipStream_t s) {
    if (!F->assembled) fail(EBBX_E_STATE, "no assembled stiffness: call ebbx_fem_assemble first");
    if (F->nv == 0) return;
    if (F->prec == EBBX_F32) launch_spmv<float>(F, u, y, accumulate, s);
    else launch_spmv<double>(F, u, y, accumulate, s);
}

// Copies of the edges relation and the blocks (FP64) for inspection.
namespace {
template <class T>
__global__ void k_blocks_f64(const T *src, int64_t n, double *dst) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (double)src[i];
}
}  // namespace

void edges_copy(ebbx_fem_s *F, int32_t *row, int32_t *col, double *blocks, hipStream_t s) {
    build_edges(F, s);
    const int64_t ne = F->n_edges, nv = F->nv;
    if (row) HIPCHK(hipMemcpyAsync(row, F->e_row.get(), (size_t)(nv + 1) * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    if (col && ne > 0) HIPCHK(hipMemcpyAsync(col, F->e_col.get(), (size_t)ne * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
    if (blocks && ne > 0) {
        if (!F->assembled) fail(EBBX_E_STATE, "no assembled stiffness: call ebbx_fem_assemble first");
        const unsigned g = (unsigned)std::min<int64_t>(grid_of(9 * ne, 256), 1 << 16);
        if (F->prec == EBBX_F32)
            hipLaunchKernelGGL((k_blocks_f64<float>), dim3(g), dim3(256), 0, s, F->e_blocks.as<float>(), 9 * ne, blocks);
        else
            hipLaunchKernelGGL((k_blocks_f64<double>), dim3(g), dim3(256), 0, s, F->e_blocks.as<double>(), 9 * ne,
                               blocks);
        HIPCHK(hipGetLastError());
    }
}

}  // namespace ebbx

// ---- C ABI --------------------------------------------------------------------------

using namespace ebbx;

extern "C" ebbx_status ebbx_fem_assemble(ebbx_fem fem, const double *d, ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *F = check_fem(fem);
    if (F->nv > 0 && !d) fail(EBBX_E_ARG, "d is NULL");
    assemble_stiffness(F, d, (hipStream_t)stream);
    EBBX_API_END
}

extern "C" ebbx_status ebbx_fem_spmv(ebbx_fem fem, const double *u, double *y, int32_t accumulate,
                                     ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *F = check_fem(fem);
    const int64_t nv = F->nv;
    if (nv > 0 && (!u || !y)) fail(EBBX_E_ARG, "u or y is NULL");
    if (nv > 0 && overlap(u, y, (size_t)(3 * nv) * sizeof(double))) fail(EBBX_E_PHASE, "y aliases u");
    assembled_spmv(F, u, y, accumulate, (hipStream_t)stream);
    EBBX_API_END
}

extern "C" ebbx_status ebbx_fem_edge_count(ebbx_fem fem, int64_t *n_edges) {
    EBBX_API_BEGIN
    auto *F = check_fem(fem);
    if (!n_edges) fail(EBBX_E_ARG, "n_edges is NULL");
    build_edges(F, nullptr);
    *n_edges = F->n_edges;
    EBBX_API_END
}

extern "C" ebbx_status ebbx_fem_edges_get(ebbx_fem fem, int32_t *row_ptr, int32_t *col, double *blocks,
                                          ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *F = check_fem(fem);
    edges_copy(F, row_ptr, col, blocks, (hipStream_t)stream);
    EBBX_API_END
}
