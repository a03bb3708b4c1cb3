// springs.hip -- the spring-mass workload of the paper's introductory example
// (a spring on every directed edge of a tet mesh; Ebb by example), on the same
// relational runtime as the FEM domain.
//
//  - rest lengths: one pass over the edges (the example's per-edge kernel);
//  - forces: each vertex loops over the edges leaving it (the grouping of the
//    edges by their tail key-field) and reduces (+=) the spring forces into its
//    force field, one division per edge and K applied to the sum.  Where
//    neighbouring vertices share neighbours, a workgroup stages the positions
//    that its 128 vertices need in LDS once (k_spring_block); elsewhere four
//    lanes per vertex gather them from memory, two edges' loads in flight per
//    lane (k_spring_forces, k_spring_step);
//  - apply: the exclusive per-vertex update (integrate, clear the force);
//  - kinetic energy: a global += as a fixed-order two-pass sum;
//  - run: nsteps replayed from a captured HIP graph of 32 steps, each step one
//    fused kernel (forces and update of a vertex together, positions ping-ponged
//    through a second buffer so that no vertex reads an advanced neighbour).
// Springs restore: edge (v -> h) adds K (dq - L dq/|dq|), dq = q_h - q_v.
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <set>
#include <vector>

#include "fem.h"
#include "sort.h"
#include "wave.h"

struct ebbx_springs_s {
    const ebbx_relation_s *edges = nullptr, *verts = nullptr;   // the relations the row copies follow
    int64_t nv = 0, ne = 0;
    double K = 0.0;
    ebbx::DevBuf row;    // int32 (nv + 1): vertex v's edges are [row[v], row[v+1]); behind them, per workgroup of
                         // k_spring_block, the place of its first vertex in its list
    ebbx::DevBuf head;   // int32 (ne): head vertex of each edge, in row order
    ebbx::DevBuf rest;   // FP64 (ne): rest length of each edge, in row order
    ebbx::DevBuf part;   // FP64 partials of the energy sum
    ebbx::DevBuf q2;     // FP64 (3 nv): the other position buffer of the fused steps of a run
    // k_spring_block (stride 0: not used), `lanes` lanes per vertex: per workgroup the sorted list of
    // the vertices it reads (-1 padded to the stride); per wave its edges, padded to the same number
    // per lane, lane-major
    int32_t stride = 0, lanes = 2;
    ebbx::DevBuf b_list, b_off, b_slot, b_rest;
    // captured steps of ebbx_springs_run
    hipGraphExec_t exec = nullptr;
    hipGraph_t graph = nullptr;
    hipStream_t cap = nullptr;
    const void *key[4] = {nullptr, nullptr, nullptr, nullptr};
    double key_dt = 0.0;
    void drop_graph() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        exec = nullptr;
        graph = nullptr;
    }
    ~ebbx_springs_s() {
        drop_graph();
        if (cap) (void)hipStreamDestroy(cap);
    }
};

namespace ebbx {

namespace {

constexpr int LANES = 4;              // lanes per vertex in the force pass (14 edges per interior vertex)
constexpr int UNROLL = 2;             // edges per lane with their loads in flight together
constexpr int RUN_CHUNK = 32;         // steps per captured graph
constexpr int EN_THREADS = 256;

std::mutex g_mu;
std::set<ebbx_springs_s *> g_springs;

}  // namespace

const char *springs_relation_user(const ebbx_relation_s *r) {
    std::lock_guard<std::mutex> lk(g_mu);
    for (const ebbx_springs_s *S : g_springs)
        if (S->edges == r || S->verts == r) return "a springs domain";
    return nullptr;
}

namespace {

ebbx_springs_s *check_springs(ebbx_springs p) {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!p || !g_springs.count(p)) fail(EBBX_E_ARG, "invalid springs handle");
    return p;
}

unsigned blocks_of(int64_t n, int per) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }

// Row-order copies of the heads and the rest lengths |X_h - X_v|.
__global__ void k_spring_setup(const int64_t *rp, const int32_t *inc, const int32_t *head_rel, const double *X,
                               int64_t nv, int32_t *row, int32_t *head, double *rest) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v > nv) return;
    row[v] = (int32_t)rp[v];
    if (v == nv) return;
    const double x0 = X[v], x1 = X[nv + v], x2 = X[2 * nv + v];
    for (int64_t p = rp[v]; p < rp[v + 1]; ++p) {
        const int32_t h = head_rel[inc[p]];
        head[p] = h;
        const double a = X[h] - x0, b = X[nv + h] - x1, c = X[2 * nv + h] - x2;
        rest[p] = sqrt(a * a + b * b + c * c);
    }
}

// len / sqrt(n2), 0 for n2 = 0 (a zero-length spring pulls with K dq), where len is finite and n2 is 0
// or in [1e-280, 1e280].  One hardware reciprocal square root (about 2^-24) serves the root and the
// quotient: two steps of Goldschmidt's coupled iteration (g to the root, h to half its reciprocal;
// Markstein 1990) and residual corrections of the root and of the quotient.  No branch, so that the
// loads of the edges after it can be issued before it.  Within one ulp (tested against exact
// arithmetic); no bit differed from len / sqrt(n2) of the library on 4M random arguments each in
// [0.5, 1.5] x [0.25, 3.25], over 9 and 17 decades and over 260 and 555 decades.
__device__ __forceinline__ double spring_scale(double len, double n2) {
    const double y = __builtin_amdgcn_rsq(n2);
    double g = n2 * y, h = 0.5 * y;   // -> sqrt(n2), 1 / (2 sqrt(n2))
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-h, g, 0.5);
    h = fma(h, r, h);
    g = fma(fma(-g, g, n2), h, g);
    const double q = len * (2.0 * h);
    const double s = fma(fma(-g, q, len), 2.0 * h, q);
    return n2 == 0.0 ? 0.0 : s;
}
__device__ __forceinline__ bool spring_in_range(double n2) { return n2 == 0.0 || (n2 >= 1e-280 && n2 <= 1e280); }
// The same for any n2 (and NaN).
__device__ __forceinline__ double spring_scale_any(double len, double n2) {
    const double n = sqrt(n2);
    return n > 0.0 ? len / n : 0.0;
}

// Sum over the edges leaving vertex v ([e0, e1) of the rows) of dq - L dq/|dq|, dq = q_h - q_v
// (K is applied once to the sum): lane `lane` of the vertex's L lanes takes edges e0 + lane,
// e0 + lane + L, ..., with the loads of U edges in flight at once; the lane sums are then
// combined by a fixed butterfly, so every lane returns the same, order-fixed total.
template <int L, int U>
__device__ __forceinline__ void spring_sum(const int32_t *head, const double *rest, const double *q, uint32_t nv,
                                           uint32_t v, int32_t e0, int32_t e1, uint32_t lane, double &f0, double &f1,
                                           double &f2) {
    const double q0 = q[v], q1 = q[nv + v], q2 = q[2 * nv + v];
    f0 = f1 = f2 = 0.0;
    for (int32_t e = e0 + (int32_t)lane; e < e1; e += U * L) {
        uint32_t h[U];
        double len[U], a[U], b[U], c[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = e + u * L < e1;
            h[u] = ok[u] ? (uint32_t)head[e + u * L] : v;
            len[u] = ok[u] ? rest[e + u * L] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = q[h[u]] - q0;
            b[u] = q[nv + h[u]] - q1;
            c[u] = q[2 * nv + h[u]] - q2;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            const double n = sqrt(a[u] * a[u] + b[u] * b[u] + c[u] * c[u]);
            const double sc = n > 0.0 ? len[u] / n : 0.0;   // a zero-length spring pulls with K dq
            f0 += fma(-sc, a[u], a[u]);
            f1 += fma(-sc, b[u], b[u]);
            f2 += fma(-sc, c[u], c[u]);
        }
    }
    f0 = lanes_sum<L>(f0);
    f1 = lanes_sum<L>(f1);
    f2 = lanes_sum<L>(f2);
}

// The exclusive update of one vertex component: a = f / m, q += qd dt + a dt^2 / 2, qd += a dt.
// Both the update pass and the fused step call it, so the two agree bit for bit.
__device__ __forceinline__ void integrate(double q, double qd, double a, double dt, double &q_new, double &qd_new) {
    q_new = q + (qd * dt + 0.5 * a * dt * dt);
    qd_new = qd + a * dt;
}

// Force pass: lanes 0..2 of each vertex's group store (or += into) the x, y, z components.
template <int L, int U>
__global__ __launch_bounds__(256) void k_spring_forces(const int32_t *row, const int32_t *head, const double *rest,
                                                       double K, const double *q, double *f, uint32_t nv,
                                                       int accumulate) {
    // XCD x takes one contiguous range of vertices (Morton-ordered), whose neighbours' positions
    // it then mostly finds in its own L2
    const uint32_t g = (xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) / L;
    const uint32_t lane = threadIdx.x % L;
    const uint32_t v = g < nv ? g : nv - 1;   // whole groups stay in the shuffles
    const int32_t e0 = row[v], e1 = g < nv ? row[v + 1] : e0;
    double f0, f1, f2;
    spring_sum<L, U>(head, rest, q, nv, v, e0, e1, lane, f0, f1, f2);
    if (g < nv && lane < 3) {
        const size_t i = (size_t)lane * nv + v;
        double fk = K * (lane == 0 ? f0 : lane == 1 ? f1 : f2);
        if (accumulate) fk += f[i];
        f[i] = fk;
    }
}

// One whole step for every vertex (forces from q, then the exclusive update) writing the new
// positions to q_out, so that no vertex reads a position already advanced.  With take_f the
// force field's contents join the spring forces and are cleared, as in the separate passes.
template <int L, int U>
__global__ __launch_bounds__(256) void k_spring_step(const int32_t *row, const int32_t *head, const double *rest,
                                                     double K, const double *mass, double dt, const double *q,
                                                     double *q_out, double *qd, double *f, int take_f, uint32_t nv) {
    // XCD x takes one contiguous range of vertices (Morton-ordered), whose neighbours' positions
    // it then mostly finds in its own L2
    const uint32_t g = (xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x) / L;
    const uint32_t lane = threadIdx.x % L;
    const uint32_t v = g < nv ? g : nv - 1;
    const int32_t e0 = row[v], e1 = g < nv ? row[v + 1] : e0;
    double f0, f1, f2;
    spring_sum<L, U>(head, rest, q, nv, v, e0, e1, lane, f0, f1, f2);
    if (g < nv && lane < 3) {
        const size_t i = (size_t)lane * nv + v;
        double fk = K * (lane == 0 ? f0 : lane == 1 ? f1 : f2);
        if (take_f) {
            fk += f[i];
            f[i] = 0.0;
        }
        integrate(q[i], qd[i], fk / mass[v], dt, q_out[i], qd[i]);
    }
}

// ---- positions staged in LDS -------------------------------------------------------------------

constexpr int SB_T = 256;                  // threads of a workgroup: 256 / L vertices, L lanes each
constexpr int SB_U = 2;                    // edges of a lane in flight together
// Lanes per vertex: four on meshes too small to fill the chip with two (8^3 cells 4.6 us per step
// with two, 3.8 with four; 32^3 5.7 and 5.0; 48^3, 118k vertices, 8.5 and 9.4).
constexpr int64_t SB_FOUR_NV = 65536;
constexpr int SB_MAX = 4096;               // edges and vertices of one workgroup (table construction)
constexpr int SB_STRIDE = 1024;            // staged vertices of one workgroup (24 KiB of LDS)

struct SpringBlocks {
    const int32_t *list, *own;   // [nwg * stride], [nwg]; the rows' offsets, nv + 1, stand before own
    const int64_t *off;          // [4 nwg + 1]: first entry of each wave, 64 per edge round
    const uint16_t *slot;        // head's place in the workgroup's list
    const double *rest;
    uint32_t stride, nv;
};

// The distinct vertices that workgroup wg's vertices and edges touch, sorted into s[0, *nu); false
// if there are more than SB_MAX of them with repeats.  The heads beyond the workgroup's own [v0, v1)
// pass through a hash table first (a vertex is the head of some 4 edges of a workgroup), so that only
// distinct ones are sorted, and the own ones go into their place among them.  With all of them sorted
// k_spring_count took 94 us in place of 59 at 64^3 cells.
__device__ __forceinline__ bool spring_list(const int32_t *row, const int32_t *head, int64_t v0, int64_t v1,
                                            uint32_t *s, int32_t *sw, int32_t *nu) {
    const int64_t e0 = row[v0], ne = row[v1] - e0;
    const int32_t own = (int32_t)(v1 - v0);
    if (ne + own > SB_MAX) return false;
    int32_t n = 64;
    while (n < ne) n <<= 1;   // a place for every head: the probing ends
    for (int32_t i = threadIdx.x; i < n; i += SB_T) s[i] = ~0u;
    __syncthreads();
    for (int32_t i0 = 0; i0 < ne; i0 += 4 * SB_T) {
        int32_t h[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t i = i0 + u * SB_T + (int32_t)threadIdx.x;
            h[u] = i < ne ? head[e0 + i] : (int32_t)v0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (h[u] >= v0 && h[u] < v1) continue;
            uint32_t at = ((uint32_t)h[u] * 2654435761u >> 16) & (uint32_t)(n - 1), was;
            while ((was = atomicCAS(s + at, ~0u, (uint32_t)h[u])) != ~0u && was != (uint32_t)h[u])
                at = (at + 1) & (uint32_t)(n - 1);
        }
    }
    __syncthreads();
    const int32_t k = lds_distinct<SB_T, SB_MAX>(s, n, sw);   // the places taken
    n = 64;
    while (n < k) n <<= 1;
    for (int32_t i = k + (int32_t)threadIdx.x; i < n; i += SB_T) s[i] = ~0u;
    lds_sort<SB_T>(s, n);
    int32_t lo = 0, hi = k;   // those below v0
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((int64_t)s[mid] < v0) lo = mid + 1;
        else hi = mid;
    }
    uint32_t up[SB_MAX / SB_T];   // the others move up; every thread reads its own before any writes
#pragma unroll
    for (int32_t u = 0; u < SB_MAX / SB_T; ++u) {
        const int32_t i = lo + u * SB_T + (int32_t)threadIdx.x;
        up[u] = i < k ? s[i] : ~0u;
    }
    __syncthreads();
#pragma unroll
    for (int32_t u = 0; u < SB_MAX / SB_T; ++u)
        if (up[u] != ~0u) s[lo + own + u * SB_T + (int32_t)threadIdx.x] = up[u];
    for (int32_t i = threadIdx.x; i < own; i += SB_T) s[lo + i] = (uint32_t)(v0 + i);
    __syncthreads();
    *nu = k + own;
    return true;
}

// A workgroup's staged vertices into *verts (2^30 if there are too many, or with a rest length that is
// not finite, for which spring_scale's quotient is not the library's); off[4 wg + w]: entries of wave w
// (its longest vertex's rounds, 64 entries each), all of them into *entries; its list, -1 padded, at
// list[SB_STRIDE wg].
template <int L>
__global__ __launch_bounds__(SB_T) void k_spring_count(const int32_t *row, const int32_t *head, const double *rest,
                                                       int64_t nv, Tally *verts, Tally *entries, int64_t *off,
                                                       int32_t *list) {
    __shared__ uint32_t s[SB_MAX];
    __shared__ int32_t sw[SB_T / 64], s_deg[4];
    constexpr int V = SB_T / L, W = 64 / L;   // vertices per workgroup and per wave
    const int64_t v0 = (int64_t)blockIdx.x * V, v1 = v0 + V < nv ? v0 + V : nv;
    if (threadIdx.x < 4) s_deg[threadIdx.x] = 0;
    int32_t nu = 0;
    bool fits = spring_list(row, head, v0, v1, s, sw, &nu);   // uniform over the workgroup
    bool finite = true;
    for (int32_t e = row[v0] + (int32_t)threadIdx.x, e1 = row[v1]; e < e1; e += SB_T) finite &= isfinite(rest[e]);
    fits = __syncthreads_and(finite) && fits && nu <= SB_STRIDE;
    const int64_t v = v0 + threadIdx.x;
    if (threadIdx.x < V && v < v1) atomicMax(&s_deg[threadIdx.x / W], row[v + 1] - row[v]);
    __syncthreads();
    auto places = [&](int w) { return fits ? (int64_t)((s_deg[w] + L - 1) / L) * 64 : 0; };
    if (threadIdx.x < 4) off[4 * (int64_t)blockIdx.x + threadIdx.x] = places(threadIdx.x);
    if (threadIdx.x == 0) {
        if (blockIdx.x + 1 == gridDim.x) off[4 * (int64_t)gridDim.x] = 0;   // scanned with the others
        verts->add(fits ? nu : 1 << 30, fits ? (unsigned long long)nu : 0);
        entries->add(0, (unsigned long long)(places(0) + places(1) + places(2) + places(3)));
    }
    if (fits)
        for (int32_t i = threadIdx.x; i < SB_STRIDE; i += SB_T)
            list[SB_STRIDE * (int64_t)blockIdx.x + i] = i < nu ? (int32_t)s[i] : -1;
}

template <int L>
__global__ __launch_bounds__(SB_T) void k_spring_fill(const int32_t *row, const int32_t *head, const double *rest,
                                                      int64_t nv, int32_t stride, const int64_t *off,
                                                      const int32_t *from, int32_t *list, int32_t *own,
                                                      uint16_t *slot, double *brest) {
    __shared__ uint32_t s[SB_STRIDE];   // the padding sorts last
    constexpr int V = SB_T / L;
    const int64_t wg = blockIdx.x, v0 = wg * V;
    for (int32_t i = threadIdx.x; i < stride; i += SB_T) {
        const int32_t v = from[SB_STRIDE * wg + i];
        s[i] = (uint32_t)v;
        list[wg * stride + i] = v;
    }
    __syncthreads();
    auto place = [&](uint32_t v) {
        int32_t lo = 0, hi = stride - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (s[mid] < v) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    const int32_t first = place((uint32_t)v0);
    if (threadIdx.x == 0) own[wg] = first;
    const int32_t lv = (int32_t)threadIdx.x / L, sub = (int32_t)threadIdx.x % L;
    const int64_t v = v0 + lv, w = 4 * wg + threadIdx.x / 64;
    const int32_t e0 = v < nv ? row[v] : 0, e1 = v < nv ? row[v + 1] : 0;
    int32_t e = e0 + sub;
    for (int64_t j = off[w] + threadIdx.x % 64; j < off[w + 1]; j += 64, e += L) {
        // a padding entry is a spring from the lane's vertex to itself: no force
        slot[j] = (uint16_t)(e < e1 ? place((uint32_t)head[e]) : v < nv ? first + lv : 0);
        brest[j] = e < e1 ? rest[e] : 0.0;
    }
}

// Forces (STEP 0) or one whole step (STEP 1; see k_spring_step) of a workgroup's 256 / L vertices, L
// lanes each.  The positions come into LDS once per workgroup (about 3 per vertex on a
// Morton-ordered tet mesh, against 14 gathers), the edges lane-major, 10 bytes each and coalesced.
// Bound by memory: 60 MB read and 14 MB written per step at 64^3 cells (275k vertices, 3.74M edges),
// 15.5 us or 4.8 TB/s, the rate of a large copy; k_spring_step, bound by its gathers, 21.3 us.
// Measured: one / two / four / eight edges in flight 17.1 / 15.5 / 16.4 / 18.2 us; with the
// library's square root and division 16.3; the rest lengths recomputed from staged rest positions
// in place of read, 18.1; 256 vertices on 512 threads no faster.
template <int STEP, int L>
__global__ __launch_bounds__(SB_T) void k_spring_block(SpringBlocks t, double K, const double *mass, double dt,
                                                       const double *q, double *q_out, double *qd, double *f,
                                                       int take_f) {
    extern __shared__ double s_q[];
    const uint32_t tid = threadIdx.x, S = t.stride, nv = t.nv;
    const uint32_t wg = xcd_block(blockIdx.x, gridDim.x);
    const uint32_t lv = tid / L, v = wg * (SB_T / L) + lv;
    const bool in = v < nv;
    const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / 64));
    const int64_t w0 = t.off[4 * (int64_t)wg + wv], j0 = w0 + (tid & 63u);
    const int32_t rounds = (int32_t)((t.off[4 * (int64_t)wg + wv + 1] - w0) / 64);
    const uint32_t me = (uint32_t)t.own[wg] + (in ? lv : 0u);
    // what the update reads, in flight while the positions are staged: lane `sub` of a vertex takes
    // the components sub, sub + L
    constexpr int NC = L >= 3 ? 1 : 2;
    const uint32_t sub = tid % L;
    double m = 1.0, vel[NC], f0[NC];
    if (in) {
        if (STEP) m = mass[v];
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if (sub + i * L < 3) {
                const size_t at = (size_t)(sub + i * L) * nv + v;
                if (STEP) vel[i] = qd[at];
                if (take_f) f0[i] = f[at];
            }
    }
    for (uint32_t i = tid; i < S; i += SB_T) {
        const int32_t g = t.list[(size_t)wg * S + i];
        if (g >= 0)
#pragma unroll
            for (int k = 0; k < 3; ++k) s_q[k * S + i] = q[(size_t)k * nv + g];
    }
    // the edges, SB_U rounds at a time, the next ones in flight while these are summed (every lane
    // of a wave has the same number of rounds)
    uint32_t h[SB_U];
    double len[SB_U];
    auto load = [&](int32_t r) {
#pragma unroll
        for (int u = 0; u < SB_U; ++u) {
            const bool on = r + u < rounds;
            h[u] = on ? t.slot[j0 + (int64_t)(r + u) * 64] : me;
            len[u] = on ? t.rest[j0 + (int64_t)(r + u) * 64] : 0.0;
        }
    };
    load(0);
    __syncthreads();
    const double q0 = s_q[me], q1 = s_q[S + me], q2 = s_q[2 * S + me];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    bool fine = true;
    for (int32_t r = 0; r < rounds; r += SB_U) {
        double a[SB_U], b[SB_U], c[SB_U], l[SB_U];
#pragma unroll
        for (int u = 0; u < SB_U; ++u) {
            a[u] = s_q[h[u]] - q0;
            b[u] = s_q[S + h[u]] - q1;
            c[u] = s_q[2 * S + h[u]] - q2;
            l[u] = len[u];
        }
        load(r + SB_U);
#pragma unroll
        for (int u = 0; u < SB_U; ++u) {
            const double n2 = a[u] * a[u] + b[u] * b[u] + c[u] * c[u];
            const double sc = spring_scale(l[u], n2);
            fine = fine && spring_in_range(n2);
            a0 += fma(-sc, a[u], a[u]);
            a1 += fma(-sc, b[u], b[u]);
            a2 += fma(-sc, c[u], c[u]);
        }
    }
    if (!fine) {   // a spring of extreme or no finite length: this lane's sum again
        a0 = a1 = a2 = 0.0;
        // its own edges alone: from a place that is not finite, a padding entry is no zero force
        const int32_t *row = t.own - (size_t)(nv + 1);
        const int32_t deg = in ? row[v + 1] - row[v] : 0, own = (deg - (int32_t)(tid % L) + L - 1) / L;
        for (int32_t r = 0; r < own; ++r) {
            const uint32_t k = t.slot[j0 + (int64_t)r * 64];
            const double x = s_q[k] - q0, y = s_q[S + k] - q1, z = s_q[2 * S + k] - q2;
            const double sc = spring_scale_any(t.rest[j0 + (int64_t)r * 64], x * x + y * y + z * z);
            a0 += fma(-sc, x, x);
            a1 += fma(-sc, y, y);
            a2 += fma(-sc, z, z);
        }
    }
    a0 = lanes_sum<L>(a0);
    a1 = lanes_sum<L>(a1);
    a2 = lanes_sum<L>(a2);
    if (!in) return;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const uint32_t c = sub + i * L;
        if (c >= 3) break;
        const size_t at = (size_t)c * nv + v;
        double fk = K * (c == 0 ? a0 : c == 1 ? a1 : a2);
        if (take_f) fk += f0[i];
        if (STEP) {
            if (take_f) f[at] = 0.0;
            double qn, vn;
            integrate(c == 0 ? q0 : c == 1 ? q1 : q2, vel[i], fk / m, dt, qn, vn);
            q_out[at] = qn;
            qd[at] = vn;
        } else {
            f[at] = fk;
        }
    }
}

SpringBlocks spring_blocks(const ebbx_springs_s *S) {
    return SpringBlocks{S->b_list.as<int32_t>(), S->row.as<int32_t>() + S->nv + 1, S->b_off.as<int64_t>(),
                        S->b_slot.as<uint16_t>(), S->b_rest.as<double>(), (uint32_t)S->stride, (uint32_t)S->nv};
}

// The tables of k_spring_block, where they pay: the workgroups' lists together hold at most half as
// many vertices as there are edges (else staging saves little), each few enough for six workgroups'
// LDS per CU, and padding the waves to their longest vertex adds at most half (else a few vertices
// of high degree make every lane of their wave wait), and every rest length is finite.  Synchronous.
template <int L> void build_spring_blocks(ebbx_springs_s *S, hipStream_t s) {
    const int64_t nv = S->nv, ne = S->ne;
    if (nv == 0 || ne == 0) return;
    const int64_t nwg = (nv + SB_T / L - 1) / (SB_T / L);
    // the lists of the counting pass; behind them its two tallies and the scratch of the scan
    const int64_t nlist = nwg * SB_STRIDE, noff = 4 * nwg + 1;
    DevBuf tmp((size_t)nlist * sizeof(int32_t) + 2 * sizeof(Tally) + (size_t)scan_scratch(noff) * sizeof(int64_t), s);
    Tally *tally = (Tally *)(tmp.as<int32_t>() + nlist);
    S->b_off.reset((size_t)noff * sizeof(int64_t), s);
    HIPCHK(hipMemsetAsync(tally, 0, 2 * sizeof(Tally), s));
    hipLaunchKernelGGL(k_spring_count<L>, dim3((unsigned)nwg), dim3(SB_T), 0, s, S->row.as<int32_t>(),
                       S->head.as<int32_t>(), S->rest.as<double>(), nv, tally, tally + 1, S->b_off.as<int64_t>(),
                       tmp.as<int32_t>());
    HIPCHK(hipGetLastError());
    exclusive_scan_i64(S->b_off.as<int64_t>(), noff, (int64_t *)(tally + 2), s);
    HIPCHK(hipStreamCreateWithFlags(&S->cap, hipStreamNonBlocking));   // while the device counts
    Tally got[2] = {};
    HIPCHK(hipMemcpyAsync(got, tally, sizeof got, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const int32_t most = (int32_t)got[0].largest();
    const int64_t staged = (int64_t)got[0].total(), entries = (int64_t)got[1].total();
    if (most > SB_STRIDE || 2 * staged > ne || 2 * entries > 3 * ne) {
        S->b_off.release();
        return;
    }
    S->b_list.reset((size_t)nwg * most * sizeof(int32_t), s);
    S->b_slot.reset((size_t)entries * sizeof(uint16_t), s);
    S->b_rest.reset((size_t)entries * sizeof(double), s);
    hipLaunchKernelGGL(k_spring_fill<L>, dim3((unsigned)nwg), dim3(SB_T), 0, s, S->row.as<int32_t>(),
                       S->head.as<int32_t>(), S->rest.as<double>(), nv, most, S->b_off.as<int64_t>(),
                       tmp.as<int32_t>(), S->b_list.as<int32_t>(), S->row.as<int32_t>() + nv + 1,
                       S->b_slot.as<uint16_t>(), S->b_rest.as<double>());
    HIPCHK(hipGetLastError());
    HIPCHK(hipStreamSynchronize(s));
    S->stride = most;
    S->lanes = L;
}

template <int STEP>
void launch_block(ebbx_springs_s *S, const double *mass, double dt, const double *q, double *q_out, double *qd,
                  double *f, int take_f, hipStream_t s) {
    const dim3 g(blocks_of(S->nv * S->lanes, SB_T));
    const size_t lds = (size_t)3 * S->stride * sizeof(double);
    if (S->lanes == 4)
        hipLaunchKernelGGL((k_spring_block<STEP, 4>), g, dim3(SB_T), lds, s, spring_blocks(S), S->K, mass, dt, q,
                           q_out, qd, f, take_f);
    else
        hipLaunchKernelGGL((k_spring_block<STEP, 2>), g, dim3(SB_T), lds, s, spring_blocks(S), S->K, mass, dt, q,
                           q_out, qd, f, take_f);
    HIPCHK(hipGetLastError());
}

__global__ void k_spring_apply(const double *mass, double dt, double *q, double *qd, double *f, int64_t nv) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x) {
        const double m = mass[v];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int64_t i = k * nv + v;
            integrate(q[i], qd[i], f[i] / m, dt, q[i], qd[i]);
            f[i] = 0.0;
        }
    }
}

__device__ __forceinline__ double block_total(double x, double *s4) {
    x = lanes_sum<64>(x);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s4[threadIdx.x >> 6] = x;
    __syncthreads();
    return (s4[0] + s4[1]) + (s4[2] + s4[3]);
}

// pass 1: one partial per workgroup (fixed order); pass 2: their fixed-order sum added to E
__global__ __launch_bounds__(EN_THREADS) void k_kinetic_part(const double *mass, const double *qd, int64_t nv,
                                                             double *part) {
    __shared__ double s4[4];
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double e = 0.0;
    if (v < nv) {
        const double a = qd[v], b = qd[nv + v], c = qd[2 * nv + v];
        e = 0.5 * mass[v] * (a * a + b * b + c * c);
    }
    e = block_total(e, s4);
    if (threadIdx.x == 0) part[blockIdx.x] = e;
}

__global__ __launch_bounds__(EN_THREADS) void k_kinetic_sum(const double *part, int n, double *E) {
    __shared__ double s4[4];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += EN_THREADS) acc += part[i];
    acc = block_total(acc, s4);
    if (threadIdx.x == 0) E[0] += acc;
}

void launch_forces(ebbx_springs_s *S, const double *q, double *f, int accumulate, hipStream_t s) {
    if (S->nv == 0) return;
    if (S->stride) {
        launch_block<0>(S, nullptr, 0.0, q, nullptr, nullptr, f, accumulate, s);
        return;
    }
    hipLaunchKernelGGL((k_spring_forces<LANES, UNROLL>), dim3(blocks_of(S->nv * LANES, 256)), dim3(256), 0, s,
                       S->row.as<int32_t>(), S->head.as<int32_t>(), S->rest.as<double>(), S->K, q, f,
                       (uint32_t)S->nv, accumulate);
    HIPCHK(hipGetLastError());
}

void launch_step(ebbx_springs_s *S, const double *mass, double dt, const double *q, double *q_out, double *qd,
                 double *f, int take_f, hipStream_t s) {
    if (S->stride) {
        launch_block<1>(S, mass, dt, q, q_out, qd, f, take_f, s);
        return;
    }
    hipLaunchKernelGGL((k_spring_step<LANES, UNROLL>), dim3(blocks_of(S->nv * LANES, 256)), dim3(256), 0, s,
                       S->row.as<int32_t>(), S->head.as<int32_t>(), S->rest.as<double>(), S->K, mass, dt, q, q_out,
                       qd, f, take_f, (uint32_t)S->nv);
    HIPCHK(hipGetLastError());
}

void launch_apply(ebbx_springs_s *S, const double *mass, double dt, double *q, double *qd, double *f, hipStream_t s) {
    if (S->nv == 0) return;
    hipLaunchKernelGGL(k_spring_apply, dim3(std::min<unsigned>(blocks_of(S->nv, 256), 16384)), dim3(256), 0, s, mass,
                       dt, q, qd, f, S->nv);
    HIPCHK(hipGetLastError());
}

// n steps ending with the positions in q: fused steps in pairs (q -> q2 -> q), the first of
// them taking the force field's contents; an odd n starts with one step of the separate passes.
void emit_steps(ebbx_springs_s *S, const double *mass, double dt, int32_t n, double *q, double *qd, double *force,
                hipStream_t s) {
    int32_t k = 0;
    if (n % 2) {
        launch_forces(S, q, force, 1, s);
        launch_apply(S, mass, dt, q, qd, force, s);
        k = 1;
    }
    double *q2 = S->q2.as<double>();
    for (; k < n; k += 2) {
        launch_step(S, mass, dt, q, q2, qd, force, k == 0, s);
        launch_step(S, mass, dt, q2, q, qd, force, 0, s);
    }
}

void check_vec(const void *p, const char *what, int64_t nv) {
    if (nv > 0 && !p) fail(EBBX_E_ARG, "%s is NULL", what);
}

}  // namespace
}  // namespace ebbx

using namespace ebbx;

extern "C" ebbx_status ebbx_springs_create(ebbx_relation edges, const char *tail, const char *head, ebbx_relation verts,
                                          const char *pos_field, double K, ebbx_springs *out) {
    EBBX_API_BEGIN
    if (!out) fail(EBBX_E_ARG, "out is NULL");
    auto *er = check_rel(edges);
    auto *vr = check_rel(verts);
    if (!tail || !head || !pos_field) fail(EBBX_E_ARG, "a field name is NULL");
    if (!std::isfinite(K)) fail(EBBX_E_ARG, "K must be finite");
    KeyField &kt = get_key(er, tail);
    KeyField &kh = get_key(er, head);
    if (kt.target != vr || kh.target != vr) fail(EBBX_E_ARG, "tail and head must target '%s'", vr->name.c_str());
    if (kt.arity != 1 || kh.arity != 1) fail(EBBX_E_SHAPE, "tail and head must have arity 1");
    const Field &X = get_field(vr, pos_field, EBBX_F64, 3);
    auto S = std::make_unique<ebbx_springs_s>();
    S->edges = er;
    S->verts = vr;
    S->nv = vr->size;
    S->ne = er->size;
    S->K = K;
    if (S->ne >= (int64_t(1) << 31)) fail(EBBX_E_ARG, "too many edges");
    auto g = build_group(er, tail, nullptr);
    S->row.reset((size_t)(S->nv + 1 + blocks_of(S->nv, SB_T / 4)) * sizeof(int32_t));
    S->head.reset((size_t)std::max<int64_t>(S->ne, 1) * sizeof(int32_t));
    S->rest.reset((size_t)std::max<int64_t>(S->ne, 1) * sizeof(double));
    S->part.reset((size_t)blocks_of(std::max<int64_t>(S->nv, 1), EN_THREADS) * sizeof(double));
    hipLaunchKernelGGL(k_spring_setup, dim3(blocks_of(S->nv + 1, 256)), dim3(256), 0, nullptr,
                       g->row_ptr.as<int64_t>(), g->inc.as<int32_t>(), kh.ptr, (const double *)X.ptr, S->nv,
                       S->row.as<int32_t>(), S->head.as<int32_t>(), S->rest.as<double>());
    HIPCHK(hipGetLastError());
    if (S->nv <= SB_FOUR_NV) build_spring_blocks<4>(S.get(), nullptr);
    else build_spring_blocks<2>(S.get(), nullptr);
    if (!S->cap) HIPCHK(hipStreamCreateWithFlags(&S->cap, hipStreamNonBlocking));
    HIPCHK(hipDeviceSynchronize());
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_springs.insert(S.get());
    }
    *out = S.release();
    EBBX_API_END
}

extern "C" ebbx_status ebbx_springs_destroy(ebbx_springs sp) {
    EBBX_API_BEGIN
    auto *S = check_springs(sp);
    HIPCHK(hipDeviceSynchronize());
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_springs.erase(S);
    }
    delete S;
    EBBX_API_END
}

extern "C" ebbx_status ebbx_springs_rest(ebbx_springs sp, double *rest_dev, ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *S = check_springs(sp);
    if (S->ne > 0 && !rest_dev) fail(EBBX_E_ARG, "rest_dev is NULL");
    if (S->ne > 0)
        HIPCHK(hipMemcpyAsync(rest_dev, S->rest.get(), (size_t)S->ne * sizeof(double), hipMemcpyDeviceToDevice,
                              (hipStream_t)stream));
    EBBX_API_END
}

extern "C" ebbx_status ebbx_springs_forces(ebbx_springs sp, const double *q, double *force, int32_t accumulate,
                                          ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *S = check_springs(sp);
    check_vec(q, "q", S->nv);
    check_vec(force, "force", S->nv);
    if (S->nv > 0 && overlap(q, force, (size_t)(3 * S->nv) * sizeof(double))) fail(EBBX_E_PHASE, "force aliases q");
    launch_forces(S, q, force, accumulate, (hipStream_t)stream);
    EBBX_API_END
}

extern "C" ebbx_status ebbx_springs_apply(ebbx_springs sp, const double *mass, double dt, double *q, double *qd,
                                         double *force, ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *S = check_springs(sp);
    const int64_t nv = S->nv;
    for (const void *p : {(const void *)mass, (const void *)q, (const void *)qd, (const void *)force})
        check_vec(p, "a vertex field", nv);
    if (!std::isfinite(dt)) fail(EBBX_E_ARG, "dt must be finite");
    const size_t b = (size_t)(3 * nv) * sizeof(double);
    if (nv > 0 && (overlap(q, qd, b) || overlap(q, force, b) || overlap(qd, force, b)))
        fail(EBBX_E_PHASE, "q, qd and force must not alias");
    launch_apply(S, mass, dt, q, qd, force, (hipStream_t)stream);
    EBBX_API_END
}

extern "C" ebbx_status ebbx_springs_kinetic_energy(ebbx_springs sp, const double *mass, const double *qd, double *E_dev,
                                                  ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *S = check_springs(sp);
    if (!E_dev) fail(EBBX_E_ARG, "E_dev is NULL");
    check_vec(mass, "mass", S->nv);
    check_vec(qd, "qd", S->nv);
    if (S->nv == 0) return EBBX_OK;
    hipStream_t s = (hipStream_t)stream;
    const unsigned nb = blocks_of(S->nv, EN_THREADS);
    hipLaunchKernelGGL(k_kinetic_part, dim3(nb), dim3(EN_THREADS), 0, s, mass, qd, S->nv, S->part.as<double>());
    hipLaunchKernelGGL(k_kinetic_sum, dim3(1), dim3(EN_THREADS), 0, s, (const double *)S->part.get(), (int)nb, E_dev);
    HIPCHK(hipGetLastError());
    EBBX_API_END
}

extern "C" ebbx_status ebbx_springs_run(ebbx_springs sp, const double *mass, double dt, int32_t nsteps, double *q,
                                       double *qd, double *force, ebbx_stream stream) {
    EBBX_API_BEGIN
    auto *S = check_springs(sp);
    const int64_t nv = S->nv;
    if (nsteps < 0) fail(EBBX_E_ARG, "nsteps must be >= 0");
    for (const void *p : {(const void *)mass, (const void *)q, (const void *)qd, (const void *)force})
        check_vec(p, "a vertex field", nv);
    if (!std::isfinite(dt)) fail(EBBX_E_ARG, "dt must be finite");
    const size_t b = (size_t)(3 * nv) * sizeof(double);
    if (nv > 0 && (overlap(q, qd, b) || overlap(q, force, b) || overlap(qd, force, b)))
        fail(EBBX_E_PHASE, "q, qd and force must not alias");
    if (nv == 0 || nsteps == 0) return EBBX_OK;
    hipStream_t s = (hipStream_t)stream;
    if (!S->q2.get()) S->q2.reset((size_t)(3 * nv) * sizeof(double), s);
    const void *key[4] = {mass, q, qd, force};
    if (nsteps >= RUN_CHUNK && (!S->exec || !std::equal(key, key + 4, S->key) || S->key_dt != dt)) {
        S->drop_graph();
        HIPCHK(hipStreamBeginCapture(S->cap, hipStreamCaptureModeThreadLocal));
        CaptureGuard guard(S->cap);
        emit_steps(S, mass, dt, RUN_CHUNK, q, qd, force, S->cap);
        guard.disarm();
        HIPCHK(hipStreamEndCapture(S->cap, &S->graph));
        HIPCHK(hipGraphInstantiate(&S->exec, S->graph, nullptr, nullptr, 0));
        std::copy(key, key + 4, S->key);
        S->key_dt = dt;
    }
    int32_t left = nsteps;
    for (; left >= RUN_CHUNK; left -= RUN_CHUNK) HIPCHK(hipGraphLaunch(S->exec, s));
    emit_steps(S, mass, dt, left, q, qd, force, s);
    EBBX_API_END
}
