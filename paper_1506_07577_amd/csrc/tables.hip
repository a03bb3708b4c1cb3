// tables.hip -- the tables of the BLOCK strategies, built on the device.
//
// Blocks of bt consecutive tets.  Per block: the sorted set of vertices it touches,
// each corner's slot in that set, the block's incidences ordered by (vertex, local
// tet, corner) with each corner's row in that order and each vertex's run of rows,
// and whether the block holds every incident tet of the vertex.  Vertices that it
// does not own outright get a place in the halo; the shared-vertex tables list each
// such vertex's halo places in block order.
//
// One workgroup sorts a block's 4 bt (vertex, incidence) pairs in LDS and counts
// (vertices per block fix the tables' stride, shared vertices the halo's places); a
// second pass writes the tables from the sorted pairs, 32 bytes per tet kept in
// memory between the two (sorting again instead took 75 us of the second pass's 80,
// 2,000 blocks).  k_blk_count takes 141 us for 6,144 blocks of 256 tets (194 with its
// tallies' atomics on one address); fewer barriers in the sort's 55 stages gained nothing.
// Measured, a new scrambled mesh of 358k tets taken in (relations, Morton order, domain,
// mass, one force; FP32): 71.9 ms with the tables built on the host and each pass of the
// radix sort waited for, 1.60 ms with these.
#include <algorithm>

#include "fem.h"
#include "sort.h"

namespace ebbx {

namespace {

constexpr int BT_THREADS = 256;

// ---- a block's pairs, sorted ---------------------------------------------------------------

// Load the pairs (vertex << 12 | 4 * local tet + corner) of block b into s[0, n), n a power of
// two >= 4 bt, absent ones as the largest value, and sort them (bitonic, ascending).
__device__ __forceinline__ void sorted_pairs(const int32_t *keys, int64_t nt, int64_t b, int32_t bt, int32_t n,
                                             unsigned long long *s) {
    const int tid = threadIdx.x;
    const int64_t t0 = b * bt;
    for (int32_t e = tid; e < n; e += BT_THREADS) {
        const int32_t c = e / bt, tl = e - c * bt;   // coalesced along each key column
        const bool in = c < 4 && t0 + tl < nt;
        const int32_t i = c < 4 ? 4 * tl + c : e;
        s[i] = in ? ((unsigned long long)(uint32_t)keys[(int64_t)c * nt + t0 + tl] << 12) | (unsigned)i : ~0ull;
    }
    lds_sort<BT_THREADS>(s, n);
}

// Thread tid's stretch of the sorted pairs, [tid * n / 256, ...): head h of a vertex's run, with
// the run's length, is passed to f(i, vertex, length, shared).
template <class F>
__device__ __forceinline__ void each_head(const unsigned long long *s, int32_t n, const int64_t *rp, F f) {
    const int32_t per = n / BT_THREADS, i0 = (int32_t)threadIdx.x * per;
    for (int32_t i = i0; i < i0 + per; ++i) {
        if (s[i] == ~0ull) break;
        const uint32_t v = (uint32_t)(s[i] >> 12);
        if (i > 0 && (uint32_t)(s[i - 1] >> 12) == v) continue;
        int32_t j = i + 1;
        while (j < n && s[j] != ~0ull && (uint32_t)(s[j] >> 12) == v) ++j;
        f(i, v, j - i, (int64_t)(j - i) != rp[v + 1] - rp[v]);
    }
}

// Pass 1: the block's shared vertices into nsh[b] and into found[1], its vertex count into found[0].
__global__ __launch_bounds__(BT_THREADS) void k_blk_count(const int32_t *keys, const int64_t *rp, int64_t nt,
                                                          int32_t bt, int32_t n, unsigned long long *pairs,
                                                          int64_t *nsh, Tally *found) {
    extern __shared__ unsigned long long s_pairs[];
    __shared__ int32_t sw[BT_THREADS / 64];
    const int64_t b = blockIdx.x;
    sorted_pairs(keys, nt, b, bt, n, s_pairs);
    for (int32_t e = threadIdx.x; e < 4 * bt; e += BT_THREADS) pairs[b * 4 * bt + e] = s_pairs[e];
    int32_t heads = 0, shared = 0;
    each_head(s_pairs, n, rp, [&](int32_t, uint32_t, int32_t, bool sh) {
        ++heads;
        shared += sh;
    });
    int32_t nb = 0, ns = 0;
    block_prefix<BT_THREADS>(heads, sw, nb);
    block_prefix<BT_THREADS>(shared, sw, ns);
    if (threadIdx.x == 0) {
        nsh[b] = ns;
        if (b + 1 == gridDim.x) nsh[b + 1] = 0;   // scanned with the others
        found[0].add(nb, (unsigned long long)nb);
        found[1].add(0, (unsigned long long)ns);
    }
}

struct BlkOut {
    int32_t *verts, *hpos;      // [nblk * S], -1 padded
    uint16_t *row;              // [nblk * (S + 1)]
    uint32_t *pos, *slot;       // [2 nt], [w nt]
    uint32_t *hkey, *hval;      // per halo place: its vertex, the place
    int32_t *cnt;               // per vertex: its halo places
};

// Pass 2: the tables of block b; its halo places start at hbase[b].
__global__ __launch_bounds__(BT_THREADS) void k_blk_fill(const unsigned long long *pairs, const int64_t *rp,
                                                         int64_t nt, int32_t bt, int32_t n, int32_t S, int32_t w,
                                                         const int64_t *hbase, BlkOut o) {
    extern __shared__ unsigned long long s_pairs[];
    uint32_t *s_at = (uint32_t *)(s_pairs + n);   // per incidence: slot << 16 | row
    __shared__ int32_t sw[BT_THREADS / 64];
    const int64_t b = blockIdx.x;
    const int tid = threadIdx.x;
    for (int32_t e = tid; e < n; e += BT_THREADS) s_pairs[e] = e < 4 * bt ? pairs[b * 4 * bt + e] : ~0ull;
    __syncthreads();
    int32_t heads = 0, shared = 0;
    each_head(s_pairs, n, rp, [&](int32_t, uint32_t, int32_t, bool sh) {
        ++heads;
        shared += sh;
    });
    int32_t nb = 0, ns = 0;
    int32_t slot = block_prefix<BT_THREADS>(heads, sw, nb);
    int64_t hp = hbase[b] + block_prefix<BT_THREADS>(shared, sw, ns);
    const int64_t left = nt - b * bt;
    const int32_t ntl = left < bt ? (int32_t)left : bt;   // tets of this block
    each_head(s_pairs, n, rp, [&](int32_t i, uint32_t v, int32_t len, bool sh) {
        const int64_t q = b * S + slot;
        o.verts[q] = (int32_t)v;
        o.row[b * (S + 1) + slot] = (uint16_t)i;
        o.hpos[q] = sh ? (int32_t)hp : -1;
        if (sh) {
            o.hkey[hp] = v;
            o.hval[hp] = (uint32_t)hp;
            atomicAdd(o.cnt + v, 1);
            ++hp;
        }
        for (int32_t j = i; j < i + len; ++j) s_at[s_pairs[j] & 4095u] = ((uint32_t)slot << 16) | (uint32_t)j;
        ++slot;
    });
    for (int32_t i = nb + tid; i <= S; i += BT_THREADS) {
        o.row[b * (S + 1) + i] = (uint16_t)(4 * ntl);
        if (i < S) {
            o.verts[b * S + i] = -1;
            o.hpos[b * S + i] = -1;
        }
    }
    __syncthreads();
    for (int32_t tl = tid; tl < ntl; tl += BT_THREADS) {
        const int64_t t = b * bt + tl;
        const uint32_t a0 = s_at[4 * tl], a1 = s_at[4 * tl + 1], a2 = s_at[4 * tl + 2], a3 = s_at[4 * tl + 3];
        o.pos[t] = (a0 & 0xffffu) | (a1 << 16);
        o.pos[nt + t] = (a2 & 0xffffu) | (a3 << 16);
        if (w == 1) {   // 4 x 8 bits: every block has at most 256 vertices
            o.slot[t] = (a0 >> 16) | ((a1 >> 16) << 8) | ((a2 >> 16) << 16) | ((a3 >> 16) << 24);
        } else {
            o.slot[t] = (a0 >> 16) | (a1 & 0xffff0000u);
            o.slot[nt + t] = (a2 >> 16) | (a3 & 0xffff0000u);
        }
    }
}

// ---- shared vertices -------------------------------------------------------------------------

// A vertex has a row in the shared-vertex table if it has halo places, or no tet at all (the halo
// pass zeroes it).  Scan inputs (rows, rows of at most 4 places, places), and the largest number of
// places of one vertex into *maxm.
__global__ void k_sh_flags(const int32_t *cnt, const int64_t *rp, int64_t nv, int64_t *flag, int64_t *few,
                           int64_t *places, int *maxm) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v > nv) return;
    const int32_t c = v < nv ? cnt[v] : 0;
    const bool on = v < nv && (c > 0 || rp[v + 1] == rp[v]);
    flag[v] = on;
    few[v] = on && c <= 4;
    places[v] = c;
    if (c > 0) atomicMax(maxm, c);
}

// The rows: nc = 0, in vertex order with offsets ptr into the places (CSR); else the n4 rows of at
// most 4 places first (one int4 of places each, -1 padded), then the others (nc int4 each), both in
// vertex order; n4 = 0: every row nc int4.
__global__ void k_sh_rows(const int32_t *cnt, const int64_t *rp, int64_t nv, const int64_t *row, const int64_t *few,
                          const int64_t *ptr, const int32_t *pos, int nc, int64_t n4, int32_t *sh_vert,
                          int32_t *sh_ptr, int32_t *sh_row, int32_t *tab) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v > nv) return;
    if (v == nv) {
        if (nc == 0) sh_ptr[row[nv]] = (int32_t)ptr[nv];
        return;
    }
    const int32_t c = cnt[v];
    if (c == 0 && rp[v + 1] != rp[v]) {
        sh_row[v] = -1;
        return;
    }
    const int64_t r = n4 == 0 ? row[v] : c <= 4 ? few[v] : n4 + row[v] - few[v];
    sh_row[v] = (int32_t)r;
    sh_vert[r] = (int32_t)v;
    if (nc == 0) {
        sh_ptr[r] = (int32_t)ptr[v];
        return;
    }
    int32_t *t = tab + 4 * (r < n4 ? r : n4 + (r - n4) * nc);
    const int32_t w = r < n4 ? 4 : 4 * nc;
    for (int32_t j = 0; j < w; ++j) t[j] = j < c ? pos[ptr[v] + j] : -1;
}

// Block-local FP32 rest positions: entry (b, i) holds X of block b's i-th vertex minus X of its
// first vertex, rounded to FP32 (three columns of nblk * S entries; padding 0).
__global__ void k_block_xf(const double *X, int64_t nv, const int32_t *bverts, int64_t n, uint32_t S, float *xf) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = bverts[e], v0 = bverts[(e / S) * S];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            xf[(int64_t)k * n + e] = v >= 0 ? (float)(X[(int64_t)k * nv + v] - X[(int64_t)k * nv + v0]) : 0.0f;
    }
}

unsigned grid_of(int64_t n, int per) { return (unsigned)std::max<int64_t>(1, (n + per - 1) / per); }

}  // namespace

void build_block_xf(ebbx_fem_s *F, hipStream_t s) {
    const int64_t n = F->nblk * (int64_t)F->blk_maxv;
    if (F->prec != EBBX_F32 || F->blk_w != 1 || F->nblk == 0) {
        F->blk_xf.release();
        return;
    }
    F->blk_xf.reset((size_t)n * 3 * sizeof(float), s);
    hipLaunchKernelGGL(k_block_xf, dim3(std::min<unsigned>(grid_of(n, 256), 16384)), dim3(256), 0, s,
                       F->Xc.as<double>(), F->nv, F->blk_verts.as<int32_t>(), n, (uint32_t)F->blk_maxv,
                       F->blk_xf.as<float>());
    HIPCHK(hipGetLastError());
}

namespace {

// What pass 1 finds about blocks of bt tets with the keys in a given order.
struct Counted {
    DevBuf hbase;         // nblk + 1: first halo place of each block
    DevBuf pairs;         // 4 bt sorted pairs per block
    int32_t maxv = 1;     // largest vertex count of a block
    int64_t halo = 0, staged = 0;
};

int32_t pairs_of(int32_t bt) {
    int32_t n = 256;
    while (n < 4 * bt) n <<= 1;
    return n;
}

Counted count_blocks(const int32_t *keys, const int64_t *rp, int64_t nt, int32_t bt, hipStream_t s) {
    Counted c;
    const int64_t nblk = (nt + bt - 1) / bt;
    const int32_t n = pairs_of(bt);
    c.hbase.reset((size_t)(nblk + 1) * sizeof(int64_t), s);
    c.pairs.reset(std::max<size_t>((size_t)nblk * 4 * bt * sizeof(unsigned long long), 16), s);
    // the two tallies and the scratch of the scan
    DevBuf found(2 * sizeof(Tally) + (size_t)scan_scratch(nblk + 1) * sizeof(int64_t), s);
    HIPCHK(hipMemsetAsync(found.get(), 0, 2 * sizeof(Tally), s));
    Tally got[2] = {};
    if (nblk > 0) {
        hipLaunchKernelGGL(k_blk_count, dim3((unsigned)nblk), dim3(BT_THREADS), (size_t)n * 8, s, keys, rp, nt, bt, n,
                           c.pairs.as<unsigned long long>(), c.hbase.as<int64_t>(), found.as<Tally>());
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(got, found.get(), sizeof got, hipMemcpyDeviceToHost, s));
        exclusive_scan_i64(c.hbase.as<int64_t>(), nblk + 1, (int64_t *)(found.as<Tally>() + 2), s);
    }
    HIPCHK(hipStreamSynchronize(s));
    c.maxv = std::max((int32_t)got[0].largest(), 1);
    c.staged = (int64_t)got[0].total();
    c.halo = (int64_t)got[1].total();
    return c;
}

}  // namespace

// Copies of the per-tet arrays that the block kernels stream, in the tables' order.
void refresh_ordered(ebbx_fem_s *F, hipStream_t s) {
    if (!F->ordered) return;
    if (F->blk_w != 1 && !F->B_ord.get()) {
        F->B_ord.reset((size_t)9 * F->nt * F->esize, s);
        permute_columns(F->B.get(), F->B_ord.get(), F->esize, F->t_order.as<int32_t>(), F->nt, 9, s);
    }
    if (F->per_tet) {
        if (!F->mat_ord.get()) F->mat_ord.reset((size_t)2 * F->nt * F->esize, s);
        permute_columns(F->mat.get(), F->mat_ord.get(), F->esize, F->t_order.as<int32_t>(), F->nt, 2, s);
    }
}

void build_blocks(ebbx_fem_s *F, int32_t bt, bool reorder, hipStream_t s) {
    if (bt < 64 || bt > 1024 || bt % 64)
        fail(EBBX_E_ARG, "block strategy: tets per block must be a multiple of 64 from 64 to 1024 (got %d)", bt);
    const int64_t nt = F->nt, nv = F->nv, nblk = (nt + bt - 1) / bt;
    const int64_t *rp = F->group->row_ptr.as<int64_t>();
    const int32_t n = pairs_of(bt);
    F->pair_tab.release();
    F->act_mesh.release();
    F->blocks_built = false;   // until the tables below are whole
    F->halo_level = -1;
    F->ordered = false;
    F->B_ord.release();
    F->mat_ord.release();
    Counted c = count_blocks(F->keys, rp, nt, bt, s);
    F->order_settled = reorder || c.maxv <= 256;
    // Blocks of more than 256 vertices share few of them between their tets (a Morton or lattice
    // order of a tet mesh has 100 to 180 in a block of 256 tets): the tables then follow a locality
    // order of the tets instead of the rows' own, if that stages at least a fifth fewer vertices and
    // needs no more LDS and halo than the rows' order (so no call meets a limit that it did not).
    // Measured, force and K u, a scrambled mesh of 635k tets, StVK FP64: 272 us in the rows' order
    // (blocks of 1,000 vertices, every vertex in some 24 of them), 55 us in the locality order.
    // Where the rows' order gives blocks of at most 256 vertices there is nothing to gain: lattice
    // rows, up to 180 vertices per block, 26.4 / 46.0 / 88.7 us at 32^3 / 48^3 / 64^3 cells, the
    // same tables reordered 26.5 / 47.6 / 88.0 us (50 CG iterations 1.04 / 1.87 / 3.34 against
    // 1.17 / 1.95 / 3.41 ms, the vertex vectors being in lattice order).
    DevBuf okeys;
    if (reorder && c.maxv > 256) {
        F->t_order.reset((size_t)nt * sizeof(int32_t), s);
        locality_order(F->Xc.as<double>(), nv, F->keys, nt, F->t_order.as<uint32_t>(), s);
        okeys.reset((size_t)4 * nt * sizeof(int32_t), s);
        permute_columns(F->keys, okeys.get(), 4, F->t_order.as<int32_t>(), nt, 4, s);
        Counted o = count_blocks(okeys.as<int32_t>(), rp, nt, bt, s);
        if (o.staged * 5 <= c.staged * 4 && o.maxv <= c.maxv && o.halo <= c.halo) {
            F->ordered = true;
            c = std::move(o);
        }
    }
    if (!F->ordered) F->t_order.release();
    const int64_t nh = c.halo;
    if (nh >= (int64_t(1) << 31)) fail(EBBX_E_ARG, "block tables exceed int32");
    const int32_t S = c.maxv, w = c.maxv <= 256 ? 1 : 2;
    DevBuf mx(16, s);
    HIPCHK(hipMemsetAsync(mx.get(), 0, 16, s));
    // pass 2
    auto room = [](int64_t count, size_t each) { return std::max<size_t>((size_t)count * each, 16); };
    F->blk_verts.reset(room(nblk * S, 4), s);
    F->blk_hpos.reset(room(nblk * S, 4), s);
    F->blk_lptr.reset(room(nblk * (S + 1), 2), s);
    F->blk_pos.reset(room(2 * nt, 4), s);
    F->blk_local.reset(room(w * nt, 4), s);
    F->sh_pos.reset(room(nh, 4), s);
    DevBuf hkey(room(nh, 4), s), cnt(room(nv, 4), s);
    HIPCHK(hipMemsetAsync(cnt.get(), 0, cnt.bytes(), s));
    if (nblk > 0) {
        const BlkOut o{F->blk_verts.as<int32_t>(), F->blk_hpos.as<int32_t>(), F->blk_lptr.as<uint16_t>(),
                       F->blk_pos.as<uint32_t>(), F->blk_local.as<uint32_t>(), hkey.as<uint32_t>(),
                       F->sh_pos.as<uint32_t>(), cnt.as<int32_t>()};
        hipLaunchKernelGGL(k_blk_fill, dim3((unsigned)nblk), dim3(BT_THREADS), (size_t)n * 12, s,
                           c.pairs.as<unsigned long long>(), rp, nt, bt, n, S, w, c.hbase.as<int64_t>(), o);
        HIPCHK(hipGetLastError());
    }
    F->blk_tets = bt;
    F->nblk = nblk;
    F->blk_maxv = S;
    // FP32 elements in the tables' own order keep streaming the stored FP32 B, as in the rows' order
    F->blk_w = F->ordered && w == 1 && F->prec == EBBX_F32 ? 3 : w;
    F->halo_n = nh;
    build_block_xf(F, s);
    refresh_ordered(F, s);
    // each shared vertex's places, ascending: a stable sort of the places by vertex
    int bits = 1;
    while ((int64_t(1) << bits) < nv) ++bits;
    radix_sort_pairs_u32(hkey.as<uint32_t>(), F->sh_pos.as<uint32_t>(), nh, bits, s);
    const size_t cols = (size_t)(nv + 1) * sizeof(int64_t);
    DevBuf row(cols, s), few(cols, s), ptr(cols, s);
    hipLaunchKernelGGL(k_sh_flags, dim3(grid_of(nv + 1, 256)), dim3(256), 0, s, cnt.as<int32_t>(), rp, nv,
                       row.as<int64_t>(), few.as<int64_t>(), ptr.as<int64_t>(), mx.as<int>());
    HIPCHK(hipGetLastError());
    exclusive_scan_i64(row.as<int64_t>(), nv + 1, s);
    exclusive_scan_i64(few.as<int64_t>(), nv + 1, s);
    exclusive_scan_i64(ptr.as<int64_t>(), nv + 1, s);
    int maxm = 0;
    int64_t sh_n = 0, n4 = 0;
    HIPCHK(hipMemcpyAsync(&maxm, mx.as<int>(), sizeof maxm, hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(&sh_n, row.as<int64_t>() + nv, sizeof sh_n, hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(&n4, few.as<int64_t>() + nv, sizeof n4, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    // fixed-width rows of halo places when no vertex has more than 16
    F->sh_n = sh_n;
    F->sh_nc = maxm <= 16 ? std::max(1, (maxm + 3) / 4) : 0;
    // Rows of two widths where seven eighths have at most 4 places.  They spare the padding of the narrow
    // rows and part the wide rows' vertices from their neighbours' lines, so the share decides, though not
    // alone.  Two widths against one, force + K u, 32^3 to 80^3 cells, Morton and lattice order, blocks of 64
    // to 512 tets, FP32 and FP64 (60 pairs): from seven eighths on 0.98 to 1.07 of the speed with rows of up
    // to 12 places (1.02 on average: 64^3 in Morton order, 89% narrow, 63.9 -> 61.2 us in FP32) and 0.97 to
    // 1.03 with up to 8 (1.00 on average: 80^3 in lattice order, 93%, 105.4 -> 107.5 us); below it 0.89 to
    // 1.03, the least at 80^3 (72%, 111.0 -> 124.6 us).
    if (F->sh_nc == 0 || n4 * 8 < sh_n * 7) n4 = 0;
    F->sh_n4 = n4;
    F->sh_vert.reset(room(sh_n, 4), s);
    F->sh_row.reset(room(nv, 4), s);
    if (F->sh_nc == 0) F->sh_ptr.reset(room(sh_n + 1, 4), s);
    else F->sh_tab.reset(room(n4 + (sh_n - n4) * F->sh_nc, 16), s);
    hipLaunchKernelGGL(k_sh_rows, dim3(grid_of(nv + 1, 256)), dim3(256), 0, s, cnt.as<int32_t>(), rp, nv,
                       row.as<int64_t>(), few.as<int64_t>(), ptr.as<int64_t>(), F->sh_pos.as<int32_t>(), F->sh_nc, n4,
                       F->sh_vert.as<int32_t>(), F->sh_ptr.as<int32_t>(), F->sh_row.as<int32_t>(),
                       F->sh_tab.as<int32_t>());
    HIPCHK(hipGetLastError());
    F->halo.reset((size_t)std::max<int64_t>(nh, 1) * 3 * sizeof(double), s);
    HIPCHK(hipStreamSynchronize(s));   // the scratch above is freed on return
    F->halo_level = 0;
    F->blocks_built = true;
}

}  // namespace ebbx
