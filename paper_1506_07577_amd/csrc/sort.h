// sort.h -- sorting and listing within one workgroup, in LDS, for the kernels that build tables.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <numeric>

namespace ebbx {

// What the workgroups of a counting kernel find together: the largest of a value and the sum of
// another.  Atomics on one address pass one by one, some 10 ns each (of 69k workgroups' two, 1.3 of the
// 1.6 ms that a count took), so both are spread over places, and only a larger value is sent.
struct Tally {
    static constexpr int PLACES = 16;
    long long most[PLACES];
    unsigned long long sum[PLACES];
    // by one thread of a workgroup
    __device__ __forceinline__ void add(long long x, unsigned long long y) {
        const unsigned i = blockIdx.x % PLACES;
        if (__hip_atomic_load(most + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < x) atomicMax(most + i, x);
        if (y) atomicAdd(sum + i, y);
    }
    long long largest() const { return *std::max_element(most, most + PLACES); }
    unsigned long long total() const { return std::accumulate(sum, sum + PLACES, 0ull); }
};

// Sort s[0, n) ascending by a workgroup of T threads (bitonic); n a power of two.  The caller's
// writes need no barrier before it, and its reads none after it.
template <int T, class K> __device__ __forceinline__ void lds_sort(K *s, int32_t n) {
    __syncthreads();
    for (int32_t k = 2; k <= n; k <<= 1)
        for (int32_t j = k >> 1; j > 0; j >>= 1) {
            for (int32_t e = threadIdx.x; e < n / 2; e += T) {
                const int32_t i = ((e & ~(j - 1)) << 1) | (e & (j - 1)), o = i | j;
                const K x = s[i], y = s[o];
                if ((x > y) == ((i & k) == 0)) {
                    s[i] = y;
                    s[o] = x;
                }
            }
            __syncthreads();
        }
}

// Exclusive prefix of x over the T threads of a workgroup and the total (sw: one entry per wave).
template <int T> __device__ __forceinline__ int32_t block_prefix(int32_t x, int32_t *sw, int32_t &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t v = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(v, o, 64);
        if (lane >= o) v += y;
    }
    __syncthreads();
    if (lane == 63) sw[wave] = v;
    __syncthreads();
    int32_t off = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
        if (w < wave) off += sw[w];
        total += sw[w];
    }
    return off + v - x;
}

// The values of s[0, n) without ~0u and repeats of the one before into s[0, total), in order; n <= MAX.
template <int T, int MAX> __device__ __forceinline__ int32_t lds_distinct(uint32_t *s, int32_t n, int32_t *sw) {
    // every thread reads its stretch before any writes
    const int32_t per = (n + T - 1) / T, i0 = (int32_t)threadIdx.x * per;
    uint32_t keep[MAX / T];
    int32_t m = 0;
#pragma unroll
    for (int32_t u = 0; u < MAX / T; ++u) {
        const int32_t i = i0 + u;
        keep[u] = ~0u;
        if (u < per && i < n && s[i] != ~0u && (i == 0 || s[i] != s[i - 1])) {
            keep[u] = s[i];
            ++m;
        }
    }
    int32_t total = 0, at = block_prefix<T>(m, sw, total);   // its barriers part the reads from the writes
#pragma unroll
    for (int32_t u = 0; u < MAX / T; ++u)
        if (keep[u] != ~0u) s[at++] = keep[u];
    __syncthreads();
    return total;
}

}  // namespace ebbx
