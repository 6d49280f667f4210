// Passes over a sector's members in order that build a trie's levels (trie.hip,
// bitmap_trie.hip): a lane takes kLevelItems consecutive members, a workgroup
// a tile of them, and running sums over all members are made of sums per
// tile (one row per level, scanned by row_scan_kernel) and within the tile.
#pragma once

#include "common.hpp"

namespace {

constexpr unsigned kLevelBlock = 256, kLevelItems = 8;
constexpr uint32_t kLevelTile = kLevelBlock * kLevelItems;

// Exclusive sum of v over the workgroup (B lanes); *all receives the total.
template <class V, unsigned B>
__device__ __forceinline__ V block_before(V v, V *red, V *all) {
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    V s = v;
    for (int o = 1; o < 64; o <<= 1) {
        const V u = __shfl_up(s, o, 64);
        if (lane >= (uint32_t)o) s += u;
    }
    __syncthreads();  // red's previous readers are done
    if (lane == 63) red[w] = s;
    __syncthreads();
    V before = 0, total = 0;
    for (uint32_t k = 0; k < B / 64; ++k) {
        if (k < w) before += red[k];
        total += red[k];
    }
    *all = total;
    return before + s - v;
}

// Row blockIdx.x of v (n values) to exclusive sums in place, its total to
// totals[row].
template <class V>
__global__ void __launch_bounds__(1024) row_scan_kernel(V *v, uint64_t n, V *totals) {
    __shared__ V red[16];
    V *row = v + (uint64_t)blockIdx.x * n;
    V run = 0;
    for (uint64_t i0 = 0; i0 < n; i0 += 1024) {
        const uint64_t i = i0 + threadIdx.x;
        const V x = i < n ? row[i] : (V)0;
        V all;
        const V e = block_before<V, 1024>(x, red, &all);
        if (i < n) row[i] = run + e;
        run += all;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = run;
}

template <class P>
__device__ __forceinline__ P low_bits(int n) {
    return n >= (int)(8 * sizeof(P)) ? (P)~(P)0 : (P)(((P)1 << n) - 1);
}

// A lane's consecutive members, and the bits in which each differs from the
// member before (dp) and after (dn), all ones at the ends.
template <class P>
__device__ __forceinline__ void load_members(const P *__restrict__ key, uint64_t n, uint64_t i0, P (&a)[kLevelItems], P (&dp)[kLevelItems],
                                             P (&dn)[kLevelItems]) {
    P e[kLevelItems + 2];
#pragma unroll
    for (unsigned k = 0; k < kLevelItems + 2; ++k) {
        const uint64_t i = i0 + k;  // member i - 1
        e[k] = i > 0 && i <= n ? key[i - 1] : (P)0;
    }
#pragma unroll
    for (unsigned k = 0; k < kLevelItems; ++k) {
        const uint64_t i = i0 + k;
        a[k] = e[k + 1];
        dp[k] = i == 0 ? (P)~(P)0 : (P)(e[k] ^ e[k + 1]);
        dn[k] = i + 1 >= n ? (P)~(P)0 : (P)(e[k + 2] ^ e[k + 1]);
    }
}

}  // namespace
