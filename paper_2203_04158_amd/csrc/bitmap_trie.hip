// Bitmap trie: a GPU layout of the radix-2^k trie of Sec. IV in which every
// node is one record {base, bitmap of its occurring chunk values}.
//
// Chunks are dispatched from the most significant end (the top chunk holds
// M mod k bits when k does not divide M), so at every level the nodes, and
// the members under each node, come in ascending numeric order.  A node's
// children are then consecutive records of the next level, and the child
// for chunk value c is record base + (number of set bits below c); at the
// last level the same count gives the rank, base being the position of the
// node's first member in the sector's list.  A clear bit means the pattern
// is not a member, so membership needs no read of the state list (the
// packed trie of trie.hip checks states[rank] == alpha after its walk).
//
// Records are 2^s bytes (8 B for k <= 5, 16 B for k = 6, 32 B for k = 7,
// 64 B for k = 8), the same size on every level (the root's short chunk
// included, one record), aligned to their size, so a record never straddles a
// 64-byte line: one line per level and query.  Up to k = 5 a record is {base,
// map}.  From k = 6 on it is made of 16-byte parts, each {child or rank of the
// part's first chunk value, 96 bits of the map}, so that a step takes one
// 16-byte load whatever the chunk value, and up to three popcounts.  (A base,
// prefix bytes and the map apart took two loads a step, and the walks are bound
// by the rate of their scattered loads: 8,000,003 lookups of 64-bit patterns
// among 7.1 M states, k = 8, 143 -> 115 us; 2^24 in 32-bit patterns of a sector
// with 242,250 leaf records 258 -> 215 us.)  Queries in ascending order find their
// records in the nearest cache, and a lookup is then bound by the issue of its vector
// instructions, 18 a step: 2^24 of them among the C(28, N) states for N = 6 to 14 take
// 53 us, with 25 a step 63 us, with base, prefix bytes and map apart 56 us.
// The top levels that fit 48 KB are staged in LDS; large batches on a trie whose
// next level fits 144 KB run with one or two workgroups of 1024 lanes per CU that
// stage that level too.  With k = 8 the sector
// M = 32, N = 16 with >= 6 of orbitals 0-7 occupied needs about 4 M leaf
// records (its packed trie holds 332 M entries).
#include <algorithm>
#include <memory>

#include "level_scan.hpp"
#include "rank_device.hpp"

namespace {

constexpr unsigned kBlock = 256;
constexpr int kQ = 4;                      // independent walks in flight per lane
constexpr size_t kLdsBudget = 48 * 1024;   // bytes of top levels staged per workgroup
constexpr unsigned kWideBlock = 1024;
constexpr size_t kWideBudget = 144 * 1024; // the same for a workgroup of kWideBlock lanes, which has a CU to itself
constexpr size_t kHalfCu = 80 * 1024;      // or shares it with one more up to here: 51 KB, 2^24 queries in order 62 -> 54 us
// Batch from which the wider staging is taken: 8,000,003 lookups (36 orbitals,
// k = 8, three levels in memory against two) 165 -> 143 us, 1,000,003 25.0 -> 24.1,
// 300,003 13.0 either way.  Queries in order gain nothing from it (98,280 states,
// k = 8: 2^24 in 53 -> 58 us, 2^22 in 17 -> 18; scattered 106 -> 83 and 30 -> 25).
constexpr uint64_t kWideMin = 1 << 19;
constexpr int kMaxH = 32;

// A level: its first word, the bit offset of its chunk, and the chunk's bits: all of
// them (8-byte records) or those above the lowest five (others).
struct alignas(16) BtLevel {
    uint32_t off, shift, wid, none;
};

struct BtArgs {
    const uint32_t *rec;      // all levels' records, level after level
    int32_t M, H, lds_levels;
    uint32_t lds_words;       // words of the staged levels
    BtLevel level[kMaxH];
};

constexpr uint32_t kPartBits = 96;  // chunk values per 16-byte part (records of 4 words and more)

// Part of a record that holds chunk value c < 256.
__host__ __device__ constexpr uint32_t part_of(uint32_t c) { return (c * 683u) >> 16; }
static_assert(part_of(95) == 0 && part_of(96) == 1 && part_of(191) == 1 && part_of(192) == 2 && part_of(255) == 2, "c / 96");

// Word of a record of rw words that holds the bit of chunk value c, and the bit.
__host__ __device__ constexpr uint32_t map_word(uint32_t rw, uint32_t c) {
    return rw == 2 ? 1 : 4 * part_of(c) + 1 + (c - kPartBits * part_of(c)) / 32;
}
__host__ __device__ constexpr uint32_t map_bit(uint32_t c) { return c % 32; }  // 96 is a multiple of 32

// What a step reads of a record: {base, map} or the 16-byte part of chunk value
// c; and its answer: whether c occurs, and the child or rank counted from one,
// base + set bits up to c.  The words are combined with masks, not chosen by
// branches, which would put the loads of the walks that advance together one after
// another; which words of the part lie below c's follows from a table with a bit per
// word of the map, its place from one with a byte per word.
template <int RW>
struct BtPart {
    uint4 v;
    uint32_t w;  // word of the map that holds c's bit
    // the record starts at rec[at]
    __device__ __forceinline__ void load(const uint32_t *rec, uint32_t at, uint32_t c, uint32_t wid) {
        if constexpr (RW == 2) {
            const uint2 h = *reinterpret_cast<const uint2 *>(rec + at);
            v = make_uint4(h.x, h.y, 0, 0);
        } else {
            w = __builtin_amdgcn_ubfe(c, 5, wid);
            if constexpr (RW > 4) at += __builtin_amdgcn_perm(0x08080404u, 0x04000000u, w);
            v = *reinterpret_cast<const uint4 *>(rec + at);
        }
    }
    __device__ __forceinline__ bool step(uint32_t c, uint32_t &next) const {
        uint32_t own = v.y;
        next = v.x;
        if constexpr (RW > 2) {
            const uint32_t past0 = (uint32_t)__builtin_amdgcn_sbfe(0xB6, w, 1);  // word 0 of the part is below c's
            own = (v.y & ~past0) | (v.z & past0);
            next += __popc(v.y & past0);
            if constexpr (RW > 4) {
                const uint32_t past1 = (uint32_t)__builtin_amdgcn_sbfe(0x24, w, 1);  // and word 1
                own = (own & ~past1) | (v.w & past1);
                next += __popc(v.z & past1);
            }
        }
        const uint32_t upto = own << (~c & 31u);  // c's bit on top, those below it
        next += __popc(upto);
        return (int32_t)upto < 0;
    }
};

template <class P, int RW, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK) bt_rank_kernel(const P *__restrict__ q, uint64_t n,
                                                         uint32_t *__restrict__ out, BtArgs a) {
    extern __shared__ __align__(16) uint32_t top[];
    stage_to_lds(top, a.rec, (uint64_t)a.lds_words * 4);
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const P beyond = a.M >= (int)(8 * sizeof(P)) ? (P)0 : (P)(~(P)0 << a.M);
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; base < n; base += stride * kQ) {
        P x[kQ];
        uint32_t node[kQ];  // counted from one
        bool ok[kQ];
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t j = base + u * stride;
            x[u] = q[j < n ? j : n - 1];  // a branch would have each load wait for the one before
        }
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            ok[u] = (x[u] & beyond) == 0;
            node[u] = 1;
        }
        // staged levels from LDS, the rest through the caches; a walk that
        // leaves the sector stays on the first record of each further level
        auto advance = [&](const uint32_t *rec, const BtLevel &v) {
            const uint32_t first = v.off - RW;
            uint32_t c[kQ];
            BtPart<RW> part[kQ];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                // the chunk; from k = 6 on with what lies above it, which the step leaves out
                c[u] = RW == 2 ? (uint32_t)(x[u] >> v.shift) & ((1u << v.wid) - 1u) : (uint32_t)(x[u] >> v.shift);
                part[u].load(rec, node[u] * RW + first, c[u], v.wid);  // words < 2^32
            }
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                uint32_t nx;
                const bool occurs = part[u].step(c[u], nx);
                ok[u] = ok[u] && occurs;
                node[u] = ok[u] ? nx : 1u;
            }
        };
        int l = 0;
        for (; l < a.lds_levels; ++l) advance(top, a.level[l]);
        for (; l < a.H; ++l) advance(a.rec, a.level[l]);
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t j = base + u * stride;
            if (j < n) out[j] = ok[u] ? node[u] - 1 : MBR_NOT_FOUND;
        }
    }
}

// Words of a record for k-bit chunks: {base, map}, or its 16-byte parts rounded
// up to a power of two.
uint32_t record_words(int w) { return w <= 5 ? 2 : w == 6 ? 4 : w == 7 ? 8 : 16; }

// ------------------------------------------------------------------ building
// The list is in ascending order, so the members under a node are consecutive
// on every level and the nodes come in the order of their records: a node
// starts where the bits above its chunk differ from the member before, and its
// record's index is the number of starts before it.  One pass counts the starts
// per tile and level, one writes each record's base (by the node's first
// member) and sets its map's bits (by the first member of each chunk value), one
// gives the later parts their bases.  7.1 M 64-bit patterns in five levels: 0.23 ms
// with the allocations; on the host, with both copies, 75 ms.
struct BtLevels {
    int32_t H;
    uint32_t rw;              // words per record
    int32_t shift[kMaxH + 1]; // bit offset of level l's chunk; shift[H] = 0 (below the last)
    uint32_t off[kMaxH];
    uint32_t cmask[kMaxH];
};

// Whether a member whose bits differ by dp from the member before starts a node
// of the level whose chunk's top lies at bit `up`.
template <class P>
__device__ __forceinline__ bool starts(P dp, int up, uint64_t i) {
    return i == 0 || (up < (int)(8 * sizeof(P)) && (dp >> up) != 0);
}

// Bit above level l's chunk.
__device__ __forceinline__ int above(const BtLevels &v, int l, int M) { return l == 0 ? M : v.shift[l - 1]; }

// Starts in tile blockIdx.x, level by level: sums[l * tiles + tile].
template <class P>
__global__ void __launch_bounds__(kLevelBlock) bt_count_kernel(const P *__restrict__ key, uint64_t n, int M, BtLevels v, uint32_t *__restrict__ sums) {
    __shared__ uint32_t red[kLevelBlock / 64];
    const uint64_t i0 = (uint64_t)blockIdx.x * kLevelTile + threadIdx.x * kLevelItems;
    P a[kLevelItems], dp[kLevelItems], dn[kLevelItems];
    load_members<P>(key, n, i0, a, dp, dn);
    for (int l = 0; l < v.H; ++l) {
        uint32_t s = 0, all;
#pragma unroll
        for (unsigned k = 0; k < kLevelItems; ++k) s += i0 + k < n && starts<P>(dp[k], above(v, l, M), i0 + k) ? 1u : 0u;
        (void)block_before<uint32_t, kLevelBlock>(s, red, &all);
        if (threadIdx.x == 0) sums[(uint64_t)l * gridDim.x + blockIdx.x] = all;
    }
}

template <class P>
__global__ void __launch_bounds__(kLevelBlock) bt_fill_kernel(const P *__restrict__ key, uint64_t n, int M, BtLevels v,
                                                              const uint32_t *__restrict__ sums, uint32_t *__restrict__ rec) {
    __shared__ uint32_t red[kLevelBlock / 64];
    const uint64_t i0 = (uint64_t)blockIdx.x * kLevelTile + threadIdx.x * kLevelItems;
    P a[kLevelItems], dp[kLevelItems], dn[kLevelItems];
    load_members<P>(key, n, i0, a, dp, dn);
    uint32_t node[kLevelItems], child[kLevelItems];
#pragma unroll
    for (unsigned k = 0; k < kLevelItems; ++k) node[k] = 0;  // the root
    for (int l = 0; l < v.H; ++l) {
        if (l + 1 < v.H) {
            uint32_t s = 0, all;
#pragma unroll
            for (unsigned k = 0; k < kLevelItems; ++k) s += i0 + k < n && starts<P>(dp[k], v.shift[l], i0 + k) ? 1u : 0u;
            uint32_t run = block_before<uint32_t, kLevelBlock>(s, red, &all) + sums[(uint64_t)(l + 1) * gridDim.x + blockIdx.x];
#pragma unroll
            for (unsigned k = 0; k < kLevelItems; ++k) {
                run += i0 + k < n && starts<P>(dp[k], v.shift[l], i0 + k) ? 1u : 0u;
                child[k] = run - 1;  // the member's node on the next level
            }
        } else {
#pragma unroll
            for (unsigned k = 0; k < kLevelItems; ++k) child[k] = (uint32_t)(i0 + k);
        }
#pragma unroll
        for (unsigned k = 0; k < kLevelItems; ++k) {
            if (i0 + k < n) {
                uint32_t *r = rec + v.off[l] + (uint64_t)node[k] * v.rw;
                if (starts<P>(dp[k], above(v, l, M), i0 + k)) r[0] = child[k];
                if (starts<P>(dp[k], v.shift[l], i0 + k)) {
                    const uint32_t c = (uint32_t)(a[k] >> v.shift[l]) & v.cmask[l];
                    atomicOr(r + map_word(v.rw, c), 1u << map_bit(c));
                }
            }
            node[k] = child[k];
        }
    }
}

// What the later parts of the records from `rec` on start from.
__global__ void __launch_bounds__(kBlock) bt_parts_kernel(uint32_t *rec, uint64_t records, uint32_t rw, uint32_t parts) {
    const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (i >= records) return;
    uint32_t *r = rec + i * rw;
    uint32_t base = r[0];
    for (uint32_t p = 1; p < parts; ++p) {
        const uint32_t *q = r + 4 * (p - 1);
        base += __popc(q[1]) + __popc(q[2]) + __popc(q[3]);
        r[4 * p] = base;
    }
}

template <class P>
mbr_status build_records(BitmapTrie &t, const mbr_sector *sec, hipStream_t s) {
    using namespace mbr;
    const int H = t.H, kw = *std::max_element(t.w, t.w + H);
    const uint64_t n = sec->n, tiles = (n + kLevelTile - 1) / kLevelTile;
    const P *key = sec->states.as<P>();
    BtLevels v{};
    v.H = H;
    v.rw = record_words(kw);  // one record size for all levels (the root's short chunk included)
    for (int l = 0; l < H; ++l) {
        v.shift[l] = t.shift[l];
        v.cmask[l] = (1u << t.w[l]) - 1u;
    }
    DevBuf scratch;  // starts per level and tile, then per level
    MBR_TRY(scratch.alloc((tiles * H + H) * 4));
    uint32_t *sums = scratch.as<uint32_t>(), *totals = sums + tiles * H;
    bt_count_kernel<P><<<(unsigned)tiles, kLevelBlock, 0, s>>>(key, n, t.M, v, sums);
    row_scan_kernel<uint32_t><<<H, 1024, 0, s>>>(sums, tiles, totals);
    MBR_HIP(hipGetLastError());
    uint32_t nodes[kMaxH] = {0};
    MBR_HIP(hipMemcpyAsync(nodes, totals, (size_t)H * 4, hipMemcpyDeviceToHost, s));
    MBR_HIP(hipStreamSynchronize(s));
    uint64_t words = 0;
    for (int l = 0; l < H; ++l) {
        t.rw[l] = v.rw;
        words = (words + 15) & ~(uint64_t)15;  // every level starts on a 64-byte line
        t.off[l] = words;
        t.nodes[l] = nodes[l];
        words += (uint64_t)nodes[l] * v.rw;
    }
    t.off[H] = words;
    if (words >= (1ull << 32)) MBR_FAIL(MBR_EUNSUPPORTED, "bitmap trie of %llu words", (unsigned long long)words);
    for (int l = 0; l < H; ++l) v.off[l] = (uint32_t)t.off[l];
    MBR_TRY(t.table.alloc(words * 4));
    uint32_t *rec = t.table.as<uint32_t>();
    MBR_HIP(hipMemsetAsync(rec, 0, words * 4, s));
    bt_fill_kernel<P><<<(unsigned)tiles, kLevelBlock, 0, s>>>(key, n, t.M, v, sums, rec);
    const uint32_t parts = kw == 8 ? 3 : kw == 7 ? 2 : 1;
    for (int l = 0; l < H && parts > 1; ++l)
        bt_parts_kernel<<<(unsigned)((nodes[l] + (uint64_t)kBlock - 1) / kBlock), kBlock, 0, s>>>(rec + t.off[l], nodes[l], v.rw, parts);
    MBR_HIP(hipGetLastError());
    uint64_t lw = 0;
    int ll = 0;
    while (ll < H && (t.off[ll + 1]) * 4 <= kLdsBudget) {
        lw = t.off[ll + 1];
        ++ll;
    }
    t.lds_levels = ll;
    t.lds_words = lw;
    while (ll < H && (t.off[ll + 1]) * 4 <= kWideBudget) {
        lw = t.off[ll + 1];
        ++ll;
    }
    t.wide_levels = ll;
    t.wide_words = lw;
    MBR_HIP(hipStreamSynchronize(s));  // the trie is ready for any stream, and the scratch is free
    return MBR_OK;
}

template <class P, int RW, unsigned BLOCK>
mbr_status run_bt(const P *q, uint64_t n, uint32_t *out, const BtArgs &a, hipStream_t s) {
    auto kern = bt_rank_kernel<P, RW, BLOCK>;
    const size_t lds = (size_t)a.lds_words * 4;
    if (lds > 64 * 1024)
        MBR_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideBudget));
    const unsigned grid = mbr::grid_for(n, BLOCK * kQ, mbr::device_cu_count() * (BLOCK == kWideBlock ? (lds > kHalfCu ? 1 : 2) : 8));
    kern<<<grid, BLOCK, lds, s>>>(q, n, out, a);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

template <class P>
mbr_status launch_bt(const mbr_ranker *r, const void *q, uint64_t n, uint32_t *out, hipStream_t s) {
    const BitmapTrie &t = *r->btrie;
    BtArgs a{};
    a.rec = t.table.as<uint32_t>();
    a.M = t.M;
    a.H = t.H;
    a.lds_levels = t.lds_levels;
    a.lds_words = (uint32_t)t.lds_words;
    for (int l = 0; l < t.H; ++l) {
        a.level[l] = {(uint32_t)t.off[l], (uint32_t)t.shift[l], (uint32_t)(t.rw[0] == 2 ? t.w[l] : std::max(t.w[l] - 5, 0)), 0};
    }
    const bool wide = t.wide_levels > t.lds_levels && n >= kWideMin;
    if (wide) {
        a.lds_levels = t.wide_levels;
        a.lds_words = (uint32_t)t.wide_words;
    }
    const P *qp = static_cast<const P *>(q);
    switch (t.rw[0]) {
    case 2: return wide ? run_bt<P, 2, kWideBlock>(qp, n, out, a, s) : run_bt<P, 2, kBlock>(qp, n, out, a, s);
    case 4: return wide ? run_bt<P, 4, kWideBlock>(qp, n, out, a, s) : run_bt<P, 4, kBlock>(qp, n, out, a, s);
    case 8: return wide ? run_bt<P, 8, kWideBlock>(qp, n, out, a, s) : run_bt<P, 8, kBlock>(qp, n, out, a, s);
    default: return wide ? run_bt<P, 16, kWideBlock>(qp, n, out, a, s) : run_bt<P, 16, kBlock>(qp, n, out, a, s);
    }
}

}  // namespace

void bitmap_trie_free(BitmapTrie *t) { delete t; }

mbr_status rank_bitmap_trie_launch(const mbr_ranker *r, const void *q, uint64_t n, uint32_t *out,
                                   hipStream_t s) {
    if (r->width_bits == 32) return launch_bt<uint32_t>(r, q, n, out, s);
    return launch_bt<uint64_t>(r, q, n, out, s);
}

extern "C" mbr_status mbr_build_bitmap_trie(const mbr_sector *sec, int32_t k, mbr_ranker **out, void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (!sec) MBR_FAIL(MBR_EINVAL, "null sector");
    if (k < 1 || k > 8) MBR_FAIL(MBR_EINVAL, "k=%d outside 1..8", k);
    if (sec->n == 0) MBR_FAIL(MBR_EINVAL, "empty sector");
    if (sec->n >= 0xFFFFFFFFull) MBR_FAIL(MBR_ERANGE, "sector of %llu states", (unsigned long long)sec->n);
    const int M = sec->M;
    const int H = (M + k - 1) / k;
    if (H > kMaxH) MBR_FAIL(MBR_EUNSUPPORTED, "%d levels (at most %d)", H, kMaxH);
    hipStream_t s = as_stream(stream);
    auto t = std::make_unique<BitmapTrie>();
    t->M = M;
    t->H = H;
    // widths from the top: the short chunk first, then k bits each
    for (int l = 0, below = M; l < H; ++l) {
        t->w[l] = l == 0 ? M - (H - 1) * k : k;
        below -= t->w[l];
        t->shift[l] = below;
    }
    if (sec->width_bits == 32) MBR_TRY(build_records<uint32_t>(*t, sec, s));
    else MBR_TRY(build_records<uint64_t>(*t, sec, s));
    auto *r = new (std::nothrow) mbr_ranker;
    if (!r) MBR_FAIL(MBR_ENOMEM, "host allocation");
    r->kind = MBR_RANKER_BITMAP_TRIE;
    r->M = M;
    r->k = k;
    r->width_bits = sec->width_bits;
    r->n_states = sec->n;
    r->sector = sec;
    (void)hipGetDevice(&r->device);
    r->btrie = t.release();
    *out = r;
    return MBR_OK;
}

extern "C" mbr_status mbr_bitmap_trie_levels(const mbr_ranker *r, uint64_t *records, uint32_t *record_bytes,
                                             int32_t cap, int32_t *levels, int32_t *lds_levels) {
    if (!r || r->kind != MBR_RANKER_BITMAP_TRIE || !r->btrie) MBR_FAIL(MBR_EINVAL, "not a bitmap trie ranker");
    const BitmapTrie &t = *r->btrie;
    if (levels) *levels = t.H;
    if (lds_levels) *lds_levels = t.lds_levels;
    for (int l = 0; l < t.H && l < cap; ++l) {
        if (records) records[l] = t.nodes[l];
        if (record_bytes) record_bytes[l] = 4 * t.rw[l];
    }
    return MBR_OK;
}
