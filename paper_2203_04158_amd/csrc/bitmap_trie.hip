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
// with 242,250 leaf records 258 -> 215 us.)
// The top levels that fit 48 KB are staged in LDS; large batches on a trie whose
// next level fits 144 KB run with one workgroup of 1024 lanes per CU that stages
// that level too.  With k = 8 the sector
// M = 32, N = 16 with >= 6 of orbitals 0-7 occupied needs about 4 M leaf
// records (its packed trie holds 332 M entries).
#include <algorithm>
#include <cstring>
#include <memory>

#include "rank_device.hpp"

namespace {

constexpr unsigned kBlock = 256;
constexpr int kQ = 4;                      // independent walks in flight per lane
constexpr size_t kLdsBudget = 48 * 1024;   // bytes of top levels staged per workgroup
constexpr unsigned kWideBlock = 1024;
constexpr size_t kWideBudget = 144 * 1024; // the same for a workgroup that has a CU to itself
// Batch from which the wider staging is taken: 8,000,003 lookups (36 orbitals,
// k = 8, three levels in memory against two) 165 -> 143 us, 1,000,003 25.0 -> 24.1,
// 300,003 13.0 either way.
constexpr uint64_t kWideMin = 1 << 19;
constexpr int kMaxH = 32;

struct BtArgs {
    const uint32_t *rec;      // all levels' records, level after level
    int32_t M, H, lds_levels;
    uint32_t lds_words;       // words of the staged levels
    uint32_t off[kMaxH];      // first word of each level
    uint32_t shift[kMaxH];    // bit offset of each level's chunk
    uint32_t cmask[kMaxH];    // chunk mask
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
// c; and its answer: whether c occurs, and the child or rank, base + set bits
// below c.  The words are combined with masks, not chosen by branches, which
// would put the loads of the walks that advance together one after another.
template <int RW>
struct BtPart {
    uint4 v;
    __device__ __forceinline__ void load(const uint32_t *rec, uint32_t c) {
        if constexpr (RW == 2) {
            const uint2 h = *reinterpret_cast<const uint2 *>(rec);
            v = make_uint4(h.x, h.y, 0, 0);
        } else {
            v = *reinterpret_cast<const uint4 *>(rec + (RW == 4 ? 0u : 4 * part_of(c)));
        }
    }
    __device__ __forceinline__ bool step(uint32_t c, uint32_t &next) const {
        const uint32_t bit = 1u << map_bit(c), below = bit - 1u;
        if constexpr (RW == 2) {
            next = v.x + __popc(v.y & below);
            return (v.y & bit) != 0;
        } else {
            const uint32_t word = RW == 4 ? c >> 5 : (c >> 5) - 3 * part_of(c);
            const uint32_t past0 = word > 0 ? ~0u : 0u, past1 = RW > 4 && word > 1 ? ~0u : 0u;  // whole words below c's
            uint32_t own = (v.y & ~past0) | (v.z & past0);
            next = v.x + __popc(v.y & past0);
            if constexpr (RW > 4) {
                own = (own & ~past1) | (v.w & past1);
                next += __popc(v.z & past1);
            }
            next += __popc(own & below);
            return (own & bit) != 0;
        }
    }
};

template <class P, int RW, unsigned BLOCK>
__global__ void __launch_bounds__(BLOCK) bt_rank_kernel(const P *__restrict__ q, uint64_t n,
                                                         uint32_t *__restrict__ out, BtArgs a) {
    extern __shared__ __align__(16) uint32_t top[];
    stage_to_lds(top, a.rec, (uint64_t)a.lds_words * 4);
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; base < n; base += stride * kQ) {
        P x[kQ];
        uint32_t node[kQ];
        bool ok[kQ];
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t j = base + u * stride;
            x[u] = j < n ? q[j] : (P)0;
            ok[u] = j < n && (a.M >= (int)(8 * sizeof(P)) || (x[u] >> a.M) == 0);
            node[u] = 0;
        }
        // staged levels from LDS, the rest through the caches; a walk that
        // leaves the sector stays on record 0 of each further level
        auto advance = [&](const uint32_t *lv, int l) {
            uint32_t c[kQ];
            BtPart<RW> part[kQ];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                c[u] = (uint32_t)(x[u] >> a.shift[l]) & a.cmask[l];
                part[u].load(lv + node[u] * RW, c[u]);  // words < 2^32
            }
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                uint32_t nx;
                const bool occurs = part[u].step(c[u], nx);
                ok[u] = ok[u] && occurs;
                node[u] = ok[u] ? nx : 0u;
            }
        };
        int l = 0;
        for (; l < a.lds_levels; ++l) {
            advance(top + a.off[l], l);
        }
        for (; l < a.H; ++l) {
            advance(a.rec + a.off[l], l);
        }
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t j = base + u * stride;
            if (j < n) out[j] = ok[u] ? node[u] : MBR_NOT_FOUND;
        }
    }
}

// Words of a record for k-bit chunks: {base, map}, or its 16-byte parts rounded
// up to a power of two.
uint32_t record_words(int w) { return w <= 5 ? 2 : w == 6 ? 4 : w == 7 ? 8 : 16; }

// Records of every level from the ascending list (one counting pass, one
// filling pass).
template <class P>
mbr_status build_records(BitmapTrie &t, const std::vector<P> &s) {
    const int H = t.H;
    std::vector<uint64_t> nodes(H, 0);
    for (int l = 0; l < H; ++l) {
        const int up = t.shift[l] + t.w[l];
        P prev = 0;
        uint64_t cnt = 0;
        for (size_t i = 0; i < s.size(); ++i) {
            const P pre = up >= (int)(8 * sizeof(P)) ? (P)0 : (P)(s[i] >> up);
            if (i == 0 || pre != prev) ++cnt;
            prev = pre;
        }
        nodes[l] = cnt;
    }
    uint64_t words = 0;
    const int kw = *std::max_element(t.w, t.w + H);
    for (int l = 0; l < H; ++l) {
        t.rw[l] = record_words(kw);  // one record size for all levels (the root's short chunk included)
        words = (words + 15) & ~(uint64_t)15;  // every level starts on a 64-byte line
        t.off[l] = words;
        t.nodes[l] = nodes[l];
        words += nodes[l] * t.rw[l];
    }
    t.off[H] = words;
    if (words >= (1ull << 32)) MBR_FAIL(MBR_EUNSUPPORTED, "bitmap trie of %llu words", (unsigned long long)words);
    std::vector<uint32_t> rec(words, 0u);
    std::vector<int64_t> cur(H, -1);
    std::vector<P> prev(H, 0);
    for (size_t i = 0; i < s.size(); ++i) {
        const P a = s[i];
        for (int l = 0; l < H; ++l) {
            const int up = t.shift[l] + t.w[l];
            const P pre = up >= (int)(8 * sizeof(P)) ? (P)0 : (P)(a >> up);
            if (cur[l] < 0 || pre != prev[l]) {
                ++cur[l];
                prev[l] = pre;
                // first child of a new node: the next record of the level
                // below (created for this member in the same pass), or at the
                // last level the position of its first member
                rec[t.off[l] + (uint64_t)cur[l] * t.rw[l]] = l + 1 < H ? (uint32_t)(cur[l + 1] + 1) : (uint32_t)i;
            }
            const uint32_t c = (uint32_t)(a >> t.shift[l]) & ((1u << t.w[l]) - 1u);
            rec[t.off[l] + (uint64_t)cur[l] * t.rw[l] + map_word(t.rw[l], c)] |= 1u << map_bit(c);
        }
    }
    // what the later parts of a record start from
    const uint32_t parts = kw == 8 ? 3 : kw == 7 ? 2 : 1;
    for (int l = 0; l < H; ++l)
        for (uint64_t nd = 0; nd < nodes[l] && parts > 1; ++nd) {
            uint32_t *r = rec.data() + t.off[l] + nd * t.rw[l];
            for (uint32_t p = 1; p < parts; ++p) {
                const uint32_t *q = r + 4 * (p - 1);
                r[4 * p] = q[0] + (uint32_t)(__builtin_popcount(q[1]) + __builtin_popcount(q[2]) + __builtin_popcount(q[3]));
            }
        }
    MBR_TRY(t.table.alloc(words * 4));
    MBR_HIP(hipMemcpy(t.table.p, rec.data(), words * 4, hipMemcpyHostToDevice));
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
    return MBR_OK;
}

template <class P, int RW, unsigned BLOCK>
mbr_status run_bt(const P *q, uint64_t n, uint32_t *out, const BtArgs &a, hipStream_t s) {
    auto kern = bt_rank_kernel<P, RW, BLOCK>;
    const size_t lds = (size_t)a.lds_words * 4;
    if (lds > 64 * 1024)
        MBR_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideBudget));
    const unsigned grid = mbr::grid_for(n, BLOCK * kQ, mbr::device_cu_count() * (BLOCK == kWideBlock ? 1 : 8));
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
        a.off[l] = (uint32_t)t.off[l];
        a.shift[l] = (uint32_t)t.shift[l];
        a.cmask[l] = (1u << t.w[l]) - 1u;
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
    mbr_status st;
    if (sec->width_bits == 32) {
        std::vector<uint32_t> h(sec->n);
        MBR_HIP(hipMemcpyAsync(h.data(), sec->states.p, sec->n * 4, hipMemcpyDeviceToHost, s));
        MBR_HIP(hipStreamSynchronize(s));
        st = build_records<uint32_t>(*t, h);
    } else {
        std::vector<uint64_t> h(sec->n);
        MBR_HIP(hipMemcpyAsync(h.data(), sec->states.p, sec->n * 8, hipMemcpyDeviceToHost, s));
        MBR_HIP(hipStreamSynchronize(s));
        st = build_records<uint64_t>(*t, h);
    }
    if (st != MBR_OK) return st;
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
