// Packed radix-2^k tries (Sec. IV) for ranking in arbitrary sectors.
//
// Dispatch order is the paper's: chunk 0 holds the k least significant bits,
// chunk l the next k bits, and a final chunk the remaining M mod k bits, so a
// lookup is the chain of the trie-lookup figure: n <- T_0[chunk_0]; n <-
// T_l[n + chunk_l] for the middle levels; rank <- T_{H-1}[n + chunk_{H-1}].
//
// Layout (GPU-specific, not the paper's single depth-first array): one array
// per level, nodes of a level contiguous in the order of their prefixes, each
// node spanning only its first..last occurring chunk value (packing), the
// parent storing start - first (the index shifted back, as in the paper's
// packed form).  Each level array starts with 2^w - 1 zeros and ends with 2^w
// zeros, so stored indices are never negative and a walk with any pattern,
// member or not, stays inside the arrays; unused slots hold 0.  The root is a
// full 2^w0 array.  Membership: the walk's rank i is accepted only when
// i < N_s and states[i] == alpha (the check of Sec. IV).
//
// Level-major arrays keep every level's nodes together: the top levels fit
// LDS and are staged there, the middle levels stay in L2/MALL and only the
// leaf level and the membership check are HBM gathers.
#include <algorithm>
#include <memory>

#include "level_scan.hpp"
#include "rank_device.hpp"

void trie_free(TrieLevels *t) { delete t; }
uint64_t trie_bytes(const TrieLevels *t) { return t ? t->entries * 4 : 0; }
int32_t trie_levels(const TrieLevels *t) { return t ? t->H : 0; }

namespace {

constexpr unsigned kBlock = 256;
constexpr size_t kLdsBudget = 48 * 1024;  // bytes of top levels staged per workgroup
constexpr int kQ = 4;                       // independent walks in flight per lane

struct TrieArgs {
    const uint32_t *tab;
    const void *states;
    uint64_t ns;
    int32_t M, H;
    uint32_t lds_entries;
    int32_t lds_levels;
    uint32_t wmask[16];
    int32_t shift[16];
    uint64_t off[17];
};

template <class P>
__device__ __forceinline__ bool fits(P x, int M) {
    return (M >= (int)(8 * sizeof(P))) ? true : (x >> M) == 0;
}

template <class P>
__global__ void __launch_bounds__(kBlock) trie_rank_kernel(const P *__restrict__ q, uint64_t n,
                                                           uint32_t *__restrict__ out, TrieArgs a) {
    extern __shared__ __align__(16) uint32_t top[];
    stage_to_lds(top, a.tab, (uint64_t)a.lds_entries * 4);
    __syncthreads();
    const P *states = static_cast<const P *>(a.states);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t base = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; base < n;
         base += stride * kQ) {
        P x[kQ];
        uint32_t node[kQ];
        bool ok[kQ];
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t j = base + u * stride;
            x[u] = j < n ? q[j] : (P)0;
            ok[u] = j < n && fits(x[u], a.M);
            if (!ok[u]) x[u] = 0;
            node[u] = 0;
        }
        // the walks of kQ queries advance level by level side by side; the
        // staged levels and the rest are separate loops, so that LDS is read
        // with LDS loads and the arrays with global loads (one loop choosing
        // per level compiles to flat loads for both)
        int l = 0;
        for (; l < a.lds_levels; ++l) {
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                const uint32_t c = (uint32_t)(x[u] >> a.shift[l]) & a.wmask[l];
                node[u] = top[a.off[l] + node[u] + c];
            }
        }
        for (; l < a.H; ++l) {
            const uint32_t *lv = a.tab + a.off[l];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                const uint32_t c = (uint32_t)(x[u] >> a.shift[l]) & a.wmask[l];
                node[u] = lv[node[u] + c];
            }
        }
        P hit[kQ];
#pragma unroll
        for (int u = 0; u < kQ; ++u) hit[u] = node[u] < a.ns ? states[node[u]] : (P)~x[u];
#pragma unroll
        for (int u = 0; u < kQ; ++u) {
            const uint64_t j = base + u * stride;
            if (j < n) out[j] = (ok[u] && hit[u] == x[u]) ? node[u] : MBR_NOT_FOUND;
        }
    }
}

// ------------------------------------------------------------------ building
// The trie is built on the device from the sector's list.  Its nodes follow the
// order of the chunk-reversed patterns (chunk 0 first): a stable radix sort by
// the chunks, last to first, starting from the list, which is already in
// order of its last chunk.  In that order the members under a node are
// consecutive at every level, a node starts where the low bits up to its level
// differ from the member before, and its first entry follows from a running
// sum over the members (node_share).  tl_fill_kernel then writes every entry of
// every level once.
//
// Bound by launches, allocations and the sort's scattered writes (841,332
// states, k = 8: three passes of 26 us, then 34 us).  On the host the same work
// (a sort and two passes per level) and the copies both ways took most of a
// sector change: list, trie and a million ranks 12.8 -> 0.68 ms.
constexpr unsigned kSortBlock = 256, kSortItems = 16;       // a wave sorts 1024 consecutive members
constexpr uint32_t kSortTile = kSortBlock * kSortItems;
constexpr int kDigits = 256;
constexpr int kMaxH = 16;

// Members of tile blockIdx.x by digit: counts[digit * tiles + tile].
template <class P>
__global__ void __launch_bounds__(kSortBlock) tl_count_kernel(const P *__restrict__ key, uint64_t n, int shift, uint32_t mask,
                                                              uint32_t *__restrict__ counts) {
    __shared__ uint32_t c[kDigits];
    for (int d = threadIdx.x; d < kDigits; d += kSortBlock) c[d] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile;
    for (unsigned k = 0; k < kSortItems; ++k) {
        const uint64_t i = base + k * kSortBlock + threadIdx.x;
        if (i < n) atomicAdd(&c[(uint32_t)(key[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < kDigits; d += kSortBlock) counts[(uint64_t)d * gridDim.x + blockIdx.x] = c[d];
}

// One stable pass: member i of a tile goes behind all members of smaller
// digits, those of its digit in earlier tiles, and those before it in its own.
// idx = nullptr: the members still stand at their positions in the list.
template <class P>
__global__ void __launch_bounds__(kSortBlock) tl_scatter_kernel(const P *__restrict__ key, const uint32_t *__restrict__ idx,
                                                                uint64_t n, int shift, uint32_t mask,
                                                                const uint32_t *__restrict__ counts, const uint32_t *__restrict__ totals,
                                                                P *__restrict__ key_out, uint32_t *__restrict__ idx_out) {
    static_assert(kSortBlock == kDigits, "a lane per digit");
    __shared__ uint32_t at[kSortBlock / 64][kDigits];  // per wave and digit: count, then next position
    __shared__ uint32_t red[kSortBlock / 64];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (uint32_t k = 0; k < kSortBlock / 64; ++k) at[k][threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile + w * (kSortTile / (kSortBlock / 64)) + lane;
    P x[kSortItems];
#pragma unroll
    for (unsigned k = 0; k < kSortItems; ++k) {
        const uint64_t i = base + k * 64;
        x[k] = i < n ? key[i] : (P)0;
        if (i < n) atomicAdd(&at[w][(uint32_t)(x[k] >> shift) & mask], 1u);
    }
    __syncthreads();
    {
        const uint32_t d = threadIdx.x;
        uint32_t all;
        uint32_t pos = block_before<uint32_t, kSortBlock>(totals[d], red, &all) + counts[(uint64_t)d * gridDim.x + blockIdx.x];
        for (uint32_t k = 0; k < kSortBlock / 64; ++k) {
            const uint32_t c = at[k][d];
            at[k][d] = pos;
            pos += c;
        }
    }
    __syncthreads();
    for (unsigned k = 0; k < kSortItems; ++k) {
        const uint64_t i = base + k * 64;
        const bool in = i < n;
        const uint32_t d = (uint32_t)(x[k] >> shift) & mask;
        uint64_t peers = __ballot(in);  // lanes of this step with the same digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t m = __ballot((d >> b) & 1);
            peers &= ((d >> b) & 1) ? m : ~m;
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0));
        const uint32_t pos = at[w][d] + before;
        wave_lds_fence();
        if (in && before == 0) at[w][d] += (uint32_t)__popcll(peers);
        wave_lds_fence();
        if (in) {
            key_out[pos] = x[k];
            idx_out[pos] = idx ? idx[i] : (uint32_t)i;
        }
    }
}

struct LevelArgs {
    int32_t H;
    int32_t shift[kMaxH + 1];  // shift[H] = M
    int32_t w[kMaxH];
    uint64_t off[kMaxH];
};

// What a member adds to the running sum of level l: the slots of its node (last
// chunk - first chunk + 1), the first chunk taken off at the node's first
// member, the rest added at its last.  `dp`, `dn` as from
// load_members.
template <class P>
__device__ __forceinline__ int64_t node_share(P a, P dp, P dn, int l, const LevelArgs &v) {
    const P lm = low_bits<P>(v.shift[l]);
    const int64_t c = (int64_t)((a >> v.shift[l]) & low_bits<P>(v.w[l]));
    return ((dn & lm) ? c + 1 : 0) - ((dp & lm) ? c : 0);
}

// Sums of node_share over tile blockIdx.x, levels 1 .. H-1: sums[(l-1) * tiles + tile].
template <class P>
__global__ void __launch_bounds__(kLevelBlock) tl_sums_kernel(const P *__restrict__ key, uint64_t n, LevelArgs v, int64_t *__restrict__ sums) {
    __shared__ int64_t red[kLevelBlock / 64];
    const uint64_t i0 = (uint64_t)blockIdx.x * kLevelTile + threadIdx.x * kLevelItems;
    P a[kLevelItems], dp[kLevelItems], dn[kLevelItems];
    load_members<P>(key, n, i0, a, dp, dn);
    for (int l = 1; l < v.H; ++l) {
        int64_t s = 0, all;
#pragma unroll
        for (unsigned k = 0; k < kLevelItems; ++k)
            if (i0 + k < n) s += node_share<P>(a[k], dp[k], dn[k], l, v);
        (void)block_before<int64_t, kLevelBlock>(s, red, &all);
        if (threadIdx.x == 0) sums[(uint64_t)(l - 1) * gridDim.x + blockIdx.x] = all;
    }
}

// Every entry of every level.  A node's index shifted back by its first chunk
// is 2^w - 1 (the front padding) plus the slots of the nodes before it minus that
// chunk, which is what the running sum stands at behind the node's first
// member.  The first member of each (node, chunk) pair writes the pair's entry:
// the child's shifted index, or at the last level its own position.
template <class P>
__global__ void __launch_bounds__(kLevelBlock) tl_fill_kernel(const P *__restrict__ key, const uint32_t *__restrict__ idx, uint64_t n,
                                                              LevelArgs v, const int64_t *__restrict__ sums, uint32_t *__restrict__ tab) {
    __shared__ int64_t red[kLevelBlock / 64];
    const uint64_t i0 = (uint64_t)blockIdx.x * kLevelTile + threadIdx.x * kLevelItems;
    P a[kLevelItems], dp[kLevelItems], dn[kLevelItems];
    load_members<P>(key, n, i0, a, dp, dn);
    uint32_t node[kLevelItems], child[kLevelItems];
#pragma unroll
    for (unsigned k = 0; k < kLevelItems; ++k) node[k] = 0;  // the root
    for (int l = 0; l < v.H; ++l) {
        const bool last = l + 1 == v.H;
        if (!last) {
            int64_t s = 0, all;
#pragma unroll
            for (unsigned k = 0; k < kLevelItems; ++k)
                if (i0 + k < n) s += node_share<P>(a[k], dp[k], dn[k], l + 1, v);
            int64_t run = block_before<int64_t, kLevelBlock>(s, red, &all) + sums[(uint64_t)l * gridDim.x + blockIdx.x];
            const P lm = low_bits<P>(v.shift[l + 1]);
            const int64_t front = ((int64_t)1 << v.w[l + 1]) - 1;
#pragma unroll
            for (unsigned k = 0; k < kLevelItems; ++k) {
                const int64_t c = (int64_t)((a[k] >> v.shift[l + 1]) & low_bits<P>(v.w[l + 1]));
                child[k] = (uint32_t)(front + run - ((dp[k] & lm) ? c : 0));
                if (i0 + k < n) run += node_share<P>(a[k], dp[k], dn[k], l + 1, v);
            }
        }
        const P pair = low_bits<P>(v.shift[l + 1]);
#pragma unroll
        for (unsigned k = 0; k < kLevelItems; ++k) {
            const uint64_t i = i0 + k;
            if (i < n && (dp[k] & pair)) {
                const uint32_t c = (uint32_t)((a[k] >> v.shift[l]) & low_bits<P>(v.w[l]));
                tab[v.off[l] + node[k] + c] = last ? (idx ? idx[i] : (uint32_t)i) : child[k];
            }
            node[k] = child[k];
        }
    }
}

template <class P>
mbr_status build_levels(TrieLevels &t, const mbr_sector *sec, hipStream_t s) {
    using namespace mbr;
    const int M = t.M, H = t.H;
    const uint64_t n = sec->n;
    const uint64_t st = (n + kSortTile - 1) / kSortTile, lt = (n + kLevelTile - 1) / kLevelTile;
    if (st > 0x7FFFFFFFull) MBR_FAIL(MBR_ERANGE, "%llu states", (unsigned long long)n);
    // scratch: level sums and totals | two copies of the patterns and of their positions | digit counts and totals
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t o_tot = al((size_t)lt * kMaxH * 8), o_key = o_tot + al(kMaxH * 8), keyb = al(n * sizeof(P)), idxb = al(n * 4);
    const size_t o_idx = o_key + 2 * keyb, o_cnt = o_idx + 2 * idxb, o_dig = o_cnt + al((size_t)st * kDigits * 4);
    DevBuf scratch;
    MBR_TRY(scratch.alloc(o_dig + kDigits * 4));
    unsigned char *base = scratch.as<unsigned char>();
    int64_t *sums = reinterpret_cast<int64_t *>(base), *level_total = reinterpret_cast<int64_t *>(base + o_tot);
    P *keys[2] = {reinterpret_cast<P *>(base + o_key), reinterpret_cast<P *>(base + o_key + keyb)};
    uint32_t *idxs[2] = {reinterpret_cast<uint32_t *>(base + o_idx), reinterpret_cast<uint32_t *>(base + o_idx + idxb)};
    uint32_t *counts = reinterpret_cast<uint32_t *>(base + o_cnt), *digit_total = reinterpret_cast<uint32_t *>(base + o_dig);
    const P *key = sec->states.as<P>();
    const uint32_t *idx = nullptr;
    int to = 0;
    for (int l = H - 2; l >= 0; --l)
        for (int b = 0; b < t.w[l]; b += 8) {
            const int shift = t.shift[l] + b;
            const uint32_t mask = (1u << std::min(8, t.w[l] - b)) - 1;
            tl_count_kernel<P><<<(unsigned)st, kSortBlock, 0, s>>>(key, n, shift, mask, counts);
            row_scan_kernel<uint32_t><<<kDigits, 1024, 0, s>>>(counts, st, digit_total);
            tl_scatter_kernel<P><<<(unsigned)st, kSortBlock, 0, s>>>(key, idx, n, shift, mask, counts, digit_total, keys[to], idxs[to]);
            key = keys[to];
            idx = idxs[to];
            to ^= 1;
        }
    LevelArgs v{};
    v.H = H;
    for (int l = 0; l < H; ++l) {
        v.shift[l] = t.shift[l];
        v.w[l] = t.w[l];
    }
    v.shift[H] = M;
    int64_t total_of[kMaxH] = {0};
    if (H > 1) {
        tl_sums_kernel<P><<<(unsigned)lt, kLevelBlock, 0, s>>>(key, n, v, sums);
        row_scan_kernel<int64_t><<<H - 1, 1024, 0, s>>>(sums, lt, level_total);
        MBR_HIP(hipGetLastError());
        MBR_HIP(hipMemcpyAsync(total_of + 1, level_total, (size_t)(H - 1) * 8, hipMemcpyDeviceToHost, s));
        MBR_HIP(hipStreamSynchronize(s));
    }
    uint64_t total = 0;
    for (int l = 0; l < H; ++l) {
        const uint64_t W = 1ull << t.w[l];
        const uint64_t pos = l == 0 ? W : W - 1 + (uint64_t)total_of[l] + W;  // padded in front and behind
        if (pos > 0xFFFFFFFFull) MBR_FAIL(MBR_ERANGE, "trie level %d has %llu entries", l, (unsigned long long)pos);
        t.off[l] = v.off[l] = total;
        total += pos;
    }
    t.off[H] = total;
    t.entries = total;
    MBR_TRY(t.table.alloc(total * 4));
    MBR_HIP(hipMemsetAsync(t.table.p, 0, total * 4, s));
    tl_fill_kernel<P><<<(unsigned)lt, kLevelBlock, 0, s>>>(key, idx, n, v, sums, t.table.as<uint32_t>());
    MBR_HIP(hipGetLastError());
    // stage the top levels in LDS while they fit
    t.lds_levels = 0;
    t.lds_entries = 0;
    for (int l = 0; l < H; ++l) {
        if (t.off[l + 1] * 4 > kLdsBudget) break;
        t.lds_levels = l + 1;
        t.lds_entries = t.off[l + 1];
    }
    MBR_HIP(hipStreamSynchronize(s));  // the trie is ready for any stream, and the scratch is free
    return MBR_OK;
}

template <class P>
mbr_status launch_trie(const mbr_ranker *r, const void *q, uint64_t n, uint32_t *out, hipStream_t s) {
    const TrieLevels &t = *r->trie;
    TrieArgs a{};
    a.tab = t.table.as<uint32_t>();
    a.states = r->sector->states.p;
    a.ns = r->sector->n;
    a.M = t.M;
    a.H = t.H;
    a.lds_entries = (uint32_t)t.lds_entries;
    a.lds_levels = (int32_t)t.lds_levels;
    for (int l = 0; l < t.H; ++l) {
        a.wmask[l] = (uint32_t)((1ull << t.w[l]) - 1);
        a.shift[l] = t.shift[l];
        a.off[l] = t.off[l];
    }
    a.off[t.H] = t.off[t.H];
    const size_t lds = t.lds_entries * 4;
    const unsigned grid = mbr::grid_for(n, kBlock * kQ, mbr::device_cu_count() * 8);
    trie_rank_kernel<P><<<grid, kBlock, lds, s>>>(static_cast<const P *>(q), n, out, a);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

}  // namespace

mbr_status rank_trie_launch(const mbr_ranker *r, const void *q, uint64_t n, uint32_t *out,
                            hipStream_t s) {
    if (r->width_bits == 32) return launch_trie<uint32_t>(r, q, n, out, s);
    return launch_trie<uint64_t>(r, q, n, out, s);
}

extern "C" mbr_status mbr_trie_level_entries(const mbr_ranker *r, uint64_t *entries, int32_t cap,
                                             int32_t *levels, int32_t *lds_levels) {
    if (!r || r->kind != MBR_RANKER_TRIE || !r->trie) MBR_FAIL(MBR_EINVAL, "not a trie ranker");
    const TrieLevels &t = *r->trie;
    if (levels) *levels = t.H;
    if (lds_levels) *lds_levels = (int32_t)t.lds_levels;
    if (entries)
        for (int l = 0; l < t.H && l < cap; ++l) entries[l] = t.off[l + 1] - t.off[l];
    return MBR_OK;
}

extern "C" mbr_status mbr_build_trie(const mbr_sector *sec, int32_t k, mbr_ranker **out,
                                     void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (!sec) MBR_FAIL(MBR_EINVAL, "null sector");
    if (k < 1 || k > 16) MBR_FAIL(MBR_EINVAL, "k=%d outside 1..16", k);
    const int M = sec->M;
    const int H = (M + k - 1) / k;
    if (H > 16) MBR_FAIL(MBR_EUNSUPPORTED, "%d levels (at most 16)", H);
    if (sec->n == 0) MBR_FAIL(MBR_EINVAL, "empty sector");
    hipStream_t s = as_stream(stream);
    auto t = std::make_unique<TrieLevels>();
    t->M = M;
    t->H = H;
    t->width_bits = sec->width_bits;
    for (int l = 0, b = 0; l < H; ++l) {
        t->w[l] = std::min(k, M - b);
        t->shift[l] = b;
        b += t->w[l];
    }
    if (sec->width_bits == 32) MBR_TRY(build_levels<uint32_t>(*t, sec, s));
    else MBR_TRY(build_levels<uint64_t>(*t, sec, s));
    auto *r = new (std::nothrow) mbr_ranker;
    if (!r) MBR_FAIL(MBR_ENOMEM, "host allocation");
    r->kind = MBR_RANKER_TRIE;
    r->M = M;
    r->k = k;
    r->width_bits = sec->width_bits;
    r->n_states = sec->n;
    r->sector = sec;
    (void)hipGetDevice(&r->device);
    r->trie = t.release();
    *out = r;
    return MBR_OK;
}
