// Generic operators from non-branching terms (App. A) applied on the fly.
//
// Every term of Eq. H, a prefactor times a product of creation and
// annihilation operators, acts on an occupation pattern as one tuple
// (v, m, l, r, x, s) (Eq. Talpha1, Eq. Talpha2).  Tuples are built on the host
// from those of the single operators (Eqs. ci) by the product rule of App. A;
// terms with equal (m, l, x, s) are merged by adding their prefactors.
//
// The product is taken in gather form from the bra side (Eq. Talpha2), each
// output row summed by one wave or workgroup, so no atomics are needed:
//   y_alpha = sum_T v [alpha AND m == l] (-1)^popcount(alpha AND s) x[rank(alpha XOR x_T)]
// with alpha = states[row].  Ranks of 32-bit patterns come from two small tables
// where the sector allows it (op_sum_tables; C^M_N always does), else from the
// packed trie (any sector; walk plus membership check).  64-bit patterns are
// ranked by the operator's ranker: a staggered table (sector C^M_N; staged in
// LDS when it fits) or a trie.
#include <algorithm>
#include <memory>
#include <tuple>

#include "rank_device.hpp"

namespace {

// ---------------------------------------------------------------- host algebra
struct Tup {
    double v;
    uint64_t m, l, r, x, s;
};

// c_i (Eqs. ci): needs orbital i occupied on the right, leaves it empty on the
// left, flips it, and picks up the parity of the orbitals below i.
Tup annihilator(int i) {
    const uint64_t b = 1ull << i;
    return Tup{1.0, b, 0, b, b, b - 1};
}

// c_i^dagger: the annihilator with its left and right requirements exchanged.
Tup creator(int i) {
    Tup t = annihilator(i);
    std::swap(t.l, t.r);
    return t;
}

// One tuple applied to a ket (Eq. Talpha1): false when it annihilates alpha,
// else the coefficient is multiplied by its signed prefactor and alpha moved to
// its image.
bool act_on(const Tup &t, uint64_t &alpha, double &coef) {
    if ((alpha & t.m) != t.r) return false;
    coef *= (__builtin_popcountll(alpha & t.s) & 1) ? -t.v : t.v;
    alpha ^= t.x;
    return true;
}

// Tuple of the product T_a T_b (T_b acts first), App. A, by running the one
// pattern that can survive through both factors.  The product touches the
// orbitals of m = m_a | m_b: on m_b a surviving pattern must hold r_b, and on
// the rest of m_a, which T_b leaves alone, it must hold r_a; outside m it is
// free.  The pattern holding exactly that (nothing outside m) is pushed
// through T_b and then T_a: if either annihilates it the product vanishes,
// otherwise its image is l and the accumulated coefficient is v.  Outside m
// each factor sees the same occupations, so an orbital there changes the sign
// once per factor whose sign mask holds it: s = (s_a ^ s_b) & ~m.
Tup product(const Tup &a, const Tup &b) {
    Tup t;
    t.m = a.m | b.m;
    t.r = b.r | (a.r & ~b.m);
    t.s = (a.s ^ b.s) & ~t.m;
    uint64_t state = t.r;
    double coef = 1.0;
    if (!act_on(b, state, coef) || !act_on(a, state, coef)) {
        t.v = 0.0;
        t.l = t.x = 0;
        return t;
    }
    t.l = state;
    t.x = t.l ^ t.r;
    t.v = coef;
    return t;
}

Tup product_of(double v, std::initializer_list<Tup> ops) {
    auto it = ops.begin();
    Tup t = *it;
    for (++it; it != ops.end(); ++it) t = product(t, *it);
    t.v *= v;
    return t;
}

// Merge tuples with equal (m, l, x, s), drop zeros; deterministic order.
std::vector<Tup> merge_terms(std::vector<Tup> ts) {
    std::sort(ts.begin(), ts.end(), [](const Tup &a, const Tup &b) {
        return std::tie(a.m, a.l, a.x, a.s) < std::tie(b.m, b.l, b.x, b.s);
    });
    std::vector<Tup> out;
    for (const Tup &t : ts) {
        if (!out.empty() && out.back().m == t.m && out.back().l == t.l && out.back().x == t.x &&
            out.back().s == t.s)
            out.back().v += t.v;
        else
            out.push_back(t);
    }
    out.erase(std::remove_if(out.begin(), out.end(), [](const Tup &t) { return t.v == 0.0; }), out.end());
    return out;
}

// ---------------------------------------------------------------- device apply
// A wave takes kOpRows consecutive rows: lane = (tuple slot, row), four tuple
// slots of sixteen rows, so one step evaluates four tuples on sixteen rows.
// Consecutive members share their high bits, and a tuple whose requirement
// fails on a bit that is the same in all of the wave's rows is dead for every
// one of them.  The wave therefore first sieves the tuples, a tuple per lane
// (64 per step, against the AND and the OR of its rows), and compacts the
// survivors into its own LDS queue; only those are evaluated row by row.  On
// the 14-site ring with total momentum 0 (841,332 rows, 2,772 tuples) about
// one tuple in four survives.
//
// Few rows leave the chip idle when every wave runs through all tuples, so a
// row group's tuples are then split over up to the 16 waves of a workgroup and
// the partial sums added in wave order (see op_split).
//
// The tuples are kept in three ranges: diagonal ones (x = 0), which need no
// rank; ones that keep every member inside the sector; and the rest, whose
// targets are checked.  Inside a range they are ordered by the high bits they
// flip, so that consecutive tuples gather from the same stretch of x, which
// then sits in L1.
//
// What bounds it: issue of the evaluation steps (19 vector instructions per
// four tuples and sixteen rows, a third of the lanes live), the SIMDs being
// about 70% busy; the gathers of x hit L1 and L2 (1.1 lines looked up per
// term).  One row per lane running through every tuple took 2,937 us on the
// ring (sum tables below, 594 us with the sieve) and 3,180 us on 15 orbitals
// half filled (6,435 rows, 11,250 tuples; 52 us).
constexpr unsigned kBlock = 256;
constexpr size_t kLdsTable = 64 * 1024;

constexpr int kOpRows = 16;                 // rows per wave
constexpr int kOpSlots = 64 / kOpRows;      // tuples evaluated side by side
constexpr int kOpUnroll = 4;                // steps issued together
constexpr int kOpWaves = 16;                // waves per workgroup
constexpr unsigned kOpBlock = 64 * kOpWaves;
constexpr unsigned kOpQueue = 128;          // survivors a wave can hold (fewer than 64 wait when a sieve step adds up to 64)

// How a target pattern is ranked.  kSum*: rank = base[high bits] + off[low
// bits], see op_sum_tables; the others are the operator's ranker.
enum RankKind { kSumLds = 0, kSumGlobal = 1, kStagLds = 2, kStagGlobal = 3, kTrie = 4 };

template <class P>
struct alignas(2 * sizeof(P)) Two {
    P a, b;
};

template <class P>
struct OpArgs {
    const P *states;
    uint64_t ns;
    int64_t n_diag, n_keep, n_all;  // ends of the three tuple ranges
    const Two<P> *ml, *xs;          // (m, l) and (x, s) of every tuple
    const double *v;
    const double *xin;
    double *out;
    uint32_t split;                 // waves that share a row group's tuples (divides kOpWaves)
    uint32_t units;                 // workgroup-sized pieces of the rows
    StagArgs stag;
    const void *stab;
    TrieWalk trie;
    const uint32_t *base;           // sum tables
    const uint16_t *off;
    uint32_t n_base, n_off;
    int32_t low_bits;
};

template <class P>
__device__ __forceinline__ int popc(P v) {
    return sizeof(P) == 8 ? __popcll((uint64_t)v) : __popc((uint32_t)v);
}

// at(): rank of a pattern known to be a member.  find(): rank of any pattern,
// or a value >= ns outside the sector.
template <class P, class E, int RK>
struct OpRank {
    static constexpr bool kFromLds = RK == kSumLds || RK == kStagLds;
    const OpArgs<P> &a;
    const E *tab;          // staggered table
    const uint32_t *base;  // sum tables
    const uint16_t *off;
    __device__ __forceinline__ uint64_t at(P be) const {
        if constexpr (RK == kSumLds || RK == kSumGlobal) {
            return base[be >> a.low_bits] + (uint32_t)off[be & (P)(a.n_off - 1)];
        } else if constexpr (RK == kTrie) {
            uint32_t node = 0;
            for (int lv = 0; lv < a.trie.H; ++lv)
                node = a.trie.tab[a.trie.off[lv] + node + ((uint32_t)(be >> a.trie.shift[lv]) & a.trie.wmask[lv])];
            return node;
        } else {
            return stag_rank<P, E>(be, tab, a.stag);
        }
    }
    __device__ __forceinline__ uint64_t find(P be) const {
        if constexpr (RK == kSumLds || RK == kSumGlobal) {
            const uint64_t r = (uint64_t)base[be >> a.low_bits] + off[be & (P)(a.n_off - 1)];
            return r < a.ns && a.states[r] == be ? r : ~0ull;
        } else if constexpr (RK == kTrie) {
            const uint32_t q = trie_rank_one<P>(be, a.trie);
            return q == MBR_NOT_FOUND ? ~0ull : q;
        } else {
            if (popc(be) != a.stag.N || !below_width(be, a.stag.M)) return ~0ull;
            return stag_rank<P, E>(be, tab, a.stag);
        }
    }
};

// A wave's queue of surviving tuples.
template <class P>
struct OpQueue {
    Two<P> ml[kOpQueue], xs[kOpQueue];
    double v[kOpQueue];
};

enum TupleRange { kDiagonal = 0, kKeeping = 1, kLeaving = 2 };

// One range of tuples on the wave's rows: sieve, queue, evaluate.  `al` is the
// pattern of the lane's row, `ref` that of any row and `same` the bits
// that agree in all rows.  kDiagonal leaves the sum of signed prefactors in acc
// and sets `any` when a tuple acted; the others add their terms to acc.
template <class P, class R, int RANGE>
__device__ __forceinline__ void op_range(const OpArgs<P> &a, const R &rk, OpQueue<P> &qu, int64_t begin, int64_t end,
                                         uint32_t part, P al, P ref, P same, double &acc, bool &any) {
    const int lane = threadIdx.x & 63;
    const uint32_t slot = (uint32_t)lane / kOpRows;
    uint32_t cnt = 0;
    auto eval = [&](uint32_t n) {  // the first n queued tuples, n a multiple of kOpSlots * kOpUnroll
        const OpQueue<P> *p = &qu;
        for (uint32_t i = slot; i < n; i += kOpSlots * kOpUnroll) {
            Two<P> xs[kOpUnroll];
            double v[kOpUnroll], xv[kOpUnroll];
            bool ok[kOpUnroll];
            uint64_t r[kOpUnroll];
#pragma unroll
            for (int u = 0; u < kOpUnroll; ++u) {
                const Two<P> ml = p->ml[i + u * kOpSlots];
                xs[u] = p->xs[i + u * kOpSlots];
                v[u] = p->v[i + u * kOpSlots];
                ok[u] = (al & ml.a) == ml.b;
            }
            // ranks, then gathers, then sums: each in flight for all the tuples of the step
            if constexpr (RANGE != kDiagonal) {
#pragma unroll
                for (int u = 0; u < kOpUnroll; ++u) {
                    if constexpr (RANGE == kKeeping) {
                        // from LDS the rank of every pattern is looked up, whether its tuple acts or not
                        r[u] = 0;
                        if (R::kFromLds || ok[u]) r[u] = rk.at(ok[u] ? al ^ xs[u].a : al);
                    } else {
                        r[u] = ok[u] ? rk.find(al ^ xs[u].a) : ~0ull;
                        ok[u] = r[u] < a.ns;
                    }
                }
#pragma unroll
                for (int u = 0; u < kOpUnroll; ++u) {
                    xv[u] = 0.0;
                    if (ok[u]) xv[u] = a.xin[r[u]];
                }
            }
#pragma unroll
            for (int u = 0; u < kOpUnroll; ++u) {
                // signed prefactor, zero when the tuple does not act
                const uint64_t bits = __builtin_bit_cast(uint64_t, v[u]);
                uint32_t hi = (uint32_t)(bits >> 32) ^ ((uint32_t)popc((P)(al & xs[u].b)) << 31), lo = (uint32_t)bits;
                hi = ok[u] ? hi : 0u;
                lo = ok[u] ? lo : 0u;
                const double c = __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
                if constexpr (RANGE == kDiagonal) {
                    acc += c;
                    any = any || ok[u];
                } else {
                    acc = __builtin_fma(c, xv[u], acc);
                }
            }
        }
    };
    const int64_t step = (int64_t)64 * a.split;
    int64_t t = begin + (int64_t)part * 64 + lane;
    const int64_t tend = end + lane;  // t < tend holds for all lanes alike
    Two<P> nx{};
    if (t < end) nx = a.ml[t];
    for (; t < tend; t += step) {
        const Two<P> ml = nx;
        const bool in = t < end;
        if (t + step < end) nx = a.ml[t + step];
        const bool live = in && (((ref ^ ml.b) & ml.a & same) == 0);
        const uint64_t b = __ballot(live);
        if (b == 0) continue;
        if (live) {
            const uint32_t q = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0));
            qu.ml[q] = ml;
            qu.xs[q] = a.xs[t];
            qu.v[q] = a.v[t];
        }
        cnt += (uint32_t)__popcll(b);
        if (cnt >= 64) {
            wave_lds_fence();
            eval(64);
            cnt -= 64;
            // the rest moves to the front
            Two<P> m2{}, x2{};
            double v2 = 0.0;
            if (lane < (int)cnt) {
                m2 = qu.ml[64 + lane];
                x2 = qu.xs[64 + lane];
                v2 = qu.v[64 + lane];
            }
            wave_lds_fence();
            if (lane < (int)cnt) {
                qu.ml[lane] = m2;
                qu.xs[lane] = x2;
                qu.v[lane] = v2;
            }
            wave_lds_fence();
        }
    }
    if (cnt) {
        // fill the last step with tuples that no pattern satisfies
        const uint32_t n = (cnt + kOpSlots * kOpUnroll - 1) / (kOpSlots * kOpUnroll) * (kOpSlots * kOpUnroll);
        if (cnt + lane < n) {
            qu.ml[cnt + lane] = Two<P>{0, 1};
            qu.xs[cnt + lane] = Two<P>{0, 0};
            qu.v[cnt + lane] = 0.0;
        }
        wave_lds_fence();
        eval(n);
        wave_lds_fence();
    }
}

template <class P>
size_t op_lds_bytes(size_t table_bytes) {
    return (table_bytes + 15) / 16 * 16 + kOpWaves * sizeof(OpQueue<P>) + kOpWaves * kOpRows * sizeof(double);
}

template <class P, class E, int RK>
__global__ void __launch_bounds__(kOpBlock) op_apply_kernel(OpArgs<P> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    // LDS: rank tables | a queue per wave | partial sums of the split
    size_t tb = 0;
    OpRank<P, E, RK> rk{a, static_cast<const E *>(a.stab), a.base, a.off};
    if constexpr (RK == kStagLds) {
        E *t = reinterpret_cast<E *>(lds_raw);
        for (uint64_t i = threadIdx.x; i < a.stag.nentries; i += blockDim.x) t[i] = rk.tab[i];
        tb = a.stag.nentries * sizeof(E);
        rk.tab = t;
    } else if constexpr (RK == kSumLds || RK == kSumGlobal) {
        if constexpr (RK == kSumLds) {
            uint32_t *b = reinterpret_cast<uint32_t *>(lds_raw);
            for (uint32_t i = threadIdx.x; i < a.n_base; i += blockDim.x) b[i] = a.base[i];
            rk.base = b;
            tb = (size_t)a.n_base * 4;
        }
        uint16_t *o = reinterpret_cast<uint16_t *>(lds_raw + tb);
        for (uint32_t i = threadIdx.x; i < a.n_off; i += blockDim.x) o[i] = a.off[i];
        rk.off = o;
        tb += (size_t)a.n_off * 2;
    }
    tb = (tb + 15) / 16 * 16;
    const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    OpQueue<P> &qu = reinterpret_cast<OpQueue<P> *>(lds_raw + tb)[w];
    double *red = reinterpret_cast<double *>(lds_raw + tb + kOpWaves * sizeof(OpQueue<P>));
    __syncthreads();
    const uint32_t groups = kOpWaves / a.split;  // row groups of a workgroup
    const uint32_t part = w % a.split;
    // workgroup b runs on XCD b mod 8: each XCD takes one contiguous stretch of
    // the rows (the grid is a multiple of 8)
    const uint32_t xcd = blockIdx.x & 7;
    const uint32_t u1 = (uint32_t)((uint64_t)a.units * (xcd + 1) / 8);
    for (uint32_t u = (uint32_t)((uint64_t)a.units * xcd / 8) + (blockIdx.x >> 3); u < u1; u += gridDim.x >> 3) {
        const uint64_t row0 = ((uint64_t)u * groups + w / a.split) * kOpRows;
        const uint64_t row = row0 + (lane & (kOpRows - 1));
        double acc = 0.0;
        if (row0 < a.ns) {
            const uint64_t own = row < a.ns ? row : a.ns - 1;  // past the end: the last row again, not stored
            const P al = a.states[own];
            P all = al, one = al;
#pragma unroll
            for (int o = 1; o < kOpRows; o <<= 1) {
                all &= (P)__shfl_xor(all, o, 64);
                one |= (P)__shfl_xor(one, o, 64);
            }
            const P same = ~(all ^ one);
            bool any = false;
            op_range<P, OpRank<P, E, RK>, kDiagonal>(a, rk, qu, 0, a.n_diag, part, al, all, same, acc, any);
            // a row no diagonal tuple acts on does not read its own x
            acc = any ? acc * a.xin[own] : 0.0;
            op_range<P, OpRank<P, E, RK>, kKeeping>(a, rk, qu, a.n_diag, a.n_keep, part, al, all, same, acc, any);
            op_range<P, OpRank<P, E, RK>, kLeaving>(a, rk, qu, a.n_keep, a.n_all, part, al, all, same, acc, any);
            // the four tuple slots of a row
#pragma unroll
            for (int o = kOpRows; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
        }
        if (a.split == 1) {
            if (lane < kOpRows && row < a.ns) a.out[row] = acc;
        } else {
            if (lane < kOpRows) red[w * kOpRows + lane] = acc;
            __syncthreads();
            if (part == 0 && lane < kOpRows && row < a.ns) {
                double s = acc;
                for (uint32_t k = 1; k < a.split; ++k) s += red[(w + k) * kOpRows + lane];
                a.out[row] = s;
            }
            __syncthreads();  // red is free again
        }
    }
}

// The product over rows that share their high part, for operators whose sector
// has sum tables (below) and whose off-diagonal tuples all keep it.  A tuple
// is a product of a factor on the high orbitals and one on the low ones, and
// in a wave of rows with one high part everything about the high factor is the
// same for all lanes: whether it acts, its sign, and the first row of the
// block it leads to.  The tuples are ordered by their low factor.  The sieve
// (a tuple per lane, as above) leaves in the queue, per surviving tuple, its
// signed prefactor and its target block; a run of equal low factors is then
// evaluated with one test, one table read and one sign per row, and a gather
// and a fused multiply-add per tuple:
//   y_row += sign_low(row) * sum_t v_t x[block_t + off[low ^ x_low]].
// The 14-site ring has 196 low factors for 2,772 tuples; the step above spends
// 19 vector instructions per tuple and 64 row slots, this one 3.
struct OpLowQueue {
    double v[kOpQueue];
    uint2 low[kOpQueue];       // low factor: m | l << 16, x | s << 16
    uint32_t block[kOpQueue];  // first row of the target block
};

struct OpTile {
    uint32_t row0, n;  // up to 64 rows of one high part
};

struct OpLowArgs {
    OpArgs<uint32_t> op;
    const OpTile *tiles;
    uint32_t n_tiles;
};

template <int RANGE, bool SPLIT>
__device__ __forceinline__ void op_low_range(const OpArgs<uint32_t> &a, const uint16_t *off, OpLowQueue &qu, int64_t begin,
                                             int64_t end, uint32_t part, uint32_t al, uint32_t ref, uint32_t same, double &acc, bool &any) {
    const int lane = threadIdx.x & 63;
    const uint32_t lmask = a.n_off - 1, low = al & lmask;
    uint32_t cnt = 0;
    auto eval = [&](uint32_t n) {
        const uint2 key = qu.low[lane], prev = qu.low[lane ? lane - 1 : 0];
        uint64_t starts = __ballot((uint32_t)lane < n && (lane == 0 || key.x != prev.x || key.y != prev.y));
        while (starts) {
            const uint32_t j = (uint32_t)__builtin_ctzll(starts);
            starts &= starts - 1;
            const uint32_t k = starts ? (uint32_t)__builtin_ctzll(starts) : n;
            const uint2 f = qu.low[j];
            if ((low & (f.x & 0xFFFFu)) == f.x >> 16) {
                double sum = 0.0;
                if constexpr (RANGE == kDiagonal) {
                    for (uint32_t e = j; e < k; ++e) sum += qu.v[e];
                    any = true;
                } else {
                    const double *px = a.xin + off[low ^ (f.y & 0xFFFFu)];
                    uint32_t e = j;
                    for (; e + 4 <= k; e += 4) {
                        const double x0 = px[qu.block[e]], x1 = px[qu.block[e + 1]], x2 = px[qu.block[e + 2]], x3 = px[qu.block[e + 3]];
                        sum = __builtin_fma(qu.v[e], x0, sum);
                        sum = __builtin_fma(qu.v[e + 1], x1, sum);
                        sum = __builtin_fma(qu.v[e + 2], x2, sum);
                        sum = __builtin_fma(qu.v[e + 3], x3, sum);
                    }
                    if (e + 2 <= k) {
                        const double x0 = px[qu.block[e]], x1 = px[qu.block[e + 1]];
                        sum = __builtin_fma(qu.v[e], x0, sum);
                        sum = __builtin_fma(qu.v[e + 1], x1, sum);
                        e += 2;
                    }
                    if (e < k) sum = __builtin_fma(qu.v[e], px[qu.block[e]], sum);
                }
                const uint64_t flip = (uint64_t)(__popc(low & (f.y >> 16)) & 1) << 63;
                acc += __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, sum) ^ flip);
            }
        }
    };
    const int64_t step = SPLIT ? (int64_t)64 * a.split : 64;
    Two<uint32_t> nx{};
    int64_t t = begin + (int64_t)part * 64 + lane;
    const int64_t tend = end + lane;
    if (t < end) nx = a.ml[t];
    for (; t < tend; t += step) {
        const Two<uint32_t> ml = nx;
        const bool in = t < end;
        if (t + step < end) nx = a.ml[t + step];
        const bool live = in && (((ref ^ ml.b) & ml.a & same) == 0);
        const uint64_t b = __ballot(live);
        if (b == 0) continue;
        if (live) {
            const uint32_t q = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0));
            const Two<uint32_t> xs = a.xs[t];
            const uint64_t flip = (uint64_t)(__popc(ref & xs.b & ~lmask) & 1) << 63;
            qu.v[q] = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, a.v[t]) ^ flip);
            qu.low[q] = make_uint2((ml.a & lmask) | (ml.b & lmask) << 16, (xs.a & lmask) | (xs.b & lmask) << 16);
            if constexpr (RANGE != kDiagonal) qu.block[q] = a.base[(ref ^ xs.a) >> a.low_bits];
        }
        cnt += (uint32_t)__popcll(b);
        if (cnt >= 64) {
            wave_lds_fence();
            eval(64);
            cnt -= 64;
            double v2 = 0.0;
            uint2 l2{};
            uint32_t b2 = 0;
            if (lane < (int)cnt) {
                v2 = qu.v[64 + lane];
                l2 = qu.low[64 + lane];
                if constexpr (RANGE != kDiagonal) b2 = qu.block[64 + lane];
            }
            wave_lds_fence();
            if (lane < (int)cnt) {
                qu.v[lane] = v2;
                qu.low[lane] = l2;
                if constexpr (RANGE != kDiagonal) qu.block[lane] = b2;
            }
            wave_lds_fence();
        }
    }
    if (cnt) {
        wave_lds_fence();
        eval(cnt);
        wave_lds_fence();
    }
}

template <bool SPLIT>
__global__ void __launch_bounds__(kOpBlock) op_low_kernel(OpLowArgs args) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const OpArgs<uint32_t> &a = args.op;
    uint16_t *off = reinterpret_cast<uint16_t *>(lds_raw);
    const size_t tb = ((size_t)a.n_off * 2 + 15) / 16 * 16;
    stage_to_lds(off, a.off, (uint64_t)a.n_off * 2);
    __syncthreads();
    const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    OpLowQueue *qu = reinterpret_cast<OpLowQueue *>(lds_raw + tb) + w;
    const uint32_t groups = SPLIT ? kOpWaves / a.split : kOpWaves, part = SPLIT ? w % a.split : 0;
    const uint32_t xcd = blockIdx.x & 7;
    const uint32_t u1 = (uint32_t)((uint64_t)a.units * (xcd + 1) / 8);
    for (uint32_t u = (uint32_t)((uint64_t)a.units * xcd / 8) + (blockIdx.x >> 3); u < u1; u += gridDim.x >> 3) {
        const uint32_t ti = u * groups + (SPLIT ? w / a.split : w);
        const bool some = ti < args.n_tiles;
        if (!SPLIT && !some) continue;
        const OpTile tl = some ? args.tiles[ti] : OpTile{0, 0};
        double acc = 0.0;
        if (some) {
            const uint32_t own = tl.row0 + (lane < tl.n ? lane : tl.n - 1);
            const uint32_t al = a.states[own];
            uint32_t all = al, one = al;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                all &= (uint32_t)__shfl_xor((int)all, o, 64);
                one |= (uint32_t)__shfl_xor((int)one, o, 64);
            }
            const uint32_t ref = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
            const uint32_t same = (uint32_t)__builtin_amdgcn_readfirstlane((int)~(all ^ one));
            bool any = false;
            op_low_range<kDiagonal, SPLIT>(a, off, *qu, 0, a.n_diag, part, al, ref, same, acc, any);
            acc = any ? acc * a.xin[own] : 0.0;
            op_low_range<kKeeping, SPLIT>(a, off, *qu, a.n_diag, a.n_keep, part, al, ref, same, acc, any);
        }
        if constexpr (!SPLIT) {
            if (lane < tl.n) a.out[tl.row0 + lane] = acc;
        } else {
            qu->v[lane] = acc;  // the queue is empty here
            __syncthreads();
            if (part == 0 && lane < tl.n) {
                double s = acc;
                for (uint32_t k = 1; k < a.split; ++k) s += qu[k].v[lane];
                a.out[tl.row0 + lane] = s;
            }
            __syncthreads();  // before the queues fill again
        }
    }
}

// Sum tables.  When the members under two different high parts are either the
// same set of low parts or share none (exact particle-number windows, and
// with them a modular weight, make it so: the high part fixes what the low
// part has to hold), the position of a low part among its siblings depends on
// the low part alone, and rank = base[high] + off[low]: two reads, both from
// LDS for up to 28 orbitals, instead of a walk through a trie or a chunk loop.
// Neighbouring rows' targets then also read neighbouring entries.  Whether a
// sector is of that kind is not guessed from its windows but checked here on
// its list: base[high] is the first position of the high part, and every
// member's position minus that has to agree for equal low parts.
constexpr uint32_t kNoEntry = 0xFFFFFFFFu;

template <class P>
__global__ void __launch_bounds__(kBlock) op_sum_base(const P *__restrict__ st, uint64_t n, int low_bits, uint32_t *base) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const P hi = st[i] >> low_bits;
        if (i == 0 || (st[i - 1] >> low_bits) != hi) base[hi] = (uint32_t)i;
    }
}

template <class P>
__global__ void __launch_bounds__(kBlock) op_sum_off(const P *__restrict__ st, uint64_t n, int low_bits,
                                                     const uint32_t *__restrict__ base, uint32_t *off, uint32_t *bad) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t o = (uint32_t)i - base[st[i] >> low_bits];
        uint32_t *e = off + (st[i] & (P)(((P)1 << low_bits) - 1));
        uint32_t cur = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == kNoEntry) cur = atomicCAS(e, kNoEntry, o);
        if (cur != kNoEntry && cur != o) *bad = 1u;
    }
}

__global__ void op_fill_kernel(uint32_t *p, uint32_t n, uint32_t v) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// 16-bit copy (a low part has fewer than 2^14 smaller siblings; low parts that
// no member has keep all ones).
__global__ void op_sum_narrow(const uint32_t *__restrict__ off, uint32_t n, uint16_t *__restrict__ o16) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) o16[i] = (uint16_t)off[i];
}

// ---------------------------------------------------------------- Lanczos
// Plain fp64 Lanczos on an operator (three vectors, no reorthogonalisation):
// alpha_j = <v_j, H v_j>; w = H v_j - alpha_j v_j - beta_{j-1} v_{j-1};
// beta_j = |w|; v_{j+1} = w / beta_j.  Dot products are fixed-order two-level
// reductions (kRedBlocks block partials, then one block), so runs repeat
// bitwise.  The recurrence stops (the remaining kernels do nothing) once
// beta_j <= tol (|alpha_j| + beta_{j-1}) or after as many steps as the sector
// has states; *len holds the steps taken.
constexpr unsigned kRedBlocks = 1024;

__device__ __forceinline__ double blk_sum(double v, double *red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += red[k];
    return s;
}

__global__ void op_start_kernel(int32_t *len, int32_t nsteps) { *len = nsteps; }

__global__ void __launch_bounds__(kBlock) op_dot_parts(const double *__restrict__ a, const double *__restrict__ b,
                                                       uint64_t n, double *parts) {
    __shared__ double red[kBlock / 64];
    double acc = 0;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        acc = __builtin_fma(a[i], b[i], acc);
    const double s = blk_sum(acc, red);
    if (threadIdx.x == 0) parts[blockIdx.x] = s;
}

// out = sum of the kRedBlocks partials (sqrt of it when root != 0).
__global__ void __launch_bounds__(kBlock) op_reduce(const double *parts, double *out, int root) {
    __shared__ double red[kBlock / 64];
    double acc = 0;
    for (unsigned i = threadIdx.x; i < kRedBlocks; i += blockDim.x) acc += parts[i];
    const double s = blk_sum(acc, red);
    if (threadIdx.x == 0) *out = root ? sqrt(s) : s;
}

__global__ void __launch_bounds__(kBlock) op_scale_kernel(const double *__restrict__ v0, double *__restrict__ v,
                                                          double *__restrict__ vp, uint64_t n, const double *norm) {
    const double c = *norm > 0 ? 1.0 / *norm : 0.0;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        v[i] = v0[i] * c;
        vp[i] = 0.0;
    }
}

__global__ void __launch_bounds__(kBlock) op_update_kernel(double *__restrict__ w, const double *__restrict__ v,
                                                           const double *__restrict__ vp, uint64_t n,
                                                           const double *al, const double *be, int j,
                                                           const int32_t *len, double *parts) {
    __shared__ double red[kBlock / 64];
    if (j >= *len) return;
    const double a = al[j], b = j > 0 ? be[j - 1] : 0.0;
    double acc = 0;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const double x = w[i] - a * v[i] - b * vp[i];
        w[i] = x;
        acc = __builtin_fma(x, x, acc);
    }
    const double s = blk_sum(acc, red);
    if (threadIdx.x == 0) parts[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kBlock) op_beta_kernel(const double *parts, const double *al, double *be, int j,
                                                         int nsteps, uint64_t dim, double tol, int32_t *len) {
    __shared__ double red[kBlock / 64];
    if (j >= *len) return;
    double acc = 0;
    for (unsigned i = threadIdx.x; i < kRedBlocks; i += blockDim.x) acc += parts[i];
    const double s = blk_sum(acc, red);
    if (threadIdx.x == 0) {
        const double b = sqrt(s);
        const double bprev = j > 0 ? be[j - 1] : 0.0;
        // the Krylov space cannot outgrow the sector
        const bool stop = b <= tol * (fabs(al[j]) + bprev) || j + 1 >= nsteps || (uint64_t)(j + 1) >= dim;
        be[j] = stop ? 0.0 : b;
        if (stop) *len = j + 1;
    }
}

// v_{j+1} = w / beta_j, in place in w's buffer (the caller rotates the buffers).
// Once the recurrence has stopped the buffer is zeroed instead, so the steps
// the host still enqueues work on zero vectors (alpha = 0, nothing grows).
__global__ void __launch_bounds__(kBlock) op_next_kernel(double *__restrict__ w, const double *__restrict__ v,
                                                         const double *__restrict__ vp, uint64_t n,
                                                         const double *be, int j, const int32_t *len) {
    const double c = (j + 1 >= *len) ? 0.0 : 1.0 / be[j];
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        w[i] *= c;
}

}  // namespace

struct mbr_operator {
    const mbr_sector *sec = nullptr;
    const mbr_ranker *rk = nullptr;
    int64_t nt = 0, n_diag = 0, n_keep = 0;  // tuples: diagonal | sector-keeping | the rest
    int32_t M = 0, width_bits = 32;
    mbr::DevBuf v, ml, xs;
    mbr::DevBuf base, off;                   // sum tables (low_bits > 0)
    int32_t low_bits = 0;
    mbr::DevBuf tiles;                       // op_low_kernel: its row tiles (n_tiles > 0)
    uint32_t n_tiles = 0;
    uint32_t split = 1, units = 1, grid = 8;
    size_t lds = 0;
    int device = 0;
};

namespace {

constexpr size_t kOpLdsMax = 160 * 1024;
constexpr size_t kOpTables = 100 * 1024;  // sum tables up to this size are staged whole

// Waves that share the tuples of one of `groups` row groups: as few as put
// `per_cu` waves on every CU, and none that would not get 64 tuples to sieve.
// op_apply_kernel is content with 16 (15 orbitals half filled, 6,435 rows and
// 11,250 tuples: 16 waves share a group, 52 us a product; unsplit 329 us).
// op_low_kernel's waves differ more in length and want 24 (13-site ring, 226,512
// rows: 156 us with two waves a tile, 184 with one).
uint32_t op_split(uint64_t groups, int64_t nt, uint32_t per_cu) {
    const uint64_t want = (uint64_t)mbr::device_cu_count() * per_cu;
    uint32_t s = 1;
    while (s < (uint32_t)kOpWaves && groups * s < want && (int64_t)s * 64 < nt) s *= 2;
    return s;
}

// Run f with the kernel instance of the operator's rank path and pattern type.
template <class P, class F>
mbr_status with_kernel(const mbr_operator *op, F f) {
    const mbr_ranker *r = op->rk;
    if constexpr (sizeof(P) == 4) {
        if (op->low_bits) {
            const size_t nb = op->base.bytes, no = op->off.bytes;
            if (nb + no <= kOpTables) return f(op_apply_kernel<P, uint16_t, kSumLds>, nb + no);
            return f(op_apply_kernel<P, uint16_t, kSumGlobal>, no);
        }
        if (r->kind == MBR_RANKER_TRIE) return f(op_apply_kernel<P, uint32_t, kTrie>, (size_t)0);
        MBR_FAIL(MBR_EUNSUPPORTED, "a staggered sector of %d orbitals without sum tables", op->M);
    } else {
        if (r->kind == MBR_RANKER_TRIE) return f(op_apply_kernel<P, uint32_t, kTrie>, (size_t)0);
        const StagTable &tb = r->stag;
        const size_t lds = ((size_t)tb.nrows << tb.k) * tb.entry_bytes;
        const bool in_lds = lds <= kLdsTable;
        switch (tb.entry_bytes) {
            case 2: return in_lds ? f(op_apply_kernel<P, uint16_t, kStagLds>, lds) : f(op_apply_kernel<P, uint16_t, kStagGlobal>, (size_t)0);
            case 4: return in_lds ? f(op_apply_kernel<P, uint32_t, kStagLds>, lds) : f(op_apply_kernel<P, uint32_t, kStagGlobal>, (size_t)0);
            default: return in_lds ? f(op_apply_kernel<P, uint64_t, kStagLds>, lds) : f(op_apply_kernel<P, uint64_t, kStagGlobal>, (size_t)0);
        }
    }
}

// Launch shape of the operator's products, fixed when it is created.
template <class P>
mbr_status plan_launch(mbr_operator *op) {
    return with_kernel<P>(op, [&](auto kern, size_t tables) -> mbr_status {
        op->lds = op_lds_bytes<P>(tables);
        MBR_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOpLdsMax));
        op->split = op_split((op->sec->n + kOpRows - 1) / kOpRows, op->nt, 16);
        const uint64_t rows = (uint64_t)kOpRows * kOpWaves / op->split;
        op->units = (uint32_t)((op->sec->n + rows - 1) / rows);
        int per_cu = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kOpBlock, op->lds) != hipSuccess || per_cu < 1) per_cu = 1;
        const uint64_t most = (uint64_t)mbr::device_cu_count() * per_cu;
        op->grid = (uint32_t)std::min<uint64_t>(most, op->units) + 7;
        op->grid -= op->grid % 8;
        return MBR_OK;
    });
}

// Sum tables of the sector split at `low` bits, when it has them;
// op->low_bits stays 0 otherwise.
mbr_status op_sum_tables(mbr_operator *op, int low, hipStream_t st) {
    using namespace mbr;
    const mbr_sector *sec = op->sec;
    const int high = sec->M - low;
    const uint32_t nb = 1u << high, no = 1u << low;
    DevBuf wide, flag;
    MBR_TRY(op->base.alloc((size_t)nb * 4));
    MBR_TRY(op->off.alloc((size_t)no * 2));
    MBR_TRY(wide.alloc((size_t)no * 4));
    MBR_TRY(flag.alloc(4));
    const unsigned grid = grid_for(sec->n, kBlock, device_cu_count() * 8);
    const uint32_t *states = sec->states.as<uint32_t>();
    op_fill_kernel<<<(nb + 255) / 256, 256, 0, st>>>(op->base.as<uint32_t>(), nb, kNoEntry);
    op_fill_kernel<<<(no + 255) / 256, 256, 0, st>>>(wide.as<uint32_t>(), no, kNoEntry);
    op_fill_kernel<<<1, 64, 0, st>>>(flag.as<uint32_t>(), 1, 0u);
    op_sum_base<uint32_t><<<grid, kBlock, 0, st>>>(states, sec->n, low, op->base.as<uint32_t>());
    op_sum_off<uint32_t><<<grid, kBlock, 0, st>>>(states, sec->n, low, op->base.as<uint32_t>(), wide.as<uint32_t>(), flag.as<uint32_t>());
    op_sum_narrow<<<(no + 255) / 256, 256, 0, st>>>(wide.as<uint32_t>(), no, op->off.as<uint16_t>());
    MBR_HIP(hipGetLastError());
    uint32_t bad = 1;
    MBR_HIP(hipMemcpyAsync(&bad, flag.p, 4, hipMemcpyDeviceToHost, st));
    MBR_HIP(hipStreamSynchronize(st));
    if (bad) {
        op->base.release();
        op->off.release();
    } else {
        op->low_bits = low;
    }
    return MBR_OK;
}

// Tiles and launch shape of op_low_kernel: the rows of every high part in
// pieces of 64.  op->n_tiles stays 0, and op_apply_kernel runs, where the work is
// too small to repay the longer chain of a wave (fewer than 2^14 rows or 2^24
// pairs of row and tuple), or where the high parts leave more than half of the
// lanes without a row.  The first two lines are a compromise: neither rows nor
// pairs alone part the kernels, and the rings of up to 10 sites give away less
// than 2 us for what 16 orbitals keep.  us per product, op_apply / op_low:
//   ring,    10 sites,   6,352 rows,  1,020 tuples: 10.7 / 9.0
//   general, 16 orbitals, 12,870 rows, 14,656 tuples: 104 / 122
//   ring,    11 sites,  19,404 rows,  1,353 tuples: 24.0 / 21.0
//   hopping, 10 sites,  63,504 rows,     50 tuples:  8.9 / 11.9
//   general, 18 orbitals, 48,620 rows, 23,733 tuples: 594 / 337
//   ring,    12 sites,  71,188 rows,  1,752 tuples: 83.6 / 50.6
//   ring,    14 sites, 841,332 rows,  2,772 tuples:  600 / 407
mbr_status plan_low(mbr_operator *op, hipStream_t st) {
    using namespace mbr;
    if (op->sec->n < (1u << 14) || op->sec->n * (uint64_t)op->nt < (1u << 24)) return MBR_OK;
    std::vector<uint32_t> base(op->base.bytes / 4);
    MBR_HIP(hipMemcpyAsync(base.data(), op->base.p, op->base.bytes, hipMemcpyDeviceToHost, st));
    MBR_HIP(hipStreamSynchronize(st));
    std::vector<OpTile> tiles;
    uint32_t row = 0;
    auto until = [&](uint32_t end) {
        for (; row < end; row += tiles.back().n) tiles.push_back(OpTile{row, std::min(64u, end - row)});
    };
    for (uint32_t b : base)
        if (b != kNoEntry) until(b);  // a block ends where the next one starts
    until((uint32_t)op->sec->n);
    if (tiles.size() * 32 > op->sec->n) return MBR_OK;
    MBR_TRY(upload(op->tiles, tiles.data(), tiles.size() * sizeof(OpTile), st));
    op->n_tiles = (uint32_t)tiles.size();
    op->split = op_split(op->n_tiles, op->nt, 24);
    const uint32_t groups = kOpWaves / op->split;
    op->units = (op->n_tiles + groups - 1) / groups;
    op->lds = (((size_t)2 << op->low_bits) + 15) / 16 * 16 + kOpWaves * sizeof(OpLowQueue);
    const auto kern = op->split > 1 ? op_low_kernel<true> : op_low_kernel<false>;
    MBR_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOpLdsMax));
    int per_cu = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kOpBlock, op->lds) != hipSuccess || per_cu < 1) per_cu = 1;
    op->grid = (uint32_t)std::min<uint64_t>((uint64_t)device_cu_count() * per_cu, op->units) + 7;
    op->grid -= op->grid % 8;
    return MBR_OK;
}

template <class P>
mbr_status apply_t(const mbr_operator *op, const double *x, double *y, hipStream_t st) {
    OpArgs<P> a{};
    a.states = op->sec->states.as<P>();
    a.ns = op->sec->n;
    a.n_diag = op->n_diag;
    a.n_keep = op->n_keep;
    a.n_all = op->nt;
    a.ml = op->ml.as<Two<P>>();
    a.xs = op->xs.as<Two<P>>();
    a.v = op->v.as<double>();
    a.xin = x;
    a.out = y;
    a.split = op->split;
    a.units = op->units;
    const mbr_ranker *r = op->rk;
    if (op->low_bits) {
        a.base = op->base.as<uint32_t>();
        a.off = op->off.as<uint16_t>();
        a.low_bits = op->low_bits;
        a.n_off = 1u << op->low_bits;
        a.n_base = 1u << (op->M - op->low_bits);
    } else if (r->kind == MBR_RANKER_TRIE) {
        const TrieLevels &t = *r->trie;
        a.trie.tab = t.table.as<uint32_t>();
        a.trie.states = op->sec->states.p;
        a.trie.ns = op->sec->n;
        a.trie.M = t.M;
        a.trie.H = t.H;
        for (int lv = 0; lv < t.H; ++lv) {
            a.trie.wmask[lv] = (uint32_t)((1ull << t.w[lv]) - 1);
            a.trie.shift[lv] = t.shift[lv];
            a.trie.off[lv] = t.off[lv];
        }
        a.trie.off[t.H] = t.off[t.H];
    } else {
        const StagTable &tb = r->stag;
        a.stag.M = tb.M;
        a.stag.k = tb.k;
        a.stag.nch = tb.nch;
        a.stag.N = r->N;
        for (int c = 0; c < tb.nch && c < 16; ++c) a.stag.rowoff[c] = tb.rowoff[c];
        a.stag.nentries = (uint64_t)tb.nrows << tb.k;
        a.stab = tb.table.p;
    }
    if constexpr (sizeof(P) == 4) {
        if (op->n_tiles) {
            const auto kern = op->split > 1 ? op_low_kernel<true> : op_low_kernel<false>;
            kern<<<op->grid, kOpBlock, op->lds, st>>>(OpLowArgs{a, op->tiles.as<OpTile>(), op->n_tiles});
            MBR_HIP(hipGetLastError());
            return MBR_OK;
        }
    }
    return with_kernel<P>(op, [&](auto kern, size_t) -> mbr_status {
        kern<<<op->grid, kOpBlock, op->lds, st>>>(a);
        MBR_HIP(hipGetLastError());
        return MBR_OK;
    });
}

}  // namespace

extern "C" {

mbr_status mbr_terms_from_hamiltonian(int32_t M, const double *t, int32_t n_u, const mbr_coulomb *u,
                                      mbr_term *out, int64_t cap, int64_t *n_out) {
    if (M < 1 || M > 64) MBR_FAIL(MBR_EINVAL, "M=%d outside 1..64", M);
    if (n_u < 0 || (n_u > 0 && !u)) MBR_FAIL(MBR_EINVAL, "bad interaction list");
    if (!n_out) MBR_FAIL(MBR_EINVAL, "null count pointer");
    std::vector<Tup> ts;
    if (t) {
        for (int i = 0; i < M; ++i)
            for (int j = 0; j < M; ++j) {
                const double a = t[(size_t)i * M + j];
                if (a != 0.0) ts.push_back(product_of(-a, {creator(i), annihilator(j)}));
            }
    }
    for (int q = 0; q < n_u; ++q) {
        const mbr_coulomb &c = u[q];
        if (c.i < 0 || c.j < 0 || c.k < 0 || c.l < 0 || c.i >= M || c.j >= M || c.k >= M || c.l >= M)
            MBR_FAIL(MBR_EINVAL, "interaction %d has an orbital outside 0..M-1", q);
        if (c.U != 0.0)
            ts.push_back(product_of(0.25 * c.U, {creator(c.i), creator(c.j), annihilator(c.l), annihilator(c.k)}));
    }
    const std::vector<Tup> mt = merge_terms(std::move(ts));
    *n_out = (int64_t)mt.size();
    if (out && cap >= (int64_t)mt.size())
        for (size_t i = 0; i < mt.size(); ++i) out[i] = mbr_term{mt[i].v, mt[i].m, mt[i].l, mt[i].r, mt[i].x, mt[i].s};
    return MBR_OK;
}

mbr_status mbr_operator_create(const mbr_sector *sec, const mbr_ranker *rk, const mbr_term *terms,
                               int64_t n_terms, mbr_operator **out, void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (!sec || !rk) MBR_FAIL(MBR_EINVAL, "null sector or ranker");
    if (n_terms < 0 || (n_terms > 0 && !terms)) MBR_FAIL(MBR_EINVAL, "bad term list");
    if (sec->n == 0) MBR_FAIL(MBR_EINVAL, "empty sector");
    if (rk->kind == MBR_RANKER_TRIE) {
        if (rk->sector != sec) MBR_FAIL(MBR_EINVAL, "the trie ranks a different sector");
    } else if (rk->kind == MBR_RANKER_STAGGERED) {
        // the sector must be exactly C^M_N of the table: one window with N set
        // bits among all M orbitals and no other constraint
        const uint64_t full = sec->M >= 64 ? ~0ull : ((1ull << sec->M) - 1);
        const bool cnm = sec->modulus == 0 && sec->cons.size() == 1 && sec->cons[0].mask == full &&
                         sec->cons[0].lo == rk->N && sec->cons[0].hi == rk->N;
        if (rk->N < 0 || rk->M != sec->M || !cnm || rk->n_states != sec->n || rk->width_bits != sec->width_bits)
            MBR_FAIL(MBR_EINVAL, "the staggered ranker does not rank this sector (C^M_N with one window)");
    } else {
        MBR_FAIL(MBR_EUNSUPPORTED, "operators rank with a staggered or trie ranker");
    }
    const uint64_t lim = sec->M >= 64 ? ~0ull : ((1ull << sec->M) - 1);
    for (int64_t i = 0; i < n_terms; ++i) {
        const mbr_term &t = terms[i];
        if ((t.m | t.l | t.x | t.s) & ~lim) MBR_FAIL(MBR_EINVAL, "term %lld touches orbitals >= M", (long long)i);
        if ((t.l & ~t.m) || (t.x & ~t.m)) MBR_FAIL(MBR_EINVAL, "term %lld: l and x must lie inside m", (long long)i);
    }
    auto op = std::make_unique<mbr_operator>();
    op->sec = sec;
    op->rk = rk;
    op->nt = n_terms;
    op->M = sec->M;
    op->width_bits = sec->width_bits;
    (void)hipGetDevice(&op->device);
    // A tuple keeps the sector when it moves no particle into or out of any
    // constraint's orbitals and leaves the modular weight unchanged: the
    // target of every member is then a member (bits outside m are untouched,
    // and inside m the row holds l and the target l ^ x).
    std::vector<uint8_t> range(n_terms);
    for (int64_t i = 0; i < n_terms; ++i) {
        const uint64_t lo = terms[i].l, hi = terms[i].l ^ terms[i].x;
        // a caller's list has no constraints to check a tuple against
        bool k = !sec->from_list;
        for (const mbr_popc_cons &c : sec->cons)
            k = k && __builtin_popcountll(lo & c.mask) == __builtin_popcountll(hi & c.mask);
        if (sec->modulus > 0) {
            int64_t dw = 0;
            for (int b = 0; b < sec->M; ++b) dw += (int64_t)(((hi >> b) & 1) - ((lo >> b) & 1)) * sec->weights[b];
            k = k && dw % sec->modulus == 0;
        }
        range[i] = terms[i].x == 0 ? kDiagonal : k ? kKeeping : kLeaving;
    }
    op->n_diag = std::count(range.begin(), range.end(), (uint8_t)kDiagonal);
    op->n_keep = op->n_diag + std::count(range.begin(), range.end(), (uint8_t)kKeeping);
    hipStream_t st = as_stream(stream);
    if (sec->width_bits == 32) {
        const int low = std::min((sec->M + 1) / 2, 14);
        MBR_TRY(op_sum_tables(op.get(), low, st));
        if (op->low_bits && op->n_keep == n_terms) MBR_TRY(plan_low(op.get(), st));
    }
    // the three ranges, each by low factor (op_low_kernel) or by the high bits its tuples flip, then as given
    std::vector<int64_t> order(n_terms);
    for (int64_t i = 0; i < n_terms; ++i) order[i] = i;
    const int half = (sec->M + 1) / 2;
    const uint64_t lm = op->n_tiles ? (1ull << op->low_bits) - 1 : 0;
    std::stable_sort(order.begin(), order.end(), [&](int64_t i, int64_t j) {
        const mbr_term &p = terms[i], &q = terms[j];
        const uint64_t fp[5] = {p.m & lm, p.l & lm, p.x & lm, p.s & lm, p.x >> half};
        const uint64_t fq[5] = {q.m & lm, q.l & lm, q.x & lm, q.s & lm, q.x >> half};
        return range[i] != range[j] ? range[i] < range[j] : std::lexicographical_compare(fp, fp + 5, fq, fq + 5);
    });
    const size_t n = (size_t)std::max<int64_t>(n_terms, 1);
    std::vector<double> v(n, 0.0);
    std::vector<uint64_t> ml(2 * n, 0), xs(2 * n, 0);
    for (int64_t i = 0; i < n_terms; ++i) {
        const mbr_term &t = terms[order[i]];
        v[i] = t.v;
        ml[2 * i] = t.m;
        ml[2 * i + 1] = t.l;
        xs[2 * i] = t.x;
        xs[2 * i + 1] = t.s;
    }
    MBR_TRY(upload(op->v, v.data(), n * 8, st));
    if (sec->width_bits == 64) {
        MBR_TRY(upload(op->ml, ml.data(), 2 * n * 8, st));
        MBR_TRY(upload(op->xs, xs.data(), 2 * n * 8, st));
        MBR_TRY(plan_launch<uint64_t>(op.get()));
    } else {
        const std::vector<uint32_t> ml32(ml.begin(), ml.end()), xs32(xs.begin(), xs.end());
        MBR_TRY(upload(op->ml, ml32.data(), 2 * n * 4, st));
        MBR_TRY(upload(op->xs, xs32.data(), 2 * n * 4, st));
        if (!op->n_tiles) MBR_TRY(plan_launch<uint32_t>(op.get()));
    }
    *out = op.release();
    return MBR_OK;
}

mbr_status mbr_operator_apply(const mbr_operator *op, const double *d_x, double *d_y, void *stream) {
    if (!op) MBR_FAIL(MBR_EINVAL, "null operator");
    if (!d_x || !d_y) MBR_FAIL(MBR_EINVAL, "null vector");
    if (d_x == d_y) MBR_FAIL(MBR_EINVAL, "x and y must not alias (gather form reads x while y is written)");
    hipStream_t st = mbr::as_stream(stream);
    if (op->width_bits == 32) return apply_t<uint32_t>(op, d_x, d_y, st);
    return apply_t<uint64_t>(op, d_x, d_y, st);
}

mbr_status mbr_operator_lanczos(const mbr_operator *op, const double *d_v0, int32_t nsteps, double tol,
                                double *e0, int32_t *steps_done, double *alpha, double *beta, void *stream) {
    using namespace mbr;
    if (!op || !d_v0) MBR_FAIL(MBR_EINVAL, "null operator or start vector");
    if (nsteps < 1 || nsteps > 100000) MBR_FAIL(MBR_EINVAL, "nsteps=%d", nsteps);
    if (!(tol >= 0.0)) MBR_FAIL(MBR_EINVAL, "tolerance must be non-negative");
    hipStream_t st = as_stream(stream);
    const uint64_t n = op->sec->n;
    DevBuf buf[3], parts, sc, d_len, d_e0;
    for (auto &b2 : buf) MBR_TRY(b2.alloc(n * 8));
    MBR_TRY(parts.alloc(kRedBlocks * 8));
    MBR_TRY(sc.alloc((2 * (size_t)nsteps + 2) * 8));
    MBR_TRY(d_len.alloc(4));
    MBR_TRY(d_e0.alloc(8));
    double *al = sc.as<double>(), *be = al + nsteps, *norm = be + nsteps;
    MBR_HIP(hipMemsetAsync(sc.p, 0, (2 * (size_t)nsteps + 2) * 8, st));
    int32_t *len = d_len.as<int32_t>();
    // v_0 = v0 / |v0|; the previous vector starts at zero
    double *vp = buf[0].as<double>(), *v = buf[1].as<double>(), *w = buf[2].as<double>();
    op_start_kernel<<<1, 1, 0, st>>>(len, nsteps);
    op_dot_parts<<<kRedBlocks, kBlock, 0, st>>>(d_v0, d_v0, n, parts.as<double>());
    op_reduce<<<1, kBlock, 0, st>>>(parts.as<double>(), norm, 1);
    op_scale_kernel<<<kRedBlocks, kBlock, 0, st>>>(d_v0, v, vp, n, norm);
    MBR_HIP(hipGetLastError());
    for (int32_t j = 0; j < nsteps; ++j) {
        MBR_TRY(mbr_operator_apply(op, v, w, stream));  // w = H v_j
        op_dot_parts<<<kRedBlocks, kBlock, 0, st>>>(v, w, n, parts.as<double>());
        op_reduce<<<1, kBlock, 0, st>>>(parts.as<double>(), al + j, 0);
        op_update_kernel<<<kRedBlocks, kBlock, 0, st>>>(w, v, vp, n, al, be, j, len, parts.as<double>());
        op_beta_kernel<<<1, kBlock, 0, st>>>(parts.as<double>(), al, be, j, nsteps, n, tol, len);
        op_next_kernel<<<kRedBlocks, kBlock, 0, st>>>(w, v, vp, n, be, j, len);
        MBR_HIP(hipGetLastError());
        double *t = vp;  // v_{j+1} now sits in w's buffer, v_j becomes the previous vector
        vp = v;
        v = w;
        w = t;
    }
    MBR_TRY(mbr_tridiag_lowest(al, be, len, nsteps, 1, d_e0.as<double>(), stream));
    int32_t hl = 0;
    double he = 0;
    MBR_HIP(hipMemcpyAsync(&hl, len, 4, hipMemcpyDeviceToHost, st));
    MBR_HIP(hipMemcpyAsync(&he, d_e0.p, 8, hipMemcpyDeviceToHost, st));
    if (alpha) MBR_HIP(hipMemcpyAsync(alpha, al, (size_t)nsteps * 8, hipMemcpyDeviceToHost, st));
    if (beta) MBR_HIP(hipMemcpyAsync(beta, be, (size_t)nsteps * 8, hipMemcpyDeviceToHost, st));
    MBR_HIP(hipStreamSynchronize(st));
    if (e0) *e0 = he;
    if (steps_done) *steps_done = hl;
    return MBR_OK;
}

mbr_status mbr_operator_destroy(mbr_operator *op) {
    delete op;
    return MBR_OK;
}

}  // extern "C"
