// Sector enumeration on the device and unrank by the stored list.
//
// A sector is every M-bit pattern passing a set of popcount windows, in
// ascending numeric order (Sec. III ordering).
//
// High part by high part (up to 32 orbitals): a wave takes all patterns of one
// high part (the low `low_bits` <= 14 bits run through, 64 at a time), and a high
// part that already breaks a window is dropped at once; see sector_block_kernel.
//
// Run by run (a fixed particle number N): the enumeration walks the C(M,N)
// patterns of that number, where each thread owns a run of consecutive combination
// indices, positions itself with a greedy combinadics unrank (inverse of Eq.
// cns) and steps to the next larger pattern of equal popcount with Gosper's rule.
// Beyond 32 orbitals this is the only way; below, runs_are_faster decides.
//
// High parts and runs are visited in increasing order, so a count pass, an
// exclusive scan of the counts and a write pass give the sorted list without
// any sort.
#include <algorithm>
#include <memory>

#include "common.hpp"

namespace {

constexpr int kMaxCons = 16;

struct ConsSet {
    uint64_t mask[kMaxCons];
    int32_t lo[kMaxCons];
    int32_t hi[kMaxCons];
    int32_t n;
    int32_t modulus, residue;  // modulus > 0: sum of the weights of the set bits = residue (mod modulus)
    int32_t weight[64];
};

__device__ __forceinline__ bool in_sector(uint64_t a, const ConsSet &cs) {
    bool ok = true;
    for (int j = 0; j < cs.n; ++j) {
        int h = __popcll(a & cs.mask[j]);
        ok = ok && (h >= cs.lo[j]) && (h <= cs.hi[j]);
    }
    if (ok && cs.modulus > 0) {
        int64_t w = 0;
        for (uint64_t m = a; m; m &= m - 1) w += cs.weight[__builtin_ctzll(m)];
        int64_t r = w % cs.modulus;
        if (r < 0) r += cs.modulus;
        ok = r == cs.residue;
    }
    return ok;
}

// Pattern with combinadics index u among N-of-M patterns (greedy inversion of
// Eq. cns: the largest c with C(c, k) <= u is c_k).
__device__ __forceinline__ uint64_t combo_at(uint64_t u, int N, int M, const uint64_t *bt) {
    uint64_t a = 0;
    int c = M - 1;
    for (int k = N; k >= 1; --k) {
        while (bt[c * 65 + k] > u) --c;
        a |= 1ull << c;
        u -= bt[c * 65 + k];
        --c;
    }
    return a;
}

// Next larger pattern with the same popcount (Gosper).
__device__ __forceinline__ uint64_t next_combo(uint64_t a) {
    uint64_t c = a & (~a + 1);
    uint64_t r = a + c;
    int tz = __builtin_ctzll(a);  // c = 2^tz, so the division by c is a shift
    return (((r ^ a) >> 2) >> tz) | r;
}

__global__ void sector_count_kernel(uint64_t S, uint64_t run, int N, int M, ConsSet cs,
                                    const uint64_t *bt, uint32_t *counts, uint64_t nruns) {
    uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (t >= nruns) return;
    uint64_t u0 = t * run;
    uint64_t len = (S - u0 < run) ? S - u0 : run;
    uint64_t a = combo_at(u0, N, M, bt);
    uint32_t cnt = 0;
    for (uint64_t j = 0; j < len; ++j) {
        cnt += in_sector(a, cs) ? 1u : 0u;
        if (j + 1 < len) a = next_combo(a);
    }
    counts[t] = cnt;
}

template <class P>
__global__ void sector_fill_kernel(uint64_t S, uint64_t run, int N, int M, ConsSet cs,
                                   const uint64_t *bt, const uint64_t *offsets, P *out,
                                   uint64_t nruns) {
    uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (t >= nruns) return;
    uint64_t u0 = t * run;
    uint64_t len = (S - u0 < run) ? S - u0 : run;
    uint64_t a = combo_at(u0, N, M, bt);
    uint64_t o = offsets[t];
    for (uint64_t j = 0; j < len; ++j) {
        if (in_sector(a, cs)) out[o++] = static_cast<P>(a);
        if (j + 1 < len) a = next_combo(a);
    }
}

// ------------------------------------------------------------ up to 32 bits
// Constraints on 32-bit patterns; weights already reduced to [0, modulus).
// The windows that hold low bits come first; those past n are open (an empty
// mask), so that NW windows can be tested per pattern from registers.
struct ConsSet32 {
    uint32_t mask[kMaxCons];
    int32_t lo[kMaxCons];
    uint32_t width[kMaxCons];  // hi - lo
    int32_t n;
    uint32_t modulus, residue;  // 1 and 0 when the sector has no modular weight
    uint32_t weight[32];
};

constexpr int kMaxLow = 14;                   // low bits a wave runs through
constexpr int kMaxHigh = 32 - kMaxLow;
constexpr unsigned kSecBlock = 512;
constexpr uint32_t kSecQueue = 512;            // high parts a workgroup looks over together
constexpr uint32_t kStepUnroll = 4;            // steps in flight (the table of step weights has room for them)
constexpr uint32_t kScanChunk = 1024;         // counts per scan workgroup
constexpr uint32_t kMaxChunks = (1u << kMaxHigh) / kScanChunk;

__device__ __forceinline__ uint32_t add_mod(uint32_t a, uint32_t b, uint32_t m) {
    const uint32_t s = a + b;  // both below m < 2^31
    return s >= m ? s - m : s;
}

// Weight of `bits` placed at bit `shift`, from the weights in LDS.
__device__ __forceinline__ uint32_t weight_of(uint32_t bits, int shift, const uint32_t *weight, uint32_t modulus) {
    uint32_t w = 0;
    for (; bits; bits &= bits - 1) w = add_mod(w, weight[shift + __builtin_ctz(bits)], modulus);
    return w;
}

// A permutation of [0, 2^bits): which high parts a workgroup takes.  Open ones are
// alike (few bits set, when there are few particles), and any regular stride
// hands them to a few workgroups.
__device__ __forceinline__ uint32_t spread(uint32_t i, int bits) {
    const uint32_t mask = (uint32_t)((1ull << bits) - 1);
    uint32_t x = (i * 0x9E3779B1u) & mask;
    x ^= x >> ((bits + 1) / 2);
    return (x * 0x9E3779B1u) & mask;
}

// A workgroup looks over `together` (up to kSecQueue) high parts and queues the
// open ones in LDS, for its waves to take in turn.  One wave per high part h: the
// patterns (h << low_bits) | p, p ascending, 64 at a time, tested against every
// window (three instructions each) and against the modular weight, which is
// split into a part per lane (bits 0-5), one per step (a table in LDS) and one
// per high part.  Without FILL the members are counted, with it they are written
// from offsets[h] on.
//
// Bound by the issue of these tests and the chain of a wave's few open high
// parts, hence the queue: with high parts dealt out to the waves at a fixed
// stride, one wave had up to all of its 32 open (32 orbitals, 4 particles: 1,382
// us, with the queue 147).  Enumerating the C(M,N) patterns of the right
// particle number one by one costs an unrank per 64 patterns and, per pattern,
// 64-bit windows, a loop over the set bits for the weight and a 64-bit
// remainder: total momentum 3 of the 14-site ring (841,332 states), both
// passes: 524 -> 83 us, and the counts no longer go through host memory.
template <class P, bool FILL, int NW>
__global__ void __launch_bounds__(kSecBlock) sector_block_kernel(int low_bits, uint32_t n_high, uint32_t together, ConsSet32 cs,
                                                                 uint32_t *__restrict__ counts,
                                                                 const uint64_t *__restrict__ chunk0, P *__restrict__ out) {
    __shared__ uint32_t weight[32];
    __shared__ __align__(16) uint32_t step_weight[1 << (kMaxLow - 6)];
    __shared__ uint2 queue[kSecQueue];
    __shared__ uint32_t queued;
    const uint32_t steps = low_bits > 6 ? 1u << (low_bits - 6) : 1u;
    const uint32_t lane = threadIdx.x & 63;
    const bool on = low_bits >= 6 || lane < (1u << low_bits);
    const uint32_t modulus = cs.modulus;  // 1 and all weights 0 without a modular weight
    if (threadIdx.x == 0) queued = 0;
    if (threadIdx.x < 32) weight[threadIdx.x] = cs.weight[threadIdx.x];
    __syncthreads();
    for (uint32_t s = threadIdx.x; s < std::max(steps, kStepUnroll); s += blockDim.x) step_weight[s] = weight_of(s, 6, weight, modulus);
    const uint32_t lane_weight = weight_of(lane, 0, weight, modulus);
    __syncthreads();
    const uint32_t low_mask = (1u << low_bits) - 1;
    const int high_bits = 31 - __builtin_clz(n_high);
    const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    for (uint64_t i0 = blockIdx.x; i0 < n_high; i0 += (uint64_t)together * gridDim.x) {
        for (uint32_t k = threadIdx.x; k < together; k += blockDim.x) {
            const uint64_t i = i0 + (uint64_t)k * gridDim.x;
            bool open = i < n_high;
            const uint32_t mh = open ? spread((uint32_t)i, high_bits) : 0u;
            uint32_t need = 0;  // weight the low bits have to bring
            if (open) {
                const uint32_t high = mh << low_bits;
                for (int j = 0; j < cs.n; ++j) {
                    const int c = __popc(high & cs.mask[j]), more = __popc(cs.mask[j] & low_mask);
                    open = open && c <= cs.lo[j] + (int)cs.width[j] && c + more >= cs.lo[j];
                }
                if (open) {
                    need = cs.residue + modulus - weight_of(mh, low_bits, weight, modulus);
                    need = need >= modulus ? need - modulus : need;
                }
                if constexpr (!FILL) {
                    if (!open) counts[mh] = 0;
                }
            }
            const uint64_t live = __ballot(open);
            if (live) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&queued, (uint32_t)__popcll(live));
                at = __builtin_amdgcn_readfirstlane(at);
                if (open) queue[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0))] = make_uint2(mh, need);
            }
        }
        __syncthreads();
        for (uint32_t q = wave; q < queued; q += waves) {
            const uint32_t h = __builtin_amdgcn_readfirstlane(queue[q].x), high = h << low_bits;
            const uint32_t need = __builtin_amdgcn_readfirstlane(queue[q].y);
            uint32_t n = 0;
            uint64_t o = 0;
            if constexpr (FILL) o = chunk0[h / kScanChunk] + counts[h];
            for (uint32_t s0 = 0; s0 < steps; s0 += kStepUnroll) {
                uint64_t b[kStepUnroll];
#pragma unroll
                for (uint32_t u = 0; u < kStepUnroll; ++u) {
                    const uint32_t s = s0 + u, a = high | (s << 6) | lane;
                    bool ok = on & (s < steps);
#pragma unroll
                    for (int j = 0; j < NW; ++j) ok = ok & ((uint32_t)(__popc(a & cs.mask[j]) - cs.lo[j]) <= cs.width[j]);
                    ok = ok & (add_mod(lane_weight, step_weight[s], modulus) == need);
                    b[u] = __ballot(ok);
                }
#pragma unroll
                for (uint32_t u = 0; u < kStepUnroll; ++u) {
                    if constexpr (FILL) {
                        if ((b[u] >> lane) & 1)
                            out[o + __builtin_amdgcn_mbcnt_hi((uint32_t)(b[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b[u], 0))] = (P)(high | ((s0 + u) << 6) | lane);
                        o += (uint64_t)__popcll(b[u]);
                    } else {
                        n += (uint32_t)__popcll(b[u]);
                    }
                }
            }
            if constexpr (!FILL) {
                if (lane == 0) counts[h] = n;
            }
        }
        if (i0 + (uint64_t)together * gridDim.x < n_high) {  // the queue fills again
            __syncthreads();
            if (threadIdx.x == 0) queued = 0;
            __syncthreads();
        }
    }
}

// Counts to offsets within chunks of kScanChunk, in place; sums[c] = the
// chunk's total.
__global__ void __launch_bounds__(kScanChunk) sector_scan_kernel(uint32_t *__restrict__ counts, uint32_t n, uint64_t *__restrict__ sums) {
    __shared__ uint32_t wave_sum[kScanChunk / 64];
    const uint32_t i = blockIdx.x * kScanChunk + threadIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t c = i < n ? counts[i] : 0u;
    uint32_t v = c;  // a chunk holds at most 2^24 patterns
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)v, o, 64);
        if (lane >= (uint32_t)o) v += u;
    }
    if (lane == 63) wave_sum[w] = v;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t k = 0; k < w; ++k) before += wave_sum[k];
    if (i < n) counts[i] = before + v - c;
    if (threadIdx.x == kScanChunk - 1) sums[blockIdx.x] = before + v;
}

// Chunk totals to chunk offsets, in place, the sector size behind them.
__global__ void __launch_bounds__(64) sector_chunks_kernel(uint64_t *sums, uint32_t n) {
    __shared__ uint64_t s[kMaxChunks];
    for (uint32_t i = threadIdx.x; i < n; i += 64) s[i] = sums[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (uint32_t i = 0; i < n; ++i) {
            const uint64_t c = s[i];
            s[i] = t;
            t += c;
        }
        sums[n] = t;
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += 64) sums[i] = s[i];
}

// First position that breaks a caller's list: for j >= 1, list[j] below its
// predecessor (code 1), equal to it (code 2), or any entry with bits at or
// above M (code 3).  The smallest (position << 2 | code) wins, so the first
// offending position decides and the result does not depend on scheduling.
template <class P>
__global__ void list_check_kernel(const P *__restrict__ a, uint64_t n, int M, unsigned long long *first) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    unsigned long long best = ~0ull;
    for (uint64_t j = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; j < n; j += stride) {
        const P v = a[j];
        unsigned code = 0;
        if (M < (int)(8 * sizeof(P)) && (v >> M) != 0) code = 3;
        if (j > 0) {
            const P u = a[j - 1];
            if (u > v) code = 1;
            else if (u == v) code = 2;
        }
        if (code) {
            const unsigned long long key = ((unsigned long long)j << 2) | code;
            best = key < best ? key : best;
            break;  // later positions of this lane cannot be smaller
        }
    }
    if (best != ~0ull) atomicMin(first, best);
}

template <class P>
__global__ void unrank_kernel(const P *__restrict__ states, uint64_t nstates,
                              const uint32_t *__restrict__ idx, uint64_t n, P *__restrict__ out) {
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; j < n; j += stride) {
        uint32_t i = idx[j];
        out[j] = (i < nstates) ? states[i] : static_cast<P>(~(P)0);
    }
}

// The fixed particle number implied by the windows, or -1.
int implied_n(int M, const std::vector<mbr_popc_cons> &cons) {
    uint64_t full = (M == 64) ? ~0ull : ((1ull << M) - 1);
    for (auto &c : cons)
        if (c.mask == full && c.lo == c.hi) return c.lo;
    uint64_t covered = 0;
    int n = 0;
    for (auto &c : cons) {
        if (c.lo != c.hi) continue;
        if (covered & c.mask) return -1;
        covered |= c.mask;
        n += c.lo;
    }
    return covered == full ? n : -1;
}

// Low bits of list_blocks: 2^10 to 2^14 patterns per high part, about 2^16 high
// parts from 26 orbitals on.
int low_bits_of(int M) { return std::min(M, std::max(10, std::min(kMaxLow, M - 16))); }

// Windows that hold one of the low bits.
int low_windows(const std::vector<mbr_popc_cons> &cons, int low) {
    return (int)std::count_if(cons.begin(), cons.end(), [&](const mbr_popc_cons &c) { return (c.mask & ((1ull << low) - 1)) != 0; });
}

// Share of the high parts that the windows leave open: exact for windows that
// share no bits (which are then independent), else by a set of such windows, the
// narrowest first.
double open_share(int M, int low, const std::vector<mbr_popc_cons> &cons) {
    std::vector<std::pair<double, uint64_t>> each;
    for (const mbr_popc_cons &c : cons) {
        const int below = __builtin_popcountll(c.mask & ((1ull << low) - 1)), above = __builtin_popcountll(c.mask) - below;
        double some = 0;
        for (int k = 0; k <= above; ++k)
            if (k <= c.hi && k + below >= c.lo) some += (double)mbr::binom(above, k);
        each.push_back({some / (double)(1ull << above), c.mask});
    }
    std::sort(each.begin(), each.end());
    double share = 1;
    uint64_t seen = 0;
    for (const auto &[part, mask] : each)
        if (!(mask & seen)) {
            share *= part;
            seen |= mask;
        }
    return share;
}

// Whether a sector of up to 32 orbitals with N particles, S = C(M,N), is listed
// sooner by its runs.  In units of one pattern tested against one window (about
// 1 us per million), high parts cost their open patterns and the chain of one
// of them, times 1.3 with two or three windows in the low bits and 5 with more
// (the kernel's instances); runs cost 23.5 per pattern, 47 with a modular weight,
// and a start that grows with the windows.  Beyond 2^28 patterns the counts
// that the runs carry through host memory double their cost.  us by runs / by
// high parts, M orbitals and N particles, one window: M = 32, N = 4 100 / 147, N = 8
// 355 / 1,497, N = 10 1,800 / 2,676, N = 16 30,600 / 3,877; M = 28, N = 6 105 / 111,
// N = 8 167 / 205, N = 10 446 / 261; M = 26, N = 8 131 / 100; 16 sites with (3, 5)
// particles 291 / 381, (3, 6) 592 / 535; nine windows, M = 26, N = 10 334 / 391.
bool runs_are_faster(int M, int N, uint64_t S, const std::vector<mbr_popc_cons> &cons, bool weighted) {
    if (N < 0 || S > (1ull << 28)) return false;
    const int low = low_bits_of(M), n_low = low_windows(cons, low);
    const double each = n_low <= 1 ? 1.0 : n_low <= 3 ? 1.3 : 5.0, chain = 2e3 * (double)(1 << low), all = (double)(1ull << M);
    const double by_runs = (weighted ? 47.0 : 23.5) * ((double)S + 1.6e6 + 0.6e6 * (double)cons.size());
    return each * (all + chain) > by_runs && each * (open_share(M, low, cons) * all + chain) > by_runs;
}

// The list of a sector of N particles, run by run.
mbr_status list_runs(mbr_sector &sec, int N, uint64_t S, hipStream_t s) {
    using namespace mbr;
    const int M = sec.M;
    const uint64_t *bt = nullptr;
    MBR_TRY(device_binom(&bt));
    uint64_t run = 64;
    while ((S + run - 1) / run > (1ull << 24)) run *= 2;
    uint64_t nruns = (S + run - 1) / run;

    ConsSet cs{};
    cs.n = (int32_t)sec.cons.size();
    for (int j = 0; j < cs.n; ++j) {
        cs.mask[j] = sec.cons[j].mask;
        cs.lo[j] = sec.cons[j].lo;
        cs.hi[j] = sec.cons[j].hi;
    }
    cs.modulus = sec.modulus;
    cs.residue = sec.residue;
    for (size_t i = 0; i < sec.weights.size(); ++i) cs.weight[i] = sec.weights[i];
    DevBuf d_counts, d_off;
    MBR_TRY(d_counts.alloc(nruns * sizeof(uint32_t)));
    unsigned blk = 256;
    unsigned grid = static_cast<unsigned>((nruns + blk - 1) / blk);
    sector_count_kernel<<<grid, blk, 0, s>>>(S, run, N, M, cs, bt, d_counts.as<uint32_t>(), nruns);
    MBR_HIP(hipGetLastError());
    std::vector<uint32_t> counts(nruns);
    MBR_HIP(hipMemcpyAsync(counts.data(), d_counts.p, nruns * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    MBR_HIP(hipStreamSynchronize(s));
    std::vector<uint64_t> off(nruns);
    uint64_t total = 0;
    for (uint64_t t = 0; t < nruns; ++t) {
        off[t] = total;
        total += counts[t];
    }
    if (total >= 0xFFFFFFFFull) MBR_FAIL(MBR_ERANGE, "sector of %llu states", (unsigned long long)total);
    sec.n = total;
    MBR_TRY(sec.states.alloc(total * (sec.width_bits / 8)));
    MBR_TRY(upload(d_off, off.data(), nruns * sizeof(uint64_t), s));
    if (total > 0) {
        if (sec.width_bits == 32)
            sector_fill_kernel<<<grid, blk, 0, s>>>(S, run, N, M, cs, bt, d_off.as<uint64_t>(), sec.states.as<uint32_t>(), nruns);
        else
            sector_fill_kernel<<<grid, blk, 0, s>>>(S, run, N, M, cs, bt, d_off.as<uint64_t>(), sec.states.as<uint64_t>(), nruns);
        MBR_HIP(hipGetLastError());
        MBR_HIP(hipStreamSynchronize(s));
    }
    return MBR_OK;
}

// The list of a sector of up to 32 orbitals, high part by high part.
mbr_status list_blocks(mbr_sector &sec, hipStream_t s) {
    using namespace mbr;
    const int M = sec.M;
    const int low = low_bits_of(M);
    const uint32_t n_high = 1u << (M - low), chunks = (n_high + kScanChunk - 1) / kScanChunk;
    ConsSet32 cs{};
    const int n_low = low_windows(sec.cons, low);  // the other windows hold or fail with the high part
    for (const bool with_low : {true, false}) {
        for (const mbr_popc_cons &c : sec.cons) {
            if (((c.mask & ((1ull << low) - 1)) != 0) != with_low) continue;
            cs.mask[cs.n] = (uint32_t)c.mask;
            cs.lo[cs.n] = c.lo;
            cs.width[cs.n++] = (uint32_t)(c.hi - c.lo);
        }
    }
    cs.modulus = sec.modulus > 0 ? (uint32_t)sec.modulus : 1u;
    cs.residue = (uint32_t)sec.residue;
    for (size_t i = 0; i < sec.weights.size(); ++i) cs.weight[i] = (uint32_t)(sec.weights[i] < 0 ? sec.weights[i] + sec.modulus : sec.weights[i]);
    DevBuf scratch;  // chunk offsets and the size, then the counts
    MBR_TRY(scratch.alloc((size_t)(chunks + 1) * 8 + (size_t)n_high * 4));
    uint64_t *sums = scratch.as<uint64_t>();
    uint32_t *counts = reinterpret_cast<uint32_t *>(sums + chunks + 1);
    // a wave for every high part while that leaves CUs idle, then up to 32 waves a CU
    const uint32_t cus = (uint32_t)device_cu_count();
    const unsigned block = 64 * std::clamp(n_high / cus, 1u, kSecBlock / 64);
    const unsigned grid = grid_for(n_high, block / 64, cus * (2048 / kSecBlock));
    const uint32_t together = std::min((n_high + grid - 1) / grid, kSecQueue);
    // windows tested per pattern
    const int nw = n_low <= 1 ? 1 : n_low <= 3 ? 3 : kMaxCons;
    const auto count = nw == 1 ? sector_block_kernel<uint32_t, false, 1> : nw == 3 ? sector_block_kernel<uint32_t, false, 3>
                                                                                    : sector_block_kernel<uint32_t, false, kMaxCons>;
    count<<<grid, block, 0, s>>>(low, n_high, together, cs, counts, nullptr, nullptr);
    sector_scan_kernel<<<chunks, kScanChunk, 0, s>>>(counts, n_high, sums);
    sector_chunks_kernel<<<1, 64, 0, s>>>(sums, chunks);
    MBR_HIP(hipGetLastError());
    uint64_t total = 0;
    MBR_HIP(hipMemcpyAsync(&total, sums + chunks, 8, hipMemcpyDeviceToHost, s));
    MBR_HIP(hipStreamSynchronize(s));
    if (total >= 0xFFFFFFFFull) MBR_FAIL(MBR_ERANGE, "sector of %llu states", (unsigned long long)total);
    sec.n = total;
    MBR_TRY(sec.states.alloc(total * (sec.width_bits / 8)));
    if (total > 0) {
        if (sec.width_bits == 32) {
            const auto fill = nw == 1 ? sector_block_kernel<uint32_t, true, 1> : nw == 3 ? sector_block_kernel<uint32_t, true, 3>
                                                                                           : sector_block_kernel<uint32_t, true, kMaxCons>;
            fill<<<grid, block, 0, s>>>(low, n_high, together, cs, counts, sums, sec.states.as<uint32_t>());
        } else {
            const auto fill = nw == 1 ? sector_block_kernel<uint64_t, true, 1> : nw == 3 ? sector_block_kernel<uint64_t, true, 3>
                                                                                           : sector_block_kernel<uint64_t, true, kMaxCons>;
            fill<<<grid, block, 0, s>>>(low, n_high, together, cs, counts, sums, sec.states.as<uint64_t>());
        }
        MBR_HIP(hipGetLastError());
        MBR_HIP(hipStreamSynchronize(s));
    }
    return MBR_OK;
}

mbr_status sector_build_impl(int32_t M, int32_t width_bits, int32_t n_cons, const mbr_popc_cons *cons,
                             const int32_t *weights, int32_t modulus, int32_t residue, mbr_sector **out,
                             void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (M < 1 || M > 64) MBR_FAIL(MBR_EINVAL, "M=%d outside 1..64", M);
    if (width_bits != 32 && width_bits != 64) MBR_FAIL(MBR_EINVAL, "width_bits=%d", width_bits);
    if (width_bits == 32 && M > 32) MBR_FAIL(MBR_EINVAL, "M=%d needs 64-bit patterns", M);
    if (n_cons < 0 || n_cons > kMaxCons) MBR_FAIL(MBR_EINVAL, "n_cons=%d outside 0..%d", n_cons, kMaxCons);
    if (n_cons > 0 && !cons) MBR_FAIL(MBR_EINVAL, "null constraint list");
    uint64_t full = (M == 64) ? ~0ull : ((1ull << M) - 1);
    std::vector<mbr_popc_cons> cv(cons, cons + n_cons);
    for (auto &c : cv) {
        if (c.mask & ~full) MBR_FAIL(MBR_EINVAL, "constraint mask has bits at or above M");
        if (c.lo < 0 || c.hi < c.lo || c.hi > 64) MBR_FAIL(MBR_EINVAL, "constraint window [%d,%d]", c.lo, c.hi);
    }
    if (modulus < 0 || (modulus > 0 && (!weights || residue < 0 || residue >= modulus)))
        MBR_FAIL(MBR_EINVAL, "modular constraint: modulus %d, residue %d", modulus, residue);
    int N = implied_n(M, cv);
    uint64_t S = 0;
    if (N >= 0) {
        if (N > M) MBR_FAIL(MBR_EINVAL, "N=%d exceeds M=%d", N, M);
        S = binom(M, N);
        if (S > (1ull << 40)) MBR_FAIL(MBR_EUNSUPPORTED, "C(%d,%d) patterns to scan", M, N);
    } else {
        if (M > 32) MBR_FAIL(MBR_EUNSUPPORTED, "M=%d without a fixed particle number", M);
    }
    hipStream_t s = as_stream(stream);
    auto sec = std::make_unique<mbr_sector>();
    sec->M = M;
    sec->width_bits = width_bits;
    sec->cons = cv;
    sec->modulus = modulus;
    sec->residue = residue;
    for (int i = 0; i < M && modulus > 0; ++i) sec->weights.push_back(weights[i] % modulus);
    MBR_HIP(hipGetDevice(&sec->device));
    if (M > 32 || runs_are_faster(M, N, S, cv, modulus > 0)) MBR_TRY(list_runs(*sec, N, S, s));
    else MBR_TRY(list_blocks(*sec, s));
    *out = sec.release();
    return MBR_OK;
}

}  // namespace

extern "C" {

mbr_status mbr_sector_build(int32_t M, int32_t width_bits, int32_t n_cons,
                            const mbr_popc_cons *cons, mbr_sector **out, void *stream) {
    return sector_build_impl(M, width_bits, n_cons, cons, nullptr, 0, 0, out, stream);
}

mbr_status mbr_sector_build_mod(int32_t M, int32_t width_bits, int32_t n_cons, const mbr_popc_cons *cons,
                                const int32_t *weights, int32_t modulus, int32_t residue,
                                mbr_sector **out, void *stream) {
    if (modulus < 1) MBR_FAIL(MBR_EINVAL, "modulus %d must be positive", modulus);
    return sector_build_impl(M, width_bits, n_cons, cons, weights, modulus, residue, out, stream);
}

mbr_status mbr_sector_from_list(int32_t M, int32_t width_bits, const void *d_states, uint64_t n,
                                mbr_sector **out, void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (M < 1 || M > 64) MBR_FAIL(MBR_EINVAL, "M=%d outside 1..64", M);
    if (width_bits != 32 && width_bits != 64) MBR_FAIL(MBR_EINVAL, "width_bits=%d", width_bits);
    if (width_bits == 32 && M > 32) MBR_FAIL(MBR_EINVAL, "M=%d needs 64-bit patterns", M);
    if (n > 0 && !d_states) MBR_FAIL(MBR_EINVAL, "null state list");
    if (n >= 0xFFFFFFFFull) MBR_FAIL(MBR_ERANGE, "list of %llu states", (unsigned long long)n);
    hipStream_t s = as_stream(stream);
    auto sec = std::make_unique<mbr_sector>();
    sec->M = M;
    sec->width_bits = width_bits;
    sec->n = n;
    sec->from_list = true;
    MBR_HIP(hipGetDevice(&sec->device));
    const size_t bytes = (size_t)n * (width_bits / 8);
    MBR_TRY(sec->states.alloc(bytes));
    if (n > 0) {
        MBR_HIP(hipMemcpyAsync(sec->states.p, d_states, bytes, hipMemcpyDeviceToDevice, s));
        const unsigned long long none = ~0ull;
        DevBuf flag;
        MBR_TRY(upload(flag, &none, sizeof none, s));
        const unsigned grid = grid_for(n, 256, device_cu_count() * 8);
        if (width_bits == 32)
            list_check_kernel<uint32_t><<<grid, 256, 0, s>>>(sec->states.as<uint32_t>(), n, M,
                                                             flag.as<unsigned long long>());
        else
            list_check_kernel<uint64_t><<<grid, 256, 0, s>>>(sec->states.as<uint64_t>(), n, M,
                                                             flag.as<unsigned long long>());
        MBR_HIP(hipGetLastError());
        unsigned long long first = 0;
        MBR_HIP(hipMemcpyAsync(&first, flag.p, sizeof first, hipMemcpyDeviceToHost, s));
        MBR_HIP(hipStreamSynchronize(s));
        if (first != ~0ull) {
            const unsigned long long pos = first >> 2;
            switch (first & 3) {
                case 1: MBR_FAIL(MBR_ENOTSORTED, "entry %llu is smaller than entry %llu", pos, pos - 1);
                case 2: MBR_FAIL(MBR_EDUP, "entry %llu repeats entry %llu", pos, pos - 1);
                default: MBR_FAIL(MBR_EINVAL, "entry %llu has bits at or above M=%d", pos, M);
            }
        }
    }
    *out = sec.release();
    return MBR_OK;
}

mbr_status mbr_sector_size(const mbr_sector *s, uint64_t *n) {
    if (!s || !n) MBR_FAIL(MBR_EINVAL, "null argument");
    *n = s->n;
    return MBR_OK;
}

mbr_status mbr_sector_states(const mbr_sector *s, const void **d_states) {
    if (!s || !d_states) MBR_FAIL(MBR_EINVAL, "null argument");
    *d_states = s->states.p;
    return MBR_OK;
}

mbr_status mbr_sector_destroy(mbr_sector *s) {
    delete s;
    return MBR_OK;
}

mbr_status mbr_unrank_batch(const mbr_sector *sec, const uint32_t *d_idx, uint64_t n, void *d_out,
                            void *stream) {
    using namespace mbr;
    if (!sec) MBR_FAIL(MBR_EINVAL, "null sector");
    if (n == 0) return MBR_OK;
    if (!d_idx || !d_out) MBR_FAIL(MBR_EINVAL, "null index or output pointer");
    hipStream_t s = as_stream(stream);
    unsigned blk = 256;
    unsigned grid = grid_for(n, blk, 65536);
    if (sec->width_bits == 32)
        unrank_kernel<uint32_t><<<grid, blk, 0, s>>>(sec->states.as<uint32_t>(), sec->n, d_idx, n,
                                                     static_cast<uint32_t *>(d_out));
    else
        unrank_kernel<uint64_t><<<grid, blk, 0, s>>>(sec->states.as<uint64_t>(), sec->n, d_idx, n,
                                                     static_cast<uint64_t *>(d_out));
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

}  // extern "C"
