// Learned index for ranking (an extension; the paper has none), in two
// stages as a recursive model index (Kraska et al., "The Case for Learned
// Index Structures", 2018):
//  * stage 1: a per-sector network 32 bit features -> 64 -> 64 -> 1 (ReLU)
//    predicts y ~ rank / N_s;
//  * stage 2: y selects one of n_leaves = 2^b leaves, leaf floor(y 2^b); each
//    leaf records the smallest and largest rank of the members the network
//    sends to it, measured with the query kernel's own arithmetic.
// A query is answered by the lower bound of the pattern in states[lo .. hi] of
// its leaf, so answers are exact: a member always lies inside its leaf's window
// and a non-member is never found.  The lower bound is found level by level
// over copies of every kSample^l-th state, l = H..1: a bisection over the top
// copy (at most kTopMax entries, staged in LDS), then at each level one over
// the at most kSample entries the level above leaves open (one 64-byte line),
// then one inside a block of kSample states, so below the top each level
// costs one line per query.  The recorded error e is the widest leaf window (hi - lo); when
// e exceeds the caller's bound the fallback ranker answers instead.  The
// single-window error max |rint(N_s y) - i| of stage 1 alone is kept as a
// statistic.
//
// Parameters (6337 fp32 masters): W1[64][32], b1[64], W2[64][64], b2[64],
// w3[64], b3.  Queries use their bf16 roundings with fp32 accumulation.
//
// Inference runs on the matrix cores, v_mfma_f32_16x16x32_bf16 (wave64, the
// gfx950 form with 32 products per lane pair and instruction): a wave
// evaluates 16 queries per product chain.  Layers are computed transposed,
// D = W * H^T (features x queries): the 16x16 fp32 output fragment of one
// layer (lane l holds features 4*(l/16)+r of query l%16 of a 16-feature
// tile) feeds the next product's B operand (K = features, N = queries)
// without shuffles, because the order in which a product sums over K is
// free: the K slot (g, j) of lane group g = l/16 and element j < 8 of a
// 32-feature chunk c takes feature 16 (2c + j/4) + 4 g + j%4, i.e. the two
// output fragments of tiles 2c and 2c+1 side by side, and the weights are
// loaded in that order.  Activations go from fp32 to bf16 in registers
// (rounded, then ReLU as a packed 16-bit integer maximum).  Training runs in
// fp32, also on the matrix cores (forward with the bf16 weights, backward,
// fixed-order batch reductions, Adam).
#include <algorithm>
#include <cmath>
#include <memory>
#include <mutex>
#include <type_traits>

#include "rank_device.hpp"

namespace {

constexpr int kIn = 32, kH = 64;
constexpr int P_W1 = 0, P_B1 = 2048, P_W2 = 2112, P_B2 = 6208, P_W3 = 6272, P_B3 = 6336;
constexpr int kParams = 6337;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 mfma_bf16x8 __attribute__((ext_vector_type(8)));

__host__ __device__ inline uint16_t f2bf(float f) {
    // round to nearest even (finite inputs)
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__host__ __device__ inline float bf2f(uint16_t b) {
    uint32_t u = (uint32_t)b << 16;
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}

// Per-lane weight fragments of the three products (A operands), biases in the
// output-fragment layout.
struct MlpFrags {
    bf16x8 w1[4];     // tile t: one 32-input chunk
    bf16x8 w2[4][2];  // tile t, 32-feature chunk c
    bf16x8 w3[2];
    f32x4 b1[4];  // the accumulators start from the biases
    f32x4 b2[4];
    f32x4 b3;
};

// Hidden feature of K slot (lane group g, element j) of 32-feature chunk c.
__device__ __forceinline__ int kslot_feature(int c, int g, int j) { return 16 * (2 * c + (j >> 2)) + 4 * g + (j & 3); }

// bf16 bits of parameter i: stored as bf16, or rounded from fp32 as the
// training kernels round them (mlp_round_kernel).
__device__ __forceinline__ uint16_t wbits(const uint16_t *__restrict__ w, int i) { return w[i]; }
__device__ __forceinline__ uint16_t wbits(const float *__restrict__ w, int i) { return f2bf(w[i]); }

// wb: bf16 weights (or fp32 parameters) in parameter order.
template <class W>
__device__ __forceinline__ void load_frags(MlpFrags &f, const W *__restrict__ wb) {
    const int l = threadIdx.x & 63;
    const int row = l & 15, g = l >> 4, kg = g * 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        // layer 1: K slot (g, j) is input bit 8 g + j
#pragma unroll
        for (int j = 0; j < 8; ++j) f.w1[t][j] = (short)wbits(wb, P_W1 + (16 * t + row) * kIn + 8 * g + j);
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                f.w2[t][c][j] = (short)wbits(wb, P_W2 + (16 * t + row) * kH + kslot_feature(c, g, j));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f.b1[t][r] = bf2f(wbits(wb, P_B1 + 16 * t + kg + r));
            f.b2[t][r] = bf2f(wbits(wb, P_B2 + 16 * t + kg + r));
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int j = 0; j < 8; ++j)
            f.w3[c][j] = row == 0 ? (short)wbits(wb, P_W3 + kslot_feature(c, g, j)) : (short)0;
    const float b3 = bf2f(wbits(wb, P_B3));
    f.b3 = (f32x4){b3, b3, b3, b3};
}

// ReLU(acc) rounded to bf16: the hardware conversion (nearest even, the
// rounding of f2bf for finite values, two values per instruction), then the
// ReLU as a packed signed 16-bit maximum with 0 on the bf16 bit patterns
// (every negative value, -0 included, has the sign bit set; rounding keeps
// the sign, so this equals rounding the ReLU).  acc already holds the bias.
typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x4 relu_bf16(const f32x4 &acc) {
    s16x2 h0 = __builtin_bit_cast(s16x2, __builtin_convertvector((f32x2){acc[0], acc[1]}, bf16v2));
    s16x2 h1 = __builtin_bit_cast(s16x2, __builtin_convertvector((f32x2){acc[2], acc[3]}, bf16v2));
    h0 = __builtin_elementwise_max(h0, (s16x2){0, 0});
    h1 = __builtin_elementwise_max(h1, (s16x2){0, 0});
    return (bf16x4){h0[0], h0[1], h1[0], h1[1]};
}

__device__ __forceinline__ f32x4 mfma32(const bf16x8 &a, const bf16x8 &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mfma_bf16x8, a),
                                                   __builtin_bit_cast(mfma_bf16x8, b), c, 0, 0, 0);
}

// Network output for the 16 queries held by lanes 16*grp .. 16*grp+15 of the
// wave (pattern in `q` of each lane).  The result is valid in lanes 0..15,
// lane n holding the output of query 16*grp + n.  All 64 lanes must call.
__device__ __forceinline__ float mlp16(const MlpFrags &f, uint32_t q, int grp) {
    const int l = threadIdx.x & 63;
    const uint32_t a = (uint32_t)__shfl((int)q, 16 * grp + (l & 15), 64);
    const uint32_t bits = (a >> (8 * (l >> 4))) & 0xFFu;  // inputs 8 g .. 8 g + 7
    bf16x8 xb;
#pragma unroll
    for (int j = 0; j < 8; ++j) xb[j] = ((bits >> j) & 1u) ? (short)0x3F80 : (short)0;
    bf16x4 h1[4], h2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) h1[t] = relu_bf16(mfma32(f.w1[t], xb, f.b1[t]));
    const bf16x8 k1[2] = {__builtin_shufflevector(h1[0], h1[1], 0, 1, 2, 3, 4, 5, 6, 7),
                          __builtin_shufflevector(h1[2], h1[3], 0, 1, 2, 3, 4, 5, 6, 7)};
#pragma unroll
    for (int t = 0; t < 4; ++t) h2[t] = relu_bf16(mfma32(f.w2[t][1], k1[1], mfma32(f.w2[t][0], k1[0], f.b2[t])));
    const bf16x8 k2[2] = {__builtin_shufflevector(h2[0], h2[1], 0, 1, 2, 3, 4, 5, 6, 7),
                          __builtin_shufflevector(h2[2], h2[3], 0, 1, 2, 3, 4, 5, 6, 7)};
    const f32x4 acc = mfma32(f.w3[1], k2[1], mfma32(f.w3[0], k2[0], f.b3));
    return acc[0];
}

// Network outputs for the 64 queries of a wave, each lane receiving its own.
// The four groups run one after another: going through each layer with all
// four together hides the latency of the dependent products but needs about
// 180 registers, which costs the ranking kernel more occupancy than it gains.
__device__ __forceinline__ float mlp64(const MlpFrags &f, uint32_t q) {
    const int l = threadIdx.x & 63;
    const float y0 = mlp16(f, q, 0), y1 = mlp16(f, q, 1), y2 = mlp16(f, q, 2), y3 = mlp16(f, q, 3);
    const float s0 = __shfl(y0, l & 15, 64), s1 = __shfl(y1, l & 15, 64);
    const float s2 = __shfl(y2, l & 15, 64), s3 = __shfl(y3, l & 15, 64);
    const int g = l >> 4;
    return g == 0 ? s0 : g == 1 ? s1 : g == 2 ? s2 : s3;
}

__device__ __forceinline__ int64_t predict_rank(float y, uint64_t n) {
    double p = rint((double)n * (double)y);
    if (!(p >= 0.0)) p = 0.0;  // also NaN
    if (p > (double)(n - 1)) p = (double)(n - 1);
    return (int64_t)p;
}

// ---------------------------------------------------------------- inference
template <class W>
__global__ void __launch_bounds__(256) mlp_forward_kernel(const W *__restrict__ wb,
                                                          const uint32_t *__restrict__ q, int B,
                                                          float *__restrict__ out) {
    MlpFrags f;
    load_frags(f, wb);
    const int waves = gridDim.x * (blockDim.x >> 6);
    for (int base = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64; base < B; base += waves * 64) {
        const int i = base + (threadIdx.x & 63);
        const uint32_t a = i < B ? q[i] : 0u;
        const float y = mlp64(f, a);
        if (i < B) out[i] = y;
    }
}

// Largest |p(alpha_i) - i| over the sector (the query kernel's arithmetic).
__global__ void __launch_bounds__(256) mlp_maxerr_kernel(const uint16_t *__restrict__ wb,
                                                         const uint32_t *__restrict__ states,
                                                         uint64_t n, unsigned long long *emax) {
    MlpFrags f;
    load_frags(f, wb);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    unsigned long long e = 0;
    for (uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64; base < n;
         base += waves * 64) {
        const uint64_t i = base + (threadIdx.x & 63);
        const uint32_t a = i < n ? states[i] : 0u;
        const float y = mlp64(f, a);
        if (i < n) {
            const int64_t p = predict_rank(y, n);
            const unsigned long long d = (unsigned long long)(p > (int64_t)i ? p - (int64_t)i : (int64_t)i - p);
            e = d > e ? d : e;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        unsigned long long v = __shfl_down(e, o, 64);
        e = v > e ? v : e;
    }
    if ((threadIdx.x & 63) == 0) atomicMax(emax, e);
}

// Leaf of a network output: floor(y n_leaves) clamped to the leaves (n_leaves
// is a power of two, so the product is exact in fp32); NaN and y <= 0 go to
// leaf 0.
__device__ __forceinline__ uint32_t leaf_of(float y, uint32_t nleaf) {
    if (!(y > 0.f)) return 0u;
    if (y >= 1.f) return nleaf - 1u;
    return (uint32_t)(y * (float)nleaf);
}

// Empty leaves: lo = all ones, hi = 0 (an empty window).
__global__ void leaf_clear_kernel(uint2 *leaf, uint32_t nleaf) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nleaf) leaf[i] = make_uint2(0xFFFFFFFFu, 0u);
}

// Stage-2 windows: every member i widens the window of its leaf to include i.
__global__ void __launch_bounds__(256) leaf_build_kernel(const uint16_t *__restrict__ wb,
                                                         const uint32_t *__restrict__ states, uint64_t n,
                                                         uint32_t nleaf, uint2 *__restrict__ leaf) {
    MlpFrags f;
    load_frags(f, wb);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    for (uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64; base < n;
         base += waves * 64) {
        const uint64_t i = base + (threadIdx.x & 63);
        const uint32_t a = i < n ? states[i] : 0u;
        const float y = mlp64(f, a);
        if (i < n) {
            uint32_t *w = reinterpret_cast<uint32_t *>(leaf + leaf_of(y, nleaf));
            atomicMin(w, (uint32_t)i);
            atomicMax(w + 1, (uint32_t)i);
        }
    }
}

// Window statistics over the members: acc[0] += hi - lo + 1 of each member's
// leaf (the mean window is acc[0] / n), acc[1] = max (hi - lo).
__global__ void __launch_bounds__(256) leaf_stats_kernel(const uint16_t *__restrict__ wb,
                                                         const uint32_t *__restrict__ states, uint64_t n,
                                                         uint32_t nleaf, const uint2 *__restrict__ leaf,
                                                         unsigned long long *acc) {
    MlpFrags f;
    load_frags(f, wb);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    unsigned long long sum = 0, mx = 0;
    for (uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64; base < n;
         base += waves * 64) {
        const uint64_t i = base + (threadIdx.x & 63);
        const uint32_t a = i < n ? states[i] : 0u;
        const float y = mlp64(f, a);
        if (i < n) {
            const uint2 w = leaf[leaf_of(y, nleaf)];
            const unsigned long long d = (unsigned long long)(w.y - w.x);
            sum += d + 1;
            mx = d > mx ? d : mx;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        sum += __shfl_down(sum, o, 64);
        const unsigned long long v = __shfl_down(mx, o, 64);
        mx = v > mx ? v : mx;
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(acc, sum);
        atomicMax(acc + 1, mx);
    }
}

constexpr uint32_t kSample = 16;     // states per sampled block (64 bytes)
constexpr uint32_t kTopMax = 8192;   // entries of the top copy (32 KB of LDS)
constexpr int kMaxLevels = 8;        // kSample^8 = 2^32 states

struct SampleLevels {
    const uint32_t *lv[kMaxLevels];  // lv[l]: states[b kSample^(l+1)]
    int32_t H;                       // copies; lv[H-1] is the top
    uint32_t top_n;                  // entries of the top copy
    uint64_t n;                      // states
};

// sample[b] = states[b stride] for b < nb, all ones up to the padded length
// npad (a multiple of kSample, so every aligned line of the copy can be read
// whole).
__global__ void sample_kernel(const uint32_t *__restrict__ states, uint32_t stride,
                              uint32_t *__restrict__ sample, uint64_t nb, uint64_t npad) {
    for (uint64_t b = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; b < npad; b += (uint64_t)gridDim.x * blockDim.x)
        sample[b] = b < nb ? states[b * stride] : 0xFFFFFFFFu;
}

// Entries [lo, hi) of v lie in the aligned line of kSample entries at base;
// their lower bound for a is lo plus the number below a (they are sorted).
// The line is read as four 16-byte loads in one round trip.
__device__ __forceinline__ uint32_t line_lower_bound(const uint32_t *__restrict__ v, uint32_t base,
                                                     uint32_t lo, uint32_t hi, uint32_t a) {
    const uint4 *p = reinterpret_cast<const uint4 *>(v + base);
    const uint4 q0 = p[0], q1 = p[1], q2 = p[2], q3 = p[3];
    const uint32_t e[kSample] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w,
                                 q2.x, q2.y, q2.z, q2.w, q3.x, q3.y, q3.z, q3.w};
    uint32_t c = 0;
#pragma unroll
    for (uint32_t i = 0; i < kSample; ++i) c += (base + i >= lo && base + i < hi && e[i] < a) ? 1u : 0u;
    return lo + c;
}

// narrow() for a copy below the top: the blocks it considers are the at most
// kSample children of the block the level above left open, one aligned line.
__device__ __forceinline__ void narrow_line(const uint32_t *__restrict__ smp, uint32_t stride, uint32_t a,
                                            uint32_t &L, uint32_t &H1) {
    const uint32_t b0 = L / stride + 1, b1 = (H1 - 1) / stride + 1;
    const uint32_t bl = b1 > b0 ? line_lower_bound(smp, (b0 - 1) & ~(kSample - 1), b0, b1, a) : b0;
    const uint32_t lo = (bl - 1) * stride, hi = bl * stride;
    L = lo > L ? lo : L;
    H1 = hi < H1 ? hi : H1;
}

// Narrow [L, H1), which holds the lower bound of a among the states of the
// window (H1 when none is >= a), to the blocks of `stride` states: among the
// blocks b with b stride in (L, H1 - 1], the first whose sampled state is not
// below a bounds the answer from above and the block before it from below.
template <class PTR>
__device__ __forceinline__ void narrow(PTR smp, uint32_t stride, uint32_t a, uint32_t &L, uint32_t &H1) {
    uint32_t bl = L / stride + 1, br = (H1 - 1) / stride + 1;
    while (bl < br) {
        const uint32_t mid = bl + ((br - bl) >> 1);
        if (smp[mid] < a) bl = mid + 1;
        else br = mid;
    }
    const uint32_t lo = (bl - 1) * stride, hi = bl * stride;
    L = lo > L ? lo : L;
    H1 = hi < H1 ? hi : H1;
}

// NET: the window comes from the network and its leaf; without it the window
// is the whole list and the search alone ranks (a static 16-ary search over
// the sampled copies).
template <bool NET>
__global__ void __launch_bounds__(256) learned_rank_kernel(const uint16_t *__restrict__ wb,
                                                           const uint32_t *__restrict__ states,
                                                           SampleLevels sl,
                                                           const uint2 *__restrict__ leaf, uint32_t nleaf,
                                                           int M, const uint32_t *__restrict__ q,
                                                           uint64_t nq, uint32_t *__restrict__ out) {
    __shared__ uint32_t top[kTopMax];
    for (uint32_t i = threadIdx.x; i < sl.top_n; i += blockDim.x) top[i] = sl.lv[sl.H - 1][i];
    __syncthreads();
    MlpFrags f;
    if constexpr (NET) load_frags(f, wb);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    for (uint64_t base = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64; base < nq;
         base += waves * 64) {
        const uint64_t j = base + (threadIdx.x & 63);
        const uint32_t a = j < nq ? q[j] : 0u;
        uint2 w = make_uint2(0u, (uint32_t)(sl.n - 1));
        if constexpr (NET) {
            const float y = mlp64(f, a);  // every lane of the wave takes part
            if (j < nq) w = leaf[leaf_of(y, nleaf)];
        }
        if (j >= nq) continue;
        const bool in_width = M >= 32 || (a >> M) == 0;
        // lower bound of a in states[lo .. hi] (empty when lo > hi)
        uint32_t L = w.x, R = w.y + 1u;
        bool hit = false;
        if (in_width && w.x <= w.y) {
            uint32_t stride = 1;
            for (int l = 0; l < sl.H; ++l) stride *= kSample;
            narrow(top, stride, a, L, R);
            for (int l = sl.H - 2; l >= 0; --l) {
                stride /= kSample;
                narrow_line(sl.lv[l], stride, a, L, R);
            }
            // [L, R) lies in one aligned block of kSample states
            const uint32_t base = L & ~(kSample - 1);
            if ((uint64_t)base + kSample <= sl.n) {
                L = line_lower_bound(states, base, L, R, a);
            } else {
                while (L < R) {
                    const uint32_t mid = L + ((R - L) >> 1);
                    if (states[mid] < a) L = mid + 1;
                    else R = mid;
                }
            }
            hit = L <= w.y && states[L] == a;
        }
        out[j] = hit ? L : MBR_NOT_FOUND;
    }
}

// ---------------------------------------------------------------- training
// SplitMix64, element k of the stream of `seed` (the generator the sample
// draws are defined by).
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t k) {
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// fp32 value of the bf16 rounding of a parameter.
__device__ __forceinline__ float rounded(float w) { return bf2f(f2bf(w)); }

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int kPart = kParams + 1;       // a workgroup's partial: gradients, then the squared error
constexpr int kPartials = 256;           // partials of a batch at most
constexpr unsigned kGradBlock = 256;     // four waves, each 16 rows of every layer
constexpr int kTileNT = 2;               // 16-sample groups of a tile

// Gradient partials of a batch, one per workgroup, each over the tiles of
// 16 NT samples that it takes in turn: forward with the bf16-rounded weights,
// squared error, backward and the products over the samples, all in fp32 and
// without leaving the workgroup.  Every product runs on the matrix cores in
// fp32 (v_mfma_f32_16x16x4_f32: lane l holds A[l%16][l/16] and B[l/16][l%16] of
// a 4-deep step, and C[4 (l/16) + r][l%16]).  Wave w owns rows 16w .. 16w+15 of
// each layer: its weights stay in registers, as do its gradients; activations
// and their gradients pass between waves through LDS, where one array serves
// both orders (rows as K of the next layer, samples as K of the gradient).
// Samples come from (q, tgt) when given, else are drawn from the sector:
// idx = splitmix64(seed, step*B + s) mod n.
//
// Bound at the batches that training uses by the chain of a tile (five
// products with a barrier between them): 4,096 samples in 11.4 us on 128
// workgroups, and 3.3 us for the sum.  One thread per sample on 64 lanes, with
// the activations through memory to a second kernel, took 132 + 39 us and its
// sum 16 us.  At 2^20 samples 0.49 ms, 80 TFLOP/s of the 138 that a large
// fp32 product reaches (12.7 ms before).  Against 64 bits the gradient is off
// by 5e-8 to 8e-8 (8e-8 to 1.7e-7 before) at 64 to 8,192 samples.  Tiles of 16
// samples gain nothing: 37.1 against 35.0 us a call at 4,096.
//
// A set input bit adds its weight and a clear one adds nothing, whatever the
// weight is, but a product with the clear bit makes NaN of an infinite one, and
// likewise of an infinite gradient.  A workgroup with such weights, or whose
// bias gradients show that there were such gradients, goes through its tiles
// once more, and non-finite values then pass the matrix cores by (CAREFUL).
template <int NT>
__global__ void __launch_bounds__(kGradBlock) mlp_grad_kernel(const float *__restrict__ w, int B,
                                                              const uint32_t *__restrict__ q,
                                                              const float *__restrict__ tgt,
                                                              const uint32_t *__restrict__ states,
                                                              uint64_t n, uint64_t seed, uint64_t step,
                                                              float *__restrict__ part) {
    constexpr int S = 16 * NT, LD = S + 1;
    __shared__ float h1[kH * LD], d1[kH * LD], d2[kH * LD];  // [feature][sample]
    __shared__ float ysum[kGradBlock / 64][S], ts[S];
    __shared__ uint32_t xs[S], again;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
    const int row = 16 * wv + 4 * g;  // this lane's rows of a C fragment: row .. row + 3
    float a1[kIn / 4], a2[kH / 4], a2t[kH / 4];
#pragma unroll
    for (int k = 0; k < kIn / 4; ++k) a1[k] = rounded(w[P_W1 + (16 * wv + c) * kIn + 4 * k + g]);
#pragma unroll
    for (int k = 0; k < kH / 4; ++k) {
        a2[k] = rounded(w[P_W2 + (16 * wv + c) * kH + 4 * k + g]);
        a2t[k] = rounded(w[P_W2 + (4 * k + g) * kH + 16 * wv + c]);
    }
    f32x4 b1, b2, w3;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        b1[r] = rounded(w[P_B1 + row + r]);
        b2[r] = rounded(w[P_B2 + row + r]);
        w3[r] = rounded(w[P_W3 + row + r]);
    }
    const float b3 = rounded(w[P_B3]);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 gw2[4], gw1[2], gb1, gb2, gw3;
    float gb3, sq;
    auto pass = [&](auto careful) {
        constexpr bool CAREFUL = decltype(careful)::value;
        gw2[0] = gw2[1] = gw2[2] = gw2[3] = gw1[0] = gw1[1] = gb1 = gb2 = gw3 = zero;
        gb3 = sq = 0.f;
        for (int tile = blockIdx.x; tile < B / S; tile += gridDim.x) {
            __syncthreads();  // the tile before is done with LDS
            if (threadIdx.x < S) {
                const int s = tile * S + threadIdx.x;
                if (q) {
                    xs[threadIdx.x] = q[s];
                    ts[threadIdx.x] = tgt[s];
                } else {
                    const uint64_t idx = splitmix64_at(seed, step * (uint64_t)B + (uint64_t)s) % n;
                    xs[threadIdx.x] = states[idx];
                    ts[threadIdx.x] = (float)((double)idx / (double)n);
                }
            }
            __syncthreads();
            // layer 1: K is the input bits
            f32x4 h[NT];
            uint32_t x[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                x[t] = xs[16 * t + c];
                h[t] = b1;
            }
#pragma unroll
            for (int k = 0; k < kIn / 4; ++k)
#pragma unroll
                for (int t = 0; t < NT; ++t) h[t] = mfma_f32(CAREFUL && !isfinite(a1[k]) ? 0.f : a1[k], (x[t] >> (4 * k + g)) & 1u ? 1.f : 0.f, h[t]);
            if constexpr (CAREFUL)
                for (int k = 0; k < kIn; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = rounded(w[P_W1 + (row + r) * kIn + k]);
                        if (!isfinite(v))
#pragma unroll
                            for (int t = 0; t < NT; ++t) h[t][r] += (x[t] >> k) & 1u ? v : 0.f;
                    }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    h[t][r] = h[t][r] > 0.f ? h[t][r] : 0.f;
                    h1[(row + r) * LD + 16 * t + c] = h[t][r];
                }
            __syncthreads();
            // layer 2, and the output's share of these rows
            f32x4 z[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) z[t] = b2;
#pragma unroll
            for (int k = 0; k < kH / 4; ++k)
#pragma unroll
                for (int t = 0; t < NT; ++t) z[t] = mfma_f32(a2[k], h1[(4 * k + g) * LD + 16 * t + c], z[t]);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float y = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    z[t][r] = z[t][r] > 0.f ? z[t][r] : 0.f;
                    y += w3[r] * z[t][r];
                }
                y += __shfl_xor(y, 16, 64);
                y += __shfl_xor(y, 32, 64);
                if (g == 0) ysum[wv][16 * t + c] = y;
            }
            __syncthreads();
            // output, its error, and back to layer 2
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int s = 16 * t + c;
                const float y = b3 + ((ysum[0][s] + ysum[1][s]) + (ysum[2][s] + ysum[3][s]));
                const float e = y - ts[s], d = 2.f * e / (float)B;
                if (wv == 0 && g == 0) {
                    sq += e * e;
                    gb3 += d;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // carefully, a non-finite error reaches the units at rest too
                    const float dz = CAREFUL ? (z[t][r] > 0.f ? 1.f : 0.f) * d * w3[r] : z[t][r] > 0.f ? d * w3[r] : 0.f;
                    gw3[r] += d * z[t][r];
                    gb2[r] += dz;
                    d2[(row + r) * LD + s] = dz;
                }
            }
            __syncthreads();
            // back to layer 1
            f32x4 u[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) u[t] = zero;
#pragma unroll
            for (int k = 0; k < kH / 4; ++k)
#pragma unroll
                for (int t = 0; t < NT; ++t) u[t] = mfma_f32(a2t[k], d2[(4 * k + g) * LD + 16 * t + c], u[t]);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float dz = h[t][r] > 0.f ? u[t][r] : 0.f;
                    gb1[r] += dz;
                    d1[(row + r) * LD + 16 * t + c] = dz;
                }
            wave_lds_fence();  // a wave reads only its own rows of d1
            // weight gradients: K is the samples
#pragma unroll
            for (int k = 0; k < S / 4; ++k) {
                const float a = d2[(16 * wv + c) * LD + 4 * k + g];
#pragma unroll
                for (int j = 0; j < 4; ++j) gw2[j] = mfma_f32(a, h1[(16 * j + c) * LD + 4 * k + g], gw2[j]);
                float e = d1[(16 * wv + c) * LD + 4 * k + g];
                if constexpr (CAREFUL) e = isfinite(e) ? e : 0.f;
                const uint32_t xk = xs[4 * k + g];
#pragma unroll
                for (int j = 0; j < 2; ++j) gw1[j] = mfma_f32(e, (xk >> (16 * j + c)) & 1u ? 1.f : 0.f, gw1[j]);
            }
            if constexpr (CAREFUL)
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = d1[(row + r) * LD + s];
                        if (!isfinite(v))
#pragma unroll
                            for (int j = 0; j < 2; ++j) gw1[j][r] += (xs[s] >> (16 * j + c)) & 1u ? v : 0.f;
                    }
        }
    };
    if (threadIdx.x == 0) again = 0;
    pass(std::false_type{});  // with barriers behind the line above
    float probe = gb3;        // not finite if any of these is not
#pragma unroll
    for (int k = 0; k < kIn / 4; ++k) probe += 0.f * a1[k];
#pragma unroll
    for (int r = 0; r < 4; ++r) probe += 0.f * w3[r] + (gb1[r] + gb2[r]);
    if (!isfinite(probe)) again = 1;
    __syncthreads();
    if (again) pass(std::true_type{});
    float *out = part + (size_t)blockIdx.x * kPart;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[P_W2 + (row + r) * kH + 16 * j + c] = gw2[j][r];
#pragma unroll
        for (int j = 0; j < 2; ++j) out[P_W1 + (row + r) * kIn + 16 * j + c] = gw1[j][r];
        // the sums over samples of the 16 lanes of a row
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            gb1[r] += __shfl_xor(gb1[r], o, 64);
            gb2[r] += __shfl_xor(gb2[r], o, 64);
            gw3[r] += __shfl_xor(gw3[r], o, 64);
        }
        if (c == 0) {
            out[P_B1 + row + r] = gb1[r];
            out[P_B2 + row + r] = gb2[r];
            out[P_W3 + row + r] = gw3[r];
        }
    }
    if (wv == 0) {
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            gb3 += __shfl_xor(gb3, o, 64);
            sq += __shfl_xor(sq, o, 64);
        }
        if (lane == 0) {
            out[P_B3] = gb3;
            out[kParams] = sq;
        }
    }
}

// Sum of the partials, fixed order: 8 waves take every 8th partial of 64
// parameters, then wave 0 adds the wave sums.  Optionally applies one Adam
// step to the fp32 masters and refreshes the rounded copies (fp32 value and
// bf16 bits); with loss, the mean squared error of the B samples.
constexpr unsigned kSumBlock = 512;

__global__ void __launch_bounds__(kSumBlock) mlp_reduce_adam_kernel(const float *__restrict__ part, int np, float *grad, float *loss, int B,
                                                                    float *w, float *m, float *v, float *wr, uint16_t *wb, float lr,
                                                                    float b1c, float b2c, int adam) {
    __shared__ float red[kSumBlock / 64][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
    float g = 0.f;
    if (p < kPart)
#pragma unroll 8
        for (int k = wave; k < np; k += kSumBlock / 64) g += part[(size_t)k * kPart + p];
    red[wave][lane] = g;
    __syncthreads();
    if (wave != 0 || p >= kPart) return;
    g = 0.f;
    for (int k = 0; k < (int)(kSumBlock / 64); ++k) g += red[k][lane];
    if (p == kParams) {
        if (loss) *loss = g / (float)B;
        return;
    }
    if (grad) grad[p] = g;
    if (!adam) return;
    const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    const float mm = beta1 * m[p] + (1.f - beta1) * g;
    const float vv = beta2 * v[p] + (1.f - beta2) * g * g;
    m[p] = mm;
    v[p] = vv;
    const float mh = mm / b1c, vh = vv / b2c;
    const float nw = w[p] - lr * mh / (sqrtf(vh) + eps);
    w[p] = nw;
    const uint16_t b = f2bf(nw);
    wb[p] = b;
    wr[p] = bf2f(b);
}

__global__ void mlp_round_kernel(const float *__restrict__ w, float *wr, uint16_t *wb) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= kParams) return;
    const uint16_t b = f2bf(w[p]);
    wb[p] = b;
    wr[p] = bf2f(b);
}

constexpr size_t part_bytes(int partials) { return (size_t)partials * kPart * 4; }
constexpr unsigned kSumGrid = (kPart + 63) / 64;

// Workgroups (and partials) of a batch of B samples (a multiple of 32).
int partials_of(int B) { return std::min(B / (16 * kTileNT), kPartials); }

// Scratch of the gradient entry points in file-scope device arrays, one for
// each of them: the partials of a batch.  Each device holds its own copies for
// the life of the process; host code uses only the address hipGetSymbolAddress
// returns for the current device (static_scratch).
constexpr int kStaticBatch = 8192;
static __device__ __align__(256) float scratch[kPartials * kPart];         // mbr_mlp_gradients_noalloc
static __device__ __align__(256) float shared_scratch[kPartials * kPart];  // mbr_mlp_gradients, one call at a time

constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
float *g_static_ptr[2][kMaxDevices] = {{nullptr}};
std::mutex g_shared_mu[kMaxDevices];  // holders of shared_scratch

// Device address of `scratch` (0) or `shared_scratch` (1) on the current
// device, looked up once per device.
mbr_status static_scratch(int which, float **out, int *device) {
    int dev = 0;
    MBR_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) MBR_FAIL(MBR_EUNSUPPORTED, "device %d beyond %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (!g_static_ptr[which][dev]) {
        void *p = nullptr;
        const hipError_t e = which ? hipGetSymbolAddress(&p, HIP_SYMBOL(shared_scratch)) : hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            MBR_FAIL(MBR_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_static_ptr[which][dev] = static_cast<float *>(p);
    }
    *out = g_static_ptr[which][dev];
    if (device) *device = dev;
    return MBR_OK;
}

// Gradient partials of one batch.
mbr_status batch_grad(const float *w, int B, const uint32_t *q, const float *tgt, const uint32_t *states, uint64_t n, uint64_t seed,
                      uint64_t step, float *part, hipStream_t s) {
    mlp_grad_kernel<kTileNT><<<partials_of(B), kGradBlock, 0, s>>>(w, B, q, tgt, states, n, seed, step, part);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

// Gradients and loss of one batch through the partials at `part`.
mbr_status batch_sum(const float *w, int B, const uint32_t *q, const float *tgt, float *grad, float *loss, float *part, hipStream_t s) {
    MBR_TRY(batch_grad(w, B, q, tgt, nullptr, 0, 0, 0, part, s));
    mlp_reduce_adam_kernel<<<kSumGrid, kSumBlock, 0, s>>>(part, partials_of(B), grad, loss, B, nullptr, nullptr, nullptr, nullptr, nullptr,
                                                          0.f, 1.f, 1.f, 0);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

}  // namespace

struct LearnedModel {
    bool net = true;              // false: sampled-copy search over the whole list
    uint64_t n = 0;
    int32_t M = 0;
    mbr::DevBuf w, m, v, wr, wb;  // masters, Adam moments, rounded fp32, bf16
    mbr::DevBuf leaf;             // stage-2 windows, uint2 {lo, hi} per leaf
    mbr::DevBuf sample[kMaxLevels];  // copy l: every kSample^(l+1)-th state of the sector
    int32_t n_sample = 0;
    uint32_t n_leaves = 0;
    uint64_t e = 0;               // widest leaf window, hi - lo
    uint64_t e_single = 0;        // max |rint(N_s y) - i| of stage 1 alone
    double mean_window = 0;       // member-weighted mean of hi - lo + 1
    int32_t uses_window = 0;
    double last_loss = 0;
};

void learned_free(LearnedModel *m) { delete m; }
int32_t learned_levels(const LearnedModel *m) { return m ? m->n_sample + 1 : 0; }
uint64_t learned_bytes(const LearnedModel *m) {
    if (!m) return 0;
    uint64_t b = m->net ? (uint64_t)kParams * 2 + (uint64_t)m->n_leaves * 8 : 0;
    for (int l = 0; l < m->n_sample; ++l) b += m->sample[l].bytes;
    return b;
}

// Sampled copies of the sector list, every kSample^l-th state, until the
// top one fits kTopMax.
static mbr_status build_samples(LearnedModel &lm, const mbr_sector *sec, hipStream_t s) {
    using namespace mbr;
    uint64_t stride = 1, nb = sec->n;
    lm.n_sample = 0;
    do {
        stride *= kSample;
        nb = (sec->n + stride - 1) / stride;
        const uint64_t npad = (nb + kSample - 1) / kSample * kSample;
        DevBuf &d = lm.sample[lm.n_sample++];
        MBR_TRY(d.alloc(npad * 4));
        sample_kernel<<<grid_for(npad, 256, device_cu_count() * 8), 256, 0, s>>>(
            sec->states.as<uint32_t>(), (uint32_t)stride, d.as<uint32_t>(), nb, npad);
    } while (nb > kTopMax && lm.n_sample < kMaxLevels);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

mbr_status rank_learned_launch(const mbr_ranker *r, const void *q, uint64_t n, uint32_t *out,
                               hipStream_t s) {
    const LearnedModel &lm = *r->learned;
    if (lm.net && !lm.uses_window) {
        if (!r->fallback) MBR_FAIL(MBR_EINVAL, "learned ranker without window or fallback");
        return mbr_rank_batch(r->fallback, q, n, out, s);
    }
    const unsigned grid = mbr::grid_for(n, 256, mbr::device_cu_count() * 8);
    SampleLevels sl{};
    sl.H = lm.n_sample;
    uint64_t stride = 1;
    for (int l = 0; l < lm.n_sample; ++l) {
        sl.lv[l] = lm.sample[l].as<uint32_t>();
        stride *= kSample;
    }
    sl.top_n = (uint32_t)((lm.n + stride - 1) / stride);
    sl.n = lm.n;
    auto kernel = lm.net ? learned_rank_kernel<true> : learned_rank_kernel<false>;
    kernel<<<grid, 256, 0, s>>>(lm.wb.as<uint16_t>(), r->sector->states.as<uint32_t>(), sl,
                                lm.leaf.as<uint2>(), lm.n_leaves, lm.M, static_cast<const uint32_t *>(q), n,
                                out);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

namespace {

// He-uniform initialisation from SplitMix64 (host), biases zero.
std::vector<float> init_params(uint64_t seed) {
    std::vector<float> p(kParams, 0.f);
    uint64_t k = 0;
    auto u01 = [&]() {
        uint64_t z = seed + (++k) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        return (double)(z >> 11) * (1.0 / 9007199254740992.0);
    };
    const double a1 = std::sqrt(6.0 / kIn), a2 = std::sqrt(6.0 / kH), a3 = std::sqrt(3.0 / kH);
    for (int i = 0; i < kH * kIn; ++i) p[P_W1 + i] = (float)((2 * u01() - 1) * a1);
    for (int i = 0; i < kH * kH; ++i) p[P_W2 + i] = (float)((2 * u01() - 1) * a2);
    for (int i = 0; i < kH; ++i) p[P_W3 + i] = (float)((2 * u01() - 1) * a3);
    p[P_B3] = 0.5f;
    return p;
}

}  // namespace

extern "C" {

mbr_status mbr_learned_train(const mbr_sector *sec, const mbr_learned_opts *o,
                             const mbr_ranker *fallback, mbr_ranker **out, void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (!sec || !o) MBR_FAIL(MBR_EINVAL, "null sector or options");
    if (sec->width_bits != 32) MBR_FAIL(MBR_EUNSUPPORTED, "learned ranking needs 32-bit patterns");
    if (sec->n < 2) MBR_FAIL(MBR_EINVAL, "sector of %llu states", (unsigned long long)sec->n);
    if (sec->n >= MBR_NOT_FOUND) MBR_FAIL(MBR_ERANGE, "ranks of %llu states do not fit below MBR_NOT_FOUND",
                                          (unsigned long long)sec->n);
    if (o->epochs < 0 || o->batch < 256 || o->batch % 256 != 0 || o->batch > (1 << 20))
        MBR_FAIL(MBR_EINVAL, "epochs=%d batch=%d (batch: multiple of 256 up to 2^20)", o->epochs, o->batch);
    if (!(o->lr > 0.f)) MBR_FAIL(MBR_EINVAL, "lr must be positive");
    if (o->log2_leaves != 0 && (o->log2_leaves < 8 || o->log2_leaves > 28))
        MBR_FAIL(MBR_EINVAL, "log2_leaves=%d (0, or 8 to 28)", o->log2_leaves);
    if (fallback && fallback->n_states != sec->n) MBR_FAIL(MBR_EINVAL, "fallback ranks a different sector");
    hipStream_t s = as_stream(stream);
    auto lm = std::make_unique<LearnedModel>();
    lm->n = sec->n;
    lm->M = sec->M;
    std::vector<float> p0 = init_params(o->seed);
    MBR_TRY(upload(lm->w, p0.data(), kParams * 4, s));
    MBR_TRY(lm->m.alloc(kParams * 4));
    MBR_TRY(lm->v.alloc(kParams * 4));
    MBR_TRY(lm->wr.alloc(kParams * 4));
    MBR_TRY(lm->wb.alloc(kParams * 2));
    MBR_HIP(hipMemsetAsync(lm->m.p, 0, kParams * 4, s));
    MBR_HIP(hipMemsetAsync(lm->v.p, 0, kParams * 4, s));
    mlp_round_kernel<<<(kParams + 255) / 256, 256, 0, s>>>(lm->w.as<float>(), lm->wr.as<float>(), lm->wb.as<uint16_t>());
    DevBuf part;
    const int np = partials_of(o->batch);
    MBR_TRY(part.alloc(part_bytes(np)));
    const uint64_t per_epoch = o->samples_per_epoch ? o->samples_per_epoch : sec->n;
    const uint64_t steps_per_epoch = (per_epoch + o->batch - 1) / o->batch;
    const uint64_t total = steps_per_epoch * (uint64_t)o->epochs;
    double b1p = 1.0, b2p = 1.0;
    for (uint64_t st = 0; st < total; ++st) {
        MBR_TRY(batch_grad(lm->wr.as<float>(), o->batch, nullptr, nullptr, sec->states.as<uint32_t>(), sec->n, o->seed, st,
                           part.as<float>(), s));
        b1p *= 0.9;
        b2p *= 0.999;
        // cosine decay of the step size over the run
        const double lr = o->lr * 0.5 * (1.0 + std::cos(3.14159265358979323846 * (double)st / (double)total));
        mlp_reduce_adam_kernel<<<kSumGrid, kSumBlock, 0, s>>>(
            part.as<float>(), np, nullptr, nullptr, o->batch, lm->w.as<float>(), lm->m.as<float>(), lm->v.as<float>(),
            lm->wr.as<float>(), lm->wb.as<uint16_t>(), (float)lr, (float)(1.0 - b1p), (float)(1.0 - b2p), 1);
        MBR_HIP(hipGetLastError());
    }
    // maximum error with the query kernel's own arithmetic
    DevBuf d_e;
    MBR_TRY(d_e.alloc(8));
    MBR_HIP(hipMemsetAsync(d_e.p, 0, 8, s));
    const unsigned grid = grid_for(sec->n, 256, device_cu_count() * 8);
    mlp_maxerr_kernel<<<grid, 256, 0, s>>>(lm->wb.as<uint16_t>(), sec->states.as<uint32_t>(), sec->n,
                                           d_e.as<unsigned long long>());
    MBR_HIP(hipGetLastError());
    // stage 2: leaf windows (about four members per leaf), then their statistics
    // Automatic: about four members per leaf, at most 2^12 leaves.  The table
    // (32 KB) then stays in every L2; with many more leaves the leaf read
    // becomes a gather from HBM that costs more than the narrower windows
    // save (2^26 leaves: 13.0 against 16.3 Granks/s on a 165.6 M sector).
    uint64_t nl = 256;
    if (o->log2_leaves) nl = 1ull << o->log2_leaves;
    else
        while (nl < sec->n / 4 && nl < (1ull << 12)) nl <<= 1;
    lm->n_leaves = (uint32_t)nl;
    MBR_TRY(lm->leaf.alloc(nl * 8));
    MBR_TRY(build_samples(*lm, sec, s));
    leaf_clear_kernel<<<(unsigned)((nl + 255) / 256), 256, 0, s>>>(lm->leaf.as<uint2>(), (uint32_t)nl);
    leaf_build_kernel<<<grid, 256, 0, s>>>(lm->wb.as<uint16_t>(), sec->states.as<uint32_t>(), sec->n,
                                           (uint32_t)nl, lm->leaf.as<uint2>());
    DevBuf d_acc;
    MBR_TRY(d_acc.alloc(16));
    MBR_HIP(hipMemsetAsync(d_acc.p, 0, 16, s));
    leaf_stats_kernel<<<grid, 256, 0, s>>>(lm->wb.as<uint16_t>(), sec->states.as<uint32_t>(), sec->n,
                                           (uint32_t)nl, lm->leaf.as<uint2>(), d_acc.as<unsigned long long>());
    MBR_HIP(hipGetLastError());
    unsigned long long e = 0, acc[2] = {0, 0};
    MBR_HIP(hipMemcpyAsync(&e, d_e.p, 8, hipMemcpyDeviceToHost, s));
    MBR_HIP(hipMemcpyAsync(acc, d_acc.p, 16, hipMemcpyDeviceToHost, s));
    MBR_HIP(hipStreamSynchronize(s));
    lm->e_single = e;
    lm->e = acc[1];
    lm->mean_window = (double)acc[0] / (double)sec->n;
    lm->uses_window = (lm->e <= o->max_window) ? 1 : 0;
    if (!lm->uses_window && !fallback)
        MBR_FAIL(MBR_ERANGE, "widest leaf window %llu exceeds max_window and no fallback was given",
                 (unsigned long long)lm->e);
    auto *r = new (std::nothrow) mbr_ranker;
    if (!r) MBR_FAIL(MBR_ENOMEM, "host allocation");
    r->kind = MBR_RANKER_LEARNED;
    r->M = sec->M;
    r->k = 0;
    r->width_bits = 32;
    r->n_states = sec->n;
    r->sector = sec;
    r->fallback = fallback;
    (void)hipGetDevice(&r->device);
    r->learned = lm.release();
    *out = r;
    return MBR_OK;
}

mbr_status mbr_build_sampled_ranker(const mbr_sector *sec, mbr_ranker **out, void *stream) {
    using namespace mbr;
    if (!out) MBR_FAIL(MBR_EINVAL, "null output handle");
    *out = nullptr;
    if (!sec) MBR_FAIL(MBR_EINVAL, "null sector");
    if (sec->width_bits != 32) MBR_FAIL(MBR_EUNSUPPORTED, "the sampled search needs 32-bit patterns");
    if (sec->n == 0) MBR_FAIL(MBR_EINVAL, "empty sector");
    if (sec->n >= MBR_NOT_FOUND) MBR_FAIL(MBR_ERANGE, "ranks of %llu states do not fit below MBR_NOT_FOUND",
                                          (unsigned long long)sec->n);
    hipStream_t s = as_stream(stream);
    auto lm = std::make_unique<LearnedModel>();
    lm->net = false;
    lm->n = sec->n;
    lm->M = sec->M;
    lm->uses_window = 1;
    MBR_TRY(build_samples(*lm, sec, s));
    MBR_HIP(hipStreamSynchronize(s));
    auto r = std::make_unique<mbr_ranker>();
    r->kind = MBR_RANKER_SAMPLED;
    r->M = sec->M;
    r->k = 0;
    r->width_bits = 32;
    r->n_states = sec->n;
    r->sector = sec;
    (void)hipGetDevice(&r->device);
    r->learned = lm.release();
    *out = r.release();
    return MBR_OK;
}

mbr_status mbr_learned_max_error(const mbr_ranker *r, uint64_t *e, int32_t *uses_window) {
    if (!r || r->kind != MBR_RANKER_LEARNED) MBR_FAIL(MBR_EINVAL, "not a learned ranker");
    if (e) *e = r->learned->e;
    if (uses_window) *uses_window = r->learned->uses_window;
    return MBR_OK;
}

mbr_status mbr_learned_autotune(mbr_ranker *r, const void *d_q, uint64_t n, int32_t reps, double *ms_window,
                                double *ms_fallback, void *stream) {
    using namespace mbr;
    if (!r || r->kind != MBR_RANKER_LEARNED || !r->learned) MBR_FAIL(MBR_EINVAL, "not a learned ranker");
    if (!r->fallback) MBR_FAIL(MBR_EINVAL, "learned ranker without a fallback");
    if (!d_q || n == 0) MBR_FAIL(MBR_EINVAL, "no queries");
    if (reps < 1 || reps > 1000) MBR_FAIL(MBR_EINVAL, "reps=%d outside 1..1000", reps);
    hipStream_t s = as_stream(stream);
    LearnedModel &lm = *r->learned;
    const int32_t keep = lm.uses_window;
    DevBuf ranks;
    MBR_TRY(ranks.alloc(n * 4));
    hipEvent_t e0, e1;
    MBR_HIP(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        MBR_FAIL(MBR_EHIP, "hipEventCreate failed");
    }
    double t[2] = {0, 0};
    mbr_status st = MBR_OK;
    for (int path = 0; path < 2 && st == MBR_OK; ++path) {
        lm.uses_window = path == 0 ? 1 : 0;  // 0: window search, 1: fallback
        st = rank_learned_launch(r, d_q, n, ranks.as<uint32_t>(), s);
        if (st != MBR_OK) break;
        (void)hipEventRecord(e0, s);
        for (int i = 0; i < reps && st == MBR_OK; ++i) st = rank_learned_launch(r, d_q, n, ranks.as<uint32_t>(), s);
        (void)hipEventRecord(e1, s);
        float ms = 0;
        hipError_t he = hipEventSynchronize(e1);
        if (he == hipSuccess) he = hipEventElapsedTime(&ms, e0, e1);
        if (st == MBR_OK && he != hipSuccess) {
            set_error("timing failed: %s", hipGetErrorString(he));
            st = MBR_EHIP;
        }
        t[path] = ms / reps;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != MBR_OK) {
        lm.uses_window = keep;
        return st;
    }
    lm.uses_window = t[0] <= t[1] ? 1 : 0;
    if (ms_window) *ms_window = t[0];
    if (ms_fallback) *ms_fallback = t[1];
    return MBR_OK;
}

mbr_status mbr_learned_stats(const mbr_ranker *r, mbr_learned_info *info) {
    if (!r || r->kind != MBR_RANKER_LEARNED || !info) MBR_FAIL(MBR_EINVAL, "not a learned ranker");
    const LearnedModel &lm = *r->learned;
    info->n_leaves = lm.n_leaves;
    info->max_window = lm.e;
    info->mean_window = lm.mean_window;
    info->single_window_error = lm.e_single;
    info->uses_window = lm.uses_window;
    return MBR_OK;
}

mbr_status mbr_learned_params(const mbr_ranker *r, float *host_out, void *stream) {
    if (!r || r->kind != MBR_RANKER_LEARNED || !host_out) MBR_FAIL(MBR_EINVAL, "bad argument");
    hipStream_t s = mbr::as_stream(stream);
    MBR_HIP(hipMemcpyAsync(host_out, r->learned->wr.p, kParams * 4, hipMemcpyDeviceToHost, s));
    MBR_HIP(hipStreamSynchronize(s));
    return MBR_OK;
}

mbr_status mbr_mlp_forward(const float *d_params, const uint32_t *d_q, int32_t B, float *d_pred,
                           void *stream) {
    using namespace mbr;
    if (!d_params || !d_q || !d_pred) MBR_FAIL(MBR_EINVAL, "null pointer");
    if (B <= 0 || B % 64 != 0) MBR_FAIL(MBR_EINVAL, "B=%d must be a positive multiple of 64", B);
    hipStream_t s = as_stream(stream);
    // each workgroup rounds the fp32 parameters to bf16 as it loads them
    mlp_forward_kernel<float><<<grid_for((uint64_t)B, 256, 4096), 256, 0, s>>>(d_params, d_q, B, d_pred);
    MBR_HIP(hipGetLastError());
    return MBR_OK;
}

mbr_status mbr_mlp_gradients(const float *d_params, const uint32_t *d_q, const float *d_tgt, int32_t B,
                             float *d_grad, float *d_loss, void *stream) {
    using namespace mbr;
    if (!d_params || !d_q || !d_tgt || !d_grad) MBR_FAIL(MBR_EINVAL, "null pointer");
    if (B <= 0 || B % 64 != 0) MBR_FAIL(MBR_EINVAL, "B=%d must be a positive multiple of 64", B);
    hipStream_t s = as_stream(stream);
    float *part = nullptr;
    int dev = 0;
    MBR_TRY(static_scratch(1, &part, &dev));
    // The call waits for its work, so whoever holds the lock has the scratch to
    // itself; a call that comes meanwhile (another thread) allocates its own.
    std::unique_lock<std::mutex> lk(g_shared_mu[dev], std::try_to_lock);
    DevBuf own;
    if (!lk.owns_lock()) {
        MBR_TRY(own.alloc(part_bytes(partials_of(B))));
        part = own.as<float>();
    }
    const mbr_status st = batch_sum(d_params, B, d_q, d_tgt, d_grad, d_loss, part, s);
    MBR_HIP(hipStreamSynchronize(s));
    return st;
}

mbr_status mbr_mlp_gradients_noalloc(const float *d_params, const uint32_t *d_q, const float *d_tgt, int32_t B,
                                     float *d_grad, float *d_loss, void *stream) {
    using namespace mbr;
    if (!d_params || !d_q || !d_tgt || !d_grad) MBR_FAIL(MBR_EINVAL, "null pointer");
    if (B <= 0 || B % 64 != 0) MBR_FAIL(MBR_EINVAL, "B=%d must be a positive multiple of 64", B);
    if (B > kStaticBatch)
        MBR_FAIL(MBR_ERANGE, "B=%d exceeds the %d samples of the static scratch", B, kStaticBatch);
    float *part = nullptr;
    MBR_TRY(static_scratch(0, &part, nullptr));
    // every scratch word the kernels read is written first in this call
    return batch_sum(d_params, B, d_q, d_tgt, d_grad, d_loss, part, as_stream(stream));
}

}  // extern "C"
