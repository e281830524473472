// gfx950 kernels of the embedding-training hot path (GraphVite, arXiv 1903.00757).
//
// Work decomposition: one 64-lane wavefront owns one positive sample at a time.
// A row of d floats is spread over the 64 lanes (d/64 floats per lane), so a row
// gather or scatter is one fully coalesced request per 64 x 16 B, the dot product
// is a per-lane partial followed by a cross-lane (DPP) reduction, and all node ids
// and coefficients of the sample are wave-uniform scalars.
//
// The file is compiled twice, side by side: plainly, and with GV_TRACK_LOSS=1 into a second object that holds
// nothing but the training kernels that also sum the running loss, under names ending in _tracked.
#include "gv_internal.hpp"

#include <algorithm>

#ifndef GV_TRACK_LOSS
#define GV_TRACK_LOSS 0
#endif
#if GV_TRACK_LOSS
#define GV_TRAIN_NAME(name) name##_tracked
#else
#define GV_TRAIN_NAME(name) name
#endif

namespace gv {
namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr bool is_atomic(int c) { return c == kAtomicAgent || c == kMixed; }
constexpr bool is_agent(int c) { return c == kAgent || c == kAtomicAgent || c == kMixed; }

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies
// and a word permutation; the key advances by the Weyl constants between rounds.
__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        c0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        c1 = (uint32_t)p1;
        c2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

// Negative k of positive sample g (Alg. 1, NegativeSampling; Sec. 4.3 alias
// table): bucket = floor(R * n / 2^64) from the first two words, accepted when
// the third word is below the bucket's threshold, else the bucket's alias.
// The table entry also carries the node of the bucket (the table may cover a partition of the nodes only) and
// the hot ranks of both candidates.
struct Drawn {
    uint32_t id;
    uint32_t rank;
};
__device__ __forceinline__ Drawn draw_ranked_negative(const uint4 *__restrict__ alias, uint32_t n, uint64_t seed,
                                                      uint64_t g, uint32_t k, uint32_t stream = 0u) {
    const uint4 r =
        philox4x32_10((uint32_t)g, (uint32_t)(g >> 32), k, stream, (uint32_t)seed, (uint32_t)(seed >> 32));
    const uint64_t R = ((uint64_t)r.x << 32) | r.y;
    const uint32_t j = (uint32_t)__umul64hi(R, (uint64_t)n);
    const uint4 e = alias[j];
    const bool keep = r.z < e.x;
    return Drawn{keep ? e.w : e.y, keep ? (e.z & 0xFFFFu) : (e.z >> 16)};
}
__device__ __forceinline__ uint32_t draw_negative(const uint4 *__restrict__ alias, uint32_t n, uint64_t seed,
                                                  uint64_t g, uint32_t k, uint32_t stream = 0u) {
    return draw_ranked_negative(alias, n, seed, g, k, stream).id;
}

// Learning rate of positive sample g (Sec. 4.3: linear decay from lr0), fp64 then fp32.
__device__ __forceinline__ float learning_rate(float lr0, float lr_min_ratio, uint64_t g, uint64_t total) {
    double f = 1.0 - (double)g / (double)total;
    if (f < (double)lr_min_ratio) f = (double)lr_min_ratio;
    return (float)((double)lr0 * f);
}

// ---------------------------------------------------------------------------
// Cross-lane sum of a wave64 with DPP moves: quad butterflies, half-row and row
// mirrors give every lane its 16-lane row sum; two row broadcasts carry the sums
// to the last row; the result is read from lane 63 as a wave-uniform scalar.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_take(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, kRowMask, 0xF, false));
}

__device__ __forceinline__ float wave_sum(float x) {
    x += dpp_take<0xB1, 0xF>(x);   // quad_perm [1,0,3,2]
    x += dpp_take<0x4E, 0xF>(x);   // quad_perm [2,3,0,1]
    x += dpp_take<0x141, 0xF>(x);  // row_half_mirror
    x += dpp_take<0x140, 0xF>(x);  // row_mirror
    x += dpp_take<0x142, 0xA>(x);  // row_bcast15 into rows 1 and 3
    x += dpp_take<0x143, 0xC>(x);  // row_bcast31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// Several of them, step by step together.
template <int kN>
__device__ __forceinline__ void wave_sums(float (&x)[kN]) {
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] += dpp_take<0xB1, 0xF>(x[n]);
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] += dpp_take<0x4E, 0xF>(x[n]);
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] += dpp_take<0x141, 0xF>(x[n]);
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] += dpp_take<0x140, 0xF>(x[n]);
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] += dpp_take<0x142, 0xA>(x[n]);
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] += dpp_take<0x143, 0xC>(x[n]);
#pragma unroll
    for (int n = 0; n < kN; ++n) x[n] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[n]), 63));
}

__device__ __forceinline__ uint32_t lane_value(uint32_t x, uint32_t lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)lane);
}

// ---------------------------------------------------------------------------
// Row <-> registers.  A lane holds kV floats of the row in segments: plain
// accesses use 16-byte segments when the row allows, device-scope accesses use
// 8-byte segments (the widest single-copy-atomic access).  Element e of segment
// s sits at row[s * 64 * W + lane * W + e], so each segment is one contiguous
// 64 * W * 4 byte request per wave.  kFull says that the row is exactly 64 * kV floats long:
// then no lane is ever past the end and the per-lane bounds tests (and the execution-mask
// bookkeeping they cost around every memory instruction) are compiled out.
template <int kV, int kCoherence, bool kFull = false>
struct RowIo {
    static constexpr int W = is_agent(kCoherence) ? (kV >= 2 ? 2 : 1) : (kV >= 4 ? 4 : kV);
    static constexpr int S = kV / W;

    // dim (a multiple of 32, at most 64 * kV) is the row length: lanes past the end hold zeros
    static __device__ __forceinline__ void load(const float *row, int lane, uint32_t dim, float (&x)[kV]) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (!kFull && (uint32_t)(s * (kWave * W) + lane * W) >= dim) {
#pragma unroll
                for (int e = 0; e < W; ++e) x[s * W + e] = 0.0f;
                continue;
            }
            const float *p = row + s * (kWave * W) + lane * W;
            if constexpr (is_agent(kCoherence)) {
                if constexpr (W == 2) {
                    const uint64_t bits =
                        __hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    x[s * W] = __uint_as_float((uint32_t)bits);
                    x[s * W + 1] = __uint_as_float((uint32_t)(bits >> 32));
                } else {
                    x[s] = __uint_as_float(
                        __hip_atomic_load((const uint32_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                }
            } else if constexpr (W == 4) {
                const f4 t = *(const f4 *)p;
                x[s * 4] = t.x; x[s * 4 + 1] = t.y; x[s * 4 + 2] = t.z; x[s * 4 + 3] = t.w;
            } else if constexpr (W == 2) {
                const f2 t = *(const f2 *)p;
                x[s * 2] = t.x; x[s * 2 + 1] = t.y;
            } else {
                x[s] = *p;
            }
        }
    }

    // row += delta without losing concurrent updates of other waves: one fp32 atomic add
    // per element.  With two floats per lane the values are first exchanged between lanes
    // (lane l takes elements l and l + 64 of the 128-float segment) so that every atomic
    // instruction covers 256 contiguous bytes instead of every other word of 512.
    static __device__ __forceinline__ void add(float *row, int lane, uint32_t dim, const float (&delta)[kV]) {
        static_assert(W <= 2, "atomic adds are used with the device-scope layouts only");
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if constexpr (W == 2) {
                const int lo = (lane >> 1) * 4, hi = (32 + (lane >> 1)) * 4;  // byte addresses of the source lanes
                const int e0 = __float_as_int(delta[s * 2]), e1 = __float_as_int(delta[s * 2 + 1]);
                const int lo0 = __builtin_amdgcn_ds_bpermute(lo, e0), lo1 = __builtin_amdgcn_ds_bpermute(lo, e1);
                const int hi0 = __builtin_amdgcn_ds_bpermute(hi, e0), hi1 = __builtin_amdgcn_ds_bpermute(hi, e1);
                const float first = __int_as_float((lane & 1) ? lo1 : lo0);
                const float second = __int_as_float((lane & 1) ? hi1 : hi0);
                float *p = row + s * (kWave * 2) + lane;
                if (kFull || (uint32_t)(s * (kWave * 2) + lane) < dim)
                    (void)__hip_atomic_fetch_add(p, first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (kFull || (uint32_t)(s * (kWave * 2) + kWave + lane) < dim)
                    (void)__hip_atomic_fetch_add(p + kWave, second, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                if (kFull || (uint32_t)(s * kWave + lane) < dim)
                    (void)__hip_atomic_fetch_add(row + s * kWave + lane, delta[s], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }

    // row += delta with returning atomic adds, x = the row right after this wave's addition
    // (whatever other waves added before it is included), delta = 0.  Same lane exchange as
    // add(), and the inverse exchange for the values that come back.
    static __device__ __forceinline__ void exchange(float *row, int lane, uint32_t dim, float (&delta)[kV],
                                                    float (&x)[kV]) {
        static_assert(W <= 2, "atomic adds are used with the device-scope layouts only");
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if constexpr (W == 2) {
                const int lo = (lane >> 1) * 4, hi = (32 + (lane >> 1)) * 4;
                const int e0 = __float_as_int(delta[s * 2]), e1 = __float_as_int(delta[s * 2 + 1]);
                const int lo0 = __builtin_amdgcn_ds_bpermute(lo, e0), lo1 = __builtin_amdgcn_ds_bpermute(lo, e1);
                const int hi0 = __builtin_amdgcn_ds_bpermute(hi, e0), hi1 = __builtin_amdgcn_ds_bpermute(hi, e1);
                float first = __int_as_float((lane & 1) ? lo1 : lo0);    // element lane of the segment
                float second = __int_as_float((lane & 1) ? hi1 : hi0);   // element 64 + lane
                float *p = row + s * (kWave * 2) + lane;
                if (kFull || (uint32_t)(s * (kWave * 2) + lane) < dim)
                    first += __hip_atomic_fetch_add(p, first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (kFull || (uint32_t)(s * (kWave * 2) + kWave + lane) < dim)
                    second += __hip_atomic_fetch_add(p + kWave, second, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // lane l wants elements 2l and 2l + 1: lanes 2l, 2l + 1 hold them in `first` when
                // l < 32, lanes 2l - 64, 2l - 63 in `second` otherwise
                const int even = ((2 * lane) & 63) * 4, odd = ((2 * lane + 1) & 63) * 4;
                const int f_even = __builtin_amdgcn_ds_bpermute(even, __float_as_int(first));
                const int f_odd = __builtin_amdgcn_ds_bpermute(odd, __float_as_int(first));
                const int s_even = __builtin_amdgcn_ds_bpermute(even, __float_as_int(second));
                const int s_odd = __builtin_amdgcn_ds_bpermute(odd, __float_as_int(second));
                x[s * 2] = __int_as_float(lane < 32 ? f_even : s_even);
                x[s * 2 + 1] = __int_as_float(lane < 32 ? f_odd : s_odd);
                delta[s * 2] = delta[s * 2 + 1] = 0.0f;
            } else {
                if (kFull || (uint32_t)(s * kWave + lane) < dim)
                    x[s] = delta[s] + __hip_atomic_fetch_add(row + s * kWave + lane, delta[s], __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                delta[s] = 0.0f;
            }
        }
    }

    static __device__ __forceinline__ void store(float *row, int lane, uint32_t dim, const float (&x)[kV]) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (!kFull && (uint32_t)(s * (kWave * W) + lane * W) >= dim) continue;
            float *p = row + s * (kWave * W) + lane * W;
            if constexpr (is_agent(kCoherence)) {
                if constexpr (W == 2) {
                    const uint64_t bits =
                        (uint64_t)__float_as_uint(x[s * W]) | ((uint64_t)__float_as_uint(x[s * W + 1]) << 32);
                    __hip_atomic_store((uint64_t *)p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    __hip_atomic_store((uint32_t *)p, __float_as_uint(x[s]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                }
            } else if constexpr (W == 4) {
                f4 t = {x[s * 4], x[s * 4 + 1], x[s * 4 + 2], x[s * 4 + 3]};
                *(f4 *)p = t;
            } else if constexpr (W == 2) {
                f2 t = {x[s * 2], x[s * 2 + 1]};
                *(f2 *)p = t;
            } else {
                *p = x[s];
            }
        }
    }
};

__device__ __forceinline__ float sigmoid(float z) { return 1.0f / (1.0f + __expf(-z)); }

// Running training loss (kernels instantiated with kTrack only): -log sigmoid(z) = log(1 + e^-z) for either
// sign of z; a positive's score s contributes minus_log_sigmoid(s), a negative's w * minus_log_sigmoid(-s).
// The scores of a chunk are laid into lanes as the wave walks it (one selection each) and the logarithms are
// taken once per chunk, lane l for sample l: taken sample by sample, the same number on all 64 lanes, they were a
// third of the walk (2048 samples of a wave at d = 96, K = 3: 5.0 ms with, 3.4 ms without the running loss).
// Lanes sum in fp32; a wave hands the sum of its lanes over every so often as one fp64 atomic add.
__device__ __forceinline__ float minus_log_sigmoid(float z) { return fmaxf(-z, 0.0f) + log1pf(__expf(-fabsf(z))); }
template <int kK>
struct ChunkScores {
    float of[kK + 1];  // lane l: the scores of sample l of the chunk
    __device__ __forceinline__ void put(int k, uint32_t i, float score) {
        of[k] = (threadIdx.x & (kWave - 1)) == i ? score : of[k];
    }
    __device__ __forceinline__ float loss(float w) const {
        float sum = minus_log_sigmoid(of[0]);
#pragma unroll
        for (int k = 1; k <= kK; ++k) sum += w * minus_log_sigmoid(-of[k]);
        return sum;
    }
};
__device__ __forceinline__ void hand_over_loss(double *slots, float &lane_loss, int lane) {
    const float total = wave_sum(lane_loss);
    if (lane == 0)
        (void)__hip_atomic_fetch_add(slots + (blockIdx.x % kLossSlots), (double)total, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    lane_loss = 0.0f;
}

// One positive sample with its K negatives (Alg. 1, the Train calls; Sec. 2.1
// scores; Sec. 4.3 negative weight): rows[0] is the positive context row v,
// rows[1..K] the negatives.  All 1+K scores come from the rows as loaded (x = vertex[u], c[k] =
// context[rows[k]]), then
//   vertex[u]      += sum_k coef_k * context[rows_k]
//   context[rows_k] += coef_k * vertex[u]
// with coef_0 = lr (1 - sigmoid(s_0)), coef_k = -lr w sigmoid(s_k).  A context
// row named more than once in the sample is written once with the summed
// coefficient.  u and rows[] are wave-uniform.  kTrack: the scores go to lane i of `scores`.

// The coefficients and the change of x; returns the score of the positive.
template <int kV, int kK, bool kTrack>
__device__ __forceinline__ float sgns_coefficients(const float (&x)[kV], const float (&c)[kK + 1][kV], float lr, float w,
                                                   ChunkScores<kK> &scores, uint32_t i, float (&coef)[kK + 1], float (&dx)[kV]) {
    float positive = 0.0f;
#pragma unroll
    for (int k = 0; k <= kK; ++k) {
        float partial = 0.0f;
#pragma unroll
        for (int j = 0; j < kV; ++j) partial = fmaf(x[j], c[k][j], partial);
        const float score = wave_sum(partial);
        if (k == 0) positive = score;
        coef[k] = k == 0 ? lr * (1.0f - sigmoid(score)) : -(lr * w) * sigmoid(score);
        if constexpr (kTrack) scores.put(k, i, score);
    }
#pragma unroll
    for (int j = 0; j < kV; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k <= kK; ++k) acc = fmaf(coef[k], c[k][j], acc);
        dx[j] = acc;
    }
    return positive;
}
// The first naming of a context row in a sample (the others are folded into it), and the coefficient of all of them.
template <int kK>
__device__ __forceinline__ bool first_naming(const uint32_t (&rows)[kK + 1], int k) {
    bool repeated = false;
#pragma unroll
    for (int k2 = 0; k2 < k; ++k2) repeated |= rows[k2] == rows[k];
    return !repeated;
}
template <int kK>
__device__ __forceinline__ float total_coefficient(const uint32_t (&rows)[kK + 1], const float (&coef)[kK + 1], int k) {
    // the sum of rounded coefficients in every kernel: joined to the product of a coefficient that happens to stand beside it,
    // the bits of deterministic training would depend on the kernel
#pragma clang fp contract(off)
    float total = coef[k];
#pragma unroll
    for (int k2 = k + 1; k2 <= kK; ++k2) total += rows[k2] == rows[k] ? coef[k2] : 0.0f;
    return total;
}

template <int kV, int kK, int kCoherence, bool kFull, bool kTrack>
__device__ __forceinline__ float sgns_step(float *__restrict__ vertex, float *__restrict__ context, uint32_t u,
                                          const uint32_t (&rows)[kK + 1], float lr, float w, int lane, uint32_t D,
                                          ChunkScores<kK> &scores, uint32_t i) {
    using Io = RowIo<kV, kCoherence, kFull>;
    float *xp = vertex + (size_t)u * D;
    float x[kV];
    float c[kK + 1][kV];
    Io::load(xp, lane, D, x);
#pragma unroll
    for (int k = 0; k <= kK; ++k) Io::load(context + (size_t)rows[k] * D, lane, D, c[k]);
    float coef[kK + 1], dx[kV];
    const float positive = sgns_coefficients<kV, kK, kTrack>(x, c, lr, w, scores, i, coef, dx);
#pragma unroll
    for (int k = 0; k <= kK; ++k) {
        if (!first_naming<kK>(rows, k)) continue;  // wave-uniform
        const float total = total_coefficient<kK>(rows, coef, k);
        if constexpr (is_atomic(kCoherence)) {
            float dc[kV];
#pragma unroll
            for (int j = 0; j < kV; ++j) dc[j] = total * x[j];
            Io::add(context + (size_t)rows[k] * D, lane, D, dc);
        } else {
#pragma unroll
            for (int j = 0; j < kV; ++j) c[k][j] = fmaf(total, x[j], c[k][j]);
            Io::store(context + (size_t)rows[k] * D, lane, D, c[k]);
        }
    }
    if constexpr (is_atomic(kCoherence)) {
        Io::add(xp, lane, D, dx);
    } else {
#pragma unroll
        for (int j = 0; j < kV; ++j) dx[j] += x[j];
        Io::store(xp, lane, D, dx);
    }
    return positive;
}

// ---------------------------------------------------------------------------
// Asynchronous (Hogwild) training of one pool.  A wave takes chunks of 64
// consecutive samples: lane l reads sample l of the chunk (one coalesced 512 B
// read), draws that sample's negatives and learning rate, and the wave then
// walks the 64 samples in order, fetching each one's ids from the owning lane.
template <int kV, int kK, int kCoherence, bool kFull, bool kTrack>
__global__ __launch_bounds__(kBlock) void k_train_hogwild(TrainArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane((blockIdx.x * kBlock + threadIdx.x) / kWave);
    const uint32_t waves = gridDim.x * (kBlock / kWave);
    const uint32_t chunks = (a.count + a.unit - 1) / a.unit;
    const uint2 *__restrict__ pairs = (const uint2 *)a.pairs;
    float lane_loss = 0.0f;
    uint32_t chunks_done = 0;
    bool diverged = false;

    for (uint32_t chunk = wave; chunk < chunks; chunk += waves) {
        const uint32_t base = chunk * a.unit;
        const uint32_t in_chunk = min(a.unit, a.count - base);
        const bool mine = (uint32_t)lane < in_chunk;
        const uint2 p = mine ? pairs[base + lane] : make_uint2(0u, 0u);
        const uint64_t g = a.first_g + (a.order && mine ? a.order[base + lane] : base + lane);
        uint32_t neg[kK];
#pragma unroll
        for (int k = 0; k < kK; ++k) neg[k] = draw_negative(a.alias, a.alias_n, a.seed, g, k);
        const float lr = learning_rate(a.lr0, a.lr_min_ratio, g, a.total);
        const bool named = mine && p.x < a.n && p.y < a.n;
        if (mine && !named) *a.error_flag = 1u;
        ChunkScores<kK> scores{};

        for (uint32_t i = 0; i < in_chunk; ++i) {
            const uint32_t u = lane_value(p.x, i);
            uint32_t rows[kK + 1];
            rows[0] = lane_value(p.y, i);
            if (u >= a.n || rows[0] >= a.n) continue;  // reported through error_flag
#pragma unroll
            for (int k = 0; k < kK; ++k) rows[k + 1] = lane_value(neg[k], i);
            const float lr_i = __uint_as_float(lane_value(__float_as_uint(lr), i));
            const float score = sgns_step<kV, kK, kCoherence, kFull, kTrack>(a.vertex, a.context, u, rows, lr_i, a.neg_weight,
                                                                             lane, a.dim, scores, i);
            diverged |= !(score == score);
        }
        if constexpr (kTrack) {
            if (named) lane_loss += scores.loss(a.neg_weight);
            if ((++chunks_done & 15u) == 0u) hand_over_loss(a.loss_slots, lane_loss, lane);
        }
    }
    if (a.report_divergence && diverged) a.error_flag[1] = 1u;
    if constexpr (kTrack) hand_over_loss(a.loss_slots, lane_loss, lane);
}

// Update of a row that is not held in registers: row += total * other.  Atomic adds keep
// every concurrent update; the plain variant writes back loaded + total * other and can
// lose an update that another wave makes between this wave's load and store.
template <int kV, int kCoherence, bool kFull>
__device__ __forceinline__ void remote_update(float *row, int lane, uint32_t D, bool warm, float total,
                                              const float (&other)[kV], const float (&loaded)[kV]) {
    using Io = RowIo<kV, kCoherence, kFull>;
    if (kCoherence == kAtomicAgent || (kCoherence == kMixed && warm)) {
        float d[kV];
#pragma unroll
        for (int j = 0; j < kV; ++j) d[j] = total * other[j];
        Io::add(row, lane, D, d);
    } else {
        float r[kV];
#pragma unroll
        for (int j = 0; j < kV; ++j) r[j] = fmaf(total, other[j], loaded[j]);
        Io::store(row, lane, D, r);
    }
}

// ---------------------------------------------------------------------------
// Tiled stationary-row training.  A workgroup takes a tile of kTile consecutive samples
// of the pool, tags every sample with the hottest of its rows (vertex[u], context[v] or the
// context row of a negative: the one of lowest hot rank, ties going to the earlier of the
// three) and sorts the tile by that row in LDS, so that samples sharing their hot row become
// adjacent.  Each of its four waves then walks a quarter of the sorted tile
// and keeps the hot row in registers for as long as consecutive samples name it: the row is
// read once per run, the run's updates are applied to the register copy in order, and the
// run's change is added to memory with fp32 atomic adds (nothing another wave adds meanwhile
// is lost): every four samples, taking in what memory holds by then, and at the end of the
// run.  The other rows of a sample are fetched and updated per sample with the given
// policy.  Accesses to one row are served one after the other by the memory system, so a
// row that a percent of all samples name -- as an endpoint or, drawn in proportion to
// degree^0.75, as a negative -- would otherwise set the pace of the whole launch.
// Tiles are taken in pool order (one workgroup per tile, started as earlier ones end, or a
// fixed number of workgroups striding over the tiles), so the launch still moves through
// the pool front to back and a row's samples stay spread over time.  Every sample keeps the
// negatives and the learning rate of its position in the pool.
template <int kTile>
__device__ __forceinline__ void sort_tile(uint32_t *word, uint32_t tile) {
    const uint32_t size = kTile > 0 ? (uint32_t)kTile : tile;
    for (uint32_t k = 2; k <= size; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t t = threadIdx.x; t < size / 2; t += kBlock) {
                const uint32_t lo = 2 * t - (t & (j - 1));  // partner pairs (lo, lo + j) of this bitonic step
                const uint32_t hi = lo + j;
                const bool ascending = (lo & k) == 0;
                const uint32_t wa = word[lo], wb = word[hi];
                if ((wa > wb) == ascending) {
                    word[lo] = wb;
                    word[hi] = wa;
                }
            }
            __syncthreads();
        }
    }
}

// bit of the pair of context rows j1 < j2 (rows 1 .. K + 1 of a sample) in a sample's `same` word
__host__ __device__ constexpr int pair_bit(int j1, int j2) { return (j1 - 1) * 6 + (j2 - 1); }

// kTile > 0: tiles of that size; 0: of a.unit samples, a power of two from kSmallestTile to kLargestTile, in LDS given
// with the launch.
template <int kV, int kK, int kCoherence, int kTile, bool kFull, bool kTrack>
__global__ __launch_bounds__(kBlock) void k_train_tiled(TrainArgs a) {
    const uint32_t D = a.dim;
    // One sort word per sample.  On top, 14 bits for its stationary row: the matrix, then either
    // the hot rank (the kGroupedRanks hottest rows: their samples must end up adjacent) or a
    // 12-bit hash of the row id (the others: they turn up less than once per tile, and the hash
    // puts their samples in an order unrelated to the pool's, where neighbours come from one
    // walk and often share a row).  Below, the number of that row within the sample (3 bits),
    // the sample's slot in the tile (13 bits) and the warm flags of u and v (2 bits).
    constexpr uint32_t kSkip = 0xFFFFFFFFu;  // word of a slot without a trainable sample (row number 7 is never used)
    constexpr uint32_t kSlotBits = 13, kGroupedRanks = 4096;
    constexpr uint32_t kRecord = kK + 3;  // words of a sample's record: u, v, K negatives, warm flags of the negatives
    static_assert(kLargestTile <= (1u << kSlotBits) && (kTile == 0 || kTile % kBlock == 0), "tile size");
    static_assert(kK + 1 < 7, "row numbers take three bits and 7 is reserved");
    const uint32_t size = kTile > 0 ? (uint32_t)kTile : a.unit;
    const uint32_t per_wave = size / (kBlock / kWave);
    // samples whose gathers are in flight together: bounded by the registers their rows take
    constexpr int kBatch = tiled_batch(kV, kK);
    const uint32_t exchange_every = a.exchange_every;  // see async_plan
    constexpr int kRows = kK + 2;  // rows of a sample: 0 = vertex[u], 1 = context[v], 2 + k = context[negative k]
    constexpr uint32_t kNoRow = 0xFFFFFFFFu;  // never a node id (ids are below n <= 2^31)
    // layout of a sample's flag word in the walk: 3 bits stationary row number, kRows warm bits, kRows
    // register-copy bits, 2 kBatch - 1 clash bits, and (K = 1 only) the one same-row bit
    constexpr uint32_t kWarmShift = 3, kTakesShift = kWarmShift + kRows, kClashShift = kTakesShift + kRows,
                       kSameShift = kClashShift + 2 * kBatch - 1;
    static_assert(kSameShift < 32, "flag word");
    using Io = RowIo<kV, kCoherence, kFull>;
    extern __shared__ uint32_t s_given[];
    __shared__ uint32_t s_fixed[kTile > 0 ? kTile : 1];
    uint32_t *const s_word = kTile > 0 ? s_fixed : s_given;  // `size` words
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave_in_group = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint2 *__restrict__ pairs = (const uint2 *)a.pairs;
    const uint32_t tiles = (a.count + size - 1) / size;
    float lane_loss = 0.0f;  // kTrack: of the samples this wave has trained since it last handed its sum over

    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t tile_base = tile * size;
        // Every tile orders the rows through its own mask, so the order in which a tile reaches
        // the hot rows differs from tile to tile.  With one common order all workgroups, started
        // together, would reach the same rows at the same moment, and a row would receive its
        // updates of thousands of tiles in one burst, all computed from the same stale value.
        const uint32_t scramble = (tile * 0x9E3779B1u) >> 18;  // 14 bits
        for (uint32_t t = threadIdx.x; t < size; t += kBlock) {
            uint32_t word = kSkip;
            if (tile_base + t < a.count) {
                const uint2 p = pairs[tile_base + t];
                if (p.x < a.n && p.y < a.n) {
                    // most nodes of a large graph have no hot rank: there a cache-resident bitmap says
                    // which do, and the rank table is read for those only
                    uint32_t ru, rv;
                    if (a.ranked) {
                        ru = (a.ranked[p.x >> 5] >> (p.x & 31u)) & 1u ? a.rank[p.x] : 0xFFFFu;
                        rv = (a.ranked[p.y >> 5] >> (p.y & 31u)) & 1u ? a.rank[p.y] : 0xFFFFu;
                    } else {
                        ru = a.rank[p.x];
                        rv = a.rank[p.y];
                    }
                    uint32_t best = ru, held = 0u, row = p.x;
                    if (rv < best) {
                        best = rv;
                        held = 1u;
                        row = p.y;
                    }
                    const uint64_t g = a.first_g + (a.order ? a.order[tile_base + t] : tile_base + t);
                    // the walk below takes the sample from this record instead of drawing it again
                    uint32_t *record = a.records + (size_t)(tile_base + t) * kRecord;
                    uint32_t warm_negatives = 0;
                    record[0] = p.x;
                    record[1] = p.y;
#pragma unroll
                    for (int k = 0; k < kK; ++k) {
                        const Drawn nk = draw_ranked_negative(a.alias, a.alias_n, a.seed, g, k);
                        record[2 + k] = nk.id;
                        warm_negatives |= (nk.rank < a.warm_ranks ? 1u : 0u) << k;
                        if (nk.rank < best) {
                            best = nk.rank;
                            held = 2u + k;
                            row = nk.id;
                        }
                    }
                    record[2 + kK] = warm_negatives;
                    const uint32_t group = (held == 0u ? 0u : 1u << 13) |
                                           (best < kGroupedRanks ? __brev(best) >> 20 : kGroupedRanks | (row * 0x9E3779B1u) >> 20);
                    const uint32_t warm_uv = (ru < a.warm_ranks ? 1u : 0u) | (rv < a.warm_ranks ? 2u : 0u);
                    word = (group ^ scramble) << 18 | held << 15 | t << 2 | warm_uv;
                } else {
                    *a.error_flag = 1u;  // the sample is skipped and reported at the next synchronisation
                }
            }
            s_word[t] = word;
        }
        __syncthreads();
        sort_tile<kTile>(s_word, size);

        float *held = nullptr;   // address of the row kept in y[]
        bool held_warm = true;   // its merge must not lose concurrent updates
        uint32_t since_exchange = 0;  // samples of the current run since memory last saw the held row
        // the held row as (matrix, id), for the lane-parallel clash tests of the next chunk; kNoRow: none
        uint32_t carried_id = kNoRow, carried_is_vertex = 0u;
        float y[kV], moved[kV];
#pragma unroll
        for (int j = 0; j < kV; ++j) y[j] = moved[j] = 0.0f;

        // Merge the held row back: add the run's total change atomically, or, for a row that
        // concurrent samples are unlikely to share (mixed policy) or under the plain
        // device-scope policy, store the register copy.
        auto flush = [&]() {
            if (!held) return;
            if (kCoherence == kAtomicAgent || (kCoherence == kMixed && held_warm))
                Io::add(held, lane, D, moved);
            else
                Io::store(held, lane, D, y);
        };

        for (uint32_t base = wave_in_group * per_wave; base < (wave_in_group + 1) * per_wave; base += kWave) {
            // ---- per chunk, lane l works out everything about sample l of the chunk, so that the walk
            // below only has to fetch ready-made scalars from the owning lane (the scalar unit of a
            // compute unit is shared by its four SIMDs and is what this kernel runs out of first).
            // a tile of fewer than 256 samples leaves a wave less than a chunk
            const bool in_quarter = kTile > 0 || (uint32_t)lane < per_wave - (base - wave_in_group * per_wave);
            const uint32_t word = in_quarter ? s_word[base + lane] : kSkip;
            const bool mine = word != kSkip;
            const uint32_t pos = tile_base + ((word >> 2) & ((1u << kSlotBits) - 1u));
            const uint32_t *record = a.records + (size_t)pos * kRecord;
            uint32_t id[kRows];  // u, v, negatives
            id[0] = mine ? record[0] : 0u;
            id[1] = mine ? record[1] : 0u;
#pragma unroll
            for (int k = 0; k < kK; ++k) id[2 + k] = mine ? record[2 + k] : 0u;
            // bit j: row j of the sample is warm (u and v from the sort word, the negatives from the record)
            const uint32_t warm = (word & 3u) | (mine ? record[2 + kK] << 2 : 0u);
            const float lr = learning_rate(a.lr0, a.lr_min_ratio, a.first_g + (a.order && mine ? a.order[pos] : pos), a.total);
            const uint32_t h = (word >> 15) & 7u;  // number of the stationary row
            uint32_t stationary_id = id[0];
#pragma unroll
            for (int j = 1; j < kRows; ++j)
                if (h == (uint32_t)j) stationary_id = id[j];
            const uint32_t is_vertex = h == 0u ? 1u : 0u;
            // bit j: row j is the stationary row, or the same context row again (a row can be named twice in
            // a sample: positive and negative, or two negatives): its value is the register copy
            uint32_t takes = 1u << h;
#pragma unroll
            for (int j = 1; j < kRows; ++j) takes |= (h != 0u && id[j] == stationary_id ? 1u : 0u) << j;
            // bit pair_bit(j1, j2): context rows j1 < j2 of the sample are the same row
            uint32_t same = 0u;
#pragma unroll
            for (int j1 = 1; j1 < kRows; ++j1)
#pragma unroll
                for (int j2 = j1 + 1; j2 < kRows; ++j2) same |= (id[j1] == id[j2] ? 1u : 0u) << pair_bit(j1, j2);
            // Clash bits.  The walk gathers up to kBatch samples at once.  A sample must not be gathered
            // while this wave still owes memory an update of one of its rows: a row that an earlier sample of
            // the batch names, or the row held when the batch starts -- unless that row is the held row simply
            // continuing from sample to sample.  It would read the row as it was before the wave's own
            // update, and under a store policy write the stale value back over it.
            //   bit d - 1           (d < kBatch):  a row of this sample is a row of the sample d places before
            //   bit kBatch - 1 + d - 1 (d <= kBatch): a row of this sample is the stationary row of that sample
            // The row held when the chunk starts stands in for "the sample before sample 0".
            uint32_t clash = 0u;
            if constexpr (kCoherence != kAtomicAgent) {
                // x of the lane d places down.  Every lane must take part in every exchange (a lane that is
                // switched off hands out nothing): the exchanges stand alone, selections follow them.
                auto from_before = [&](uint32_t x, int d) {
                    return (uint32_t)__builtin_amdgcn_ds_bpermute((lane - d) * 4, (int)x);
                };
                // run[d]: this sample and the d before it all have the same stationary row
                const uint32_t id_before = from_before(stationary_id, 1), is_vertex_before = from_before(is_vertex, 1);
                const uint32_t prev_id = lane >= 1 ? id_before : carried_id;
                const uint32_t prev_is_vertex = lane >= 1 ? is_vertex_before : carried_is_vertex;
                const uint32_t same_as_before = prev_id == stationary_id && prev_is_vertex == is_vertex ? 1u : 0u;
                uint32_t run[kBatch + 1];
                run[0] = 1u;
                run[1] = same_as_before;
#pragma unroll
                for (int d = 2; d <= kBatch; ++d) {
                    const uint32_t same_there = from_before(same_as_before, d - 1);
                    run[d] = run[d - 1] & (lane >= d - 1 ? same_there : 0u);
                }
#pragma unroll
                for (int d = 1; d <= kBatch; ++d) {
                    // the stationary row of the sample d before (the carried row for the sample "before sample 0")
                    const bool real = lane >= d;
                    const uint32_t stationary_there = from_before(stationary_id, d), is_vertex_there = from_before(is_vertex, d);
                    const uint32_t their_stationary = real ? stationary_there : (lane == d - 1 ? carried_id : kNoRow);
                    const uint32_t their_is_vertex = real ? is_vertex_there : carried_is_vertex;
                    bool names_their_stationary = false;
#pragma unroll
                    for (int j = 0; j < kRows; ++j)
                        names_their_stationary |= id[j] == their_stationary && (j == 0) == (their_is_vertex != 0u) &&
                                                  !(run[d] != 0u && h == (uint32_t)j);
                    clash |= (names_their_stationary && their_stationary != kNoRow ? 1u : 0u) << (kBatch - 1 + d - 1);
                    if (d < kBatch) {
                        uint32_t theirs[kRows];
#pragma unroll
                        for (int j = 0; j < kRows; ++j) theirs[j] = from_before(id[j], d);
                        const uint32_t their_h = from_before(h, d);
                        bool shares = id[0] == theirs[0] && !(run[d] != 0u && h == 0u && their_h == 0u);
#pragma unroll
                        for (int j1 = 1; j1 < kRows; ++j1)
#pragma unroll
                            for (int j2 = 1; j2 < kRows; ++j2)
                                shares |= id[j1] == theirs[j2] &&
                                          !(run[d] != 0u && h == (uint32_t)j1 && their_h == (uint32_t)j2);
                        clash |= (real && shares ? 1u : 0u) << (d - 1);
                    }
                }
            }
            // one word for the walk: stationary row number, warm bits, register-copy bits, clash bits
            const uint32_t flags = h | warm << kWarmShift | takes << kTakesShift | clash << kClashShift |
                                   (kK == 1 ? ((same >> pair_bit(1, 2)) & 1u) << kSameShift : 0u);
            // sorted order puts the skipped slots last: the first one ends this wave's work
            const uint64_t live = __ballot(mine);
            const uint32_t in_chunk = live == ~0ull ? (uint32_t)kWave : (uint32_t)__builtin_ctzll(~live);

            // ---- the walk: wave-uniform copies of one sample's scalars
            struct Sample {
                float *row[kRows];   // addresses of vertex[u], context[v], context[negative k]
                float *stationary;   // the one of them that is kept in registers
                uint32_t flags, same;
                float lr;
            };
            auto decode = [&](uint32_t i) {
                Sample s;
                s.flags = lane_value(flags, i);
                s.row[0] = a.vertex + (size_t)lane_value(id[0], i) * D;
#pragma unroll
                for (int j = 1; j < kRows; ++j) s.row[j] = a.context + (size_t)lane_value(id[j], i) * D;
                const size_t stationary_at = (size_t)lane_value(stationary_id, i) * D;
                s.stationary = (s.flags & 7u) == 0u ? a.vertex + stationary_at : a.context + stationary_at;
                s.same = kK > 1 ? lane_value(same, i) : ((s.flags >> kSameShift) & 1u) << pair_bit(1, 2);
                s.lr = __uint_as_float(lane_value(__float_as_uint(lr), i));
                return s;
            };
            // Issue the loads of a sample: every row whose value is not the register copy, and the
            // stationary row when that is not the row the wave will be holding at that point.
            auto fetch = [&](const Sample &s, const float *held_then, float (&loaded)[kRows][kV], float (&fresh)[kV]) {
#pragma unroll
                for (int j = 0; j < kRows; ++j)
                    if (!((s.flags >> (kTakesShift + j)) & 1u)) Io::load(s.row[j], lane, D, loaded[j]);
                if (s.stationary != held_then) Io::load(s.stationary, lane, D, fresh);
            };

            // One sample (same arithmetic as sgns_step): switch the held row if needed, then all
            // scores and coefficients from the rows as they are before the sample, then the updates:
            // into the register copy for the held row, to memory for the others.
            ChunkScores<kK> scores{};
            auto train_one = [&](const Sample &cur, uint32_t i, const float (&loaded)[kRows][kV], const float (&fresh)[kV]) {
                if (cur.stationary != held) {
                    flush();
#pragma unroll
                    for (int e = 0; e < kV; ++e) {
                        y[e] = fresh[e];
                        moved[e] = 0.0f;
                    }
                    held = cur.stationary;
                    held_warm = ((cur.flags >> kWarmShift >> (cur.flags & 7u)) & 1u) != 0;
                }
                const float lrw = cur.lr * a.neg_weight;
                // x = vertex[u], c[k] = context row 1 + k: the register copy where the flags say so
                float x[kV], c[kK + 1][kV];
                bool held_row[kRows];
#pragma unroll
                for (int j = 0; j < kRows; ++j) held_row[j] = ((cur.flags >> (kTakesShift + j)) & 1u) != 0;
#pragma unroll
                for (int e = 0; e < kV; ++e) x[e] = held_row[0] ? y[e] : loaded[0][e];
#pragma unroll
                for (int k = 0; k <= kK; ++k)
#pragma unroll
                    for (int e = 0; e < kV; ++e) c[k][e] = held_row[1 + k] ? y[e] : loaded[1 + k][e];
                float coef[kK + 1];
#pragma unroll
                for (int k = 0; k <= kK; ++k) {
                    float partial = 0.0f;
#pragma unroll
                    for (int e = 0; e < kV; ++e) partial = fmaf(x[e], c[k][e], partial);
                    const float score = wave_sum(partial);
                    coef[k] = k == 0 ? cur.lr * (1.0f - sigmoid(score)) : -lrw * sigmoid(score);
                    if constexpr (kTrack) scores.put(k, i, score);
                }
                // context rows first (they take the vertex row as it was), each distinct row once
#pragma unroll
                for (int k = 0; k <= kK; ++k) {
                    bool repeated = false;
#pragma unroll
                    for (int k2 = 0; k2 < k; ++k2) repeated |= ((cur.same >> pair_bit(1 + k2, 1 + k)) & 1u) != 0;
                    if (repeated) continue;
                    float total = coef[k];
#pragma unroll
                    for (int k2 = k + 1; k2 <= kK; ++k2)
                        total += (cur.same >> pair_bit(1 + k, 1 + k2)) & 1u ? coef[k2] : 0.0f;
                    if (held_row[1 + k]) {
#pragma unroll
                        for (int e = 0; e < kV; ++e) {
                            const float d = total * x[e];
                            y[e] += d;
                            moved[e] += d;
                        }
                    } else {
                        remote_update<kV, kCoherence, kFull>(cur.row[1 + k], lane, D,
                                                             (cur.flags >> (kWarmShift + 1 + k)) & 1u, total, x, c[k]);
                    }
                }
                float dx[kV];
#pragma unroll
                for (int e = 0; e < kV; ++e) {
                    float acc = 0.0f;
#pragma unroll
                    for (int k = 0; k <= kK; ++k) acc = fmaf(coef[k], c[k][e], acc);
                    dx[e] = acc;
                }
                if (held_row[0]) {
#pragma unroll
                    for (int e = 0; e < kV; ++e) {
                        y[e] += dx[e];
                        moved[e] += dx[e];
                    }
                } else {
                    remote_update<kV, kCoherence, kFull>(cur.row[0], lane, D, (cur.flags >> kWarmShift) & 1u, 1.0f, dx, x);
                }
            };

            // Samples go through in batches of up to kBatch: all gathers of a batch are issued first,
            // then the samples are computed one after the other (a later sample of the batch sees
            // the held row as the earlier ones left it), so one memory round trip serves kBatch
            // samples instead of one.  A sample whose clash bits name a sample of the batch, or the row
            // held when the batch starts, is left for the next batch (and that held row is merged first).
            for (uint32_t i0 = 0; i0 < in_chunk;) {
                Sample batch[kBatch];
                float loaded[kBatch][kRows][kV], fresh[kBatch][kV];
                batch[0] = decode(i0);
                // A run that goes on trades with memory before its staleness would pass exchange_every
                // samples: its change so far is added and the register copy takes in what other waves
                // added meanwhile, so a held row is never more than that many samples behind the other
                // holders of that row.
                if (held && held == batch[0].stationary && since_exchange > 0u &&
                    since_exchange + kBatch > exchange_every &&
                    (kCoherence == kAtomicAgent || (kCoherence == kMixed && held_warm))) {
                    Io::exchange(held, lane, D, moved, y);
                    since_exchange = 0;
                }
                if constexpr (kCoherence != kAtomicAgent) {
                    if (held && ((batch[0].flags >> (kClashShift + kBatch - 1)) & 1u)) {
                        flush();
                        held = nullptr;
                    }
                }
                const float *then = held;
                uint32_t taken = 0;
#pragma unroll
                for (int b = 0; b < kBatch; ++b) {
#pragma unroll
                    for (int e = 0; e < kV; ++e) fresh[b][e] = 0.0f;
                    if (taken == (uint32_t)b && i0 + b < in_chunk) {
                        if (b > 0) {
                            batch[b] = decode(i0 + b);
                            // earlier samples of the batch (b places at most), and the row held at its start
                            const uint32_t kEarlier = ((1u << b) - 1u) | 1u << (kBatch - 1 + b);
                            if (kCoherence != kAtomicAgent && ((batch[b].flags >> kClashShift) & kEarlier)) continue;
                        }
                        fetch(batch[b], then, loaded[b], fresh[b]);
                        then = batch[b].stationary;
                        taken = b + 1;
                    }
                }
                // All gathers of the batch are awaited here, once, whichever of them were issued: the
                // counter of outstanding vector memory operations also counts stores and atomic adds, so a
                // wait placed between the samples would sit out the previous sample's updates as well.
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), the other counters untouched
#pragma unroll
                for (int b = 0; b < kBatch; ++b)
                    if ((uint32_t)b < taken) {
                        since_exchange = batch[b].stationary == held ? since_exchange + 1u : 1u;
                        train_one(batch[b], i0 + b, loaded[b], fresh[b]);
                    }
                i0 += taken;
            }
            if constexpr (kTrack)
                if ((uint32_t)lane < in_chunk) lane_loss += scores.loss(a.neg_weight);
            // what the next chunk's clash tests compare with: the row held now
            if (in_chunk > 0u) {
                carried_id = lane_value(stationary_id, in_chunk - 1u);
                carried_is_vertex = lane_value(is_vertex, in_chunk - 1u);
            }
            if (in_chunk < (uint32_t)kWave) break;
        }
        // a row that is no number any more: training has diverged (reported by the next synchronising call)
        if (held && !(y[0] == y[0])) a.error_flag[1] = 1u;
        flush();
        if constexpr (kTrack) hand_over_loss(a.loss_slots, lane_loss, lane);
        __syncthreads();  // the next tile overwrites the LDS arrays
    }
}

// Deterministic mode.  The samples of a pool are sorted into levels (gv_api.cpp): those of one level share no vertex
// row and no context row (Def. 1, Sec. 3.2: such samples commute), and samples that share a row keep their order from
// level to level, so the result equals the sequential order up to fp32 rounding inside a sample.  A record holds
// what a wave needs of its sample: u, v, the K negatives, and its place in the pool.
template <int kK>
struct LevelSample {
    uint32_t u, rows[kK + 1], place;
};
template <int kK>
__device__ __forceinline__ LevelSample<kK> level_sample(const uint32_t *__restrict__ records, uint32_t i) {
    const uint32_t *record = records + (size_t)i * (kK + 3);
    LevelSample<kK> s;
    s.u = record[0];
#pragma unroll
    for (int k = 0; k <= kK; ++k) s.rows[k] = record[1 + k];
    s.place = record[kK + 2];
    return s;
}

// A level too wide for one workgroup: wave i trains sample i.
template <int kV, int kK, bool kFull, bool kTrack>
__global__ __launch_bounds__(kBlock) void k_train_level(TrainArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t i = __builtin_amdgcn_readfirstlane((blockIdx.x * kBlock + threadIdx.x) / kWave);
    if (i >= a.count) return;
    const LevelSample<kK> s = level_sample<kK>(a.records, i);
    const float lr = learning_rate(a.lr0, a.lr_min_ratio, a.first_g + s.place, a.total);
    ChunkScores<kK> scores{};
    (void)sgns_step<kV, kK, kPlain, kFull, kTrack>(a.vertex, a.context, s.u, s.rows, lr, a.neg_weight, lane, a.dim, scores, 0u);
    if constexpr (kTrack) {
        float lane_loss = lane == 0 ? scores.loss(a.neg_weight) : 0.0f;
        hand_over_loss(a.loss_slots, lane_loss, lane);
    }
}

// Consecutive narrow levels in one launch: one workgroup of 16 waves walks level after level, a barrier between them (its
// waves share their L1 cache, so rows stored before the barrier are read after it).  A level costs the latency of
// gathering, storing and the barrier, at d = 128, K = 1 0.8 us with one sample, 1.0 with four and 1.5 with sixteen (the host's
// levelling of these among it), where a launch of its own takes 3 us; the record of a wave's first sample of the next level is
// on its way meanwhile.
constexpr int kLevelBlock = 1024;
template <int kV, int kK, bool kFull, bool kTrack>
__global__ __launch_bounds__(kLevelBlock) void k_train_levels(TrainArgs a) {
    constexpr uint32_t kWaves = kLevelBlock / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    float lane_loss = 0.0f;
    uint32_t end = a.level_starts[0], i = end + wave;
    const uint32_t last = a.level_starts[a.levels] - 1u;  // a record to read where a wave has no sample left
    LevelSample<kK> s = level_sample<kK>(a.records, min(i, last));
    for (uint32_t level = 0; level < a.levels; ++level) {
        const uint32_t start = end;
        end = a.level_starts[level + 1];
        for (i = start + wave; i < end; i += kWaves) {
            const float lr = learning_rate(a.lr0, a.lr_min_ratio, a.first_g + s.place, a.total);
            const LevelSample<kK> now = s;
            s = level_sample<kK>(a.records, min(i + kWaves < end ? i + kWaves : end + wave, last));
            ChunkScores<kK> scores{};
            (void)sgns_step<kV, kK, kPlain, kFull, kTrack>(a.vertex, a.context, now.u, now.rows, lr, a.neg_weight, lane,
                                                           a.dim, scores, 0u);
            if constexpr (kTrack) lane_loss += lane == 0 ? scores.loss(a.neg_weight) : 0.0f;
        }
        if (start + wave >= end) s = level_sample<kK>(a.records, min(end + wave, last));  // nothing here: the next level's
        __syncthreads();
    }
    if constexpr (kTrack) hand_over_loss(a.loss_slots, lane_loss, lane);
}

// Rows in the order of lanes of the cached accesses (16-byte segments where the row allows), at device scope, in the
// 8-byte words that such accesses come in: a sample is computed as in the level kernels.  `row` is the same in all lanes
// (a scalar address), `at` the lane's byte offset in it.
template <int kV, bool kFull>
struct HandedRow {
    static constexpr int W = kV >= 4 ? 4 : kV, S = kV / W;
    static __device__ __forceinline__ uint32_t lane_offset(int lane) { return (uint32_t)lane * (W * 4); }
    static __device__ __forceinline__ void load(const char *row, uint32_t at, uint32_t bytes, float (&x)[kV]) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t here = at + (uint32_t)s * (kWave * W * 4);
            const bool inside = kFull || here < bytes;
            if constexpr (W == 1) {
                x[s] = inside ? __uint_as_float(__hip_atomic_load((const uint32_t *)(row + here), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0.0f;
            } else {
#pragma unroll
                for (int e = 0; e < W; e += 2) {
                    const uint64_t bits =
                        inside ? __hip_atomic_load((const uint64_t *)(row + here + 4 * e), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
                    x[s * W + e] = __uint_as_float((uint32_t)bits);
                    x[s * W + e + 1] = __uint_as_float((uint32_t)(bits >> 32));
                }
            }
        }
    }
    static __device__ __forceinline__ void store(char *row, uint32_t at, uint32_t bytes, const float (&x)[kV]) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t here = at + (uint32_t)s * (kWave * W * 4);
            if (!kFull && here >= bytes) continue;
            if constexpr (W == 1) {
                __hip_atomic_store((uint32_t *)(row + here), __float_as_uint(x[s]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
#pragma unroll
                for (int e = 0; e < W; e += 2)
                    __hip_atomic_store((uint64_t *)(row + here + 4 * e),
                                       (uint64_t)__float_as_uint(x[s * W + e]) | ((uint64_t)__float_as_uint(x[s * W + e + 1]) << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
};

// A pool in one launch, every sample as soon as the earlier samples that name one of its rows are done.  a.places holds,
// for every row that a sample names, the place of that naming among all of them, sorted by row and then by sample; a row's
// turn is the place of the naming that comes next.  A wave takes the next a.unit samples of the pool, lane l looks after
// sample l: it polls the turns of its rows, and the samples whose turns have all come are trained (those of different
// lanes share no row), their rows stored, the stores waited for, and the turns of their rows passed on.
//
// What bounds it is the chain of samples that share the hottest rows, each link the latency of one wave.  A row goes from
// one wave to another in 1.0 us (store, wait, turn, poll, load; the same within a die and across dies), with the
// arithmetic 1.5 us a sample (K = 5: 2.3; a chain of 8000, one in eight samples of its pool), about 1.9 with a whole pool polling.  So
// each of the kFlowHubs rows named most has a wave of its own, which trains the samples that name it one after the other with the row
// in registers: a link of such a chain takes 0.52 us at d = 128, K = 1 where nothing else is waited for, 0.87 at K = 5 (flow_hub).
// 2*10^5 samples on 10^4 nodes, d = 128, K = 1: 4.1 ms as launches of levels, 2.0 without chains, 1.59 now (three contexts in turn: 3.4,
// 0.87, 0.63 ms a pool), this kernel 1.44 of it.  Its longest path, counted with links of 0.52 us in a chain and 1.5 to 1.9 from wave
// to wave, is 1.2 to 1.47 ms: some 750 links through rows that have no wave of their own, 80 in a chain, 3 that hand a hub's row on.
// 1.5*10^5 pairs drawn by degree on 10^5 nodes, exponent 2.5: 1.43 ms; 5*10^4 on 10^4 nodes, the hottest row in 4 % of them, 1.95, and
// 5.03 at d = 256, K = 5 (2.57 and 6.48 with the slower chains that are named at flow_hub).
// 1024 waves of 8 samples: 16 or more samples a wave wait for each other in the wave, and twice as many waves only poll more (3.4 ms
// with 1024 waves of 64, 6.2 with 2048, before samples far from their turn were left alone).
//
// Every wait ends: the waves of the hubs are those of one workgroup, the first that runs, together with one that takes
// samples as all others do; samples are taken in pool order, so the first sample of the pool that is not done is at
// the head of a hub's chain, or has been taken by a wave that runs, or is taken by the next one that has finished
// its own, and its turns have come.  Should they fail to (memory overwritten by the caller), a wave gives up and says so
// (FlowPatience).
constexpr uint32_t kFlowStep = 2000;  // cycles, about half of what a row takes from wave to wave
constexpr int kFlowBlock = 512, kFlowHubs = kFlowBlock / kWave - 1;
__device__ __forceinline__ uint32_t flow_progress(const FlowState *state) {
    return __hip_atomic_load(&state->next_chunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
           __hip_atomic_load(&state->chained, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int flow_batch(int V, int K) { return V * (K + 2) <= 14 ? 2 : 1; }
// The rows of two samples of a chain fit the 256 registers of a wave, with 226 used at most, 242 where the loss is tracked (with
// those of longer ones kept in memory, 20000 samples at d = 512, K = 5 take 19 ms, without chains 5.5); without chains there are no
// hubs.  Beyond 128 registers a compute unit has room for one workgroup only, and pools of three contexts wait for each other: 2*10^4
// samples on 2000 nodes, d = 64, K = 3, three contexts in turn 470 us a pool with 153 registers, 400 with 112; 5*10^4 on 10^4 nodes, the
// hottest row in 4 % of them, d = 256, K = 1 922 with 133, 751 with 109 (on 2*10^5 nodes without hubs 174 and 187).
constexpr bool flow_has_hubs(int V, int K) { return V * (K + 2) < 40; }

// One sample in registers: the rows after their updates stand where they were.  A chain is as fast as one wave goes through
// its instructions, so the sigmoids of the K + 1 scores are taken together, score k in lane k.
template <int kV, int kK, bool kTrack>
__device__ __forceinline__ void sgns_in_place(float (&x)[kV], float (&c)[kK + 1][kV], const uint32_t (&rows)[kK + 1], float lr, float w,
                                              int lane, ChunkScores<kK> &scores, uint32_t i) {
    float score = 0.0f;
#pragma unroll
    for (int k = 0; k <= kK; ++k) {
        float partial = 0.0f;
#pragma unroll
        for (int j = 0; j < kV; ++j) partial = fmaf(x[j], c[k][j], partial);
        const float score_k = wave_sum(partial);
        score = lane == k ? score_k : score;
        if constexpr (kTrack) scores.put(k, i, score_k);
    }
    const float s = sigmoid(score), each = lane == 0 ? lr * (1.0f - s) : -(lr * w) * s;
    float coef[kK + 1];
#pragma unroll
    for (int k = 0; k <= kK; ++k) coef[k] = __uint_as_float(lane_value(__float_as_uint(each), k));
    float dx[kV];
#pragma unroll
    for (int j = 0; j < kV; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k <= kK; ++k) acc = fmaf(coef[k], c[k][j], acc);
        dx[j] = acc;
    }
#pragma unroll
    for (int k = 0; k <= kK; ++k) {
        if (!first_naming<kK>(rows, k)) continue;
        const float total = total_coefficient<kK>(rows, coef, k);
#pragma unroll
        for (int j = 0; j < kV; ++j) c[k][j] = fmaf(total, x[j], c[k][j]);
    }
#pragma unroll
    for (int j = 0; j < kV; ++j) x[j] += dx[j];
}

// Every load has come and every store is in memory (vmcnt(0), the other counters untouched).
__device__ __forceinline__ void memory_is_done() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
}

// The same (bit for bit) of a sample whose rows are all different, the sums of its scores side by side.
template <int kV, int kK, bool kTrack>
__device__ __forceinline__ void sgns_plain(float (&x)[kV], float (&c)[kK + 1][kV], float lr, float w, int lane,
                                           ChunkScores<kK> &scores, uint32_t i) {
    float part[kK + 1];
#pragma unroll
    for (int k = 0; k <= kK; ++k) {
        part[k] = 0.0f;
#pragma unroll
        for (int j = 0; j < kV; ++j) part[k] = fmaf(x[j], c[k][j], part[k]);
    }
    wave_sums<kK + 1>(part);
    float score = 0.0f;
#pragma unroll
    for (int k = 0; k <= kK; ++k) {
        score = lane == k ? part[k] : score;
        if constexpr (kTrack) scores.put(k, i, part[k]);
    }
    const float s = sigmoid(score), each = lane == 0 ? lr * (1.0f - s) : -(lr * w) * s;
    float coef[kK + 1];
#pragma unroll
    for (int k = 0; k <= kK; ++k) coef[k] = __uint_as_float(lane_value(__float_as_uint(each), k));
#pragma unroll
    for (int j = 0; j < kV; ++j) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k <= kK; ++k) {
            acc = fmaf(coef[k], c[k][j], acc);
            c[k][j] = fmaf(k < kK ? coef[k] + 0.0f : coef[k], x[j], c[k][j]);  // (total_coefficient adds nothing to it)
        }
        x[j] += acc;
    }
}

// What lane l knows of the sample that it looks after.
template <int kK>
struct FlowSample {
    static constexpr int kRows = kK + 2;
    uint32_t key[kRows];        // its rows (context row v is n + v)
    uint32_t waits_for[kRows];  // the place of its naming (the first, where it names a row twice)
    uint32_t hands_on[kRows];   // the place behind it (so the last one's stays)
    uint32_t level = 0;         // the highest level of the samples before it at its rows

    __device__ __forceinline__ void take(const FlowArgs &a, uint32_t sample, bool mine) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            key[j] = mine ? a.keys[(size_t)sample * kRows + j] : 0u;
            waits_for[j] = mine ? a.places[(size_t)sample * kRows + j] : 0u;
            hands_on[j] = waits_for[j] + 1u;
        }
#pragma unroll
        for (int j = 1; j < kRows; ++j)
#pragma unroll
            for (int j2 = j - 1; j2 >= 0; --j2) waits_for[j] = key[j2] == key[j] ? waits_for[j2] : waits_for[j];
    }
    // The turns of the first kN rows.
    template <int kN>
    __device__ __forceinline__ void read(uint64_t *turns, bool looks, uint64_t (&is)[kN]) const {
        if (looks) {
#pragma unroll
            for (int j = 0; j < kN; ++j) is[j] = __hip_atomic_load(turns + key[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // How many samples come first at the row where most do (0: its turns have come).
    template <int kN>
    __device__ __forceinline__ uint32_t seen(const uint64_t (&is)[kN]) {
        uint32_t away = 0, highest = 0;
#pragma unroll
        for (int j = 0; j < kN; ++j) {
            away = max(away, waits_for[j] - (uint32_t)is[j]);
            highest = max(highest, (uint32_t)(is[j] >> 32));
        }
        level = highest;
        return away;
    }
    __device__ __forceinline__ void hand_on(uint64_t *turns) const {
#pragma unroll
        for (int j = 0; j < kRows; ++j)
            __hip_atomic_store(turns + key[j], (uint64_t)(level + 1u) << 32 | hands_on[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// The same value, from which nothing is worked out ahead of a loop to be kept in registers over it.
template <class T>
__device__ __forceinline__ T *afresh(T *x) {
    asm volatile("" : "+s"(x));
    return x;
}
__device__ __forceinline__ uint32_t afresh(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// The rows that have a wave of their own: lane h < kFlowHubs holds the hub h, most namings first.
struct FlowHubs {
    uint32_t key, begin, namings;  // namings 0: none
    __device__ __forceinline__ void find(const FlowArgs &a, int lane) {
        unsigned long long slot = a.flow->slots[lane], mine = 0ull;
        for (int h = 0; h < kFlowHubs; ++h) {
            unsigned long long most = slot;
            for (int d = kWave / 2; d > 0; d /= 2) {
                const unsigned long long other = __shfl_xor(most, d);
                most = other > most ? other : most;
            }
            if (lane == h) mine = most;
            if (slot == most) slot = 0ull;  // slots are different or empty: they hold where a row's namings begin
        }
        namings = (uint32_t)(mine >> 32);
        begin = (uint32_t)mine;
        key = namings > 0u ? a.sorted[begin] : 0u;
    }
    // The first hub among the rows of a sample (kFlowHubs: none).  Every lane must take part: the values of other lanes are
    // read, and a register that had to be kept in memory comes back for the lanes that take part only.
    template <int kRows>
    __device__ __forceinline__ uint32_t owner(const uint32_t (&rows)[kRows]) const {
        uint32_t first = kFlowHubs;
        for (int h = kFlowHubs - 1; h >= 0; --h) {
            if (lane_value(namings, h) == 0u) continue;
            const uint32_t hub = lane_value(key, h);
            bool named = false;
#pragma unroll
            for (int j = 0; j < kRows; ++j) named |= rows[j] == hub;
            first = named ? (uint32_t)h : first;
        }
        return first;
    }
};

// Scalar addresses of the rows by key.
struct FlowRows {
    char *vertex, *context;  // of keys 0
    uint32_t bytes;
    __device__ __forceinline__ explicit FlowRows(const FlowArgs &a)
        : vertex((char *)a.vertex), context((char *)a.context - (uint64_t)a.n * a.dim * sizeof(float)), bytes(a.dim * (uint32_t)sizeof(float)) {}
    __device__ __forceinline__ char *of(int j, uint32_t key) const { return (j == 0 ? vertex : context) + (uint64_t)key * bytes; }
};

// The chain of hub h: its samples, except those that name a hub before it (the row is handed to the wave of that hub and
// awaited back).  The row stays in registers y; the other rows of the next sample are on their way while one is computed,
// and its stores are waited for after the next one's arithmetic.  What a link takes are the loads of the next sample's other rows
// and the instructions of one wave beside them (one every five cycles or so, a branch more), so the samples that name the hub once
// and their other rows once have a loop without branches on the rows, with the addresses of the rows worked out by the lanes, 64
// samples at once.  A link, in pools of 4*10^4 samples that all name one row and no other twice: d = 128, K = 1 0.90 us with one loop
// for every kind of sample, 0.52 now; d = 96, K = 3 1.14 and 0.71; d = 128, K = 5 1.44 and 0.87; d = 256, K = 5 1.80 and 1.08.  The other
// samples wait for their rows: 0.1 to 0.4 % of those that name a hub at K = 1, 1 to 2 % at K = 5, in pools that take this way.
// false: gave up.
template <int kV, int kK, bool kFull, bool kTrack>
__device__ __forceinline__ bool flow_hub(const FlowArgs &a, const FlowHubs &hubs, uint32_t h, int lane, uint32_t &deepest,
                                         float &lane_loss) {
    constexpr int kRows = kK + 2, kOthers = kK + 1;
    constexpr uint32_t kNone = 0xFFFFFFFFu, kAhead = 16;  // samples ahead whose turns are looked at
    using Io = HandedRow<kV, kFull>;
    const FlowRows matrix(a);
    const uint32_t at = Io::lane_offset(lane);
    const uint32_t hub = lane_value(hubs.key, h), begin = lane_value(hubs.begin, h), end = begin + lane_value(hubs.namings, h);
    char *const row = matrix.of(hub < a.n ? 0 : 1, hub);
    float y[kV];
#pragma unroll
    for (int e = 0; e < kV; ++e) y[e] = 0.0f;
    bool held = false;
    uint32_t level = 0, sample_before = kNone;  // of the row in registers; the sample of the naming before
    for (uint32_t base = begin; base < end; base += kWave) {
        const bool inside = (uint32_t)lane < end - base;
        const uint32_t sample = inside ? a.namings[base + lane] / (uint32_t)kRows : kNone;
        FlowSample<kK> s;
        s.take(a, sample, inside);
        const uint32_t lane_before = (uint32_t)__builtin_amdgcn_ds_bpermute((lane - 1) * 4, (int)sample);
        const bool again = sample == (lane > 0 ? lane_before : sample_before);  // the second naming of the row by a sample
        sample_before = lane_value(sample, kWave - 1);
        uint32_t takes = 0u;  // bit j: row j is the hub
#pragma unroll
        for (int j = 0; j < kRows; ++j) takes |= (s.key[j] == hub ? 1u : 0u) << j;
        const uint32_t owner = hubs.owner<kRows>(s.key);
        const uint64_t own = __ballot(inside && owner == h);
        uint64_t todo = __ballot(inside && !again), come = 0;  // samples to do; those of which all other turns have come
        const float lr = learning_rate(a.lr0, a.lr_min_ratio, a.first_g + (inside ? sample : 0u), a.total);
        // Most samples name the hub once and kOthers other rows, all different: what the wave needs of those, one after the other.
        bool differ = (takes & (takes - 1u)) == 0u;
#pragma unroll
        for (int j1 = 1; j1 < kRows; ++j1)
#pragma unroll
            for (int j2 = j1 + 1; j2 < kRows; ++j2) differ &= s.key[j1] != s.key[j2];
        const uint64_t plain = own & __ballot(differ);
        // From here on a sample's rows are those beside its first naming of the hub, in their order, and the first of them stands
        // where it names the hub again, whose turn is neither waited for nor handed on.  (In place, the addresses of turns worked
        // out where they are used: with copies in the chain's order kept beside them, 16 to 100 registers more, see flow_has_hubs.)
        const uint32_t first_other = takes & 1u ? s.key[1] : s.key[0], first_waits_for = takes & 1u ? s.waits_for[1] : s.waits_for[0];
        uint64_t other_at[kOthers];
#pragma unroll
        for (int m = 0; m < kOthers; ++m) {
            const bool behind = (takes & ((2u << m) - 1u)) != 0u;  // the hub comes first: the row was number m + 1
            const bool again_hub = behind && ((takes >> (m + 1)) & 1u);
            s.key[m] = again_hub ? first_other : behind ? s.key[m + 1] : s.key[m];
            s.waits_for[m] = again_hub ? first_waits_for : behind ? s.waits_for[m + 1] : s.waits_for[m];
            other_at[m] = (uint64_t)matrix.of(m == 0 && !behind ? 0 : 1, s.key[m]);
        }
        ChunkScores<kK> scores{};
        uint32_t unhanded = kNone;  // the sample whose turns are to be passed on once its rows are in memory
        auto hand_on = [&]() {
            if ((uint32_t)lane != unhanded) return;
            uint64_t *const turns = afresh(a.turns);
            if ((plain >> lane) & 1u) {
#pragma unroll
                for (int m = 0; m < kOthers; ++m)
                    __hip_atomic_store(turns + s.key[m], (uint64_t)(s.level + 1u) << 32 | (s.waits_for[m] + 1u), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            } else {
                const uint32_t takes_it = afresh(takes);
                uint32_t key[kOthers];
                bool hubs_own[kOthers];
#pragma unroll
                for (int m = 0; m < kOthers; ++m) {
                    key[m] = afresh(s.key[m]);
                    hubs_own[m] = (takes_it & ((2u << m) - 1u)) != 0u && ((takes_it >> (m + 1)) & 1u);
                    uint32_t next = s.waits_for[m] + 1u;  // the namings of a row by one sample have places one behind the other
#pragma unroll
                    for (int m2 = 0; m2 < m; ++m2) next += key[m2] == key[m] && !hubs_own[m2] ? 1u : 0u;
                    if (!hubs_own[m])
                        __hip_atomic_store(turns + key[m], (uint64_t)(s.level + 1u) << 32 | next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        };
        uint64_t is[kOthers];
        auto looked = [&](bool looks) {
            bool came = false;
            if (looks) came = s.seen(is) == 0u;
            come |= __ballot(came);
        };
        auto waits = [&](uint32_t first) {
            return (uint32_t)lane >= first && (uint32_t)lane <= first + kAhead && inside && !((come >> lane) & 1u);
        };
        while (todo) {
            uint32_t i = (uint32_t)__builtin_ctzll(todo);
            memory_is_done();
            hand_on();
            unhanded = kNone;
            if (!((own >> i) & 1u)) {  // another hub's: the row has to be in memory when its turn comes
                if (held) {
                    Io::store(row, at, matrix.bytes, y);
                    memory_is_done();
                    if (lane == 0)
                        __hip_atomic_store(a.turns + hub, (uint64_t)level << 32 | (base + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    held = false;
                }
                todo &= todo - 1;
                continue;
            }
            if (!held || !((come >> i) & 1u)) {
                bool here = held;
                for (FlowPatience patience;;) {
                    const uint64_t hub_turn = __hip_atomic_load(a.turns + hub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const bool looks = waits(i);
                    s.read(afresh(a.turns), looks, is);
                    looked(looks);
                    if (!here && __builtin_amdgcn_readfirstlane((uint32_t)hub_turn) == base + i) {
                        here = true;
                        level = __builtin_amdgcn_readfirstlane((uint32_t)(hub_turn >> 32));
                    }
                    if (here && ((come >> i) & 1u)) break;
                    if (patience.ends([&] { return __builtin_amdgcn_readfirstlane(flow_progress(a.flow)); })) {
                        if (lane == 0) a.flow->stalled = 1u;
                        return false;
                    }
                }
                asm volatile("" ::: "memory");
                if (!held) Io::load(row, at, matrix.bytes, y);
                held = true;
            }
            if (!((plain >> i) & 1u)) {
                const uint32_t takes_i = lane_value(takes, i), u = lane_value(s.key[0], i);
                float x[kV], c[kK + 1][kV];
                uint32_t rows[kK + 1];
#pragma unroll
                for (int e = 0; e < kV; ++e) x[e] = 0.0f;
                if (!(takes_i & 1u)) Io::load(matrix.of(0, u), at, matrix.bytes, x);
#pragma unroll
                for (int k = 0; k <= kK; ++k) {
                    const uint32_t here = lane_value(s.key[min(1 + k, kK)], i), before = lane_value(s.key[k], i);
                    rows[k] = (takes_i >> (1 + k)) & 1u ? hub : (takes_i & ((2u << k) - 1u)) != 0u ? before : here;
#pragma unroll
                    for (int e = 0; e < kV; ++e) c[k][e] = 0.0f;
                    if (!((takes_i >> (1 + k)) & 1u)) Io::load(matrix.of(1, rows[k]), at, matrix.bytes, c[k]);
                }
                memory_is_done();
#pragma unroll
                for (int e = 0; e < kV; ++e) x[e] = takes_i & 1u ? y[e] : x[e];
#pragma unroll
                for (int k = 0; k <= kK; ++k)
#pragma unroll
                    for (int e = 0; e < kV; ++e) c[k][e] = (takes_i >> (1 + k)) & 1u ? y[e] : c[k][e];
                sgns_in_place<kV, kK, kTrack>(x, c, rows, __uint_as_float(lane_value(__float_as_uint(lr), i)), a.neg_weight, lane, scores, i);
                if (!(takes_i & 1u)) {
                    Io::store(matrix.of(0, u), at, matrix.bytes, x);
                } else {
#pragma unroll
                    for (int e = 0; e < kV; ++e) y[e] = x[e];
                }
#pragma unroll
                for (int k = 0; k <= kK; ++k) {
                    if (!first_naming<kK>(rows, k)) continue;
                    if (!((takes_i >> (1 + k)) & 1u)) {
                        Io::store(matrix.of(1, rows[k]), at, matrix.bytes, c[k]);
                    } else {
#pragma unroll
                        for (int e = 0; e < kV; ++e) y[e] = c[k][e];
                    }
                }
                level = max(level, lane_value(s.level, i));
                if ((uint32_t)lane == i) s.level = level;
                unhanded = i;
                level += 1u;
                todo &= todo - 1;
                continue;
            }
            // The chain: from here on as long as the next sample is one of these and its turns have come (then it shares none of
            // its other rows with this one).
            float o[kOthers][kV];
            char *o_at[kOthers];
            auto fetch = [&](uint32_t sample, float (&rows)[kOthers][kV], char *(&rows_at)[kOthers]) {
#pragma unroll
                for (int m = 0; m < kOthers; ++m) {
                    rows_at[m] = (char *)((uint64_t)lane_value((uint32_t)(other_at[m] >> 32), sample) << 32 | lane_value((uint32_t)other_at[m], sample));
                    Io::load(rows_at[m], at, matrix.bytes, rows[m]);
                }
            };
            fetch(i, o, o_at);
            memory_is_done();
            for (;;) {
                const uint64_t rest = todo & (todo - 1), next = rest & (0 - rest), behind = rest ^ next;
                const bool goes_on = (next & plain & come) != 0;
                // the turns of those behind it, unless the next two are known to have come
                const bool look = ((next | (behind & (0 - behind))) & own & ~come) != 0;
                const bool looks = look && waits(i + 1u);
                if (look) s.read(afresh(a.turns), looks, is);
                float ahead[kOthers][kV];
                char *ahead_at[kOthers];
                const uint32_t n = goes_on ? (uint32_t)__builtin_ctzll(next) : i;
                if (goes_on) fetch(n, ahead, ahead_at);
                level = max(level, lane_value(s.level, i));
                const float lr_i = __uint_as_float(lane_value(__float_as_uint(lr), i));
                // where the hub stands among the context rows; 0 and none of them where it is a vertex row
                const uint32_t stands = lane_value(takes, i) >> 1;
                float x[kV], c[kK + 1][kV];
#pragma unroll
                for (int e = 0; e < kV; ++e) {
                    x[e] = stands == 0u ? y[e] : o[0][e];
#pragma unroll
                    for (int k = 0; k <= kK; ++k) {
                        // rows before the hub are one further back among the others, for u comes first there
                        c[k][e] = k < kK ? (stands >> (k + 1) ? o[k + 1 <= kK ? k + 1 : kK][e] : o[k][e]) : o[k][e];
                        c[k][e] = (stands >> k) & 1u ? y[e] : c[k][e];
                    }
                }
                sgns_plain<kV, kK, kTrack>(x, c, lr_i, a.neg_weight, lane, scores, i);
                // (without this the compiler moves the wait up into the sums, and the rows of the next sample come before, not
                // beside them: 1678 -> 1612 us the pool on 10^4 nodes that is named above k_train_flow)
#pragma unroll
                for (int e = 0; e < kV; ++e) {
                    asm volatile("" : "+v"(x[e]));
#pragma unroll
                    for (int k = 0; k <= kK; ++k) asm volatile("" : "+v"(c[k][e]));
                }
                // the rows of the sample before are in memory, and so the turns can go on
                memory_is_done();
                hand_on();
#pragma unroll
                for (int e = 0; e < kV; ++e) {
                    y[e] = x[e];
                    o[0][e] = stands == 0u ? c[0][e] : x[e];
#pragma unroll
                    for (int k = 0; k <= kK; ++k) y[e] = (stands >> k) & 1u ? c[k][e] : y[e];
#pragma unroll
                    for (int m = 1; m <= kK; ++m) o[m][e] = stands >> m ? c[m - 1][e] : c[m][e];
                }
#pragma unroll
                for (int m = 0; m < kOthers; ++m) Io::store(o_at[m], at, matrix.bytes, o[m]);
                if (look) looked(looks);
                if ((uint32_t)lane == i) s.level = level;
                level += 1u;
                unhanded = i;
                todo = rest;
                if (!goes_on) break;
                i = n;
#pragma unroll
                for (int m = 0; m < kOthers; ++m) {
                    o_at[m] = ahead_at[m];
#pragma unroll
                    for (int e = 0; e < kV; ++e) o[m][e] = ahead[m][e];
                }
            }
        }
        memory_is_done();
        hand_on();
        if (lane == 0) (void)__hip_atomic_fetch_add(&a.flow->chained, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        deepest = max(deepest, level);
        if constexpr (kTrack) {
            if ((own >> lane) & 1u) lane_loss += again ? 0.0f : scores.loss(a.neg_weight);
            hand_over_loss(a.loss_slots, lane_loss, lane);
        }
    }
    if (held) Io::store(row, at, matrix.bytes, y);
    return true;
}

template <int kV, int kK, bool kFull, bool kTrack>
__global__ __launch_bounds__(kFlowBlock) void k_train_flow(FlowArgs a) {
    constexpr int kRows = kK + 2, kBatch = flow_batch(kV, kK);
    using Io = HandedRow<kV, kFull>;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    FlowState *const state = a.flow;
    float lane_loss = 0.0f;
    uint32_t deepest = 0, chunks_done = 0;
    bool goes_on = true;
    FlowHubs hubs{};
    if constexpr (flow_has_hubs(kV, kK)) {
        __shared__ uint32_t s_started;
        hubs.find(a, lane);
        if (threadIdx.x == 0) s_started = __hip_atomic_fetch_add(&state->started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_started == 0u && wave < (uint32_t)kFlowHubs && lane_value(hubs.namings, wave) > 0u)
            goes_on = flow_hub<kV, kK, kFull, kTrack>(a, hubs, wave, lane, deepest, lane_loss);
    }
    const FlowRows matrix(a);
    const uint32_t at = Io::lane_offset(lane);
    const uint32_t chunks = (a.count + a.unit - 1) / a.unit;
    while (goes_on) {
        uint32_t chunk = 0;
        if (lane == 0) chunk = __hip_atomic_fetch_add(&state->next_chunk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        chunk = __builtin_amdgcn_readfirstlane(chunk);
        if (chunk >= chunks) break;
        const uint32_t base = chunk * a.unit;
        const bool inside = (uint32_t)lane < min(a.unit, a.count - base);
        FlowSample<kK> s;
        s.take(a, base + lane, inside);
        uint32_t owner = kFlowHubs;
        if constexpr (flow_has_hubs(kV, kK)) owner = hubs.owner<kRows>(s.key);
        const bool mine = inside && owner == (uint32_t)kFlowHubs;
        const float lr = learning_rate(a.lr0, a.lr_min_ratio, a.first_g + base + lane, a.total);
        ChunkScores<kK> scores{};
        FlowPatience patience;
        uint64_t pending = __ballot(mine), ready = 0;            // samples to do; those of which all turns have come
        uint32_t due = (uint32_t)__builtin_readcyclecounter();  // lane l: when its turns are looked at again
        while (pending) {
            if ((uint32_t)__popcll(ready) < (uint32_t)kBatch) {
                const uint32_t now = (uint32_t)__builtin_readcyclecounter();
                const bool waits = (pending & ~ready) >> lane & 1u, looks = waits && (int32_t)(now - due) >= 0;
                uint64_t is[kRows];
                s.read(a.turns, looks, is);
                bool came = false;
                if (looks) {
                    const uint32_t away = s.seen(is);
                    came = away == 0u;
                    // a sample that others come before is not looked at again before they can be done; `due` is never far
                    // behind `now` while the lane waits (their difference has 31 bits)
                    if (away > 0u) due = now + min(away - 1u, 64u) * kFlowStep;
                }
                ready |= __ballot(came);
                if (!ready) {
                    if (__ballot(looks) && patience.ends([&] { return __builtin_amdgcn_readfirstlane(flow_progress(state)); })) {
                        if (lane == 0) state->stalled = 1u;
                        break;
                    }
                    if (!__ballot(waits && (int32_t)(due - now) < (int32_t)kFlowStep)) __builtin_amdgcn_s_sleep(8);
                    continue;
                }
            }
            patience = FlowPatience{};
            asm volatile("" ::: "memory");
            uint64_t taken = 0;
            float x[kBatch][kV], c[kBatch][kK + 1][kV];
            uint32_t u[kBatch], rows[kBatch][kK + 1], of[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                if (ready == 0) continue;
                of[b] = (uint32_t)__builtin_ctzll(ready);
                ready &= ready - 1;
                taken |= 1ull << of[b];
                u[b] = lane_value(s.key[0], of[b]);
#pragma unroll
                for (int k = 0; k <= kK; ++k) rows[b][k] = lane_value(s.key[1 + k], of[b]);
                Io::load(matrix.of(0, u[b]), at, matrix.bytes, x[b]);
#pragma unroll
                for (int k = 0; k <= kK; ++k) Io::load(matrix.of(1, rows[b][k]), at, matrix.bytes, c[b][k]);
            }
            const uint32_t batch = (uint32_t)__popcll(taken);
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
                if ((uint32_t)b < batch) {
                    const float lr_b = __uint_as_float(lane_value(__float_as_uint(lr), of[b]));
                    sgns_in_place<kV, kK, kTrack>(x[b], c[b], rows[b], lr_b, a.neg_weight, lane, scores, of[b]);
#pragma unroll
                    for (int k = 0; k <= kK; ++k)
                        if (first_naming<kK>(rows[b], k)) Io::store(matrix.of(1, rows[b][k]), at, matrix.bytes, c[b][k]);
                    Io::store(matrix.of(0, u[b]), at, matrix.bytes, x[b]);
                }
            memory_is_done();
            if ((taken >> lane) & 1u) {
                s.hand_on(a.turns);
                deepest = max(deepest, s.level + 1u);
            }
            pending &= ~taken;
        }
        goes_on = !pending;
        if constexpr (kTrack) {
            if (mine) lane_loss += scores.loss(a.neg_weight);
            if ((++chunks_done & 15u) == 0u) hand_over_loss(a.loss_slots, lane_loss, lane);
        }
    }
    for (int d = kWave / 2; d > 0; d /= 2) deepest = max(deepest, (uint32_t)__shfl_xor((int)deepest, d));
    if (lane == 0 && deepest > 0u) (void)__hip_atomic_fetch_max(&state->deepest, deepest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (kTrack) hand_over_loss(a.loss_slots, lane_loss, lane);
}

#if !GV_TRACK_LOSS
// ---------------------------------------------------------------------------
// Evaluation (no training runs meanwhile, so plain cached loads are fine).
//
// Mean of the per-sample loss  -log sigmoid(x_u . c_v) - w sum_k log sigmoid(-x_u . c_k)
// over an evaluation pool; the negatives of sample i come from Philox stream 2, counter
// (i, k).  Dot products in fp32, the logarithms and the sum in fp64.
__device__ __forceinline__ double log_sigmoid(double z) { return z >= 0.0 ? -log1p(exp(-z)) : z - log1p(exp(z)); }

//
// A wave takes a.unit samples at a time, lane l the ids and draws of sample l, gathers the rows of a few samples together
// and lays their scores into lanes; the logarithms are taken once per chunk, lane l for sample l.  Every workgroup
// leaves one partial sum.  (2^18 samples, d = 128, K = 1: 224 us with one sample at a time, the logarithms on all 64
// lanes and one fp64 atomic add a wave to one address -- 4096 of them, one after the other -- and 58 us
// now, 7.0 TB/s of rows, with the pairs on the device; in two pieces read from pinned memory 46 us each.)
constexpr int eval_batch(int V, int K) { return V * (K + 2) <= 6 ? 4 : (V * (K + 2) <= 14 ? 2 : 1); }

template <int kV, int kK, bool kFull>
__global__ __launch_bounds__(kBlock) void k_eval_loss(TrainArgs a, double *__restrict__ partial) {
    using Io = RowIo<kV, kPlain, kFull>;
    constexpr int kBatch = eval_batch(kV, kK);
    __shared__ double s_sum[kBlock / kWave];
    const uint32_t D = a.dim;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane((blockIdx.x * kBlock + threadIdx.x) / kWave);
    const uint32_t waves = gridDim.x * (kBlock / kWave);
    const uint32_t chunks = (uint32_t)(((uint64_t)a.count + a.unit - 1) / a.unit);
    const uint2 *__restrict__ pairs = (const uint2 *)a.pairs;
    double sum = 0.0;
    for (uint32_t chunk = wave; chunk < chunks; chunk += waves) {
        const uint32_t base = chunk * a.unit;
        const uint32_t in_chunk = min(a.unit, a.count - base);
        const bool mine = (uint32_t)lane < in_chunk;
        uint2 p = mine ? pairs[base + lane] : make_uint2(0u, 0u);
        const bool named = mine && p.x < a.n && p.y < a.n;
        if (mine && !named) *a.error_flag = 1u;
        if (!named) p = make_uint2(0u, 0u);  // row 0 is read in its place, and its scores are dropped
        uint32_t neg[kK];
#pragma unroll
        for (int k = 0; k < kK; ++k)
            neg[k] = mine ? draw_negative(a.alias, a.alias_n, a.seed, a.first_g + base + lane, k, 2u) : 0u;
        ChunkScores<kK> scores{};
        for (uint32_t i0 = 0; i0 < in_chunk; i0 += kBatch) {
            float x[kBatch][kV], c[kBatch][kK + 1][kV];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const uint32_t i = min(i0 + b, in_chunk - 1u);  // past the end: the last sample again
                Io::load(a.vertex + (size_t)lane_value(p.x, i) * D, lane, D, x[b]);
                Io::load(a.context + (size_t)lane_value(p.y, i) * D, lane, D, c[b][0]);
#pragma unroll
                for (int k = 0; k < kK; ++k) Io::load(a.context + (size_t)lane_value(neg[k], i) * D, lane, D, c[b][1 + k]);
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
#pragma unroll
                for (int k = 0; k <= kK; ++k) {
                    float dot = 0.0f;
#pragma unroll
                    for (int j = 0; j < kV; ++j) dot = fmaf(x[b][j], c[b][k][j], dot);
                    scores.put(k, min(i0 + b, in_chunk - 1u), wave_sum(dot));
                }
        }
        if (named) {
            sum -= log_sigmoid((double)scores.of[0]);
#pragma unroll
            for (int k = 1; k <= kK; ++k) sum -= (double)a.neg_weight * log_sigmoid(-(double)scores.of[k]);
        }
    }
    for (int d = kWave / 2; d > 0; d /= 2) sum += __shfl_xor(sum, d);
    if (lane == 0) s_sum[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) sum += s_sum[w];
        partial[blockIdx.x] = sum;
    }
}

// out[i] = cosine of vertex rows first[i], second[i] (0 when a row is zero), the score of
// an edge in link prediction (Sec. 4.5).  A wave takes `unit` pairs at a time, lane l the ids of pair l, gathers the rows
// of a few pairs together and lays their sums into lanes, which take the roots and the quotients once per chunk.
// (5*10^5 pairs, d = 128, a million nodes: 93 us with one pair at a time, 5.5 TB/s of rows, and 66 now, 7.7 TB/s, what a read of
// random rows reaches.)
constexpr int cosine_batch(int V) { return V <= 2 ? 4 : (V == 4 ? 2 : 1); }
template <int kV, bool kFull>
__global__ __launch_bounds__(kBlock) void k_cosine(const float *__restrict__ vertex, uint32_t n, uint32_t dim,
                                                   const uint32_t *__restrict__ first,
                                                   const uint32_t *__restrict__ second, uint32_t count, uint32_t unit,
                                                   float *__restrict__ out, uint32_t *error_flag) {
    using Io = RowIo<kV, kPlain, kFull>;
    constexpr int kBatch = cosine_batch(kV);
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t waves = gridDim.x * (kBlock / kWave), chunks = (uint32_t)(((uint64_t)count + unit - 1) / unit);
    for (uint32_t chunk = __builtin_amdgcn_readfirstlane((blockIdx.x * kBlock + threadIdx.x) / kWave); chunk < chunks; chunk += waves) {
        const uint32_t base = chunk * unit, in_chunk = min(unit, count - base);
        const bool mine = (uint32_t)lane < in_chunk;
        uint32_t ra = mine ? first[base + lane] : 0u, rb = mine ? second[base + lane] : 0u;
        const bool named = mine && ra < n && rb < n;
        if (mine && !named) *error_flag = 1u;
        if (!named) ra = rb = 0u;  // row 0 is read in its place, and its score dropped
        float xy = 0.0f, xx = 0.0f, yy = 0.0f;
        for (uint32_t i0 = 0; i0 < in_chunk; i0 += kBatch) {
            float x[kBatch][kV], y[kBatch][kV];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const uint32_t i = min(i0 + b, in_chunk - 1u);  // past the end: the last pair again
                Io::load(vertex + (size_t)lane_value(ra, i) * dim, lane, dim, x[b]);
                Io::load(vertex + (size_t)lane_value(rb, i) * dim, lane, dim, y[b]);
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                float pxy = 0.0f, pxx = 0.0f, pyy = 0.0f;
#pragma unroll
                for (int j = 0; j < kV; ++j) {
                    pxy = fmaf(x[b][j], y[b][j], pxy);
                    pxx = fmaf(x[b][j], x[b][j], pxx);
                    pyy = fmaf(y[b][j], y[b][j], pyy);
                }
                const bool here = (uint32_t)lane == i0 + b;
                const float sxy = wave_sum(pxy), sxx = wave_sum(pxx), syy = wave_sum(pyy);
                xy = here ? sxy : xy;
                xx = here ? sxx : xx;
                yy = here ? syy : yy;
            }
        }
        if (mine) out[base + lane] = named && xx > 0.0f && yy > 0.0f ? xy / (sqrtf(xx) * sqrtf(yy)) : 0.0f;
    }
}

// ---------------------------------------------------------------------------
// Rank statistic (gv_link_prediction_auc): twice the sum over all positives of (negatives below it + half of the
// negatives equal to it).  The negatives are sorted (least significant digit first, eight bits a pass) and every
// positive is looked up among them; whole numbers throughout, so the result is that of sorting all scores on the host.
// 250000 + 250000 scores: 75 us with three launches a pass, all of it latency of short launches, so a workgroup owns as few keys as
// it takes at a time and up to 256 of them do without a launch for the places (own_places; the whole call 263 -> 252)
// (segments of 4096 keys, one workgroup for the places, all of a search in memory: 105 us); std::sort of the pairs on the host
// took 29 ms.
constexpr int kSortBlock = 1024, kSortWaves = kSortBlock / kWave, kDigits = 256;

// A score as an unsigned integer of the same order (the two zeros are one value).
__device__ __forceinline__ uint32_t score_key(uint32_t x) {
    if ((x & 0x7FFFFFFFu) == 0u) x = 0u;
    return x & 0x80000000u ? ~x : x | 0x80000000u;
}
__device__ __forceinline__ bool not_a_number(uint32_t x) { return (x & 0x7F800000u) == 0x7F800000u; }  // or an infinity

// One pass: workgroup b owns the keys b * segment .. (b + 1) * segment - 1 and counts their digits (by_block: digit after digit
// of one workgroup, for own_places; kScores: of the scores
// still to be made keys; *not_finite is set where one is no number) ...
template <bool kScores>
__global__ __launch_bounds__(kSortBlock) void k_radix_count(const uint32_t *__restrict__ keys, uint32_t count, uint32_t segment,
                                                            uint32_t shift, bool by_block, uint32_t *__restrict__ counts,
                                                            unsigned long long *__restrict__ not_finite) {
    __shared__ uint32_t s_count[kDigits];
    if (threadIdx.x < kDigits) s_count[threadIdx.x] = 0u;
    __syncthreads();
    const uint64_t begin = (uint64_t)blockIdx.x * segment, end = min(begin + segment, (uint64_t)count);
    for (uint64_t i = begin + threadIdx.x; i < end; i += kSortBlock) {
        uint32_t key = keys[i];
        if constexpr (kScores) {
            if (not_a_number(key)) *not_finite = 1ull;
            key = score_key(key);
        }
        atomicAdd(&s_count[(key >> shift) & (kDigits - 1)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < kDigits)
        counts[by_block ? (size_t)blockIdx.x * kDigits + threadIdx.x : (size_t)threadIdx.x * gridDim.x + blockIdx.x] = s_count[threadIdx.x];
}

// ... the counts, digit after digit and workgroup after workgroup, become places: a workgroup adds up the counts before its
// part, and scans the part, a thread the sixteen bytes that follow each other ...
__global__ __launch_bounds__(kSortBlock) void k_radix_places(const uint32_t *__restrict__ counts, uint32_t entries,
                                                             uint32_t *__restrict__ places) {
    __shared__ uint32_t s_before[kSortWaves], s_total[kSortWaves];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t fours = entries / 4u, part = (fours + gridDim.x - 1) / gridDim.x;  // entries is a multiple of the 256 digits
    const uint32_t part_begin = min(blockIdx.x * part, fours), part_end = min(part_begin + part, fours);
    const uint4 *const four = (const uint4 *)counts;
    auto sum_of = [](uint4 c) { return c.x + c.y + c.z + c.w; };
    uint32_t before = 0u;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < part_begin; i += kSortBlock) before += sum_of(four[i]);
    for (int d = kWave / 2; d > 0; d /= 2) before += __shfl_xor(before, d);
    if (lane == 0) s_before[wave] = before;
    for (uint32_t first = part_begin; first < part_end; first += kSortBlock) {
        const uint32_t i = first + threadIdx.x;
        const uint4 c = i < part_end ? four[i] : make_uint4(0u, 0u, 0u, 0u);
        const uint32_t own = sum_of(c);
        uint32_t upto = own;
        for (uint32_t d = 1; d < (uint32_t)kWave; d *= 2) {
            const uint32_t x = __shfl_up(upto, d);
            upto += lane >= d ? x : 0u;
        }
        if (lane == kWave - 1) s_total[wave] = upto;
        __syncthreads();
        uint32_t place = upto - own, all = 0u;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            place += s_before[w] + ((uint32_t)w < wave ? s_total[w] : 0u);
            all += s_total[w];
        }
        if (i < part_end) ((uint4 *)places)[i] = make_uint4(place, place + c.x, place + c.x + c.y, place + c.x + c.y + c.z);
        __syncthreads();
        if (threadIdx.x == 0) s_before[0] += all;  // of what follows in this part
        __syncthreads();
    }
}

// ... or, of few workgroups, each adds up the places of its own keys: a wave takes whole rows of counts, a lane four digits of
// each, into s_next[digit] = the counts of lower digits, and of this one in the workgroups before.  (A launch of
// k_radix_places takes 5 to 8 us with the way to it, a pass: link prediction of 10000 against 10000 pairs 95 -> 83 us, of 80000 155 ->
// 147, of 150000 207 -> 194; deterministic pools of 10000 samples 148 -> 138, of 50000 200 -> 189.)
__device__ __forceinline__ void own_places(const uint32_t *__restrict__ counts, uint32_t (&s_part)[kSortWaves][kDigits],
                                           uint32_t (&s_next)[kDigits]) {
    __shared__ uint32_t s_before[kSortWaves][kDigits], s_total[kDigits / kWave];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint4 all = make_uint4(0u, 0u, 0u, 0u), before = all;
#pragma unroll 8
    for (uint32_t b = wave; b < gridDim.x; b += kSortWaves) {
        const uint4 c = ((const uint4 *)counts)[(size_t)b * (kDigits / 4) + lane];
        const uint32_t earlier = b < blockIdx.x ? ~0u : 0u;
        all = make_uint4(all.x + c.x, all.y + c.y, all.z + c.z, all.w + c.w);
        before = make_uint4(before.x + (c.x & earlier), before.y + (c.y & earlier), before.z + (c.z & earlier), before.w + (c.w & earlier));
    }
    ((uint4 *)s_part[wave])[lane] = all;
    ((uint4 *)s_before[wave])[lane] = before;
    __syncthreads();
    uint32_t own = 0u, next = 0u, upto = 0u;
    if (threadIdx.x < kDigits) {  // whole waves
        for (int w = 0; w < kSortWaves; ++w) {
            own += s_part[w][threadIdx.x];
            next += s_before[w][threadIdx.x];
        }
        upto = own;
        for (uint32_t d = 1; d < (uint32_t)kWave; d *= 2) {
            const uint32_t x = __shfl_up(upto, d);
            upto += lane >= d ? x : 0u;
        }
        if (lane == kWave - 1) s_total[wave] = upto;
    }
    __syncthreads();
    if (threadIdx.x < kDigits) {
        for (uint32_t w = 0; w < wave; ++w) next += s_total[w];
        s_next[threadIdx.x] = next + upto - own;
    }
    __syncthreads();  // s_part is used again
}

// ... and the keys go there in their order: 1024 at a time, a wave finds the lanes with its lane's digit by eight ballots.
// kCarried: each key takes a word with it, the one beside it in `words`, or, where that is null, its own place.  kScores:
// scores come in, their keys go out.
// kOwnPlaces: `places` are the counts, workgroup after workgroup, and each workgroup adds up its own places (own_places).
template <bool kCarried, bool kScores, bool kOwnPlaces>
__global__ __launch_bounds__(kSortBlock) void k_radix_scatter(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ words,
                                                              uint32_t count, uint32_t segment, uint32_t shift,
                                                              const uint32_t *__restrict__ places, uint32_t *__restrict__ out,
                                                              uint32_t *__restrict__ words_out) {
    __shared__ uint32_t s_next[kDigits];               // place of the workgroup's next key of a digit
    __shared__ uint32_t s_place[kSortWaves][kDigits];  // keys of a digit in a wave, then the place of the first of them
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if constexpr (kOwnPlaces)
        own_places(places, s_place, s_next);
    else if (threadIdx.x < kDigits)
        s_next[threadIdx.x] = places[(size_t)threadIdx.x * gridDim.x + blockIdx.x];
    const uint64_t begin = (uint64_t)blockIdx.x * segment, end = min(begin + segment, (uint64_t)count);
    for (uint64_t base = begin; base < end; base += kSortBlock) {
        for (uint32_t i = threadIdx.x; i < kSortWaves * kDigits; i += kSortBlock) (&s_place[0][0])[i] = 0u;
        __syncthreads();
        const bool mine = base + threadIdx.x < end;
        uint32_t key = mine ? keys[base + threadIdx.x] : 0u;
        if constexpr (kScores) key = score_key(key);
        const uint32_t digit = (key >> shift) & (kDigits - 1);
        uint64_t same = __ballot(mine);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t set = __ballot((digit >> b) & 1u);
            same &= (digit >> b) & 1u ? set : ~set;
        }
        const uint32_t rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        if (mine && rank == 0u) s_place[wave][digit] = (uint32_t)__popcll(same);
        __syncthreads();
        if (threadIdx.x < kDigits) {
            uint32_t next = s_next[threadIdx.x];
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t here = s_place[w][threadIdx.x];
                s_place[w][threadIdx.x] = next;
                next += here;
            }
            s_next[threadIdx.x] = next;
        }
        __syncthreads();
        if (mine) {
            const uint32_t to = s_place[wave][digit] + rank;
            out[to] = key;
            if constexpr (kCarried) words_out[to] = words ? words[base + threadIdx.x] : (uint32_t)(base + threadIdx.x);
        }
        __syncthreads();
    }
}

// twice[workgroup] = sum over its positives of 2 (sorted keys below) + (sorted keys equal).  The search begins among 1024
// of the keys at equal distances, in LDS: a search of all in memory is twice as many dependent loads (20 us instead of 16).
constexpr uint32_t kRankMarks = 1024;
__global__ __launch_bounds__(kSortBlock) void k_rank_sum(const uint32_t *__restrict__ positives, uint64_t num_pos,
                                                         const uint32_t *__restrict__ sorted, uint32_t num_neg,
                                                         unsigned long long *__restrict__ twice,
                                                         unsigned long long *__restrict__ not_finite) {
    __shared__ uint32_t s_mark[kRankMarks];
    __shared__ unsigned long long s_sum[kSortWaves];
    const uint32_t step = (num_neg + kRankMarks - 1) / kRankMarks, marks = (num_neg + step - 1) / step;  // the last key of each step
    if (threadIdx.x < marks) s_mark[threadIdx.x] = sorted[min((uint64_t)(threadIdx.x + 1) * step, (uint64_t)num_neg) - 1];
    __syncthreads();
    unsigned long long sum = 0ull;
    for (uint64_t i = (uint64_t)blockIdx.x * kSortBlock + threadIdx.x; i < num_pos; i += (uint64_t)gridDim.x * kSortBlock) {
        const uint32_t score = positives[i], key = score_key(score);
        if (not_a_number(score)) *not_finite = 1ull;
        // first place that is not `before`: among the marks, then in the step that ends with the mark
        auto first_not = [&](auto &&before) {
            uint32_t begin = 0, length = marks;
            while (length > 0u) {
                const uint32_t half = length / 2u;
                const bool less = before(s_mark[begin + half]);
                begin = less ? begin + half + 1u : begin;
                length = less ? length - half - 1u : half;
            }
            if (begin == marks) return num_neg;
            begin *= step;
            length = min(step, num_neg - begin) - 1u;  // the step's last key is not before
            while (length > 0u) {
                const uint32_t half = length / 2u;
                const bool less = before(sorted[begin + half]);
                begin = less ? begin + half + 1u : begin;
                length = less ? length - half - 1u : half;
            }
            return begin;
        };
        const uint32_t below = first_not([&](uint32_t x) { return x < key; });
        uint32_t upto = below;
        if (below < num_neg && sorted[below] == key) upto = first_not([&](uint32_t x) { return x <= key; });
        sum += (unsigned long long)below + upto;
    }
    for (int d = kWave / 2; d > 0; d /= 2) sum += __shfl_xor(sum, d);
    if ((threadIdx.x & (kWave - 1)) == 0) s_sum[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kSortWaves; ++w) sum += s_sum[w];
        twice[blockIdx.x] = sum;
    }
}

__global__ __launch_bounds__(kBlock) void k_draw_negatives(const uint4 *__restrict__ alias, uint32_t n, uint64_t seed,
                                                           uint64_t first_g, uint64_t count, uint32_t num_neg,
                                                           uint32_t *__restrict__ out) {
    const uint64_t total = count * num_neg;
    for (uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x; t < total; t += (uint64_t)gridDim.x * kBlock) {
        const uint64_t i = t / num_neg;
        const uint32_t k = (uint32_t)(t - i * num_neg);
        out[t] = draw_negative(alias, n, seed, first_g + i, k);
    }
}

// The records of a deterministic launch (see k_train_level): record i is sample order[i] of the pool.
__global__ __launch_bounds__(kBlock) void k_level_records(const uint2 *__restrict__ pairs,
                                                          const uint32_t *__restrict__ negatives,
                                                          const uint32_t *__restrict__ order, uint32_t count,
                                                          uint32_t num_neg, uint32_t *__restrict__ records) {
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (uint64_t)gridDim.x * kBlock) {
        const uint32_t place = order[i];
        const uint2 p = pairs[place];
        uint32_t *record = records + i * (num_neg + 3);
        record[0] = p.x;
        record[1] = p.y;
        for (uint32_t k = 0; k < num_neg; ++k) record[2 + k] = negatives[(size_t)place * num_neg + k];
        record[2 + num_neg] = place;
    }
}

// Preparation of k_train_flow.  The state of a part: what the part before counted is folded into `batches`; of a pool: no
// id is bad so far.
__global__ __launch_bounds__(kWave) void k_flow_begin(FlowState *state, bool new_pool, bool fresh) {
    state->slots[threadIdx.x] = 0ull;
    if (threadIdx.x != 0) return;
    if (fresh) {
        state->batches = 0ull;
        state->deepest = state->stalled = 0u;
    }
    state->started = state->chained = 0u;
    state->batches += state->deepest;
    state->deepest = 0u;
    state->next_chunk = 0u;
    if (new_pool) state->first_bad = UINT32_MAX;
}
// The rows that a sample names, K + 2 words: u, n + v, n + every negative (row 0 in the place of a bad id: the sort and the
// turns go over such a pool, the training does not).
__device__ __forceinline__ void flow_keys(uint2 p, const uint4 *__restrict__ alias, uint32_t n, uint64_t seed, uint64_t g, uint32_t num_neg,
                                          uint32_t *__restrict__ key) {
    key[0] = p.x < n ? p.x : 0u;
    key[1] = n + (p.y < n ? p.y : 0u);
    for (uint32_t k = 0; k < num_neg; ++k) key[2 + k] = n + draw_negative(alias, n, seed, g, k);
}
// first_bad = the first sample that names an id that is no node, if any does; `named`: see launch_flow_check
__global__ __launch_bounds__(kBlock) void k_flow_check(const uint2 *__restrict__ pairs, uint64_t count, const uint4 *__restrict__ alias,
                                                       uint32_t n, uint64_t seed, uint64_t first_g, uint32_t num_neg, FlowState *state,
                                                       uint32_t *__restrict__ named) {
    const uint32_t thread = blockIdx.x * kBlock + threadIdx.x;
    for (uint32_t t = thread; t < flow_looked_at(count); t += gridDim.x * kBlock) {
        const uint64_t i = flow_look(t, count);
        flow_keys(pairs[i], alias, n, seed, first_g + i, num_neg, named + (size_t)t * (num_neg + 2));
    }
    for (uint64_t i = thread; i < count; i += (uint64_t)gridDim.x * kBlock) {
        const uint2 p = pairs[i];
        if (p.x >= n || p.y >= n) atomicMin(&state->first_bad, (uint32_t)i);
    }
}
__global__ __launch_bounds__(kBlock) void k_flow_keys(const uint2 *__restrict__ pairs, const uint4 *__restrict__ alias, uint32_t n,
                                                      uint64_t seed, uint64_t first_g, uint32_t count, uint32_t num_neg,
                                                      uint32_t *__restrict__ keys) {
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += (uint64_t)gridDim.x * kBlock)
        flow_keys(pairs[i], alias, n, seed, first_g + i, num_neg, keys + i * (num_neg + 2));
}
// From the sorted namings: the place of every naming; where a row's namings begin, the row's first turn, and, if there
// are many, an entry {namings, begin} in one of 64 slots, which keeps the largest (FlowHubs takes the first of them).
__global__ __launch_bounds__(kBlock) void k_flow_places(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ namings,
                                                        uint32_t count, uint32_t *__restrict__ places, uint64_t *__restrict__ turns,
                                                        FlowState *state) {
    constexpr uint32_t kMany = 32;
    for (uint64_t j = (uint64_t)blockIdx.x * kBlock + threadIdx.x; j < count; j += (uint64_t)gridDim.x * kBlock) {
        places[namings[j]] = (uint32_t)j;
        const uint32_t key = keys[j];
        if (j > 0 && keys[j - 1] == key) continue;
        turns[key] = j;
        if (j + kMany > count || keys[j + kMany - 1] != key) continue;
        uint64_t last = j + kMany - 1, step = kMany;  // a naming of the row; the last one is less than `step` on
        while (last + step < count && keys[last + step] == key) {
            last += step;
            step *= 2;
        }
        for (; step > 1; step /= 2)
            if (last + step / 2 < count && keys[last + step / 2] == key) last += step / 2;
        atomicMax(&state->slots[(key * 0x9E3779B1u) >> 26], (unsigned long long)(last - j + 1) << 32 | j);
    }
}

// Negatives restricted to a partition (Sec. 3.2): sample i draws from the alias table of the partition of its
// context node v[i].
__global__ __launch_bounds__(kBlock) void k_draw_negatives_partitioned(const uint4 *__restrict__ tables,
                                                                       const uint64_t *__restrict__ offsets,
                                                                       const uint8_t *__restrict__ part,
                                                                       const uint32_t *__restrict__ v, uint64_t seed,
                                                                       uint64_t first_g, uint64_t count, uint32_t num_neg,
                                                                       uint32_t *__restrict__ out) {
    const uint64_t total = count * num_neg;
    for (uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x; t < total; t += (uint64_t)gridDim.x * kBlock) {
        const uint64_t i = t / num_neg;
        const uint32_t k = (uint32_t)(t - i * num_neg);
        const uint32_t j = part[v[i]];
        out[t] = draw_negative(tables + offsets[j], (uint32_t)(offsets[j + 1] - offsets[j]), seed, first_g + i, k);
    }
}

// vertex[row][4b .. 4b+3] from the four words of Philox block (row, b) of stream 1:
// ((word + 0.5) / 2^32 - 0.5) / d, evaluated in fp64.
__global__ __launch_bounds__(kBlock) void k_init_vertex(float *__restrict__ vertex, uint64_t rows, uint32_t dim,
                                                        uint64_t seed) {
    const uint32_t blocks_per_row = dim / 4;
    const uint64_t total = rows * blocks_per_row;
    for (uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x; t < total; t += (uint64_t)gridDim.x * kBlock) {
        const uint64_t row = t / blocks_per_row;
        const uint32_t b = (uint32_t)(t - row * blocks_per_row);
        const uint4 r = philox4x32_10((uint32_t)row, (uint32_t)(row >> 32), b, 1u, (uint32_t)seed,
                                      (uint32_t)(seed >> 32));
        const double inv = 1.0 / 4294967296.0;
        f4 out;
        out.x = (float)((((double)r.x + 0.5) * inv - 0.5) / (double)dim);
        out.y = (float)((((double)r.y + 0.5) * inv - 0.5) / (double)dim);
        out.z = (float)((((double)r.z + 0.5) * inv - 0.5) / (double)dim);
        out.w = (float)((((double)r.w + 0.5) * inv - 0.5) / (double)dim);
        *(f4 *)(vertex + row * dim + 4 * (uint64_t)b) = out;
    }
}

// ---------------------------------------------------------------------------
// Producer on the device: online augmentation (Sec. 3.1, Alg. 2) with the pseudo shuffle of
// the same section, one thread per random walk.  Walk w departs at the owner of a uniformly
// chosen half-edge (probability proportional to degree), takes `length` uniform steps over the
// CSR adjacency (on a weighted graph both are alias draws, see below) and emits every ordered pair (w_i, w_j), i < j <= i + window, in order of i then
// j; sample number t of the pool (walks concatenated) goes to position t, or, pseudo-shuffled,
// to block t mod window at offset t / window.  Random numbers: Philox stream 4, counter
// (walk number, step): the pool depends on nothing but the seed and the walk numbers.
constexpr int kMaxWalkLength = 64;

__device__ __forceinline__ uint64_t pick_below(uint4 r, uint64_t range) {
    return __umul64hi(((uint64_t)r.x << 32) | r.y, range);
}
// the same for a range below 2^32
__device__ __forceinline__ uint32_t pick_below(uint4 r, uint32_t range) {
    return (uint32_t)(((uint64_t)r.x * range + (((uint64_t)r.y * range) >> 32)) >> 32);
}

// What a step of a walk needs of the node it reaches, in one 16-byte load: node, degree, first half-edge.  Read from the
// neighbour id and then from the offsets, the same takes two dependent loads a step (a million nodes, 40 steps:
// 2.4 us a step, now 1.75).
__global__ __launch_bounds__(kBlock) void k_pack_steps(const uint64_t *__restrict__ offsets, const uint32_t *__restrict__ adj,
                                                       uint64_t half_edges, uint4 *__restrict__ steps) {
    for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < half_edges; e += (uint64_t)gridDim.x * kBlock) {
        const uint32_t x = adj[e];
        const uint64_t begin = offsets[x];
        steps[e] = make_uint4(x, (uint32_t)(offsets[x + 1] - begin), (uint32_t)begin, (uint32_t)(begin >> 32));
    }
}

// The same of a weighted graph, for both outcomes of the alias draw, in 32 bytes: {threshold, neighbour, degree, first
// half-edge} and {the alias's neighbour, degree, first half-edge, 0}; half-edges are below 2^32 there.  (The alias
// table, then the step: 3*10^5 nodes, 40 steps: 1.4 us a step instead of 0.9.)
__global__ __launch_bounds__(kBlock) void k_pack_weighted_steps(const uint64_t *__restrict__ offsets,
                                                                const uint32_t *__restrict__ adj,
                                                                const uint2 *__restrict__ nbr_table, uint32_t n,
                                                                uint4 *__restrict__ steps) {
    // a wave takes a row at a time: an alias is a place within the row
    const uint32_t lane = threadIdx.x & (kWave - 1), waves = gridDim.x * (kBlock / kWave);
    for (uint32_t x = __builtin_amdgcn_readfirstlane((blockIdx.x * kBlock + threadIdx.x) / kWave); x < n; x += waves) {
        const uint64_t begin = offsets[x], end = offsets[x + 1];
        for (uint64_t e = begin + lane; e < end; e += kWave) {
            const uint2 entry = nbr_table[e];
            const uint32_t self = adj[e], other = adj[begin + entry.y];
            const uint64_t self_begin = offsets[self], other_begin = offsets[other];
            steps[2 * e] = make_uint4(entry.x, self, (uint32_t)(offsets[self + 1] - self_begin), (uint32_t)self_begin);
            steps[2 * e + 1] = make_uint4(other, (uint32_t)(offsets[other + 1] - other_begin), (uint32_t)other_begin, 0u);
        }
    }
}

// last node of lo .. hi - 1 whose first half-edge is at or before e, where the node lo is such
__device__ __forceinline__ uint32_t owner_of(const uint64_t *__restrict__ offsets, uint64_t e, uint32_t lo, uint32_t hi) {
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (offsets[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
}

// owners[j] = owner of half-edge j << shift; owners[entries - 1] = n - 1: the search for a departure starts between two
// of them (4 turns instead of 20 at a million nodes).
__global__ __launch_bounds__(kBlock) void k_departure_guide(const uint64_t *__restrict__ offsets, uint32_t n, uint64_t half_edges,
                                                            uint32_t shift, uint32_t entries, uint32_t *__restrict__ owners) {
    const uint32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= entries) return;
    const uint64_t e = (uint64_t)j << shift;
    owners[j] = e < half_edges ? owner_of(offsets, e, 0u, n) : n - 1u;
}

// The pool position of sample number t (generation order): t itself, or, pseudo-shuffled, block t mod s at
// offset t / s (block b holds the samples b, b + s, b + 2s, ...: the blocks before it hold
// ceil((count - b') / s) samples each, i.e. the first count mod s blocks hold one more).
__device__ __forceinline__ uint64_t place_of(uint64_t t, uint32_t s, uint64_t count, bool pseudo_shuffle) {
    if (!pseudo_shuffle) return t;
    const uint64_t b = t % s, q = t / s, whole = count / s, extra = count % s;
    return b * whole + (b < extra ? b : extra) + q;
}

// A workgroup of kThreads threads makes kWalks walks, a thread each, and all of its threads write their pairs.  Where walks are
// few, what they cost is latency: of the steps, and of the writing, a thread some 600 pairs with as many threads as walks.  So
// below 2^16 walks and 2^23 pairs there are 64 walks to a workgroup, on more compute units, and four threads to each; us among other
// launches (alone), 128 walks and threads -> 64 and 256: 10^6 nodes, 40 steps, window 5, 1053 walks 13.0 (51) -> 8.3 (36), 21053 24.3
// (68) -> 22.1 (55), 42106 40.6 (78) -> 40.4 (65); 10^4 nodes, 64 steps, window 10, 7050 walks 32.4 (104) -> 17.7 (60); weighted, window
// 2, 37975 walks 35.9 (54) -> 31.9 (49).  With more of them the reads of the steps and the pairs written fill the memory, and
// the four threads gain nothing: 88301 walks, 2^24 pairs, 89.8 (124) and 101 (120); weighted 75950 walks 60.2 and 61.3.  Between 2^23
// and 2^24 pairs of few walks the pools differ, by what is not known: 63158 walks of 40 steps, window 5, 59.9 (90) -> 59.4 (86), 28197 of
// 64 steps, window 10, 61.7 (134) -> 61.0 (93), another 48.9 -> 57.3; so those keep the larger workgroups.
// Walks of few pairs leave three of the four threads idle, which shows once the chip is full: window 1, 65535 walks of 5 steps 12.4 ->
// 12.9 on 10^6 nodes, 2 to 5 % more on all graphs, of 2 steps 6.5 -> 6.8; 40000 walks gain or keep their time (5 steps 8.5 -> 8.3).  So
// those are few up to 3 * 2^14 only.  With 8 to 11 pairs a walk, 55000 and more lose 2 to 4 % on 10^6 nodes and gain 3 to 7 % on 10^4;
// with 15 and more none loses.
constexpr uint64_t kFewWalks = 1u << 16, kFewShortWalks = 3u << 14, kShortWalk = 8, kFewPairs = 1u << 23;
template <int kWalks, int kThreads>
__global__ __launch_bounds__(kThreads) void k_augment(AugmentArgs a) {
    // a walk's nodes, one row per thread (65 words: the rows start in different banks)
    __shared__ uint32_t s_path[kWalks][kMaxWalkLength + 1];
    // the pairs of a walk in order: i << 8 | j of pair number t (i < j <= i + s, in order of i then j)
    __shared__ uint16_t s_pair[(kMaxWalkLength + 1) * kMaxWalkLength / 2];
    const uint64_t w0 = (uint64_t)blockIdx.x * kWalks, w = w0 + threadIdx.x;
    const uint32_t L = a.length, s = a.window;
    for (uint32_t i = threadIdx.x; i < L; i += kThreads) {
        uint32_t start = 0;  // pairs of the nodes before i
        for (uint32_t before = 0; before < i; ++before) start += min(s, L - before);
        for (uint32_t j = i + 1; j <= L && j - i <= s; ++j) s_pair[start + (j - i - 1)] = (uint16_t)(i << 8 | j);
    }
    if (threadIdx.x < kWalks && w < a.walks) {
        const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
        const uint64_t walk = a.first_walk + w;
        uint32_t x;
        const uint4 r0 = philox4x32_10((uint32_t)walk, (uint32_t)(walk >> 32), 0u, 4u, k0, k1);
        if (a.node_table) {
            // weighted graph (Sec. 4.3): departure by an alias draw over the nodes, weights = weighted degrees
            const uint32_t j = pick_below(r0, a.n);
            const uint2 entry = a.node_table[j];
            x = r0.z < entry.x ? j : entry.y;
        } else {
            // departure: last node whose first half-edge is at or before the chosen one
            const uint64_t e = pick_below(r0, a.half_edges);
            const uint32_t bucket = (uint32_t)(e >> a.guide_shift);
            x = a.guide ? owner_of(a.offsets, e, a.guide[bucket], a.guide[bucket + 1] + 1u) : owner_of(a.offsets, e, 0u, a.n);
        }
        s_path[threadIdx.x][0] = x;
        uint64_t begin = a.offsets[x];
        uint32_t degree = (uint32_t)(a.offsets[x + 1] - begin);
        uint4 r = philox4x32_10((uint32_t)walk, (uint32_t)(walk >> 32), 1u, 4u, k0, k1);
        for (uint32_t t = 1; t <= L; ++t) {
            uint32_t at = pick_below(r, degree);
            // the next step's random words are worked out while this one's neighbour is on its way
            if (a.weighted_steps) {
                const uint4 self = a.weighted_steps[2 * (begin + at)], other = a.weighted_steps[2 * (begin + at) + 1];
                const uint32_t decides = r.z;
                r = philox4x32_10((uint32_t)walk, (uint32_t)(walk >> 32), t + 1u, 4u, k0, k1);
                const bool keep = decides < self.x;
                x = keep ? self.y : other.x;
                degree = keep ? self.z : other.y;
                begin = keep ? self.w : other.z;
                s_path[threadIdx.x][t] = x;
                continue;
            }
            if (a.nbr_table) {  // weighted step: alias draw over the row's edge weights
                const uint2 entry = a.nbr_table[begin + at];
                at = r.z < entry.x ? at : entry.y;
            }
            if (a.steps) {
                const uint4 step = a.steps[begin + at];
                r = philox4x32_10((uint32_t)walk, (uint32_t)(walk >> 32), t + 1u, 4u, k0, k1);
                x = step.x;
                degree = step.y;
                begin = (uint64_t)step.w << 32 | step.z;
            } else {
                x = a.adj[begin + at];
                r = philox4x32_10((uint32_t)walk, (uint32_t)(walk >> 32), t + 1u, 4u, k0, k1);
                begin = a.offsets[x];
                degree = (uint32_t)(a.offsets[x + 1] - begin);
            }
            s_path[threadIdx.x][t] = x;
        }
    }
    __syncthreads();
    // The workgroup's walks cover the samples t_lo .. t_hi - 1 of the pool; the workgroup writes them together, a
    // thread per sample, in the order of their places in the pool, so that neighbouring threads write
    // neighbouring pairs (one thread writing its own walk's 190 pairs scatters 8-byte stores over the pool).
    const uint32_t here = (uint32_t)min((uint64_t)kWalks, a.walks - w0);
    const uint64_t t_lo = w0 * a.per_walk;
    const uint64_t t_hi = min(t_lo + (uint64_t)here * a.per_walk, a.count);
    if (t_lo >= t_hi) return;
    const uint32_t per_walk = (uint32_t)a.per_walk, span = (uint32_t)(t_hi - t_lo);
    // t_rel / per_walk by a multiplication: exact, as t_rel * per_walk is below 2^32 (128 walks of at most 2080 pairs)
    const uint32_t inverse = (uint32_t)(0xFFFFFFFFu / per_walk) + 1u;
    auto emit = [&](uint32_t t_rel, uint64_t place) {  // sample t_lo + t_rel goes to pairs[place]
        const uint32_t walk = per_walk > 1u ? __umulhi(t_rel, inverse) : t_rel, pair = s_pair[t_rel - walk * per_walk];
        a.pairs[place] = make_uint2(s_path[walk][pair >> 8], s_path[walk][pair & 0xFFu]);
    };
    if (!a.pseudo_shuffle) {
        for (uint32_t t_rel = threadIdx.x; t_rel < span; t_rel += kThreads) emit(t_rel, t_lo + t_rel);
    } else if (s > span) {
        for (uint32_t t_rel = threadIdx.x; t_rel < span; t_rel += kThreads)
            emit(t_rel, place_of(t_lo + t_rel, s, a.count, true));
    } else {
        // block after block: within block b the workgroup's samples are b + q s for consecutive q
        const uint64_t q_lo = t_lo / s, whole = a.count / s, extra = a.count % s;
        const uint32_t steps = (uint32_t)((t_hi - 1) / s - q_lo) + 1u, skip = (uint32_t)(t_lo - q_lo * s);  // skip < s
        for (uint32_t b = 0; b < s; ++b) {
            const uint64_t first = b * whole + (b < extra ? b : extra) + q_lo;
#pragma unroll 4
            for (uint32_t q = threadIdx.x; q < steps; q += kThreads) {
                const uint32_t t_rel = q * s + b - skip;  // wraps below t_lo, and is past the end there as well
                if (t_rel < span) emit(t_rel, first + q);
            }
        }
    }
}

#endif  // !GV_TRACK_LOSS

// A row that fills its lanes exactly (d = 64, 128, 256, 512) takes the kernels without per-lane bounds tests.
template <int kV, int kK, bool kFull, bool kTrack>
hipError_t launch_hogwild_vkft(const TrainArgs &a, uint32_t coherence, uint32_t blocks, hipStream_t stream) {
    switch (coherence) {
        case kAgent:
            hipLaunchKernelGGL((k_train_hogwild<kV, kK, kAgent, kFull, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
            break;
        case kAtomicAgent:
        case kMixed:  // the per-row choice exists in the tiled kernel only
            hipLaunchKernelGGL((k_train_hogwild<kV, kK, kAtomicAgent, kFull, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
            break;
        default:
            hipLaunchKernelGGL((k_train_hogwild<kV, kK, kPlain, kFull, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
    }
    return hipGetLastError();
}

// the kernels that also sum the running loss are separate instantiations (in an object of their own): the ones
// that do not carry none of it
template <int kV, int kK, bool kFull>
hipError_t launch_hogwild_vkf(const TrainArgs &a, uint32_t coherence, uint32_t blocks, hipStream_t stream) {
    if ((a.loss_slots != nullptr) != (GV_TRACK_LOSS != 0)) return hipErrorInvalidValue;
    return launch_hogwild_vkft<kV, kK, kFull, GV_TRACK_LOSS != 0>(a, coherence, blocks, stream);
}

template <int kV, int kK>
hipError_t launch_hogwild_vk(const TrainArgs &a, uint32_t coherence, hipStream_t stream) {
    if (a.count == 0) return hipSuccess;
    if (a.unit == 0 || a.unit > (uint32_t)kWave || a.blocks == 0) return hipErrorInvalidValue;
    return a.dim == (uint32_t)(kWave * kV) ? launch_hogwild_vkf<kV, kK, true>(a, coherence, a.blocks, stream)
                                           : launch_hogwild_vkf<kV, kK, false>(a, coherence, a.blocks, stream);
}

template <int kV, int kK, bool kFull, bool kTrack>
hipError_t launch_tiled_vkft(const TrainArgs &a, uint32_t coherence, uint32_t blocks, hipStream_t stream) {
    constexpr int tile = (int)kLargestTile;
    if (a.unit != kLargestTile) {  // smaller tiles come with atomic adds for all rows, or with the mixed policy on short ones
        if (coherence == kAtomicAgent) {
            hipLaunchKernelGGL((k_train_tiled<kV, kK, kAtomicAgent, 0, kFull, kTrack>), dim3(blocks), dim3(kBlock),
                               a.unit * sizeof(uint32_t), stream, a);
            return hipGetLastError();
        }
        if constexpr (short_rows(kV, kK)) {
            if (coherence == kMixed) {
                hipLaunchKernelGGL((k_train_tiled<kV, kK, kMixed, 0, kFull, kTrack>), dim3(blocks), dim3(kBlock),
                                   a.unit * sizeof(uint32_t), stream, a);
                return hipGetLastError();
            }
        }
        return hipErrorInvalidValue;
    }
    if (coherence == kAgent) {
        hipLaunchKernelGGL((k_train_tiled<kV, kK, kAgent, tile, kFull, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
    } else if (coherence == kMixed) {
        hipLaunchKernelGGL((k_train_tiled<kV, kK, kMixed, tile, kFull, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
    } else {
        hipLaunchKernelGGL((k_train_tiled<kV, kK, kAtomicAgent, tile, kFull, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
    }
    return hipGetLastError();
}

template <int kV, int kK, bool kFull>
hipError_t launch_tiled_vkf(const TrainArgs &a, uint32_t coherence, uint32_t blocks, hipStream_t stream) {
    if ((a.loss_slots != nullptr) != (GV_TRACK_LOSS != 0)) return hipErrorInvalidValue;
    return launch_tiled_vkft<kV, kK, kFull, GV_TRACK_LOSS != 0>(a, coherence, blocks, stream);
}

template <int kV, int kK>
hipError_t launch_tiled_vk(const TrainArgs &a, uint32_t coherence, hipStream_t stream) {
    if (a.count == 0) return hipSuccess;
    if (a.rank == nullptr || a.records == nullptr || a.blocks == 0) return hipErrorInvalidValue;
    if (a.unit < kSmallestTile || a.unit > kLargestTile || (a.unit & (a.unit - 1u)) || a.exchange_every == 0)
        return hipErrorInvalidValue;
    return a.dim == (uint32_t)(kWave * kV) ? launch_tiled_vkf<kV, kK, true>(a, coherence, a.blocks, stream)
                                           : launch_tiled_vkf<kV, kK, false>(a, coherence, a.blocks, stream);
}

template <int kV, int kK>
hipError_t launch_levels_vk(const TrainArgs &a, hipStream_t stream) {
    if (a.count == 0) return hipSuccess;
    if ((a.loss_slots != nullptr) != (GV_TRACK_LOSS != 0) || a.records == nullptr) return hipErrorInvalidValue;
    constexpr bool kTrack = GV_TRACK_LOSS != 0;
    const bool full = a.dim == (uint32_t)(kWave * kV);
    if (a.levels > 0) {
        if (full)
            hipLaunchKernelGGL((k_train_levels<kV, kK, true, kTrack>), dim3(1), dim3(kLevelBlock), 0, stream, a);
        else
            hipLaunchKernelGGL((k_train_levels<kV, kK, false, kTrack>), dim3(1), dim3(kLevelBlock), 0, stream, a);
        return hipGetLastError();
    }
    const uint32_t blocks = (a.count + (kBlock / kWave) - 1) / (kBlock / kWave);
    if (full)
        hipLaunchKernelGGL((k_train_level<kV, kK, true, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
    else
        hipLaunchKernelGGL((k_train_level<kV, kK, false, kTrack>), dim3(blocks), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
}

template <int kV, int kK>
hipError_t launch_flow_vk(const FlowArgs &a, hipStream_t stream) {
    if (a.count == 0) return hipSuccess;
    if ((a.loss_slots != nullptr) != (GV_TRACK_LOSS != 0) || a.unit == 0 || a.unit > (uint32_t)kWave || a.blocks == 0)
        return hipErrorInvalidValue;
    constexpr bool kTrack = GV_TRACK_LOSS != 0;
    if (a.dim == (uint32_t)(kWave * kV))
        hipLaunchKernelGGL((k_train_flow<kV, kK, true, kTrack>), dim3(a.blocks), dim3(kFlowBlock), 0, stream, a);
    else
        hipLaunchKernelGGL((k_train_flow<kV, kK, false, kTrack>), dim3(a.blocks), dim3(kFlowBlock), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

#define GV_DISPATCH_K(V, CALL)                 \
    switch (num_neg) {                         \
        case 1: return CALL(V, 1);             \
        case 2: return CALL(V, 2);             \
        case 3: return CALL(V, 3);             \
        case 4: return CALL(V, 4);             \
        case 5: return CALL(V, 5);             \
        default: return hipErrorInvalidValue;  \
    }
// a lane holds V floats of a row: the smallest V in {1, 2, 4, 8} with 64 V >= dim
#define GV_DISPATCH(CALL)                                                   \
    if (!supported_shape(dim, num_neg) || a.dim != dim) return hipErrorInvalidValue; \
    if (dim <= 64) { GV_DISPATCH_K(1, CALL) }                               \
    if (dim <= 128) { GV_DISPATCH_K(2, CALL) }                              \
    if (dim <= 256) { GV_DISPATCH_K(4, CALL) }                              \
    GV_DISPATCH_K(8, CALL)

hipError_t GV_TRAIN_NAME(launch_train_hogwild)(const TrainArgs &a, uint32_t dim, uint32_t num_neg, uint32_t coherence,
                                               hipStream_t stream) {
#define GV_CALL(V, K) launch_hogwild_vk<V, K>(a, coherence, stream)
    GV_DISPATCH(GV_CALL)
#undef GV_CALL
}

hipError_t GV_TRAIN_NAME(launch_train_tiled)(const TrainArgs &a, uint32_t dim, uint32_t num_neg, uint32_t coherence,
                                             hipStream_t stream) {
#define GV_CALL(V, K) launch_tiled_vk<V, K>(a, coherence, stream)
    GV_DISPATCH(GV_CALL)
#undef GV_CALL
}

hipError_t GV_TRAIN_NAME(launch_train_levels)(const TrainArgs &a, uint32_t dim, uint32_t num_neg, hipStream_t stream) {
#define GV_CALL(V, K) launch_levels_vk<V, K>(a, stream)
    GV_DISPATCH(GV_CALL)
#undef GV_CALL
}

hipError_t GV_TRAIN_NAME(launch_train_flow)(FlowArgs a, uint32_t dim, uint32_t num_neg, hipStream_t stream) {
    a.unit = 8;
    const uint32_t per_block = a.unit * (kFlowBlock / kWave);
    a.blocks = std::min((a.count + per_block - 1) / per_block, 128u);
#define GV_CALL(V, K) launch_flow_vk<V, K>(a, stream)
    GV_DISPATCH(GV_CALL)
#undef GV_CALL
}

#if !GV_TRACK_LOSS
template <int kV, int kK>
hipError_t launch_eval_vk(const TrainArgs &a, double *partial, hipStream_t stream) {
    if (a.count == 0 || a.blocks == 0 || a.unit == 0 || a.unit > (uint32_t)kWave) return hipErrorInvalidValue;
    if (a.dim == (uint32_t)(kWave * kV))
        hipLaunchKernelGGL((k_eval_loss<kV, kK, true>), dim3(a.blocks), dim3(kBlock), 0, stream, a, partial);
    else
        hipLaunchKernelGGL((k_eval_loss<kV, kK, false>), dim3(a.blocks), dim3(kBlock), 0, stream, a, partial);
    return hipGetLastError();
}

hipError_t launch_eval_loss(TrainArgs a, uint32_t dim, uint32_t num_neg, double *partial, uint32_t *blocks, hipStream_t stream) {
    // Chunks of 64 samples, or of fewer (down to 4) as long as that brings more waves to work: 2048, for the pairs lie in host
    // memory, where reads of 64 bytes are slow (50000 samples, d = 128, K = 5: 65 us, with 8192 waves 73), and 8192 of the
    // larger pieces, which read 256 bytes a wave then (2^20 samples in pieces of 2^18: 428 us, with 2048 waves 471).
    auto chunks = [&](uint32_t unit) { return (uint32_t)(((uint64_t)a.count + unit - 1) / unit); };
    const uint32_t waves = a.count > 1u << 17 ? 8192u : kWavesOnHostPairs;
    a.unit = kWave;
    while (a.unit > 4u && chunks(a.unit) < waves) a.unit /= 2u;
    a.blocks = *blocks = std::min((chunks(a.unit) + kBlock / kWave - 1u) / (kBlock / kWave), kEvalBlocks);
#define GV_CALL(V, K) launch_eval_vk<V, K>(a, partial, stream)
    GV_DISPATCH(GV_CALL)
#undef GV_CALL
}

template <int kV>
void launch_cosine_v(const float *vertex, uint32_t n, uint32_t dim, const uint32_t *first, const uint32_t *second, uint32_t count,
                     uint32_t unit, uint32_t blocks, float *out, uint32_t *error_flag, hipStream_t stream) {
    if (dim == (uint32_t)(kWave * kV))
        hipLaunchKernelGGL((k_cosine<kV, true>), dim3(blocks), dim3(kBlock), 0, stream, vertex, n, dim, first, second, count, unit, out,
                           error_flag);
    else
        hipLaunchKernelGGL((k_cosine<kV, false>), dim3(blocks), dim3(kBlock), 0, stream, vertex, n, dim, first, second, count, unit, out,
                           error_flag);
}
hipError_t launch_cosine(const float *vertex, uint32_t n, uint32_t dim, const uint32_t *first, const uint32_t *second,
                         uint32_t count, uint32_t waves, float *out, uint32_t *error_flag, hipStream_t stream) {
    if (count == 0) return hipSuccess;
    // as in launch_eval_loss; pairs on the device are read as well in short pieces (gv_cosine of 3*10^5 pairs, d = 512: 400 us
    // with 8192 waves, 411 with 2048)
    auto chunks = [&](uint32_t unit) { return (uint32_t)(((uint64_t)count + unit - 1) / unit); };
    uint32_t unit = kWave;
    while (unit > 4u && chunks(unit) < waves) unit /= 2u;
    const uint32_t blocks = std::min((chunks(unit) + kBlock / kWave - 1u) / (kBlock / kWave), 4096u);
    if (dim <= 64)
        launch_cosine_v<1>(vertex, n, dim, first, second, count, unit, blocks, out, error_flag, stream);
    else if (dim <= 128)
        launch_cosine_v<2>(vertex, n, dim, first, second, count, unit, blocks, out, error_flag, stream);
    else if (dim <= 256)
        launch_cosine_v<4>(vertex, n, dim, first, second, count, unit, blocks, out, error_flag, stream);
    else
        launch_cosine_v<8>(vertex, n, dim, first, second, count, unit, blocks, out, error_flag, stream);
    return hipGetLastError();
}

// Segments of whole sub-tiles of 1024 keys: one, more where that would be over 1024 workgroups.
static uint32_t sort_segment(uint32_t count) {
    const uint32_t tiles = (uint32_t)(((uint64_t)count + kSortBlock - 1u) / kSortBlock);
    return (tiles + 1023u) / 1024u * kSortBlock;
}
static uint32_t sort_blocks(uint32_t count) { return (uint32_t)(((uint64_t)count + sort_segment(count) - 1u) / sort_segment(count)); }
// counts and places of a pass
static uint64_t sort_count_words(uint32_t count) { return 2ull * kDigits * sort_blocks(count); }
// Every workgroup reads the counts of all of them: a megabyte each and more from 1024 on (10^6 against 10^6 pairs 850 us, 908 with
// own places; 500000, 489 workgroups, 453 and 462; 256 workgroups and fewer are faster that way).
constexpr uint32_t kOwnPlacesBlocks = 256;
// One pass over `from`, and the words that go along if `words_out` is given; counts at a multiple of 16 bytes.
template <bool kScores>
static void sort_pass(const uint32_t *from, const uint32_t *words, uint32_t count, uint32_t shift, uint32_t *counts, uint32_t *to,
                      uint32_t *words_out, unsigned long long *not_finite, hipStream_t stream) {
    const uint32_t segment = sort_segment(count), blocks = sort_blocks(count), entries = kDigits * blocks;
    uint32_t *const places = counts + entries;
    const bool own = blocks <= kOwnPlacesBlocks;
    hipLaunchKernelGGL(k_radix_count<kScores>, dim3(blocks), dim3(kSortBlock), 0, stream, from, count, segment, shift, own, counts,
                       not_finite);
    if (!own)
        hipLaunchKernelGGL(k_radix_places, dim3((entries + 4u * kSortBlock - 1u) / (4u * kSortBlock)), dim3(kSortBlock), 0, stream,
                           counts, entries, places);
    const auto scatter = words_out ? (own ? k_radix_scatter<true, kScores, true> : k_radix_scatter<true, kScores, false>)
                                   : (own ? k_radix_scatter<false, kScores, true> : k_radix_scatter<false, kScores, false>);
    hipLaunchKernelGGL(scatter, dim3(blocks), dim3(kSortBlock), 0, stream, from, words, count, segment, shift, own ? counts : places, to,
                       words_out);
}

static uint64_t rank_counts_at(uint32_t num_neg) { return ((uint64_t)num_neg + 3u) & ~3ull; }  // behind the keys, for 16-byte reads
uint64_t rank_scratch_words(uint32_t num_neg) { return rank_counts_at(num_neg) + sort_count_words(num_neg); }

hipError_t launch_rank_sort(uint32_t *negatives, uint32_t num_neg, uint32_t *scratch, unsigned long long *not_finite, hipStream_t stream) {
    if (num_neg == 0) return hipErrorInvalidValue;
    uint32_t *const counts = scratch + rank_counts_at(num_neg);
    // four passes: the keys end where the scores were
    sort_pass<true>(negatives, nullptr, num_neg, 0u, counts, scratch, nullptr, not_finite, stream);
    sort_pass<false>(scratch, nullptr, num_neg, 8u, counts, negatives, nullptr, nullptr, stream);
    sort_pass<false>(negatives, nullptr, num_neg, 16u, counts, scratch, nullptr, nullptr, stream);
    sort_pass<false>(scratch, nullptr, num_neg, 24u, counts, negatives, nullptr, nullptr, stream);
    return hipGetLastError();
}
hipError_t launch_rank_sum(const uint32_t *scores, uint32_t num_pos, uint32_t num_neg, unsigned long long *twice,
                           unsigned long long *not_finite, hipStream_t stream) {
    if (num_pos == 0 || num_neg == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rank_sum, dim3(kRankBlocks), dim3(kSortBlock), 0, stream, scores, (uint64_t)num_pos, scores + num_pos, num_neg,
                       twice, not_finite);
    return hipGetLastError();
}

// Keys, the sorted keys with their namings (twice, for the passes of the sort), the places and the counts of the sort.
uint64_t flow_scratch_words(uint32_t count, uint32_t num_neg) {
    const uint64_t namings = (uint64_t)count * (num_neg + 2);
    return 6 * ((namings + 3u) & ~3ull) + sort_count_words((uint32_t)namings);
}

hipError_t launch_flow_check(const TrainArgs &pool, uint64_t count, uint32_t num_neg, FlowState *state, bool fresh, uint32_t *named,
                             hipStream_t stream) {
    hipLaunchKernelGGL(k_flow_begin, dim3(1), dim3(kWave), 0, stream, state, true, fresh);
    const uint64_t wanted = (count + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_flow_check, dim3((uint32_t)std::min<uint64_t>(wanted, 4096u)), dim3(kBlock), 0, stream, (const uint2 *)pool.pairs,
                       count, pool.alias, pool.n, pool.seed, pool.first_g, num_neg, state, named);
    return hipGetLastError();
}

hipError_t launch_flow_prepare(FlowArgs &a, uint32_t num_neg, uint32_t *scratch, uint64_t *turns, hipStream_t stream) {
    if (a.count == 0 || a.n > 0x80000000u) return hipErrorInvalidValue;
    const uint32_t namings = a.count * (num_neg + 2);
    const uint64_t stride = ((uint64_t)namings + 3u) & ~3ull;
    uint32_t *const keys = scratch, *const places = scratch + stride;
    uint32_t *to = scratch + 2 * stride, *other = scratch + 4 * stride, *const counts = scratch + 6 * stride;
    hipLaunchKernelGGL(k_flow_begin, dim3(1), dim3(kWave), 0, stream, a.flow, false, false);
    const uint32_t by_sample = std::min((a.count + kBlock - 1u) / kBlock, 65536u);
    hipLaunchKernelGGL(k_flow_keys, dim3(by_sample), dim3(kBlock), 0, stream, (const uint2 *)a.pairs, a.alias, a.n, a.seed, a.first_g,
                       a.count, num_neg, keys);
    const uint32_t *from = keys, *words = nullptr;
    for (uint32_t shift = 0; (2ull * a.n - 1u) >> shift; shift += 8u) {
        sort_pass<false>(from, words, namings, shift, counts, to, to + stride, nullptr, stream);
        from = to;
        words = to + stride;
        std::swap(to, other);
    }
    hipLaunchKernelGGL(k_flow_places, dim3(std::min((namings + kBlock - 1u) / kBlock, 65536u)), dim3(kBlock), 0, stream, from, words,
                       namings, places, turns, a.flow);
    a.sorted = from;
    a.namings = words;
    a.keys = keys;
    a.places = places;
    a.turns = turns;
    return hipGetLastError();
}

hipError_t launch_draw_negatives(const uint4 *alias, uint32_t n, uint64_t seed, uint64_t first_g, uint64_t count,
                                 uint32_t num_neg, uint32_t *out, hipStream_t stream) {
    const uint64_t total = count * num_neg;
    if (total == 0) return hipSuccess;
    const uint64_t wanted = (total + kBlock - 1) / kBlock;
    const uint32_t blocks = (uint32_t)(wanted < 65536 ? wanted : 65536);
    hipLaunchKernelGGL(k_draw_negatives, dim3(blocks), dim3(kBlock), 0, stream, alias, n, seed, first_g, count,
                       num_neg, out);
    return hipGetLastError();
}

hipError_t launch_level_records(const uint32_t *pairs, const uint32_t *negatives, const uint32_t *order, uint32_t count,
                                uint32_t num_neg, uint32_t *records, hipStream_t stream) {
    if (count == 0) return hipSuccess;
    const uint32_t wanted = (uint32_t)(((uint64_t)count + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_level_records, dim3(std::min(wanted, 65536u)), dim3(kBlock), 0, stream, (const uint2 *)pairs,
                       negatives, order, count, num_neg, records);
    return hipGetLastError();
}

hipError_t launch_draw_negatives_partitioned(const uint4 *tables, const uint64_t *offsets, const uint8_t *part,
                                             const uint32_t *v, uint64_t seed, uint64_t first_g, uint64_t count,
                                             uint32_t num_neg, uint32_t *out, hipStream_t stream) {
    const uint64_t total = count * num_neg;
    if (total == 0) return hipSuccess;
    const uint64_t wanted = (total + kBlock - 1) / kBlock;
    const uint32_t blocks = (uint32_t)(wanted < 65536 ? wanted : 65536);
    hipLaunchKernelGGL(k_draw_negatives_partitioned, dim3(blocks), dim3(kBlock), 0, stream, tables, offsets, part, v, seed,
                       first_g, count, num_neg, out);
    return hipGetLastError();
}

hipError_t launch_init_vertex(float *vertex, uint64_t rows, uint32_t dim, uint64_t seed, hipStream_t stream) {
    const uint64_t total = rows * (dim / 4);
    if (total == 0) return hipSuccess;
    const uint64_t wanted = (total + kBlock - 1) / kBlock;
    const uint32_t blocks = (uint32_t)(wanted < 65536 ? wanted : 65536);
    hipLaunchKernelGGL(k_init_vertex, dim3(blocks), dim3(kBlock), 0, stream, vertex, rows, dim, seed);
    return hipGetLastError();
}

hipError_t launch_pack_steps(const uint64_t *offsets, const uint32_t *adj, uint64_t half_edges, uint4 *steps, hipStream_t stream) {
    if (half_edges == 0) return hipSuccess;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((half_edges + kBlock - 1) / kBlock, 65536u);
    hipLaunchKernelGGL(k_pack_steps, dim3(blocks), dim3(kBlock), 0, stream, offsets, adj, half_edges, steps);
    return hipGetLastError();
}

hipError_t launch_pack_weighted_steps(const uint64_t *offsets, const uint32_t *adj, const uint2 *nbr_table, uint32_t n,
                                      uint4 *steps, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint32_t blocks = std::min((n + kBlock / kWave - 1u) / (kBlock / kWave), 65536u);
    hipLaunchKernelGGL(k_pack_weighted_steps, dim3(blocks), dim3(kBlock), 0, stream, offsets, adj, nbr_table, n, steps);
    return hipGetLastError();
}

uint32_t guide_shift(uint64_t half_edges) {
    uint32_t shift = 0;
    while ((half_edges >> shift) >= 65536u) ++shift;
    return shift;
}

hipError_t launch_departure_guide(const uint64_t *offsets, uint32_t n, uint64_t half_edges, uint32_t *owners, hipStream_t stream) {
    const uint32_t shift = guide_shift(half_edges), entries = (uint32_t)(half_edges >> shift) + 2u;
    hipLaunchKernelGGL(k_departure_guide, dim3((entries + kBlock - 1) / kBlock), dim3(kBlock), 0, stream, offsets, n, half_edges,
                       shift, entries, owners);
    return hipGetLastError();
}

hipError_t launch_augment(const AugmentArgs &a, hipStream_t stream) {
    if (a.walks == 0) return hipSuccess;
    if (a.length == 0 || a.length > (uint32_t)kMaxWalkLength || a.window == 0) return hipErrorInvalidValue;
    const uint64_t few = a.count >= kShortWalk * a.walks ? kFewWalks : kFewShortWalks;
    const uint64_t of_block = a.walks < few && a.count <= kFewPairs ? 64u : 128u, blocks = (a.walks + of_block - 1) / of_block;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (of_block == 64u)
        hipLaunchKernelGGL((k_augment<64, 256>), dim3((uint32_t)blocks), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((k_augment<128, 128>), dim3((uint32_t)blocks), dim3(128), 0, stream, a);
    return hipGetLastError();
}

#endif  // !GV_TRACK_LOSS

}  // namespace gv
