// cat.hip -- gfx950 kernels of the categorical mask sampler, the
// parameterization the paper compares with (appendix, "Optimization
// Efficiency"): one logit alpha_c per feasible n-hot mask c of a group,
// Pr(c) = softmax(alpha)_c, sampled with Gumbel-Softmax.
//
// One lane per group of m in {4, 8} weights (up to 8 candidates), or the
// candidates of a group over up to three waves (28 to 70); the C = binom(m, n)
// candidate masks are compile-time bitmasks in lexicographic order of their
// index sets.
// Keys kappa_c = alpha_c / lambda + g_c with the noise of element 4 B Q + c
// (B = ceil(C / 4) Philox blocks per group Q).  The hard sample is the
// candidate of largest key (ties to the lower candidate), the relaxed mask
// S_j = sum_c y_c [j in c] with y = softmax(kappa / tau), and the backward is
// the straight-through derivative through that softmax.  As in the item
// sampler: the forward without S decides with the hardware-log keys when the
// top two are further apart than their error margin (else with the exact
// keys); S and the backward use the exact keys.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "host.hpp"
#include "noise.hpp"
#include "relax.hpp"
#include "roi.h"

namespace roi {
namespace {

constexpr int binom(int m, int n)
{
    int r = 1;
    for (int k = 1; k <= n; ++k) r = r * (m - n + k) / k;
    return r;
}

template <int M, int N>
struct Candidates {
    static constexpr int C = binom(M, N);
    uint8_t mask[C];
};

// The n-subsets of {0..m-1} in lexicographic order, as bitmasks.
template <int M, int N>
constexpr Candidates<M, N> make_candidates()
{
    Candidates<M, N> t{};
    int idx[8] = {0, 1, 2, 3, 4, 5, 6, 7};
    for (int c = 0; c < Candidates<M, N>::C; ++c) {
        int mask = 0;
        for (int k = 0; k < N; ++k) mask |= 1 << idx[k];
        t.mask[c] = (uint8_t)mask;
        int k = N - 1;
        while (k >= 0 && idx[k] == M - N + k) --k;
        if (k < 0) break;
        ++idx[k];
        for (int r = k + 1; r < N; ++r) idx[r] = idx[r - 1] + 1;
    }
    return t;
}

template <int M, int N>
constexpr Candidates<M, N> kCand = make_candidates<M, N>();

// Philox words for a 64-bit block index (the block of a candidate need not
// share its high word with the rest of the launch).
__device__ __forceinline__ uint4 philox_block64(uint64_t blk, const NoiseKey& key)
{
    return philox4x32_10((uint32_t)blk, (uint32_t)(blk >> 32), key.step_lo, key.step_hi, key.k0,
                         key.k1);
}

// The C logits of a group (fp32, contiguous, 4C bytes from a 4C-byte stride).
template <int C>
__device__ __forceinline__ void load_cat_logits(const float* p, float (&a)[C])
{
    if constexpr (C % 4 == 0) {
#pragma unroll
        for (int t = 0; t < C / 4; ++t) {
            const f32x4 v = stream_load(reinterpret_cast<const f32x4*>(p) + t);
            a[4 * t] = v.x; a[4 * t + 1] = v.y; a[4 * t + 2] = v.z; a[4 * t + 3] = v.w;
        }
    } else if constexpr (C % 2 == 0) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int t = 0; t < C / 2; ++t) {
            const f32x2 v = stream_load(reinterpret_cast<const f32x2*>(p) + t);
            a[2 * t] = v.x; a[2 * t + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int c = 0; c < C; ++c) a[c] = stream_load(p + c);
    }
}

template <int C>
__device__ __forceinline__ void store_cat(float* p, const float (&a)[C])
{
    if constexpr (C % 4 == 0) {
#pragma unroll
        for (int t = 0; t < C / 4; ++t) {
            const f32x4 v = {a[4 * t], a[4 * t + 1], a[4 * t + 2], a[4 * t + 3]};
            stream_store(v, reinterpret_cast<f32x4*>(p) + t);
        }
    } else if constexpr (C % 2 == 0) {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int t = 0; t < C / 2; ++t) {
            const f32x2 v = {a[2 * t], a[2 * t + 1]};
            stream_store(v, reinterpret_cast<f32x2*>(p) + t);
        }
    } else {
#pragma unroll
        for (int c = 0; c < C; ++c) stream_store(a[c], p + c);
    }
}

// Threads (and groups) per block of the kernels with one lane per group.
constexpr int kCatBlock = 256;
// Groups of 8 logits (32 bytes; the largest that take these kernels) are staged:
// read per lane from global memory, their stride would touch twice the cache
// lines per load instruction of a contiguous 16-byte-per-lane stream.
constexpr bool cat_staged(int C) { return C >= 8; }
// The backward stages 6 candidates (2:4) as well: per lane, its 24-byte
// strides leave every gradient store instruction covering only part of its
// cache lines.  Measured in one session, the backward was 11% faster staged
// and 6-7% faster with only its stores staged; the forward, which reads
// those strides and stores nothing of them, was 23% slower staged.
constexpr bool cat_staged_bwd(int C) { return C >= 6 && C % 2 == 0; }

// Coalesced copies between global memory and a block's LDS tile, in 8-byte
// chunks (every staged C is even, so a group's logits start 8-byte aligned).
typedef float f32x2v __attribute__((ext_vector_type(2)));

template <int B>
__device__ __forceinline__ void tile_in(const float* g, float* lds, int count)
{
    const f32x2v* src = reinterpret_cast<const f32x2v*>(g);
    f32x2v* dst = reinterpret_cast<f32x2v*>(lds);
    for (int i = threadIdx.x; i < count / 2; i += B) dst[i] = stream_load(src + i);
}

template <int B>
__device__ __forceinline__ void tile_out(const float* lds, float* g, int count)
{
    const f32x2v* src = reinterpret_cast<const f32x2v*>(lds);
    f32x2v* dst = reinterpret_cast<f32x2v*>(g);
    for (int i = threadIdx.x; i < count / 2; i += B) stream_store(src[i], dst + i);
}

struct CatArgs {
    const uint16_t* W;
    const float* alpha;
    const uint16_t* G; // backward
    uint16_t* Wm;      // forward
    float* S;
    uint8_t* choice;
    float* dalpha;     // backward
    int64_t ngroups;
    uint64_t group0;   // global index of group 0
    NoiseKey key;      // block_hi unused
    float lambda;
    float div_y;       // 1 / lambda for quotients() (noise.hpp), or 0
    float key_c;       // fl(log2(e) / lambda)
    float inv_lambda;
    float inv_tau;
};

// The exact keys of one group (the words x come from its B Philox blocks).
template <int C>
__device__ __forceinline__ void cat_exact_keys(const float (&alpha)[C], const uint32_t (&x)[C],
                                               float lambda, float div_y, const float2* tab,
                                               float (&k)[C])
{
    // a wave-uniform branch, so that lambda = 1 does not run the division
    if (__builtin_amdgcn_readfirstlane(__float_as_uint(lambda)) == 0x3F800000u) {
#pragma unroll
        for (int c = 0; c < C; ++c) k[c] = alpha[c] - neg_gumbel_from_word(x[c], tab);
    } else {
        quotients<C>(alpha, lambda, div_y, k);
#pragma unroll
        for (int c = 0; c < C; ++c) k[c] -= neg_gumbel_from_word(x[c], tab);
    }
}

template <int C>
__device__ __forceinline__ void cat_words(uint64_t Q, const NoiseKey& key, uint32_t (&x)[C])
{
    constexpr int B = (C + 3) / 4;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const uint4 v = philox_block64(Q * B + b, key);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (4 * b + t < C) x[4 * b + t] = w[t];
    }
}

// y = softmax(kappa * scale) in place (scale turns key differences into log2
// units over tau).
template <int C>
__device__ __forceinline__ void cat_softmax(float (&k)[C], float scale)
{
    float mx = k[0];
#pragma unroll
    for (int c = 1; c < C; ++c) mx = fmaxf(mx, k[c]);
    float t = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        k[c] = __builtin_amdgcn_exp2f((k[c] - mx) * scale);
        t += k[c];
    }
    const float r = __builtin_amdgcn_rcpf(t);
#pragma unroll
    for (int c = 0; c < C; ++c) k[c] *= r;
}

template <int M, int N, bool kSoft>
__global__ __launch_bounds__(kCatBlock) void cat_fwd_kernel(CatArgs a)
{
    constexpr int C = Candidates<M, N>::C;
    constexpr int B = kCatBlock;
    constexpr bool kStage = cat_staged(C);
    // The log cells in LDS only when every group takes the exact keys (kSoft);
    // otherwise they serve groups whose top two keys are close and are read
    // from global memory, where they stay cached.
    __shared__ float2 tab_lds[kSoft ? kLogCells : 1];
    __shared__ float tile[kStage ? B * C : 2];
    const float2* tab = kSoft ? tab_lds : kLogCellTable.cell;
    if constexpr (kSoft) {
        fill_log_table(tab_lds);
        __syncthreads();
    }
    // The loop bound is uniform over the block (the tile copies are cooperative).
    for (int64_t base = (int64_t)blockIdx.x * B; base < a.ngroups; base += (int64_t)gridDim.x * B) {
        const int here = (int)(a.ngroups - base < B ? a.ngroups - base : B);
        const int64_t q = base + threadIdx.x;
        float alpha[C];
        if constexpr (kStage) {
            tile_in<B>(a.alpha + base * C, tile, here * C);
            __syncthreads();
            if ((int)threadIdx.x < here) {
#pragma unroll
                for (int c = 0; c < C; ++c) alpha[c] = tile[threadIdx.x * C + c];
            }
            __syncthreads(); // the tile is refilled next iteration
        }
        if ((int)threadIdx.x >= here) continue;
        if constexpr (!kStage) load_cat_logits<C>(a.alpha + q * C, alpha);
        uint32_t w[M];
        load_bf16<M>(a.W + q * M, w);
        uint32_t x[C];
        cat_words<C>(a.group0 + (uint64_t)q, a.key, x);
        float k[C];
        int best = 0;
        bool exact = true;
        if constexpr (!kSoft) {
            // hardware-log keys; decided when the top two are further apart
            // than the error margin of two keys (noise.hpp)
            // (scanned like the exact argmax: a NaN or infinite key leaves the
            // gap undefined or the margin infinite, so the exact keys decide)
#pragma unroll
            for (int c = 0; c < C; ++c) k[c] = fast_key_log2(alpha[c], a.key_c, x[c]);
            float top = k[0], second = -INFINITY, big = fabsf(k[0]);
#pragma unroll
            for (int c = 1; c < C; ++c) {
                big = fmaxf(big, fabsf(k[c]));
                const bool better = k[c] > top;
                second = better ? top : fmaxf(second, k[c]);
                best = better ? c : best;
                top = better ? k[c] : top;
            }
            const float margin = __builtin_fmaf(big, 0x1p-20f, kFastPairMargin);
            exact = C > 1 && !(top - second > margin);
        }
        if (exact) {
            cat_exact_keys<C>(alpha, x, a.lambda, a.div_y, tab, k);
            float top = k[0];
            best = 0;
#pragma unroll
            for (int c = 1; c < C; ++c) {
                const bool better = k[c] > top; // strict: ties keep the lower candidate
                best = better ? c : best;
                top = better ? k[c] : top;
            }
        }
        {
            uint32_t mask = 0;
#pragma unroll
            for (int c = 0; c < C; ++c) mask = best == c ? kCand<M, N>.mask[c] : mask;
            uint32_t out[M];
#pragma unroll
            for (int j = 0; j < M; ++j) out[j] = ((mask >> j) & 1u) ? w[j] : 0u;
            if constexpr (M == 4) {
                const u32x2 v = {out[0] | (out[1] << 16), out[2] | (out[3] << 16)};
                stream_store(v, reinterpret_cast<u32x2*>(a.Wm + q * M));
            } else {
                const u32x4 v = {out[0] | (out[1] << 16), out[2] | (out[3] << 16),
                                 out[4] | (out[5] << 16), out[6] | (out[7] << 16)};
                stream_store(v, reinterpret_cast<u32x4*>(a.Wm + q * M));
            }
            if (a.choice) stream_store((uint8_t)best, a.choice + q);
        }
        if constexpr (kSoft) {
            cat_softmax<C>(k, kLog2e * a.inv_tau);
            float S[M];
#pragma unroll
            for (int j = 0; j < M; ++j) S[j] = 0.0f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
#pragma unroll
                for (int j = 0; j < M; ++j)
                    if ((kCand<M, N>.mask[c] >> j) & 1) S[j] += k[c];
            }
            if (a.S) store_f32<M>(a.S + q * M, S);
        }
    }
}

// The keys from the logits and the noise ng = -g of a group's candidates,
// kappa = fl(fl(alpha / lambda) + g); lambda = 1 is a wave-uniform branch
// without the division.
template <int C>
__device__ __forceinline__ void cat_keys_from_noise(const float (&alpha)[C], const float (&ng)[C],
                                                    float lambda, float div_y, float (&k)[C])
{
    if (__builtin_amdgcn_readfirstlane(__float_as_uint(lambda)) == 0x3F800000u) {
#pragma unroll
        for (int c = 0; c < C; ++c) k[c] = alpha[c] - ng[c];
    } else {
        quotients<C>(alpha, lambda, div_y, k);
#pragma unroll
        for (int c = 0; c < C; ++c) k[c] -= ng[c];
    }
}

// One chunk of B groups of the categorical backward.  The loads go out first:
// the group's W and dL/dW_masked, its logits (per lane, or for the staged
// tile this thread's share of the block's contiguous logits), and the log
// cells.  The noise -- C Philox words and 2C logarithms per group, most of the
// arithmetic -- needs none of them and runs while they are in flight.  kFull:
// all B groups are inside the array, so no per-lane condition makes the
// compiler wait for every load at a join.
template <int M, int N, bool kFull>
__device__ __forceinline__ void cat_bwd_chunk(const CatArgs& a, float* tile, float2* tab,
                                              int64_t base)
{
    constexpr int C = Candidates<M, N>::C;
    constexpr int B = kCatBlock;
    constexpr bool kStage = cat_staged_bwd(C);
    constexpr int kShare = kStage ? C / 2 : 1; // 8-byte tile pieces per thread
    const int here = kFull ? B : (int)(a.ngroups - base);
    const int64_t q = base + threadIdx.x;
    const bool live = kFull || (int)threadIdx.x < here;
    uint32_t w[M / 2], g[M / 2];
    float alpha[C];
    f32x2v share[kShare];
    if (live) {
        load_bf16_pairs<M>(a.W + q * M, w);
        load_bf16_pairs<M>(a.G + q * M, g);
    }
    if constexpr (kStage) {
        if constexpr (kFull) {
            const f32x2v* src = reinterpret_cast<const f32x2v*>(a.alpha + base * C);
#pragma unroll
            for (int i = 0; i < kShare; ++i) share[i] = stream_load(src + threadIdx.x + i * B);
        }
    } else if (live) {
        load_cat_logits<C>(a.alpha + q * C, alpha);
    }
    const float4 cells = log_cells_of_lane();
    __builtin_amdgcn_sched_barrier(0);
    float ng[C];
    uint32_t x[C];
    cat_words<C>(a.group0 + (uint64_t)q, a.key, x);
    publish_log_table(tab, cells);
#pragma unroll
    for (int c = 0; c < C; ++c) ng[c] = neg_gumbel_from_word(x[c], tab);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kStage) {
        if constexpr (kFull) {
            f32x2v* dst = reinterpret_cast<f32x2v*>(tile);
#pragma unroll
            for (int i = 0; i < kShare; ++i) dst[threadIdx.x + i * B] = share[i];
        } else {
            tile_in<B>(a.alpha + base * C, tile, here * C);
        }
        __syncthreads();
        if (live) {
#pragma unroll
            for (int c = 0; c < C; ++c) alpha[c] = tile[threadIdx.x * C + c];
        }
        __syncthreads(); // the gradients go into the same tile
    }
    float d[C];
    if (live) {
        // the keys the forward sampled, and their softmax
        float y[C];
        cat_keys_from_noise<C>(alpha, ng, a.lambda, a.div_y, y);
        cat_softmax<C>(y, kLog2e * a.inv_tau);
        // Straight-through: dL/dS = dL/dW_masked (.) W; ybar_c = sum_{j in c} sbar_j.
        float sbar[M];
#pragma unroll
        for (int i = 0; i < M / 2; ++i) {
            sbar[2 * i] = bf16_bits_to_float(g[i] & 0xFFFFu) * bf16_bits_to_float(w[i] & 0xFFFFu);
            sbar[2 * i + 1] = bf16_bits_to_float(g[i] >> 16) * bf16_bits_to_float(w[i] >> 16);
        }
        float ybar[C], dot = 0.0f;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < M; ++j)
                if ((kCand<M, N>.mask[c] >> j) & 1) acc += sbar[j];
            ybar[c] = acc;
            dot = __builtin_fmaf(y[c], acc, dot);
        }
        const float s = a.inv_tau * a.inv_lambda;
#pragma unroll
        for (int c = 0; c < C; ++c) d[c] = y[c] * (ybar[c] - dot) * s;
    }
    if constexpr (kStage) {
        if (live) {
#pragma unroll
            for (int c = 0; c < C; ++c) tile[threadIdx.x * C + c] = d[c];
        }
        __syncthreads();
        tile_out<B>(tile, a.dalpha + base * C, here * C);
        __syncthreads(); // before the next chunk overwrites the tile
    } else if (live) {
        store_cat<C>(a.dalpha + q * C, d);
    }
}

template <int M, int N>
__global__ __launch_bounds__(kCatBlock) void cat_bwd_kernel(CatArgs a)
{
    constexpr int C = Candidates<M, N>::C;
    constexpr int B = kCatBlock;
    __shared__ float tile[cat_staged_bwd(C) ? B * C : 2];
    // Every group takes the exact keys; the block's waves share one copy of
    // the log cells in LDS (noise.hpp).
    __shared__ float4 tab4[kLogCells / 2];
    float2* tab = reinterpret_cast<float2*>(tab4);
    // The loop bound and the full / partial choice are uniform over the block
    // (the tile copies are cooperative).
    for (int64_t base = (int64_t)blockIdx.x * B; base < a.ngroups; base += (int64_t)gridDim.x * B) {
        if (base + B <= a.ngroups)
            cat_bwd_chunk<M, N, true>(a, tile, tab, base);
        else
            cat_bwd_chunk<M, N, false>(a, tile, tab, base);
    }
}

// ---- groups with many candidates (C = 28, 56, 70: m = 8, n = 2 .. 6)
//
// One lane per group would hold C noise values, keys and gradients in
// registers and one wave 64 C logits in LDS: two waves per SIMD at 4:8, each
// waiting in turn for its logits, its arithmetic and its stores.  Here the
// candidates of a group are split over kParts waves of a block: lane l of
// wave (row, part) takes the 4 kBlocks candidates of Philox blocks
// part kBlocks .. of group 64 row + l, so that every lane has the same work
// (70 candidates are 18 Philox blocks: three parts of six).  The block's
// logits are one contiguous span, staged through LDS, and the noise -- most of
// the arithmetic, and independent of every input -- is computed while they are
// in flight.
// Group maxima, sums and dot products go through small LDS arrays.
// 1.5B-class layer at 4:8 (5.85e6 groups) on MI355X: forward 924 us with one
// lane per group, 363 us so (284 us at the streaming-copy rate); backward
// 1433 us and 601 us (537 us).
// Waves per SIMD the split kernels are compiled for (at most 128 VGPRs; five
// spill in most of them).
constexpr int kSplitWaves = 4;
// Up to 8 candidates fit one lane's registers beside their noise, and take
// the kernels above; 28 is the next count.
constexpr bool cat_split(int C) { return C >= 28; }
constexpr int cat_parts(int C) { return C > 64 ? 3 : (C > 32 ? 2 : 1); }
// Rows of 64 groups per block.
constexpr int cat_rows(int C) { return C > 64 ? 1 : 2; }

template <int M, int N>
struct CatSplit {
    static constexpr int C = Candidates<M, N>::C;
    static constexpr int kParts = cat_parts(C);
    static constexpr int kRows = cat_rows(C);
    static constexpr int kPhilox = (C + 3) / 4;      // Philox blocks per group
    static constexpr int kBlocks = kPhilox / kParts; // per part
    static constexpr int K = 4 * kBlocks;            // candidates per lane
    static constexpr int kPad = kParts * K - C;      // past the end, in the last part
    static constexpr int kGroups = 64 * kRows;       // groups per block
    static constexpr int kThreads = kGroups * kParts;
    static constexpr int kFloats = kGroups * C;      // logits per block
    // 16-byte vectors per thread, and the tile they fill.
    static constexpr int kShare = (kFloats / 4 + kThreads - 1) / kThreads;
    static constexpr int kTile = kShare * kThreads * 4;
    static_assert(kPhilox % kParts == 0 && C % 2 == 0 && kPad % 2 == 0 && kPad < K, "split");
};

// The logits of a full block (kFloats floats, 16-byte aligned): each thread
// loads its share, 16 bytes at a time, ahead of the noise, and stores it to
// the tile after.  The last loads may lie half beyond the span: they read the
// last vector again, into the tile's padding, so that no load stands under a
// condition (after which the compiler would wait for all of them).  Loads
// that write LDS themselves would need no registers, but the compiler waits
// for them before the next access to LDS, and the noise reads its table there.
template <typename Sp>
__device__ __forceinline__ void load_share(const float* g, f32x4 (&share)[Sp::kShare])
{
    constexpr int kVecs = Sp::kFloats / 4;
#pragma unroll
    for (int i = 0; i < Sp::kShare; ++i) {
        const int v = i * Sp::kThreads + (int)threadIdx.x;
        share[i] = stream_load(reinterpret_cast<const f32x4*>(g) + (v < kVecs ? v : kVecs - 1));
    }
}

template <typename Sp>
__device__ __forceinline__ void store_share(const f32x4 (&share)[Sp::kShare], float* tile)
{
#pragma unroll
    for (int i = 0; i < Sp::kShare; ++i)
        reinterpret_cast<f32x4*>(tile)[i * Sp::kThreads + (int)threadIdx.x] = share[i];
}

// The lane's place: its group's row in the block, and its first candidate.
template <typename Sp>
struct CatLane {
    int part, row, c0;
    __device__ __forceinline__ CatLane()
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        part = wave / Sp::kRows;
        row = (wave % Sp::kRows) * 64 + (int)(threadIdx.x & 63);
        c0 = part * Sp::K;
    }
    // candidate i of the lane exists (known at compile time for most i)
    __device__ __forceinline__ bool has(int i) const
    {
        return i < Sp::K - Sp::kPad || part + 1 < Sp::kParts;
    }
};

// The noise of the lane's candidates: f(word) for each.  One Philox block at
// a time, finished where it is written (pin, and the barrier that keeps the
// compiler from interleaving the blocks), so that the kernel's registers are
// those of the keys, not of the noise in the making.
template <typename Sp, typename F>
__device__ __forceinline__ void split_noise(uint64_t Q, int part, const NoiseKey& key,
                                            float (&v)[Sp::K], F f)
{
    const uint64_t first = Q * Sp::kPhilox + (uint32_t)(part * Sp::kBlocks);
#pragma unroll
    for (int b = 0; b < Sp::kBlocks; ++b) {
        const uint4 x = philox_block64(first + b, key);
        v[4 * b] = f(x.x);
        v[4 * b + 1] = f(x.y);
        v[4 * b + 2] = f(x.z);
        v[4 * b + 3] = f(x.w);
#pragma unroll
        for (int i = 4 * b; i < 4 * b + 4; ++i) pin(v[i]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The lane's logits from the tile (8-byte reads: rows of an odd number of
// 8-byte words at C = 70, so a wave's reads spread over the banks).
template <typename Sp>
__device__ __forceinline__ void split_logits(const float* tile, const CatLane<Sp>& ln,
                                             float (&alpha)[Sp::K])
{
    const f32x2v* p = reinterpret_cast<const f32x2v*>(tile + ln.row * Sp::C + ln.c0);
#pragma unroll
    for (int i = 0; i < Sp::K; i += 2) {
        const f32x2v v = ln.has(i) ? p[i / 2] : f32x2v{0.0f, 0.0f};
        alpha[i] = v.x;
        alpha[i + 1] = v.y;
    }
}

// Exact keys in place, kappa = fl(fl(alpha / lambda) + g), from the noise k =
// -g (lambda = 1 is a wave-uniform branch without the division); entries past
// the end are -inf (below every key, weight 0).
template <typename Sp>
__device__ __forceinline__ void split_keys(const CatLane<Sp>& ln, const float (&alpha)[Sp::K],
                                           float lambda, float div_y, float (&k)[Sp::K])
{
    if (__builtin_amdgcn_readfirstlane(__float_as_uint(lambda)) == 0x3F800000u) {
#pragma unroll
        for (int i = 0; i < Sp::K; ++i) k[i] = alpha[i] - k[i];
    } else {
#pragma unroll
        for (int i = 0; i < Sp::K; i += 4) {
            const float a4[4] = {alpha[i], alpha[i + 1], alpha[i + 2], alpha[i + 3]};
            float q4[4];
            quotients<4>(a4, lambda, div_y, q4);
#pragma unroll
            for (int e = 0; e < 4; ++e) k[i + e] = q4[e] - k[i + e];
            __builtin_amdgcn_sched_barrier(0); // few quotients in the making
        }
    }
#pragma unroll
    for (int i = Sp::K - Sp::kPad; i < Sp::K; ++i) k[i] = ln.has(i) ? k[i] : -INFINITY;
}

// Whether candidate c (none past the last) holds element j.
template <int M, int N>
constexpr bool in_candidate(int c, int j)
{
    return c < Candidates<M, N>::C && ((kCand<M, N>.mask[c] >> j) & 1) != 0;
}

// Calls f with each part's candidate numbers as compile-time constants:
// f(integral_constant<int, c0>) runs for the wave's own part.
template <typename Sp, int P = 0, typename F>
__device__ __forceinline__ void for_part(int part, F&& f)
{
    if constexpr (P + 1 < Sp::kParts) {
        if (part == P)
            f(std::integral_constant<int, P * Sp::K>{});
        else
            for_part<Sp, P + 1>(part, f);
    } else {
        f(std::integral_constant<int, P * Sp::K>{});
    }
}

// Reads the kParts values that the parts of a group stored at x[part][row].
template <typename Sp, typename Op>
__device__ __forceinline__ float over_parts(const float (*x)[Sp::kGroups], int row, Op op)
{
    float v = x[0][row];
#pragma unroll
    for (int p = 1; p < Sp::kParts; ++p) v = op(v, x[p][row]);
    return v;
}

// The expanded masks of the candidates: entry c clears the elements outside
// c's subset from a group's eight bf16 values.
struct alignas(16) Keep8 {
    uint32_t w[4];
};
template <int N>
struct Keep8Table {
    Keep8 e[Candidates<8, N>::C];
};
template <int N>
constexpr Keep8Table<N> make_keep8()
{
    Keep8Table<N> t{};
    for (int c = 0; c < Candidates<8, N>::C; ++c)
        for (int j = 0; j < 8; ++j)
            if ((kCand<8, N>.mask[c] >> j) & 1)
                t.e[c].w[j / 2] |= j % 2 ? 0xFFFF0000u : 0x0000FFFFu;
    return t;
}
template <int N>
__device__ const Keep8Table<N> kKeep8 = make_keep8<N>();

// The candidate of largest key among the parts' (key, candidate) pairs, ties
// to the lower candidate (parts hold ascending candidates).
template <typename Sp>
__device__ __forceinline__ int best_of_parts(const float (*top)[Sp::kGroups],
                                             const int (*best)[Sp::kGroups], int row)
{
    float t = top[0][row];
    int b = best[0][row];
#pragma unroll
    for (int p = 1; p < Sp::kParts; ++p) {
        const bool better = top[p][row] > t;
        b = better ? best[p][row] : b;
        t = better ? top[p][row] : t;
    }
    return b;
}

// The lane's largest key, ties to the lower candidate.  A NaN never wins, as in
// a scan over the group's candidates in order, where only candidate 0 can hold
// the lead with one: a later part that starts with a NaN starts below every key.
template <typename Sp>
__device__ __forceinline__ void lane_argmax(const CatLane<Sp>& ln, const float (&k)[Sp::K],
                                            float& top, int& best)
{
    top = ln.part > 0 && k[0] != k[0] ? -INFINITY : k[0];
    best = 0;
#pragma unroll
    for (int i = 1; i < Sp::K; ++i) {
        const bool better = k[i] > top;
        best = better ? i : best;
        top = better ? k[i] : top;
    }
    best += ln.c0;
}

template <int M, int N, bool kSoft>
struct CatFwdShared {
    using Sp = CatSplit<M, N>;
    alignas(16) float tile[Sp::kTile];
    float4 tab[kLogCells / 2];
    float x_top[Sp::kParts][Sp::kGroups];
    float x_second[kSoft ? 1 : Sp::kParts][Sp::kGroups];
    int x_best[Sp::kParts][Sp::kGroups];
    float x_sum[kSoft ? Sp::kParts : 1][kSoft ? M + 1 : 1][Sp::kGroups];
};

// The forward of kGroups groups from `base` (kFull: all are inside the array).
template <int M, int N, bool kSoft, bool kFull>
__device__ __forceinline__ void cat_fwd_split_tile(const CatArgs& a, CatFwdShared<M, N, kSoft>& sh,
                                                   int64_t base)
{
    using Sp = CatSplit<M, N>;
    constexpr int K = Sp::K;
    const CatLane<Sp> ln;
    const int here = kFull ? Sp::kGroups : (int)(a.ngroups - base);
    const bool live = kFull || ln.row < here;
    const int64_t q = base + ln.row;
    const bool writes = ln.part == 0 && live; // one part stores the group's outputs
    const float4 cells = log_cells_of_lane();
    __builtin_amdgcn_sched_barrier(0);
    uint32_t w[M / 2];
    f32x4 share[Sp::kShare];
    if constexpr (kFull) load_share<Sp>(a.alpha + base * Sp::C, share);
    if (live) load_bf16_pairs<M>(a.W + q * M, w); // by every part: no condition
    float2* tab = reinterpret_cast<float2*>(sh.tab);
    publish_log_table(tab, cells);
    const uint64_t Q = a.group0 + (uint64_t)q;
    const auto exact_noise = [&](uint32_t x) { return neg_gumbel_from_word(x, tab); };
    float k[K]; // the noise, then the keys
    if constexpr (kSoft)
        split_noise<Sp>(Q, ln.part, a.key, k, exact_noise);
    else
        split_noise<Sp>(Q, ln.part, a.key, k, [](uint32_t x) { return fast_noise_log2(x); });
    if constexpr (kFull)
        store_share<Sp>(share, sh.tile);
    else
        tile_in<Sp::kThreads>(a.alpha + base * Sp::C, sh.tile, here * Sp::C);
    __syncthreads();
    float alpha[K];
    split_logits<Sp>(sh.tile, ln, alpha);
    bool exact = true;
    int best = 0;
    if constexpr (!kSoft) {
        // Hardware-log keys: decided when the top two of the group are
        // further apart than the error of two keys (noise.hpp); a lower
        // key's larger |K| widens the margin by less than its distance.
        // The sum tells a NaN, and an infinite key makes the margin so.
        float sum = 0.0f, top = -INFINITY, second = -INFINITY;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (!ln.has(i)) continue;
            const float v = __builtin_fmaf(alpha[i], a.key_c, k[i]);
            sum += v;
            second = __builtin_amdgcn_fmed3f(top, second, v);
            const bool better = v > top;
            best = better ? i : best;
            top = better ? v : top;
        }
        sh.x_top[ln.part][ln.row] = sum == sum ? top : NAN;
        sh.x_second[ln.part][ln.row] = second;
        sh.x_best[ln.part][ln.row] = ln.c0 + best;
        __syncthreads();
        // the same in every part of the group
        best = best_of_parts<Sp>(sh.x_top, sh.x_best, ln.row);
        top = -INFINITY;
        second = -INFINITY;
        float nan = 0.0f;
#pragma unroll
        for (int p = 0; p < Sp::kParts; ++p) {
            const float t = sh.x_top[p][ln.row], s = sh.x_second[p][ln.row];
            nan += t;
            second = fmaxf(fmaxf(second, s), fminf(top, t));
            top = fmaxf(top, t);
        }
        const float margin = __builtin_fmaf(fmaxf(fabsf(top), fabsf(second)), 0x1p-20f,
                                            kFastPairMargin);
        exact = nan != nan || !(top - second > margin);
        exact = __syncthreads_or(live && exact) != 0;
    }
    if (exact) { // uniform over the block
        if constexpr (!kSoft) { // rare: words and logits anew, not held in registers
            uint64_t again = Q;
            asm volatile("" : "+v"(again));
            split_noise<Sp>(again, ln.part, a.key, k, exact_noise);
            split_logits<Sp>(sh.tile, ln, alpha);
        }
        split_keys<Sp>(ln, alpha, a.lambda, a.div_y, k);
        float top;
        lane_argmax<Sp>(ln, k, top, best);
        sh.x_top[ln.part][ln.row] = top;
        sh.x_best[ln.part][ln.row] = best;
        __syncthreads();
        best = best_of_parts<Sp>(sh.x_top, sh.x_best, ln.row);
    }
    if (writes) {
        const Keep8 keep = kKeep8<N>.e[best];
        const u32x4 v = {w[0] & keep.w[0], w[1] & keep.w[1], w[2] & keep.w[2],
                         w[3] & keep.w[3]};
        stream_store(v, reinterpret_cast<u32x4*>(a.Wm + q * M));
        if (a.choice) stream_store((uint8_t)best, a.choice + q);
    }
    if constexpr (kSoft) {
        const auto larger = [](float u, float v) { return fmaxf(u, v); };
        const float mx = over_parts<Sp>(sh.x_top, ln.row, larger);
        const float scale = kLog2e * a.inv_tau;
        float t = 0.0f, S[M];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            k[i] = __builtin_amdgcn_exp2f((k[i] - mx) * scale);
            t += k[i];
        }
        for_part<Sp>(ln.part, [&](auto c0) {
#pragma unroll
            for (int j = 0; j < M; ++j) S[j] = 0.0f;
#pragma unroll
            for (int i = 0; i < K; ++i) {
#pragma unroll
                for (int j = 0; j < M; ++j)
                    if (in_candidate<M, N>(c0 + i, j))
                        S[j] += k[i];
            }
        });
#pragma unroll
        for (int j = 0; j < M; ++j) sh.x_sum[ln.part][j][ln.row] = S[j];
        sh.x_sum[ln.part][M][ln.row] = t;
        __syncthreads();
        if (writes && a.S) {
            float total = 0.0f;
#pragma unroll
            for (int j = 0; j < M; ++j) S[j] = 0.0f;
#pragma unroll
            for (int p = 0; p < Sp::kParts; ++p) {
                total += sh.x_sum[p][M][ln.row];
#pragma unroll
                for (int j = 0; j < M; ++j) S[j] += sh.x_sum[p][j][ln.row];
            }
            const float r = __builtin_amdgcn_rcpf(total);
#pragma unroll
            for (int j = 0; j < M; ++j) S[j] *= r;
            store_f32<M>(a.S + q * M, S);
        }
    }
    __syncthreads(); // the tile and the exchange arrays are used again
}

template <int M, int N, bool kSoft>
__global__ __launch_bounds__((CatSplit<M, N>::kThreads), kSplitWaves) void cat_fwd_split_kernel(
    CatArgs a)
{
    constexpr int G = CatSplit<M, N>::kGroups;
    __shared__ CatFwdShared<M, N, kSoft> sh;
    for (int64_t base = (int64_t)blockIdx.x * G; base < a.ngroups; base += (int64_t)gridDim.x * G) {
        if (base + G <= a.ngroups) // uniform over the block
            cat_fwd_split_tile<M, N, kSoft, true>(a, sh, base);
        else
            cat_fwd_split_tile<M, N, kSoft, false>(a, sh, base);
    }
}

template <int M, int N>
struct CatBwdShared {
    using Sp = CatSplit<M, N>;
    alignas(16) float tile[Sp::kTile];
    float4 tab[kLogCells / 2];
    float x_top[Sp::kParts][Sp::kGroups];
    float x_sum[Sp::kParts][Sp::kGroups];
    float x_dot[Sp::kParts][Sp::kGroups];
};

// The backward of kGroups groups from `base` (kFull: all are inside the array).
template <int M, int N, bool kFull>
__device__ __forceinline__ void cat_bwd_split_tile(const CatArgs& a, CatBwdShared<M, N>& sh,
                                                   int64_t base)
{
    using Sp = CatSplit<M, N>;
    constexpr int K = Sp::K;
    const CatLane<Sp> ln;
    const int here = kFull ? Sp::kGroups : (int)(a.ngroups - base);
    const bool live = kFull || ln.row < here;
    const int64_t q = base + ln.row;
    const float4 cells = log_cells_of_lane();
    __builtin_amdgcn_sched_barrier(0);
    uint32_t w[M / 2] = {}, g[M / 2] = {};
    f32x4 share[Sp::kShare];
    if constexpr (kFull) load_share<Sp>(a.alpha + base * Sp::C, share);
    if (live) { // every part of a group reads them; all but one hit the cache
        load_bf16_pairs<M>(a.W + q * M, w);
        load_bf16_pairs<M>(a.G + q * M, g);
    }
    float k[K]; // -g, then the keys, then the weights
    {
        float2* tab = reinterpret_cast<float2*>(sh.tab);
        publish_log_table(tab, cells);
        split_noise<Sp>(a.group0 + (uint64_t)q, ln.part, a.key, k,
                        [&](uint32_t x) { return neg_gumbel_from_word(x, tab); });
    }
    if constexpr (kFull)
        store_share<Sp>(share, sh.tile);
    else
        tile_in<Sp::kThreads>(a.alpha + base * Sp::C, sh.tile, here * Sp::C);
    __syncthreads();
    {
        float alpha[K];
        split_logits<Sp>(sh.tile, ln, alpha);
        split_keys<Sp>(ln, alpha, a.lambda, a.div_y, k);
    }
    float mx = k[0];
#pragma unroll
    for (int i = 1; i < K; ++i) mx = fmaxf(mx, k[i]);
    sh.x_top[ln.part][ln.row] = mx;
    if constexpr (Sp::kParts > 1) __syncthreads();
    mx = over_parts<Sp>(sh.x_top, ln.row, [](float u, float v) { return fmaxf(u, v); });
    // Straight-through: dL/dS = dL/dW_masked (.) W; ybar_c = sum_{j in c} sbar_j.
    float sbar[M];
#pragma unroll
    for (int i = 0; i < M / 2; ++i) {
        sbar[2 * i] = bf16_bits_to_float(g[i] & 0xFFFFu) * bf16_bits_to_float(w[i] & 0xFFFFu);
        sbar[2 * i + 1] = bf16_bits_to_float(g[i] >> 16) * bf16_bits_to_float(w[i] >> 16);
    }
    const float scale = kLog2e * a.inv_tau;
    float t = 0.0f, dot = 0.0f, ybar[K];
    for_part<Sp>(ln.part, [&](auto c0) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < M; ++j)
                if (in_candidate<M, N>(c0 + i, j))
                    acc += sbar[j];
            ybar[i] = acc;
        }
    });
#pragma unroll
    for (int i = 0; i < K; ++i) {
        k[i] = __builtin_amdgcn_exp2f((k[i] - mx) * scale);
        t += k[i];
        dot = __builtin_fmaf(k[i], ybar[i], dot);
    }
    sh.x_sum[ln.part][ln.row] = t;
    sh.x_dot[ln.part][ln.row] = dot;
    if constexpr (Sp::kParts > 1) __syncthreads();
    const auto add = [](float u, float v) { return u + v; };
    const float r = __builtin_amdgcn_rcpf(over_parts<Sp>(sh.x_sum, ln.row, add));
    // ybar - <y, ybar> in two steps, first from the rounded <y, ybar>, then from
    // the mean of what is left: where one candidate dominates, its ybar is
    // close to <y, ybar>, and their difference would keep only the rounding.
    dot = over_parts<Sp>(sh.x_dot, ln.row, add) * r;
    float left = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        ybar[i] -= dot;
        left = __builtin_fmaf(k[i], ybar[i], left);
    }
    sh.x_top[ln.part][ln.row] = left; // every part has read the maxima before the last barrier
    if constexpr (Sp::kParts > 1) __syncthreads();
    left = over_parts<Sp>(sh.x_top, ln.row, add) * r;
    const float s = r * (a.inv_tau * a.inv_lambda);
    f32x2v* out = reinterpret_cast<f32x2v*>(sh.tile + ln.row * Sp::C + ln.c0);
#pragma unroll
    for (int i = 0; i < K; i += 2) {
        if (!ln.has(i)) continue;
        out[i / 2] = f32x2v{(k[i] * s) * (ybar[i] - left), (k[i + 1] * s) * (ybar[i + 1] - left)};
    }
    __syncthreads();
    if constexpr (kFull) {
        const f32x4* src = reinterpret_cast<const f32x4*>(sh.tile);
        f32x4* dst = reinterpret_cast<f32x4*>(a.dalpha + base * Sp::C);
        for (int i = threadIdx.x; i < Sp::kFloats / 4; i += Sp::kThreads)
            stream_store(src[i], dst + i);
    } else {
        tile_out<Sp::kThreads>(sh.tile, a.dalpha + base * Sp::C, here * Sp::C);
    }
    __syncthreads(); // before the next block of groups overwrites the tile
}

template <int M, int N>
__global__ __launch_bounds__((CatSplit<M, N>::kThreads), kSplitWaves) void cat_bwd_split_kernel(
    CatArgs a)
{
    constexpr int G = CatSplit<M, N>::kGroups;
    __shared__ CatBwdShared<M, N> sh;
    for (int64_t base = (int64_t)blockIdx.x * G; base < a.ngroups; base += (int64_t)gridDim.x * G) {
        if (base + G <= a.ngroups) // uniform over the block
            cat_bwd_split_tile<M, N, true>(a, sh, base);
        else
            cat_bwd_split_tile<M, N, false>(a, sh, base);
    }
}

template <int M, int N>
void* pick_cat_fwd(bool soft)
{
    if constexpr (cat_split(Candidates<M, N>::C))
        return soft ? (void*)cat_fwd_split_kernel<M, N, true>
                    : (void*)cat_fwd_split_kernel<M, N, false>;
    else
        return soft ? (void*)cat_fwd_kernel<M, N, true> : (void*)cat_fwd_kernel<M, N, false>;
}

template <int M, int N>
void* pick_cat_bwd()
{
    if constexpr (cat_split(Candidates<M, N>::C))
        return (void*)cat_bwd_split_kernel<M, N>;
    else
        return (void*)cat_bwd_kernel<M, N>;
}

template <int M, int... Ns>
void* cat_fwd_for_n(int n, bool soft, std::integer_sequence<int, Ns...>)
{
    void* f = nullptr;
    ((n == Ns + 1 ? (f = pick_cat_fwd<M, Ns + 1>(soft), 0) : 0), ...);
    return f;
}

template <int M, int... Ns>
void* cat_bwd_for_n(int n, std::integer_sequence<int, Ns...>)
{
    void* f = nullptr;
    ((n == Ns + 1 ? (f = pick_cat_bwd<M, Ns + 1>(), 0) : 0), ...);
    return f;
}

} // namespace
} // namespace roi

using namespace roi;

extern "C" int roi_cat_num_candidates(int n, int m)
{
    if ((m != 4 && m != 8) || n < 1 || n > m) return -1;
    return binom(m, n);
}

namespace roi {
namespace {
int cat_run(bool fwd, const uint16_t* W, const float* alpha, const uint16_t* G, int64_t rows,
            int64_t cols, int n, int m, float tau, float lambda, uint64_t seed, uint64_t step,
            uint64_t group_offset, uint16_t* W_masked, float* S, uint8_t* choice, float* dalpha,
            hipStream_t stream)
{
    const char* what = fwd ? "roi_cat_mask_fwd" : "roi_cat_mask_bwd";
    int64_t ngroups;
    int C;
    if (int st = validate_cat(fwd, W, alpha, G, rows, cols, n, m, tau, lambda, group_offset,
                              W_masked, S, choice, dalpha, &ngroups, &C))
        return st;
    if (ngroups == 0) return ok();
    void* fn = m == 4 ? (fwd ? cat_fwd_for_n<4>(n, S != nullptr, std::make_integer_sequence<int, 4>{})
                             : cat_bwd_for_n<4>(n, std::make_integer_sequence<int, 4>{}))
                      : (fwd ? cat_fwd_for_n<8>(n, S != nullptr, std::make_integer_sequence<int, 8>{})
                             : cat_bwd_for_n<8>(n, std::make_integer_sequence<int, 8>{}));
    if (!fn) return fail(ROI_E_UNSUPPORTED, "no kernel for %d:%d", n, m);
    CatArgs a{};
    a.W = W;
    a.alpha = alpha;
    a.G = G;
    a.Wm = W_masked;
    a.S = S;
    a.choice = choice;
    a.dalpha = dalpha;
    a.ngroups = ngroups;
    a.group0 = group_offset;
    a.key = make_key(seed, step, 0);
    a.lambda = lambda;
    a.div_y = quotient_reciprocal(lambda);
    a.key_c = (float)(1.4426950408889634 / (double)lambda);
    a.inv_lambda = (float)(1.0 / (double)lambda);
    a.inv_tau = (float)(1.0 / (double)tau);
    void* args[] = {&a};
    // groups and threads per block; a dispatch holds fewer than 2^32 threads
    const int groups = cat_split(C) ? 64 * cat_rows(C) : kCatBlock;
    const int threads = cat_split(C) ? groups * cat_parts(C) : kCatBlock;
    const int64_t need = (ngroups + groups - 1) / groups;
    const unsigned grid = (unsigned)std::min<int64_t>(need, 0xFFFFFFFFu / (unsigned)threads);
    if (hipLaunchKernel(fn, dim3(grid), dim3(threads), args, 0, stream) != hipSuccess)
        return launch_status(what);
    return launch_status(what);
}
} // namespace
} // namespace roi

extern "C" int roi_cat_mask_fwd(const uint16_t* W, const float* cat_logits, int64_t rows,
                                int64_t cols, int n, int m, float tau, float lambda, uint64_t seed,
                                uint64_t step, uint64_t group_offset, uint16_t* W_masked,
                                float* soft_mask, uint8_t* choice, hipStream_t stream)
{
    return cat_run(true, W, cat_logits, nullptr, rows, cols, n, m, tau, lambda, seed, step,
                   group_offset, W_masked, soft_mask, choice, nullptr, stream);
}

extern "C" int roi_cat_mask_bwd(const uint16_t* grad_W_masked, const uint16_t* W,
                                const float* cat_logits, int64_t rows, int64_t cols, int n, int m,
                                float tau, float lambda, uint64_t seed, uint64_t step,
                                uint64_t group_offset, float* grad_cat_logits, hipStream_t stream)
{
    return cat_run(false, W, cat_logits, grad_W_masked, rows, cols, n, m, tau, lambda, seed, step,
                   group_offset, nullptr, nullptr, nullptr, grad_cat_logits, stream);
}
