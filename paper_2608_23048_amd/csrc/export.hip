// export.hip -- gfx950 kernel of the final-mask export.
//
// After training, the sampling temperature lambda has been annealed towards
// 0 (§4.2.3); the sampler's lambda -> 0 limit keeps the n largest logits of
// each group (ties to the lower index, as in the sampler).  This kernel writes
// that mask in the forms a deployment needs: the dense masked weights, the
// compressed weights (the kept values of each group in increasing index
// order) with their indices, and for 2:4 the indices as 2-bit fields, the
// metadata a sparse-matrix core consumes next to the compressed values.
//
// One lane per group at m = 4 and 8, four consecutive elements per lane at m =
// 16 and 32; no noise.  The 2:4 metadata word of 8 consecutive groups is
// assembled across 8 adjacent lanes.
#include <hip/hip_runtime.h>

#include <utility>

#include "common.hpp"
#include "relax.hpp"
#include "roi.h"
#include "wide.hpp"

namespace roi {

namespace {

// m bf16 values of a group (16-bit patterns in the low half of each word).
template <int M>
__device__ __forceinline__ void load_group_bf16(const uint16_t* p, uint32_t (&w)[M])
{
    if constexpr (M == 4) {
        const u32x2 v = stream_load(reinterpret_cast<const u32x2*>(p));
        w[0] = v.x & 0xFFFFu; w[1] = v.x >> 16; w[2] = v.y & 0xFFFFu; w[3] = v.y >> 16;
    } else {
#pragma unroll
        for (int t = 0; t < M / 8; ++t) {
            const u32x4 v = stream_load(reinterpret_cast<const u32x4*>(p) + t);
            w[8 * t + 0] = v.x & 0xFFFFu; w[8 * t + 1] = v.x >> 16;
            w[8 * t + 2] = v.y & 0xFFFFu; w[8 * t + 3] = v.y >> 16;
            w[8 * t + 4] = v.z & 0xFFFFu; w[8 * t + 5] = v.z >> 16;
            w[8 * t + 6] = v.w & 0xFFFFu; w[8 * t + 7] = v.w >> 16;
        }
    }
}

template <int M>
__device__ __forceinline__ void store_group_bf16(uint16_t* p, const uint32_t (&w)[M])
{
    if constexpr (M == 4) {
        const u32x2 v = {w[0] | (w[1] << 16), w[2] | (w[3] << 16)};
        stream_store(v, reinterpret_cast<u32x2*>(p));
    } else {
#pragma unroll
        for (int t = 0; t < M / 8; ++t) {
            const u32x4 v = {w[8 * t] | (w[8 * t + 1] << 16), w[8 * t + 2] | (w[8 * t + 3] << 16),
                             w[8 * t + 4] | (w[8 * t + 5] << 16),
                             w[8 * t + 6] | (w[8 * t + 7] << 16)};
            stream_store(v, reinterpret_cast<u32x4*>(p) + t);
        }
    }
}

template <int M, int N>
__global__ __launch_bounds__(kBlock) void export_kernel(ExportArgs a)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    // The loop bound is uniform over the block, so every lane of a wave takes
    // part in the cross-lane metadata assembly, live or not.
    for (int64_t base = (int64_t)blockIdx.x * kBlock; base < a.ngroups; base += stride) {
        const int64_t q = base + threadIdx.x;
        const bool live = q < a.ngroups;
        uint32_t nib = 0;
        if (live) {
            float phi[M];
            uint32_t w[M];
            load_logits<M>(a.phi + q * M, phi);
            // W is read only when a weight output is requested (it may be NULL
            // otherwise)
            if (a.Wm || a.vals) {
                load_group_bf16<M>(a.W + q * M, w);
            } else {
#pragma unroll
                for (int j = 0; j < M; ++j) w[j] = 0;
            }
            int rank[M];
            rank_keys<M>(phi, rank);
            if (a.Wm) {
                uint32_t wm[M];
#pragma unroll
                for (int j = 0; j < M; ++j) wm[j] = rank[j] < N ? w[j] : 0u;
                store_group_bf16<M>(a.Wm + q * M, wm);
            }
            // kept entries in increasing index order, in registers
            uint32_t kv[N], ki[N];
#pragma unroll
            for (int p = 0; p < N; ++p) kv[p] = ki[p] = 0;
            int pos = 0;
#pragma unroll
            for (int j = 0; j < M; ++j) {
                const bool keep = rank[j] < N;
#pragma unroll
                for (int p = 0; p < N; ++p) {
                    kv[p] = (keep && pos == p) ? w[j] : kv[p];
                    ki[p] = (keep && pos == p) ? (uint32_t)j : ki[p];
                }
                pos += keep ? 1 : 0;
            }
            if (a.vals) {
                if constexpr (N % 2 == 0) {
#pragma unroll
                    for (int p = 0; p < N; p += 2)
                        stream_store(kv[p] | (kv[p + 1] << 16),
                                     reinterpret_cast<uint32_t*>(a.vals + q * N + p));
                } else {
#pragma unroll
                    for (int p = 0; p < N; ++p) a.vals[q * N + p] = (uint16_t)kv[p];
                }
            }
            if (a.idx) {
#pragma unroll
                for (int p = 0; p < N; ++p) a.idx[q * N + p] = (uint8_t)ki[p];
            }
            if constexpr (M == 4 && N == 2) nib = ki[0] | (ki[1] << 2);
        }
        if constexpr (M == 4 && N == 2) {
            if (a.meta) { // uniform: the same for every lane
                uint32_t word = nib << (4 * (threadIdx.x & 7));
                word |= (uint32_t)__shfl_xor((int)word, 1);
                word |= (uint32_t)__shfl_xor((int)word, 2);
                word |= (uint32_t)__shfl_xor((int)word, 4);
                if (live && (threadIdx.x & 7) == 0) stream_store(word, a.meta + q / 8);
            }
        }
    }
}

// ---- m = 16 and 32: four consecutive elements per lane, the layout of the
// wide kernels.
//
// The n-th largest logit of each group comes from a sort of order-preserving
// integers (wide.hpp); the kept entries are those at or above it.  Where the
// n-th and the next logit tie (logits that were never trained, for one), the
// entries equal to it are kept in index order while there is room.  A wave with
// a NaN counts, for every entry, the entries that beat it (rank_keys' rule).
// The kept values and indices of a block are gathered in LDS and leave as
// contiguous 16-byte stores.  One lane per group instead reads and writes at
// strides of a whole group, its compressed outputs 1 or 2 bytes at a time, and
// compares all pairs.  1.5B-class layer (46.8e6 weights), values and indices:
// 16:32 207 us one lane per group, 71 us so; 8:16 126 and 65 us; 1:16 79 and
// 68 us (54 us at the streaming-copy rate for 16:32); with every logit equal,
// 16:32 172 and 71 us, 8:16 102 and 69 us, 1:16 65 and 66 us.  At m = 8 the lane kernel
// stays: its group is 32 bytes, and it was faster, 4:8 57 and 63 us, 1:8 51 and
// 58 us.

// p[i], without indexing registers.
__device__ __forceinline__ int pick4(const int (&p)[4], int i)
{
    const int a = i & 1 ? p[1] : p[0], b = i & 1 ? p[3] : p[2];
    return i & 2 ? b : a;
}

// Copies `count` entries from LDS to a 16-byte aligned place, 16 bytes per
// thread, and one entry per thread past the last whole 16 bytes.
template <typename T>
__device__ __forceinline__ void copy_out(const T* lds, T* dst, int count)
{
    constexpr int kPer = 16 / (int)sizeof(T);
    const int vecs = count / kPer;
    for (int i = threadIdx.x; i < vecs; i += kBlock)
        stream_store(reinterpret_cast<const u32x4*>(lds)[i], reinterpret_cast<u32x4*>(dst) + i);
    const int i = vecs * kPer + (int)threadIdx.x;
    if (i < count) dst[i] = lds[i];
}

template <int M>
__global__ __launch_bounds__(kBlock) void export_wide_kernel(ExportArgs a)
{
    constexpr int L = M / 4;
    constexpr int kGroups = kBlock / L; // per block; kGroups n is a multiple of 16
    __shared__ __attribute__((aligned(16))) uint16_t vals[kBlock * 4];
    __shared__ __attribute__((aligned(16))) uint8_t idx[kBlock * 4];
    const int n = a.n;
    const int part = (int)(threadIdx.x % L), lane = (int)(threadIdx.x & 63);
    const bool want_w = a.Wm || a.vals; // uniform; W may be NULL otherwise
    // The loop bound is uniform over the block: every lane takes part in the
    // exchanges, live or not (a group's lanes are all live or none).
    for (int64_t g0 = (int64_t)blockIdx.x * kGroups; g0 < a.ngroups;
         g0 += (int64_t)gridDim.x * kGroups) {
        const int here = (int)(a.ngroups - g0 < kGroups ? a.ngroups - g0 : kGroups);
        const int row = (int)threadIdx.x / L;
        const bool live = row < here;
        const int64_t slot = g0 * L + threadIdx.x;
        f32x4 pv{};
        u32x2 wv{};
        if (live) {
            if (n < M) pv = stream_load(reinterpret_cast<const f32x4*>(a.phi + slot * 4));
            if (want_w) wv = stream_load(reinterpret_cast<const u32x2*>(a.W + slot * 4));
        }
        const float phi[4] = {pv.x, pv.y, pv.z, pv.w};
        uint32_t nib = 0xFu; // n = m keeps every entry
        if (n < M) { // uniform
            int own[4], p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                own[e] = sortable_int(phi[e] + 0.0f); // -0 and +0 tie
                p[e] = own[e];
            }
            sort_group<M>(p, part);
            const int first = lane - part; // the group's first lane
            const int kth = __shfl(pick4(p, n - 1), first + (n - 1) / 4);
            const bool tied = __shfl(pick4(p, n), first + n / 4) == kth;
            const float sum = (phi[0] + phi[1]) + (phi[2] + phi[3]);
            nib = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) nib |= own[e] >= kth ? 1u << e : 0u;
            if (__any(tied || !(sum == sum))) { // rare
                // Hidden, so that nothing of this is computed ahead of the branch.
                int at = part, top = kth;
                asm volatile("" : "+v"(at), "+v"(top));
                uint32_t above = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) above |= own[e] > top ? 1u << e : 0u;
                const int room = n - __popc(group_or<L>(above << (4 * at)));
                const uint32_t equal = group_or<L>((nib ^ above) << (4 * at));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t before = equal & ((1u << (4 * at + e)) - 1u);
                    if (__popc(before) >= room) nib &= ~(1u << e) | above;
                }
                // the sum is NaN for opposite infinities too: look at each logit
                if (__any(phi[0] != phi[0] || phi[1] != phi[1] || phi[2] != phi[2] ||
                          phi[3] != phi[3])) {
                    int rank[4] = {0, 0, 0, 0};
#pragma unroll 1
                    for (int t = 0; t < L; ++t) {
#pragma unroll
                        for (int f = 0; f < 4; ++f) {
                            const float v = __shfl(phi[f], first + t);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int i = 4 * t + f, j = 4 * at + e;
                                // the earlier of two entries wins when it is >= the later
                                if (i < j) rank[e] += v >= phi[e] ? 1 : 0;
                                if (i > j) rank[e] += phi[e] >= v ? 0 : 1;
                            }
                        }
                    }
                    nib = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) nib |= rank[e] < n ? 1u << e : 0u;
                }
            }
        }
        const uint32_t kept = group_or<L>(nib << (4 * part));
        if (a.Wm && live) {
            const u32x2 v = {wv.x & ((nib & 1u ? 0x0000FFFFu : 0u) | (nib & 2u ? 0xFFFF0000u : 0u)),
                             wv.y & ((nib & 4u ? 0x0000FFFFu : 0u) | (nib & 8u ? 0xFFFF0000u : 0u))};
            stream_store(v, reinterpret_cast<u32x2*>(a.Wm + slot * 4));
        }
        if (!a.vals && !a.idx) continue; // uniform
        // the kept entries in increasing index order
        int pos = __popc(kept & ((1u << (4 * part)) - 1u));
        const uint32_t w[4] = {wv.x & 0xFFFFu, wv.x >> 16, wv.y & 0xFFFFu, wv.y >> 16};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // pos < n unless a NaN left a group's ranks without an order
            if (((nib >> e) & 1u) && pos < n) {
                vals[row * n + pos] = (uint16_t)w[e];
                idx[row * n + pos] = (uint8_t)(4 * part + e);
                ++pos;
            }
        }
        if (__any(__popc(kept) < n)) { // NaN
#pragma unroll 1
            for (int r = __popc(kept) + part; r < n; r += L) {
                vals[row * n + r] = 0;
                idx[row * n + r] = 0;
            }
        }
        __syncthreads();
        if (a.vals) copy_out(vals, a.vals + g0 * n, here * n);
        if (a.idx) copy_out(idx, a.idx + g0 * n, here * n);
        __syncthreads(); // before the next groups' entries
    }
}

template <int M, int... Ns>
ExportFn export_for_n(int n, std::integer_sequence<int, Ns...>)
{
    ExportFn f = nullptr;
    ((n == Ns + 1 ? (f = export_kernel<M, Ns + 1>, 0) : 0), ...);
    return f;
}

} // namespace

ExportFn select_export(int m, int n)
{
    if (m == 4) return export_for_n<4>(n, std::make_integer_sequence<int, 4>{});
    if (m == 8) return export_for_n<8>(n, std::make_integer_sequence<int, 8>{});
    if (m == 16) return export_wide_kernel<16>;
    if (m == 32) return export_wide_kernel<32>;
    return nullptr;
}

int64_t export_block_groups(int m) { return m <= 8 ? kBlock : kBlock / (m / 4); }

} // namespace roi
