// wide.hpp -- device helpers of the gfx950 kernels for groups of m = 16 and 32
// weights (wide_fwd.hip, wide_bwd.hip), and of the backward for m = 8.
//
// Four consecutive elements per lane (one Philox call, one 16-byte logits load
// and one 8-byte bf16 load per lane), a group spread over L = m / 4 adjacent
// lanes of one wave.  Group-wide maxima and "sum over the other lanes" use
// cross-lane butterflies: DPP quad permutations for lane distances 1..3 and
// the DPP half-row mirror for distances 4..7.  Every group is whole inside a
// wave and either all its lanes are active or none is, so the butterflies
// never read a lane outside the group.  Same arithmetic as the per-lane
// kernels: the noise of noise.hpp, ranks with ties to the lower index, and the
// relaxation of relax.hpp in its "all entries but j" form.
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"
#include "noise.hpp"
#include "relax.hpp"

namespace roi {
namespace {


// Value held by lane (lane ^ D) of the same group (D < 8), with DPP only:
// quad permutations for D < 4; for D >= 4, the half-row mirror (lane i of an
// 8-lane half to lane 7 - i, i.e. xor 7) followed by the quad permutation of
// D ^ 7.
template <int D>
__device__ __forceinline__ float lane_xor(float v)
{
    static_assert(D > 0 && D < 8, "lane distance");
    int x = __float_as_int(v);
    if constexpr ((D & 4) != 0) x = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true);
    constexpr int lo = ((D & 4) != 0 ? (D ^ 7) : D) & 3;
    if constexpr (lo == 1) x = __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true); // [1,0,3,2]
    if constexpr (lo == 2) x = __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true); // [2,3,0,1]
    if constexpr (lo == 3) x = __builtin_amdgcn_update_dpp(0, x, 0x1B, 0xF, 0xF, true); // [3,2,1,0]
    return __int_as_float(x);
}

// Value of the group's other quad of lanes, for a v that is the same in every
// lane of a quad (lane xor 7 is then as good as xor 4, and one DPP less).
__device__ __forceinline__ float other_quad(float v) { return lane_xor<7>(v); }

template <int L>
__device__ __forceinline__ float group_max(float v)
{
    v = fmaxf(v, lane_xor<1>(v));
    if constexpr (L >= 4) v = fmaxf(v, lane_xor<2>(v));
    if constexpr (L >= 8) v = fmaxf(v, other_quad(v));
    return v;
}

// Sum of t over the other L - 1 lanes of the group (never includes this lane's
// own t, so a dominant lane does not swamp the others).
template <int L>
__device__ __forceinline__ float sum_other_lanes(float t)
{
    const float o1 = lane_xor<1>(t);
    if constexpr (L == 2) return o1;
    const float s1 = t + o1; // pair sum
    float other = o1 + lane_xor<2>(s1);
    if constexpr (L == 8) {
        const float s2 = s1 + lane_xor<2>(s1); // quad sum, the same bits in the quad's lanes
        other += other_quad(s2);
    }
    return other;
}

__device__ __forceinline__ float max4(const float (&x)[4])
{
    return fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
}

template <int L>
__device__ __forceinline__ float group_min(float v)
{
    v = fminf(v, lane_xor<1>(v));
    if constexpr (L >= 4) v = fminf(v, lane_xor<2>(v));
    if constexpr (L >= 8) v = fminf(v, other_quad(v));
    return v;
}

// The OR of a value over the group.
template <int L>
__device__ __forceinline__ uint32_t group_or(uint32_t v)
{
    const auto bits = [](float f) { return __float_as_uint(f); };
    v |= bits(lane_xor<1>(__uint_as_float(v)));
    if constexpr (L >= 4) v |= bits(lane_xor<2>(__uint_as_float(v)));
    if constexpr (L >= 8) v |= bits(other_quad(__uint_as_float(v)));
    return v;
}

__device__ __forceinline__ float min4(const float (&x)[4])
{
    return fminf(fminf(x[0], x[1]), fminf(x[2], x[3]));
}

// Hard top-n of keys that may tie, by a bitonic sort of the group
// (descending), entry i = 4 part + e of the group at lane `part`, slot e.  Each
// key travels with its index.  An entry beats another when its key is larger,
// or equal with a lower index.  A stage (kk, j) pairs entry i with i ^ j; the
// pair is ordered descending when (i & kk) == 0 and ascending otherwise, the
// lower entry of a descending pair keeping the entry that beats.  j = 1, 2
// pair slots of one lane; j >= 4 pairs lane part with lane part ^ (j / 4),
// each lane keeping one side of its four pairs.  This is the fallback of
// wide_top_packed, which orders almost every wave.
__device__ __forceinline__ bool beats(float ka, int ia, float kb, int ib)
{
    return ka > kb || (ka == kb && ia < ib);
}

template <int KK, int J>
__device__ __forceinline__ void bitonic_stage(float (&k)[4], int (&ix)[4], int part)
{
    if constexpr (J < 4) {
#pragma unroll
        for (int lo = 0; lo < 4; ++lo) {
            if ((lo & J) != 0) continue;
            const int hi = lo | J;
            // direction of the pair: (i & KK) with i = 4 part + lo
            const bool desc = KK < 4 ? ((lo & KK) == 0) : ((part & (KK >> 2)) == 0);
            const bool sw = beats(k[hi], ix[hi], k[lo], ix[lo]) == desc;
            const float kl = k[lo], kh = k[hi];
            const int il = ix[lo], ih = ix[hi];
            k[lo] = sw ? kh : kl;
            k[hi] = sw ? kl : kh;
            ix[lo] = sw ? ih : il;
            ix[hi] = sw ? il : ih;
        }
    } else {
        constexpr int D = J / 4; // lane distance
        const bool lower = (part & D) == 0;
        const bool desc = (part & (KK >> 2)) == 0;
        const bool keep_max = lower == desc;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float o = lane_xor<D>(k[e]);
            const int oi = __float_as_int(lane_xor<D>(__int_as_float(ix[e])));
            const bool take = beats(o, oi, k[e], ix[e]) == keep_max;
            k[e] = take ? o : k[e];
            ix[e] = take ? oi : ix[e];
        }
    }
}

template <int M, int KK, int J>
__device__ __forceinline__ void bitonic_from(float (&k)[4], int (&ix)[4], int part)
{
    bitonic_stage<KK, J>(k, ix, part);
    if constexpr (J > 1)
        bitonic_from<M, KK, J / 2>(k, ix, part);
    else if constexpr (KK < M)
        bitonic_from<M, KK * 2, KK>(k, ix, part);
}

// Sorts the group's keys (four per lane, kf) and sets keep[e] (is this lane's
// entry e among the n that beat the others) and sidx[e] (the index within the
// group of the entry at sorted position 4 part + e, i.e. of rank 4 part + e).
template <int L, int N>
__device__ __forceinline__ void wide_top_ties(const float (&kf)[4], int part, bool (&keep)[4],
                                              int (&sidx)[4])
{
    constexpr int M = 4 * L;
    float k[4] = {kf[0], kf[1], kf[2], kf[3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) sidx[e] = 4 * part + e;
    bitonic_from<M, 2, 1>(k, sidx, part);
    const int lane = (int)(threadIdx.x & 63);
    // the entry of rank n - 1, held by lane (n - 1) / 4 of the group
    const int src = lane - part + (N - 1) / 4;
    const float kth = __shfl(k[(N - 1) % 4], src);
    const int ith = __shfl(sidx[(N - 1) % 4], src);
#pragma unroll
    for (int e = 0; e < 4; ++e) keep[e] = !beats(kth, ith, kf[e], 4 * part + e);
}

// The median of three: max(a, b) for c = INT32_MAX, min(a, b) for c =
// INT32_MIN (one v_med3_i32).
__device__ __forceinline__ int med3(int a, int b, int c)
{
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    const int m = hi < c ? hi : c;
    return lo > m ? lo : m;
}

// One stage of the packed sort below: entry i is paired with i ^ X, the lower
// entry keeping the larger key.  X < 4 pairs slots of a lane; a larger X pairs
// lane part with part ^ (X / 4) and slot e with e ^ (X % 4), `bound` being
// INT32_MAX in the lanes that hold the lower entries and INT32_MIN elsewhere.
template <int X>
__device__ __forceinline__ void packed_stage(int (&p)[4], int bound)
{
    if constexpr (X < 4) {
#pragma unroll
        for (int lo = 0; lo < 4; ++lo) {
            if ((lo ^ X) < lo) continue;
            const int a = p[lo], b = p[lo ^ X];
            p[lo] = a > b ? a : b;
            p[lo ^ X] = a > b ? b : a;
        }
    } else {
        int o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = __float_as_int(lane_xor<X / 4>(__int_as_float(p[e ^ (X % 4)])));
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = med3(p[e], o[e], bound);
    }
}

// Float bits to integers of the same order (and back: the map is its own
// inverse): the magnitude bits of a negative number are complemented.
__device__ __forceinline__ int sortable_int(float f)
{
    const uint32_t u = __float_as_uint(f);
    // a ^ (b & c)
    return (int)__builtin_amdgcn_bitop3_b32(u, (uint32_t)((int32_t)u >> 31), 0x7FFFFFFFu, 0x78);
}

__device__ __forceinline__ float float_of_sortable_int(int v)
{
    return __int_as_float(sortable_int(__int_as_float(v)));
}

// Sorts a group's integers (four per lane, entry 4 part + e) in descending
// order.  Every merge of KK entries starts by pairing i with i ^ (KK - 1),
// after which all comparisons point the same way and every lane exchange is
// one DPP permutation (xor 1, 2, 3 or 7).
template <int M>
__device__ __forceinline__ void sort_group(int (&p)[4], int part)
{
    static_assert(M == 16 || M == 32, "group size");
    constexpr int kMax = 0x7FFFFFFF, kMin = -0x7FFFFFFF - 1;
    const int b1 = (part & 1) == 0 ? kMax : kMin;
    const int b2 = (part & 2) == 0 ? kMax : kMin;
    const int b4 = (part & 4) == 0 ? kMax : kMin;
    packed_stage<1>(p, 0);
    packed_stage<3>(p, 0);
    packed_stage<1>(p, 0);
    packed_stage<7>(p, b1); // 8: lane xor 1
    packed_stage<2>(p, 0);
    packed_stage<1>(p, 0);
    if constexpr (M >= 16) {
        packed_stage<15>(p, b2); // 16: lane xor 3
        packed_stage<4>(p, b1);
        packed_stage<2>(p, 0);
        packed_stage<1>(p, 0);
    }
    if constexpr (M == 32) {
        packed_stage<31>(p, b4); // 32: lane xor 7
        packed_stage<8>(p, b2);
        packed_stage<4>(p, b1);
        packed_stage<2>(p, 0);
        packed_stage<1>(p, 0);
    }
}

// Hard top-n by a bitonic sort of one 32-bit integer per key: the key's
// order-preserving integer with its low log2(m) bits replaced by the entry's
// index, so that an exchange is a minimum and a maximum (in a lane) or a DPP
// move and a median (across lanes), and the index travels for free.  On MI355X
// the minimum, maximum, median and DPP each issue in 4.2 cycles per wave: 16:32
// sorts with 350 issue cycles per wave instead of 940 with keys and indices
// carried apart.
//
// Replacing the low bits moves a key by less than m ulps, m 2^-23 |K|.  The
// result is decided -- the order of ranks 0 .. n-1 and the kept set are those
// of the unpacked keys' exact counterparts -- when each of those ranks is
// further from the next rank than the error of two keys:
//   kExact: the keys are the exact ones, and packing is monotone, so the
//     packed keys only have to differ above the index bits;
//   else: hardware-log keys, kFastPairMargin + 2^-20 |K| (noise.hpp) plus the
//     packing's m 2^-23 |K|, |K| the larger of the pair.
// Ranks past n need no order among themselves.  Returns whether this lane's
// ranks are decided (a group is when all its lanes are); a NaN anywhere in the
// group, equal exact keys and an infinite hardware-log key among the checked
// ranks are not.
template <int L, int N, bool kExact>
__device__ __forceinline__ bool wide_top_packed(const float (&kf)[4], int part, bool (&keep)[4],
                                                int (&sidx)[4])
{
    constexpr int M = 4 * L;
    constexpr int kIdx = M - 1;
    int own[4], p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        // +0.0f: exact keys of -0 and +0 tie
        const int v = sortable_int(kExact ? kf[e] + 0.0f : kf[e]);
        // (a & b) | c
        own[e] = (int)__builtin_amdgcn_bitop3_b32((uint32_t)v, (uint32_t)~kIdx,
                                                  (uint32_t)(4 * part + e), 0xEA);
        p[e] = own[e];
    }
    sort_group<M>(p, part);
    const int lane = (int)(threadIdx.x & 63);
    const int kth = __shfl(p[(N - 1) % 4], lane - part + (N - 1) / 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        keep[e] = own[e] >= kth;
        sidx[e] = p[e] & kIdx;
    }
    // the next lane's first rank, by the DPP row shift (the group's last lane
    // reads a value that it does not use)
    const int next = __builtin_amdgcn_update_dpp(0, p[0], 0x101, 0xF, 0xF, true);
    // rank 4 part + e needs no check past n, nor past the last pair
    const auto unchecked = [&](int e) { return 4 * part + e >= (N < M ? N : M - 1); };
    const float sum = (kf[0] + kf[1]) + (kf[2] + kf[3]);
    bool sep = sum == sum; // no NaN (opposite infinities count as one)
    if constexpr (kExact) {
        const int q[5] = {p[0], p[1], p[2], p[3], next};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            sep &= unchecked(e) | ((uint32_t)(q[e] ^ q[e + 1]) > (uint32_t)kIdx);
    } else {
        float k[5];
#pragma unroll
        for (int e = 0; e < 4; ++e) k[e] = float_of_sortable_int(p[e] & ~kIdx);
        k[4] = float_of_sortable_int(next & ~kIdx);
        // sorted: the largest magnitude of the four pairs is at an end
        const float big = unchecked(3) ? fmaxf(fabsf(k[0]), fabsf(k[3]))
                                       : fmaxf(fabsf(k[0]), fabsf(k[4]));
        const float margin =
            __builtin_fmaf(big, 0x1p-20f + (float)M * 0x1p-23f, kFastPairMargin);
#pragma unroll
        for (int e = 0; e < 4; ++e) sep &= unchecked(e) | (k[e] - k[e + 1] > margin);
    }
    return sep;
}

// After wide_top_packed left some group of the wave undecided (sep: its result):
// groups whose keys are all equal, as a masked row's are where the mask's value
// swallows the noise, keep their first n entries.  Returns whether every group
// of the wave is decided now.  Over 46.8e6 weights of equal keys on MI355X,
// forward with S at tau = 1, keys and indices sorted apart at once, after the
// packed sort, and so: 16:32 210, 236 and 194 us, 8:16 153, 171 and 152 us, 1:16
// 126, 145 and 123 us.  A check of the whole keys in sorted order, which would
// also decide ties among some of a group's entries, made untied waves 7% slower.
// So a group with fewer than n unmasked entries still sorts twice: 16:32 354 and
// 383 us, 8:16 197 and 217 us.
template <int L, int N>
__device__ __forceinline__ bool wide_top_equal(const float (&kappa)[4], int part, bool sep,
                                               bool (&keep)[4], int (&sidx)[4])
{
    const float first = __shfl(kappa[0], (int)(threadIdx.x & 63) - part);
    const bool same = (kappa[0] == first) & (kappa[1] == first) & (kappa[2] == first) &
                      (kappa[3] == first);
    const uint32_t flags = group_or<L>((sep ? 0u : 1u) | (same ? 0u : 2u));
    if (!__all(flags != 3u)) return false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4 * part + e;
        keep[e] = flags & 2u ? keep[e] : i < N;
        sidx[e] = flags & 2u ? sidx[e] : i;
    }
    return true;
}

// Relaxation over the group (§3.2 recursion, Algorithm 1), four entries per
// lane: the exp-domain recursion of relax_forward_exp when the group's key
// span is at most exp_span (the host's bound, relax.hpp), else the log-domain
// loop of relax_forward, with sums over the group's other lanes.  The choice
// is the group's own (all its lanes agree), so its outputs do not depend on
// which groups share its wave.  Returns true when this group took the
// exp-domain path (its omegas then never reach the floor).
template <int L, int N, bool kKeep, int kQ>
__device__ __forceinline__ bool wide_relax_forward(const float (&kappa)[4], float key_scale,
                                                   float inv_tau, float exp_span, bool want_s,
                                                   float (&S)[4], StepRec<4> (&rec)[N])
{
    // b = kappa * key_scale unshifted, each step subtracting its own largest b
    // (see scaled_keys in relax.hpp)
    const float kmax = group_max<L>(max4(kappa));
    const float c = key_scale;
    const float bmax0 = kmax * c;
    float b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        b[e] = kappa[e] * c;
        S[e] = 0.0f;
    }
    // kQ < 0: the exp-domain form is off at this temperature (no span needed)
    const float span = kQ < 0 ? 0.0f : (kmax - group_min<L>(min4(kappa))) * c;
    if (kQ >= 0 && span <= exp_span) { // the same on all lanes of the group
        float ex[4];
        first_exps<4>(kappa, c, bmax0, [&] { return group_max<L>(max4(kappa)); }, ex);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            float others[4], t;
            sums_but_one<4>(ex, others, t);
            const float ext = sum_other_lanes<L>(t);
            const float inv_total = __builtin_amdgcn_rcpf(t + ext);
            const float ext_w = ext * inv_total; // the other lanes' weight
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float mu = ex[e] * inv_total;
                const float om = __builtin_fmaf(others[e], inv_total, ext_w);
                if (want_s) S[e] += mu;
                if (kKeep) {
                    rec[k].mu[e] = mu;
                    rec[k].om[e] = om;
                }
                if (k + 1 < N) ex[e] = mu * pow_q<kQ < 0 ? 0 : kQ>(om, inv_tau);
            }
        }
        return true;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        float ex[4];
        const float bmax = k == 0 ? bmax0 : group_max<L>(max4(b));
#pragma unroll
        for (int e = 0; e < 4; ++e) ex[e] = __builtin_amdgcn_exp2f(b[e] - bmax);
        float others[4], t;
        sums_but_one<4>(ex, others, t);
        const float ext = sum_other_lanes<L>(t);
        const float inv_total = __builtin_amdgcn_rcpf(t + ext);
        const float ext_w = ext * inv_total; // the other lanes' weight
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float mu = ex[e] * inv_total;
            const float om = __builtin_fmaf(others[e], inv_total, ext_w);
            if (want_s) S[e] += mu;
            if (kKeep) {
                rec[k].mu[e] = mu;
                rec[k].om[e] = om;
            }
            if (k + 1 < N)
                b[e] = __builtin_fmaf(__builtin_amdgcn_logf(fmaxf(om, kFltMin)), inv_tau, b[e]);
        }
    }
    return false;
}

// Reverse sweep over the group: relax_backward of relax.hpp (one form for
// every entry; with kFloor, floored logs pass no derivative), with the sum over
// the other entries taken across the group's lanes.
template <int L, int N, bool kTauIsOne, bool kFloor>
__device__ __forceinline__ void wide_relax_backward(const StepRec<4> (&rec)[N],
                                                    const float (&sbar)[4], float inv_tau,
                                                    float (&abar)[4])
{
#pragma unroll
    for (int k = N - 1; k >= 0; --k) {
        const bool has_next = (k + 1 < N);
        float t[4], mubar[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mubar[e] = sbar[e];
            if (has_next) {
                const float om = rec[k].om[e];
                const bool live = !kFloor || om >= kFltMin;
                // 1/inf = 0 for a floored entry.  Selecting the reciprocal's
                // input, not its result, leaves the two copies of the sweep
                // (with and without the selects) no reciprocal in common, so
                // the compiler does not compute them ahead of the choice and
                // hold them in registers beside the records.
                const float rinv = __builtin_amdgcn_rcpf(live ? om : __builtin_inff());
                mubar[e] = __builtin_fmaf(-abar[e], rinv, sbar[e]);
            }
            t[e] = rec[k].mu[e] * mubar[e];
        }
        // Sum over the group's entries but e: the other lanes' sum enters the
        // two pair sums of this lane, so each is one add from them (no
        // subtraction).
        const float pa = t[0] + t[1], pb = t[2] + t[3];
        const float ext = sum_other_lanes<L>(pa + pb);
        const float pae = pa + ext, pbe = pb + ext;
        const float q[4] = {t[1] + pbe, t[0] + pbe, pae + t[3], pae + t[2]};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = __builtin_fmaf(rec[k].om[e], mubar[e], -q[e]);
            const float m_t = kTauIsOne ? rec[k].mu[e] : rec[k].mu[e] * inv_tau;
            abar[e] = has_next ? __builtin_fmaf(m_t, x, abar[e]) : m_t * x;
        }
    }
}

__device__ __forceinline__ void wide_keys(const float (&phi)[4], uint32_t block, const NoiseKey& key,
                                          float lambda, float div_y, const float2* tab,
                                          float (&kappa)[4])
{
    const uint4 x = philox_block(block, key);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    float phi_bar[4];
    scaled_logits4(phi, lambda, div_y, phi_bar);
#pragma unroll
    for (int e = 0; e < 4; ++e) kappa[e] = phi_bar[e] - neg_gumbel_from_word(w[e], tab);
}

} // namespace
} // namespace roi
