// The end of a one-launch select + attention workgroup: the sixteen waves' online-softmax
// states (xw[w][g] = (acc[D], m, l), log2 domain) are folded into the split's partial;
// when a (sequence, kv head) has several splits the partial is published and the workgroup
// that arrives last combines them (see select_attention.hip for the protocol).  Every lane
// of the 1024-lane workgroup calls this.
#pragma once
#include "attention_common.h"
#include "select_core.h"

namespace leoam {

constexpr int kFusedWaves = kSelWaves;                 // 16
constexpr int kFusedMergeBatch = 16;                   // one state per lane of a 16-lane row

// Online-softmax states of one (head, channel) that are folded by a lane: (m, l) of state i sits in lane i of
// every 16-lane row (m = -inf: no such state), column(i) gives its accumulator of this lane's channel for
// i < kStates.  Broadcasts inside the row hand the weights round: a lane reads (or loads) one (m, l) and not
// all of them, and takes one exponential instead of sixteen.
struct FoldedState {
    float m = -INFINITY, l = 0.f, o = 0.f;
    template <int kStates, typename Column> __device__ __forceinline__ void fold(float m_i, float l_i, Column&& column) {
        float top = m_i;
        top = fmaxf(top, dpp_f<0xB1>(top));
        top = fmaxf(top, dpp_f<0x4E>(top));
        top = fmaxf(top, dpp_f<0x141>(top));
        top = fmaxf(top, dpp_f<0x140>(top));
        const float m_new = fmaxf(m, top), c = exp2_or_zero(m, m_new), a = exp2_or_zero(m_i, m_new);
        m = m_new;
        l = l * c + row16_sum(a * l_i);
        o *= c;
        static_for<0, kStates>([&](auto i) { o = fmaf(row_bcast<decltype(i)::value>(a), column(decltype(i)::value), o); });
    }
};

// `exchange` (two splits only, else nullptr): one 64-bit word per (b, q head, channel), zero between calls.
// The two workgroups of a (sequence, kv head) then combine without a ticket and without waiting for
// store acknowledgements: every lane swaps its normalised result (o / l, m + log2 l) into the word
// with ONE atomic exchange; the lane that finds the other split's pair there combines the two, in
// split order, writes the output and puts the word back to zero.  The value travels inside the atomic
// itself, so nothing depends on the order of separate memory operations.
//
// A wave carries kHeads of the group's G heads: xw[w][j] is head j of part w / (waves per part).
// n_splits of the launch's `stride` splits take part (partials are laid out for `stride`).
template <int G, int kHeads>
__device__ __forceinline__ void fused_tail(float (*xw)[kHeads][kPartStride], int32_t& sh_last, float* partial,
                                           int32_t* arrivals, float* __restrict__ out, float* __restrict__ lse,
                                           size_t bh, int split, int n_splits, int stride,
                                           unsigned long long* exchange = nullptr) {
    constexpr int kWaves = kFusedWaves * kHeads / G;       // waves that hold a head
    const int tid = threadIdx.x;
    // ---- fold the waves: lane (g, d) gets the split's (m, l, o[d]) ----------------
    const int g = tid >> 7, d = tid & (LEOAM_D - 1);
    const bool owner = tid < G * LEOAM_D;
    FoldedState state;
    if (owner) {      // (whole waves: a head is two of them)
        const float(*x)[kHeads][kPartStride] = xw + (g / kHeads) * kWaves;
        const int j = g % kHeads, w = lane_id() & (kFusedMergeBatch - 1);
        const float m_w = w < kWaves ? x[w][j][LEOAM_D] : -INFINITY, l_w = w < kWaves ? x[w][j][LEOAM_D + 1] : 0.f;
        state.fold<kWaves>(m_w, l_w, [&](int i) { return x[i][j][d]; });
    }
    float m = state.m, l = state.l, o = state.o;
    const size_t bj = bh * G + g;
    if (n_splits == 2 && exchange != nullptr) {
        if (!owner) return;
        // w = log2 of this split's softmax denominator, on = its normalised output; the high word of a
        // published pair is never zero (+0 travels as -0), which is what marks the word as taken
        const float w = (l > 0.f) ? m + log2f(l) : -INFINITY;
        const float on = (l > 0.f) ? o / l : 0.f;
        uint32_t wb = float_to_bits(w);
        if (wb == 0u) wb = 0x80000000u;
        const unsigned long long mine = ((unsigned long long)wb << 32) | float_to_bits(on);
        unsigned long long* slot = exchange + bj * LEOAM_D + d;
        const unsigned long long other = __hip_atomic_exchange(slot, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)(other >> 32) == 0u) return;          // first to arrive: the other split's lane combines
        __hip_atomic_store(slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float w_o = bits_to_float((uint32_t)(other >> 32)), on_o = bits_to_float((uint32_t)other);
        // operands in split order, so that the result does not depend on which split arrived last
        const float w0 = split == 0 ? w : w_o, w1 = split == 0 ? w_o : w;
        const float o0 = split == 0 ? on : on_o, o1 = split == 0 ? on_o : on;
        const float wm = fmaxf(w0, w1);
        const float e0 = exp2_or_zero(w0, wm), e1 = exp2_or_zero(w1, wm);
        const float den = e0 + e1;
        out[bj * LEOAM_D + d] = (den > 0.f) ? (o0 * e0 + o1 * e1) / den : 0.f;
        if (lse && d == 0) lse[bj] = (den > 0.f) ? (wm + log2f(den)) * kLn2 : -INFINITY;
        return;
    }
    if (n_splits > 1) {
        // publish the partial, take a ticket; the last workgroup to arrive merges
        float* mine = partial + (bj * (size_t)stride + split) * kPartStride;
        if (owner) {
            __hip_atomic_store(&mine[d], o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (d == 0) {
                __hip_atomic_store(&mine[LEOAM_D], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&mine[LEOAM_D + 1], l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this wave's stores have been acknowledged
        __syncthreads();
        if (tid == 0) {
            const int ticket = __hip_atomic_fetch_add(&arrivals[bh], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int is_last = ticket == n_splits - 1;
            sh_last = is_last;
        }
        __syncthreads();
        if (!sh_last || !owner) return;
        const float* base = partial + bj * (size_t)stride * kPartStride;
        state = FoldedState{};
        // a batch of partials is one memory round trip: (m, l) of a split per lane, its column from each
        auto merge_batch = [&](int s0, auto width, auto full) {
            constexpr int kW = decltype(width)::value;
            constexpr bool kFull = decltype(full)::value;
            const int own = s0 + (lane_id() & (kFusedMergeBatch - 1));
            const bool real = own < n_splits && own < s0 + kW;
            const unsigned long long ml = __hip_atomic_load(
                reinterpret_cast<const unsigned long long*>(base + (size_t)min(own, n_splits - 1) * kPartStride + LEOAM_D),
                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            float os[kW];
#pragma unroll
            for (int i = 0; i < kW; ++i)
                os[i] = __hip_atomic_load(&base[(size_t)(kFull ? s0 + i : min(s0 + i, n_splits - 1)) * kPartStride + d],
                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if constexpr (!kFull) {      // past the end the weight is 0, but the last split's value may be infinite
#pragma unroll
                for (int i = 0; i < kW; ++i)
                    if (s0 + i >= n_splits) os[i] = 0.f;
            }
            state.fold<kW>(real ? bits_to_float((uint32_t)ml) : -INFINITY, real ? bits_to_float((uint32_t)(ml >> 32)) : 0.f,
                           [&](int i) { return os[i]; });
        };
        if (n_splits <= 4) {
            merge_batch(0, std::integral_constant<int, 4>{}, std::false_type{});
        } else if (n_splits <= 8) {
            merge_batch(0, std::integral_constant<int, 8>{}, std::false_type{});
        } else {
            const std::integral_constant<int, kFusedMergeBatch> width{};
            int s0 = 0;
            for (; s0 + width() <= n_splits; s0 += width()) merge_batch(s0, width, std::true_type{});
            if (s0 < n_splits) merge_batch(s0, width, std::false_type{});
        }
        m = state.m;
        l = state.l;
        o = state.o;
        // (behind the loads: the memory counter is in order, a store before them would be waited for)
        if (tid == 0) __hip_atomic_store(&arrivals[bh], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!owner) return;
    out[bj * LEOAM_D + d] = (l > 0.f) ? o / l : 0.f;
    if (lse && d == 0) lse[bj] = (l > 0.f) ? (m + log2f(l)) * kLn2 : -INFINITY;
}

}  // namespace leoam
