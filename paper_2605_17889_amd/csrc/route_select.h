// Selection and gates of one token by a group of 16 lanes or by a wavefront (device code; included by route.hip,
// permute.hip and the expert GEMMs).
#pragma once
#include "common.h"

namespace moe {

// Logits as unsigned keys of the same order: -0 counts as +0, NaN as -infinity; 0 is below every key and
// stands for an expert that is selected already or does not exist.
__device__ __forceinline__ uint32_t logit_key(float l) {
    const uint32_t u = __float_as_uint(l != l ? -INFINITY : l + 0.0f);
    return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ __forceinline__ float key_logit(uint32_t key) {
    return __uint_as_float(key ^ ((key >> 31) ? 0x80000000u : 0xffffffffu));
}

// v combined with its value in the lane that CTRL names, inside a row of 16 lanes; after rotations by 8
// and 4 and swaps inside quads at distance 2 and 1 every lane of the row has seen all 16.
template <class Op>
__device__ __forceinline__ uint32_t over_16_lanes(uint32_t v, Op&& op) {
#define MOE_ROW(CTRL) static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xf, 0xf, false))
    v = op(v, MOE_ROW(0x128));     // row_ror:8
    v = op(v, MOE_ROW(0x124));     // row_ror:4
    v = op(v, MOE_ROW(0x4e));      // quad_perm:[2,3,0,1]
    v = op(v, MOE_ROW(0xb1));      // quad_perm:[1,0,3,2]
#undef MOE_ROW
    return v;
}

// Lane g of a token's group holds the logits of experts g, g+16, g+32, ... (EW of them). Each of
// the k rounds takes the largest remaining logit of the group (ties -> lower expert index, NaN
// below every number): the largest key over the lane and over the 16 lanes, then the lowest index that
// has it. A round is a chain of dependent instructions that nothing hides when there are few tokens,
// so it is kept short: integer maxima and minima of single values, no compare-and-select of
// (value, index) pairs (with those: 12.3 us for the launch that selects 8 of 128 and permutes for one
// token, now 8.6; 9.2 against 7.2 us for 8192 tokens). The gates are the softmax over the selected logits,
// accumulated in slot order like select_and_gate(). All lanes of the wavefront call it together;
// emit(slot, expert, gate) is called for every slot of a live token, by one of its lanes.
template <int EW, class Emit>
__device__ __forceinline__ void select_by_16_lanes(const float* __restrict__ logits, int t, bool live, int g,
                                                   int E, int k, Emit&& emit) {
    constexpr int G = 16;
    uint32_t key[EW];
#pragma unroll
    for (int w = 0; w < EW; ++w) {
        const int e = w * G + g;
        key[w] = (live && e < E) ? logit_key(logits[static_cast<size_t>(t) * E + e]) : 0u;
    }
    float top = 0.f, den = 0.f;
    float my_w[4] = {0.f, 0.f, 0.f, 0.f};                 // lane g keeps slots g, g+16, g+32, g+48
    int my_idx[4] = {0, 0, 0, 0};
    for (int s = 0; s < k; ++s) {
        uint32_t best = key[0];
#pragma unroll
        for (int w = 1; w < EW; ++w) best = max(best, key[w]);
        best = over_16_lanes(best, [](uint32_t a, uint32_t b) { return max(a, b); });
        // lowest index with that key: k <= E, so there is one
        uint32_t e = 0xffffffffu;
#pragma unroll
        for (int w = 0; w < EW; ++w) e = min(e, key[w] == best ? static_cast<uint32_t>(w * G + g) : 0xffffffffu);
        e = over_16_lanes(e, [](uint32_t a, uint32_t b) { return min(a, b); });
#pragma unroll
        for (int w = 0; w < EW; ++w) key[w] = e == static_cast<uint32_t>(w * G + g) ? 0u : key[w];
        const float bv = key_logit(best);
        if (s == 0) top = bv;
        const float w = expf(bv - top);
        den += w;
        if ((s & (G - 1)) == g) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((s >> 4) == j) { my_w[j] = w; my_idx[j] = static_cast<int>(e); }
        }
    }
    if (!live) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int s = j * G + g;
        if (s < k) emit(s, my_idx[j], my_w[j] / den);
    }
}

// The same for a few tokens, a wavefront per token: lane g holds experts g, g + 64, ... (EW of them). A round is
// shorter: six row moves to the maximum, then the lowest index that has it by ballots on the scalar unit. The same keys,
// order and gates, so the same results. emit(slot, expert, gate) is called once for every slot.
template <int EW, class Emit>
__device__ __forceinline__ void select_by_wavefront(const float* __restrict__ logits, int t, int lane, int E, int k,
                                                    Emit&& emit) {
    uint32_t key[EW];
#pragma unroll
    for (int w = 0; w < EW; ++w) {
        const int e = w * kWave + lane;
        key[w] = e < E ? logit_key(logits[static_cast<size_t>(t) * E + e]) : 0u;
    }
    float top = 0.f, den = 0.f, my_w = 0.f;               // lane s keeps slot s: k <= 64
    int my_e = 0;
    for (int s = 0; s < k; ++s) {
        uint32_t v = key[0];
#pragma unroll
        for (int w = 1; w < EW; ++w) v = max(v, key[w]);
#define MOE_UP(CTRL, ROWS) \
    v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xf, false)))
        MOE_UP(0x111, 0xf);        // from the lanes 1, 2, 4, 8 below inside rows of 16; 0 is below every key
        MOE_UP(0x112, 0xf);
        MOE_UP(0x114, 0xf);
        MOE_UP(0x118, 0xf);
        MOE_UP(0x142, 0xa);        // lane 15 of a row to the row behind it, lane 31 to the upper half
        MOE_UP(0x143, 0xc);
#undef MOE_UP
        const uint32_t best = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), kWave - 1));
        int e = -1;                // k <= E, so there is one
#pragma unroll
        for (int w = EW - 1; w >= 0; --w) {
            const uint64_t has = __ballot(key[w] == best);
            e = has != 0 ? w * kWave + __builtin_ctzll(has) : e;
        }
#pragma unroll
        for (int w = 0; w < EW; ++w) key[w] = e == w * kWave + lane ? 0u : key[w];
        const float bv = key_logit(best);
        if (s == 0) top = bv;
        const float g = expf(bv - top);
        den += g;
        my_w = s == lane ? g : my_w;
        my_e = s == lane ? e : my_e;
    }
    if (lane < k) emit(lane, my_e, my_w / den);
}

}  // namespace moe
