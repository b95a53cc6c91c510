// Selection and gates of one token by a group of 16 lanes (device code; included by route.hip and
// permute.hip).
#pragma once
#include "common.h"

namespace moe {

// Lane g of a token's group holds the logits of experts g, g+16, g+32, ... (EW of them). Each of
// the k rounds takes the largest remaining logit of the group (ties -> lower expert index, NaN
// below every number): first inside the lane, ascending, then by four exchange steps of
// (value, index) pairs over the 16 lanes; "larger value, then lower index" is a total order, so
// the result does not depend on how the lanes are paired. The gates are the softmax over the selected logits,
// accumulated in slot order like select_and_gate(). All lanes of the wavefront call it together;
// emit(slot, expert, gate) is called for every slot of a live token, by one of its lanes.
template <int EW, class Emit>
__device__ __forceinline__ void select_by_16_lanes(const float* __restrict__ logits, int t, bool live, int g,
                                                   int E, int k, Emit&& emit) {
    constexpr int G = 16;
    float v[EW];
#pragma unroll
    for (int w = 0; w < EW; ++w) {
        const int e = w * G + g;
        const float l = (live && e < E) ? logits[static_cast<size_t>(t) * E + e] : -INFINITY;
        v[w] = (l != l) ? -INFINITY : l;
    }
    unsigned taken = 0;                                   // bit w: expert w*16+g is selected
    float top = 0.f, den = 0.f;
    float my_w[4] = {0.f, 0.f, 0.f, 0.f};                 // lane g keeps slots g, g+16, g+32, g+48
    int my_idx[4] = {0, 0, 0, 0};
    for (int s = 0; s < k; ++s) {
        // best of this lane: ascending expert index, strict '>' keeps the lower index on ties
        float bv = 0.f;
        int be = -1;
#pragma unroll
        for (int w = 0; w < EW; ++w) {
            const int e = w * G + g;
            if (e < E && !((taken >> w) & 1u) && (be < 0 || v[w] > bv)) { bv = v[w]; be = e; }
        }
        // best of the group: larger value, then lower index; lanes without a candidate lose
        // (data-parallel-primitive moves inside a row of 16 lanes: rotate by 8, by 4, then swap
        // inside quads at distance 2 and 1; after the four steps every lane has seen all 16)
        auto take = [&](float ov, int oe) {
            const bool other = oe >= 0 && (be < 0 || ov > bv || (ov == bv && oe < be));
            if (other) { bv = ov; be = oe; }
        };
#define MOE_DPP_STEP(CTRL)                                                                        \
        take(__int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(bv), CTRL, 0xf, 0xf, false)), \
             __builtin_amdgcn_update_dpp(0, be, CTRL, 0xf, 0xf, false))
        MOE_DPP_STEP(0x128);      // row_ror:8
        MOE_DPP_STEP(0x124);      // row_ror:4
        MOE_DPP_STEP(0x4e);       // quad_perm:[2,3,0,1]
        MOE_DPP_STEP(0xb1);       // quad_perm:[1,0,3,2]
#undef MOE_DPP_STEP
        if ((be & (G - 1)) == g) taken |= 1u << (be >> 4);    // be >= 0 because k <= E
        if (s == 0) top = bv;
        const float w = expf(bv - top);
        den += w;
        if ((s & (G - 1)) == g) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((s >> 4) == j) { my_w[j] = w; my_idx[j] = be; }
        }
    }
    if (!live) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int s = j * G + g;
        if (s < k) emit(s, my_idx[j], my_w[j] / den);
    }
}

}  // namespace moe
