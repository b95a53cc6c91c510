// The permutation of a few ids by one workgroup (device code; included by permute.hip and by the expert GEMMs,
// whose few-token kernel makes the tables on the side).
#pragma once
#include "common.h"

namespace moe {

constexpr int kExpertWords = kMaxExperts / kWave;   // experts per lane: 4

__device__ __forceinline__ uint64_t lanemask_lt(int lane) { return (1ull << lane) - 1ull; }

// Lanes of the wavefront that hold the same value as this lane (values in [0, 256), or -1 for
// "none", which matches nothing): one ballot per bit of the value instead of one per expert.
__device__ __forceinline__ uint64_t same_value_lanes(int my) {
    uint64_t m = __ballot(my >= 0);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const uint64_t bit = __ballot((my >> b) & 1);
        m &= ((my >> b) & 1) ? bit : ~bit;
    }
    return my >= 0 ? m : 0ull;
}

// off[e] = sum of tot[0..e), off[E] = the sum of all; by one wavefront, four experts per lane.
__device__ __forceinline__ void expert_offsets(const int32_t* tot, int E, int32_t* off) {
    const int lane = threadIdx.x & (kWave - 1);
    int mine[kExpertWords], sum = 0;
#pragma unroll
    for (int w = 0; w < kExpertWords; ++w) {
        const int x = lane * kExpertWords + w;
        mine[w] = x < E ? tot[x] : 0;
        sum += mine[w];
    }
    int incl = sum;
    for (int s = 1; s < kWave; s <<= 1) {
        const int up = __shfl_up(incl, s, kWave);
        if (lane >= s) incl += up;
    }
    int run = incl - sum;
#pragma unroll
    for (int w = 0; w < kExpertWords; ++w) {
        const int x = lane * kExpertWords + w;
        if (x < E) off[x] = run;
        run += mine[w];
    }
    if (lane == kWave - 1) off[E] = incl;
}

// All three steps of the permutation in one workgroup of WAVES wavefronts, with the per-wavefront tables in LDS
// instead of segment tables in global memory: one launch, not three. Wavefront w owns the KEEP * 64 consecutive
// ids from w * KEEP * 64 on and holds them in registers from the count to the scatter. The workgroup
// takes the ids [first, last) of at most WAVES * 64 * KEEP: all of them, or with PART a part, whose first
// position of every expert the caller has put into sm.off.
template <int WAVES>
struct SmallTables {
    int32_t table[WAVES][kMaxExperts];              // per wavefront: count, then start position
    int32_t tot[kMaxExperts];
    int32_t off[kMaxExperts + 1];
};
template <int WAVES, int KEEP, bool PART>
__device__ __forceinline__ void permute_block(SmallTables<WAVES>& sm, const int32_t* ids, int first, int last, int E,
                                              int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                              int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm) {
    static_assert(WAVES * kWave >= kMaxExperts, "a thread per expert");
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = tid / kWave;
    const int base = first + wv * KEEP * kWave;
    const int waves = min(WAVES, (last - first + KEEP * kWave - 1) / (KEEP * kWave));   // that own any id
    volatile int32_t* mine = sm.table[wv];    // read and written across lanes: never cached
    int my[KEEP];
    uint64_t same[KEEP];
#pragma unroll
    for (int r = 0; r < KEEP; ++r) {
        const int i = base + r * kWave + lane;
        my[r] = (i < last) ? ids[i] : -1;
    }
    if (wv < waves) {                         // the tables of the others are not read
        for (int e = lane; e < E; e += kWave) mine[e] = 0;
#pragma unroll
        for (int r = 0; r < KEEP; ++r) {
            if (my[r] < 0 || my[r] >= E) my[r] = -1;
            same[r] = same_value_lanes(my[r]);
            if (my[r] >= 0 && (same[r] & lanemask_lt(lane)) == 0) mine[my[r]] += __popcll(same[r]);
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    if (tid < E) {                            // wavefronts' counts of one expert, in order
        int run = 0;
        for (int g = 0; g < waves; ++g) {
            const int v = sm.table[g][tid];
            sm.table[g][tid] = run;
            run += v;
        }
        sm.tot[tid] = run;
    }
    __syncthreads();
    if constexpr (!PART) {
        if (tid < kWave) expert_offsets(sm.tot, E, sm.off);
        __syncthreads();
        if (tid < E) {
            counts[tid] = sm.tot[tid];
            offsets[tid] = sm.off[tid];
        }
        if (tid == 0) offsets[E] = sm.off[E];
    }
    if (wv >= waves) return;
    for (int e = lane; e < E; e += kWave) mine[e] += sm.off[e];   // start positions of this wavefront's ids
#pragma unroll
    for (int r = 0; r < KEEP; ++r) {
        const int i = base + r * kWave + lane;
        int pos = -1;
        if (my[r] >= 0) pos = mine[my[r]] + __popcll(same[r] & lanemask_lt(lane));
        __builtin_amdgcn_wave_barrier();      // every lane of a set has read before its first lane writes
        if (my[r] >= 0 && (same[r] & lanemask_lt(lane)) == 0) mine[my[r]] = pos + __popcll(same[r]);
        __builtin_amdgcn_wave_barrier();
        if (i < last) {
            inv_perm[i] = pos;
            if (pos >= 0) perm[pos] = i;
        }
    }
}

}  // namespace moe
