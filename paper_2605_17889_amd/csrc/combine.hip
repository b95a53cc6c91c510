// Gate-weighted combine of expert outputs:  y[t,:] = sum_{s<k} g[t,s] * y_perm[inv_perm[t*k+s],:]
// (the layer's defining sum over the selected experts). A per-token gather with a fixed slot
// order in fp32, so the result is deterministic; no scatter, no atomics.
//
// HBM traffic per token: 2*d_model*k bytes read (4*d_model*k when the expert outputs were kept
// in fp32), 2*d_model bytes written.
#include "common.h"

namespace moe {
namespace {

constexpr int kMaxSlots = 64;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One block per token; each thread owns 8 consecutive columns per step (one 16-byte vector of
// bf16 expert outputs, or two of fp32 ones with YF32).
template <bool YF32>
__global__ __launch_bounds__(256) void combine_kernel(const void* __restrict__ y_perm,
                                                      const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ topk_w, int R,
                                                      int d, int k, uint16_t* __restrict__ y) {
    const int t = blockIdx.x;
    __shared__ int32_t row[kMaxSlots];
    __shared__ float gate[kMaxSlots];
    if (threadIdx.x < k) {
        row[threadIdx.x] = inv_perm[static_cast<size_t>(t) * k + threadIdx.x];
        gate[threadIdx.x] = topk_w[static_cast<size_t>(t) * k + threadIdx.x];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < d / 8; c += blockDim.x) {
        float acc[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) acc[v] = 0.f;
        // the rows of four slots are on their way together; slots are still added one after the other
        for (int s0 = 0; s0 < k; s0 += 4) {
            constexpr int N = YF32 ? 2 : 1;
            u32x4 q[4][N];
            bool on[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = s0 + i < k ? row[s0 + i] : -1;
                on[i] = static_cast<unsigned>(p) < static_cast<unsigned>(R);         // else a dropped row
                const size_t at = static_cast<size_t>(on[i] ? p : 0) * d;
                if (!on[i]) continue;
                if constexpr (YF32) {                // (non-temporal loads measured 3 % slower here)
                    const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const float*>(y_perm) + at) + 2 * c;
                    q[i][0] = src[0];
                    q[i][1] = src[1];
                } else {
                    // each expert-output row is read once, by this block: a non-temporal load (9 % faster
                    // with 8 rows of 4 KB per token, and the next call's router finds its rows cached)
                    q[i][0] = __builtin_nontemporal_load(
                        reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(y_perm) + at) + c);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!on[i]) continue;
                const float g = gate[s0 + i];
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    float w;
                    if constexpr (YF32) w = __uint_as_float(q[i][v >> 2][v & 3]);
                    else w = __uint_as_float((v & 1) ? (q[i][0][v >> 1] & 0xffff0000u) : (q[i][0][v >> 1] << 16));
                    acc[v] = fmaf(g, w, acc[v]);
                }
            }
        }
        uint4 o;
        o.x = f32_to_bf16(acc[0]) | (static_cast<uint32_t>(f32_to_bf16(acc[1])) << 16);
        o.y = f32_to_bf16(acc[2]) | (static_cast<uint32_t>(f32_to_bf16(acc[3])) << 16);
        o.z = f32_to_bf16(acc[4]) | (static_cast<uint32_t>(f32_to_bf16(acc[5])) << 16);
        o.w = f32_to_bf16(acc[6]) | (static_cast<uint32_t>(f32_to_bf16(acc[7])) << 16);
        reinterpret_cast<uint4*>(y + static_cast<size_t>(t) * d)[c] = o;
    }
}

}  // namespace

int launch_combine(const void* y_perm, bool y_f32, const int32_t* inv_perm, const float* topk_w, int T,
                   int d, int k, moe_bf16* y, hipStream_t s) {
    if (T == 0) return MOE_OK;
    if (y_f32)
        hipLaunchKernelGGL(combine_kernel<true>, dim3(T), dim3(256), 0, s, y_perm, inv_perm, topk_w,
                           T * k, d, k, y);
    else
        hipLaunchKernelGGL(combine_kernel<false>, dim3(T), dim3(256), 0, s, y_perm, inv_perm, topk_w,
                           T * k, d, k, y);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

}  // namespace moe
