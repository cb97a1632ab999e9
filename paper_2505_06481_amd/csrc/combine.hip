// Step C: Y[t,:] = sum_j topk_w[t,j] * Yg[inv_perm[t*k+j], :]  (section 3.2: the gate's
// weighted-averaging coefficients applied to the selected experts' outputs).
// Gather-side and therefore deterministic: one thread owns four elements of an output row, sums their k
// contributions in fp32 in ascending j and rounds once to the storage type.
#include "mmoe_internal.h"

namespace mmoe {

constexpr int kCombThreads = 256;

// Bound by HBM for large batches, by the chain of loads for small ones.  Rows that the caches cannot hold anyway are read past
// them (kNT), and a small batch's row is shared out to a workgroup for every 1024 elements.  Before : now, us, two picks: 1 token of
// 4096 3.05 : 2.06, 64 tokens 3.31 : 2.31, 8192 65.4 : 57.9 (5.8 TB/s), 16384 132 : 113; either way round 777 tokens past the caches 7.1 :
// 7.6, 1037 of 2048, four picks, shared out 7.7 : 8.2.
constexpr int kCombSmall = 512;                           // tokens
constexpr int64_t kCombLarge = (int64_t)128 << 20;        // bytes of expert outputs: half of the last-level cache

template <bool kBf16, bool kNT>
__global__ __launch_bounds__(kCombThreads) void combine_kernel(const f32x4* __restrict__ Yg,
                                                               const int32_t* __restrict__ inv_perm,
                                                               const float* __restrict__ topk_w,
                                                               void* __restrict__ Y, int d4, int k)
{
    const int t = blockIdx.x;
    int rows[kMaxTopK];
    float w[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j)
        if (j < k) {
            // without a permutation the expert outputs are indexed by pair id (self-grouping expert stage)
            rows[j] = inv_perm ? inv_perm[(size_t)t * k + j] : t * k + j;
            w[j] = topk_w[(size_t)t * k + j];
        }
    for (int c = blockIdx.y * kCombThreads + threadIdx.x; c < d4; c += kCombThreads * gridDim.y) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k) {
                const f32x4* row = Yg + (size_t)rows[j] * d4 + c;
                const f32x4 y = kNT ? __builtin_nontemporal_load(row) : *row;
                acc += w[j] * y;
            }
        if (kBf16) {
            u32x2 o;
            o[0] = (uint32_t)f32_to_bf16_bits(acc[0]) | ((uint32_t)f32_to_bf16_bits(acc[1]) << 16);
            o[1] = (uint32_t)f32_to_bf16_bits(acc[2]) | ((uint32_t)f32_to_bf16_bits(acc[3]) << 16);
            reinterpret_cast<u32x2*>(Y)[(size_t)t * d4 + c] = o;
        } else {
            reinterpret_cast<f32x4*>(Y)[(size_t)t * d4 + c] = acc;
        }
    }
}

int launch_combine(const mmoe_shape& s, const float* Yg, const int32_t* inv_perm, const float* topk_w, void* Y,
                   hipStream_t st)
{
    const int d4 = s.d_model / 4;
    const dim3 grid(s.T, s.T < kCombSmall ? (d4 + kCombThreads - 1) / kCombThreads : 1), block(kCombThreads);
    const bool large = (int64_t)s.T * s.top_k * s.d_model * 4 > kCombLarge;
    const auto kernel = s.dtype == MMOE_BF16 ? (large ? combine_kernel<true, true> : combine_kernel<true, false>)
                                             : (large ? combine_kernel<false, true> : combine_kernel<false, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, st, (const f32x4*)Yg, inv_perm, topk_w, Y, d4, s.top_k);
    return launch_status();
}

}  // namespace mmoe
