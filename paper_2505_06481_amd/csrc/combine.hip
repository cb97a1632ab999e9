// Step C: Y[t,:] = sum_j topk_w[t,j] * Yg[inv_perm[t*k+j], :]  (section 3.2: the gate's
// weighted-averaging coefficients applied to the selected experts' outputs).
// Gather-side and therefore deterministic: one thread owns four elements of an output row, sums their k
// contributions in fp32 in ascending j and rounds once to the storage type.
#include "mmoe_internal.h"

namespace mmoe {

constexpr int kCombThreads = 256;

// Bound by HBM for large batches, by the chain of loads for small ones.  A small batch's row is shared out to a workgroup for every 1024
// elements.  Before : now, us, two picks: 1 token of 4096 3.05 : 2.06, 64 tokens 3.31 : 2.31; either way round 1037 of 2048, four picks 7.7 :
// 8.2.  Rows that the product before cannot have left in the last-level cache (256 MB) are read past the caches (kNT): of what
// still is there they would be read from memory.  Through : past, us in the layer, by MB of expert outputs:
//   two picks of 4096   150 34.9 : 37.3   172 39.5 : 39.9   219 49.9 : 49.6   231 54.5 : 51.8   256 63.2 : 58.2   375 90.3 : 80.8   512 124.9 : 112.5
//   four of 2048        141 30.2 : 31.8   172 34.3 : 36.5   203 43.7 : 43.8   225 48.0 : 45.6   269 65.7 : 55.9   500 120.7 : 106.8
//   four of 4096        144 33.1 : 35.6   188 38.6 : 42.8   219 43.7 : 45.1   244 50.7 : 52.7   262 62.3 : 60.2   375 97.0 : 76.5
constexpr int kCombSmall = 512;                           // tokens
constexpr int64_t kCombLarge = (int64_t)224 << 20;        // bytes of expert outputs
bool combine_past_the_caches(const mmoe_shape& s) { return (int64_t)s.T * s.top_k * s.d_model * 4 > kCombLarge; }

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
    const bool large = combine_past_the_caches(s);
    const auto kernel = s.dtype == MMOE_BF16 ? (large ? combine_kernel<true, true> : combine_kernel<true, false>)
                                             : (large ? combine_kernel<false, true> : combine_kernel<false, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, st, (const f32x4*)Yg, inv_perm, topk_w, Y, d4, s.top_k);
    return launch_status();
}

}  // namespace mmoe
