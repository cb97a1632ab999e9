// One-time repacking of the expert pool.  Runs when the pool is loaded (section 3.1: the
// loader runs once, before serving), never on the serving path.
//
// Every product of the expert stage is  out[r, n] = sum_k A[r, k] * W[n][k]  with W given
// "in x out", i.e. as W[k][n].
//
// fp32: W is transposed to [S, N, K] (reduction dimension contiguous).
//
// bf16: W is stored as matrix-core fragments.  A fragment is the 32-row x 16-k operand of
// v_mfma_f32_32x32x16_bf16 exactly as the 64 lanes hold it: 64 pieces of 16 bytes, piece
// `lane` = 8 consecutive k of row lane%32, for the lane half h = lane/32.  Fragments of one
// 32-row block follow each other along k, so a wavefront streams a block's weights with
// fully contiguous 1 KB loads straight into registers: no LDS, no shuffle.  The k values a
// fragment covers are permuted inside each run of 64 so that a lane's four consecutive
// fragments read 64 contiguous bytes of the activation row:
//     fragment ks = 4m + kk (kk < 4), lane half h  <->  k = 64m + 32h + 8kk + [0, 8).
// Element (n, k) of slot s lives at
//     ((((s*(N/32) + n/32) * (K/16) + ks) * 64 + 32h + n%32) * 8 + k%8.
#include "mmoe_internal.h"

namespace mmoe {

constexpr int kTile = 64;

__global__ __launch_bounds__(256) void transpose_kernel(const float* __restrict__ in, float* __restrict__ out, int R,
                                                        int C)
{
    __shared__ float tile[kTile][kTile + 2];
    // backwards and past the caches, as the fragment packing below
    const size_t mat = (size_t)(gridDim.z - 1 - blockIdx.z) * R * C;
    const int c0 = (gridDim.x - 1 - blockIdx.x) * kTile, r0 = (gridDim.y - 1 - blockIdx.y) * kTile;
    const int tx = threadIdx.x % kTile, ty = threadIdx.x / kTile;  // 64 x 4
    for (int i = ty; i < kTile; i += 4) {
        int r = r0 + i, c = c0 + tx;
        if (r < R && c < C) tile[i][tx] = in[mat + (size_t)r * C + c];
    }
    __syncthreads();
    for (int i = ty; i < kTile; i += 4) {
        int c = c0 + i, r = r0 + tx;
        if (r < R && c < C) __builtin_nontemporal_store(tile[tx][i], &out[mat + (size_t)c * R + r]);
    }
}

// bf16 fragment packing.  Bound by HBM.  A workgroup packs 64 k x 256 n: rows are read 512 bytes at a time into LDS, a
// thread then gathers the 8 k of a piece from LDS and writes it, a wavefront the pieces of a fragment (1 KB).  A program
// packs the pool that it has just assembled, so the pool is walked backwards, last matrix first, and the packed copy,
// which nobody reads soon, is written past the caches: the end of the pool is then still in the last-level cache.
// (768 x 3072, 12 layers of 20 slots on average, assembly and packing of 2.26 GB: 1749 us with a 16-byte piece gathered
// by eight 2-byte loads, forwards; 1570 backwards and past the caches; 1500 with rows read into LDS.)
constexpr int kPackN = 256, kPackK = 64;
__global__ __launch_bounds__(256) void pack_fragments_kernel(const uint16_t* __restrict__ in, u32x4* __restrict__ out, int K, int N)
{
    __shared__ __attribute__((aligned(16))) uint16_t tile[kPackK][kPackN];
    // workgroup -> (slot, block of 256 n, block of 64 k), `in` is [S, K, N]
    const unsigned b = gridDim.x - 1 - blockIdx.x;
    const unsigned km = K / kPackK, nn = N / kPackN;
    const unsigned m = b % km, rest = b / km, nb8 = rest % nn;
    const size_t s = rest / nn;
    const int tid = threadIdx.x;
    const uint16_t* src = in + (s * K + (size_t)m * kPackK) * N + nb8 * kPackN;
    u32x4 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const u32x4*>(src + (size_t)(i * 8 + tid / 32) * N + (tid % 32) * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(&tile[i * 8 + tid / 32][((tid % 32) * 8) ^ (i < 4 ? 0 : 32)]) = v[i];  // the upper 32 k in other banks
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6;  // wave = fragment kk of the 64-k step; i = block of 32 n
    const int k0 = (lane >> 5) * 32 + wave * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int n = (i * 32 + (lane & 31)) ^ (lane & 32);
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (uint32_t)tile[k0 + 2 * e][n] | ((uint32_t)tile[k0 + 2 * e + 1][n] << 16);
        const size_t frag = (s * (N / 32) + nb8 * 8 + i) * (K / 16) + m * 4 + wave;
        __builtin_nontemporal_store((u32x4{w[0], w[1], w[2], w[3]}), &out[frag * 64 + lane]);
    }
}

static void pack_fragments(const void* in, void* out, int S, int K, int N, hipStream_t st)
{
    const size_t blocks = (size_t)S * (N / kPackN) * (K / kPackK);
    hipLaunchKernelGGL(pack_fragments_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const uint16_t*)in, (u32x4*)out, K, N);
}

static void transpose(const void* in, void* out, int S, int R, int C, hipStream_t st)
{
    dim3 grid((C + kTile - 1) / kTile, (R + kTile - 1) / kTile, S), block(256);
    hipLaunchKernelGGL(transpose_kernel, grid, block, 0, st, (const float*)in, (float*)out, R, C);
}

int launch_pack(const mmoe_shape& s, const void* W1, const void* W3, const void* W2, void* W1p, void* W3p,
                void* W2p, hipStream_t st)
{
    if (s.dtype == MMOE_BF16) {
        pack_fragments(W2, W2p, s.S, s.d_ff, s.d_model, st);
        if (W3) pack_fragments(W3, W3p, s.S, s.d_model, s.d_ff, st);
        pack_fragments(W1, W1p, s.S, s.d_model, s.d_ff, st);
    } else {
        transpose(W2, W2p, s.S, s.d_ff, s.d_model, st);
        if (W3) transpose(W3, W3p, s.S, s.d_model, s.d_ff, st);
        transpose(W1, W1p, s.S, s.d_model, s.d_ff, st);
    }
    return launch_status();
}

}  // namespace mmoe
