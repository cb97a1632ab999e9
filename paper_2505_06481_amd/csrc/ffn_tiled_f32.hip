// Step F in fp32 where slots hold more rows than one pass of the streaming kernel takes: the grouped
// expert FFN on v_mfma_f32_16x16x4f32 (Algorithm 2, "expert[iL][iE](act)").
//
// Both products are  out[r, n] = sum_k A[r, k] * W[s][n][k]  over the transposed pool [S, N, K].
//
// Products with many rows per slot and enough tiles run on bf16 parts instead (ffn_split_f32.hip).
//
// What bounds it: the fp32 matrix rate (256 flop per cycle and compute unit), a sixteenth of bf16's, so a
// tile moves little per flop and the design is plain.  Tile: up to 96 token rows x 64 output features x
// 32 k per step, four wavefronts, 16 features each (of both weight matrices for the gated product, so that
// SiLU(gate)*up is lane-local) and all rows; three workgroups per compute unit (two of the gated product), one's barriers
// and epilogue behind the others' matrix instructions.  64 features rather than 128: the down product of a 768-wide
// layer has 12 feature tiles a slot, 6 would leave a third of the chip idle in the last round.
//   weights   global -> registers, a row's 128 bytes per step by four lanes, two steps ahead;
//   tokens    global -> registers two steps ahead -> LDS (three stages, 16-byte pieces xor-swizzled by
//             row & 7) -> fragments, shared by the four wavefronts.  The one barrier of a step stands
//             between its two halves, so the next step's first fragments are fetched, and this step's second
//             ones were, while matrix instructions run.
// The streaming kernel (ffn_skinny.hip) reads the weights again, and every wavefront its own copy of the token
// rows, for each 32 rows of a slot; here once for 96.
// Measured against the streaming kernel, rows spread evenly (768 x 3072, top-1, 13 slots): 260 tokens 85 -> 70 us, 416 tokens
// 117 -> 81; 1024 x 2048 SwiGLU, top-2, 13 slots, 208 tokens 141 -> 121; 2048 x 4096 SwiGLU, 8 slots, 128 tokens 281 -> 203.  At 2000
// tokens of 768 x 3072 (which run on bf16 parts) each product reached 80 of 157 TFLOP/s with the matrix pipes busy for 74 % of
// the cycles in which their compute unit had work (SQ_VALU_MFMA_BUSY_CYCLES / 4 / SQ_BUSY_CU_CYCLES).
//
// Summation: a chain of matrix instructions runs over kChain k values from zero and is then added to
// the running total, so rounding errors do not build up over the whole reduction dimension (as in the
// streaming kernel).
#include <type_traits>

#include "mmoe_internal.h"
#include "tile_table.h"

namespace mmoe {

// What a product writes: as in ffn_tiled.hip, with H in fp32.
enum { kModeReluH = 0, kModeSwigluH = 1, kModePlainF32 = 2, kModeGeluH = 3, kModeGatedY = 4 };

constexpr int kFThreads = 256;
constexpr int kFK = 32;            // k per step
constexpr int kFRing = 4;          // weight steps in registers (static indexes of an unrolled loop; two are ahead)
constexpr int kChain = 256;        // k per chain of matrix instructions
static_assert(kChain % (kFK * kFRing) == 0, "tile and unrolling");

// Workgroups per compute unit: three, as many as the token stages and the registers allow (168 of them; the tallest
// tile spills 8 to 12 more); two for the gated product, whose accumulators are twice as many (three with tiles of 64 rows
// instead: 4 to 30 % slower).
constexpr int resident(int mode) { return mode == kModeSwigluH ? 2 : 3; }

template <int MODE>
__global__ __launch_bounds__(kFThreads, resident(MODE)) void tiled_f32_kernel(
    const float* __restrict__ A, const int32_t* __restrict__ perm, int kdiv, const int32_t* __restrict__ tab, int hdr,
    int list_at, int list_stride, const float* __restrict__ W0, const float* __restrict__ W1, float* __restrict__ out,
    int K, int N, const int32_t* __restrict__ sink_perm, const float* __restrict__ sink_w)
{
    constexpr int kStage = kFRows * kFK * 4;  // bytes of a token tile
    __shared__ __attribute__((aligned(128))) char lds[3 * kStage];

    // workgroup id -> tile: entry blockIdx.x / 8 of this XCD's list
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const int4* list = reinterpret_cast<const int4*>(tab) + list_at + xcd * list_stride;
    const int n_mine = tab[hdr + xcd];
    const int4 ent = list[local];  // in bounds for every workgroup of the grid
    if (local >= n_mine) return;   // uniform over the workgroup
    const int s = ent.x & kSlotMask;
    const int nt = list_stride ? ent.y : ent.y * kXcds + xcd;
    const int r0 = ent.z, cnt = ent.w;  // first row, rows (1..96)

    constexpr int NW = MODE == kModeSwigluH ? 2 : 1;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int li = lane & 15, g = lane >> 4;
    const int n0 = nt * kFeatF32 + wave * 16;

    // Weights: lane (li, g) holds, for piece q of a step, the 4 k values 16 q + 4 g .. of feature n0 + li;
    // element c of the piece feeds matrix instruction c.  Tokens use the same order.
    const float* wrow[NW];
    wrow[0] = W0 + ((size_t)s * N + n0 + li) * K + 4 * g;
    if (NW == 2) wrow[NW - 1] = W1 + ((size_t)s * N + n0 + li) * K + 4 * g;

    auto run = [&](auto njc) {
        constexpr int NJ = decltype(njc)::value;         // 16-row fragments of the tile that hold rows
        constexpr int NP = (NJ * 16 * 8 + 255) / 256;    // 16-byte pieces of a step's tokens per thread
        // Piece i*256 + tid of a step: row (i*256 + tid) / 8, 16 bytes (tid % 8) of its 128.  Rows past the end
        // re-read the last one (never stored).
        const float* asrc[NP];
        int adst[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int row = i * 32 + (tid >> 3), q = tid & 7;
            const int r = r0 + min(row, cnt - 1);
            asrc[i] = A + (size_t)(perm ? perm[r] / kdiv : r) * K + 4 * q;
            adst[i] = row * 128 + ((q ^ (row & 7)) << 4);
        }
        int fsrc[2];  // this lane's two pieces of a fragment row
#pragma unroll
        for (int q = 0; q < 2; ++q) fsrc[q] = li * 128 + (((4 * q + g) ^ (li & 7)) << 4);

        f32x4 tot[NJ][NW], acc[NJ][NW];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                tot[j][w] = f32x4{0.f, 0.f, 0.f, 0.f};
                acc[j][w] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        const int steps = K / kFK, last = steps - 1;  // a multiple of 8
        f32x4 wr[kFRing][NW][2], ar[2][NP];
        auto load_w = [&](int slot, int t) {
            const int tt = min(t, last);  // past the end: a harmless reload
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    wr[slot][w][q] = *reinterpret_cast<const f32x4*>(wrow[w] + (size_t)tt * kFK + 16 * q);
        };
        auto load_a = [&](int slot, int t) {
            const int tt = min(t, last);
#pragma unroll
            for (int i = 0; i < NP; ++i) ar[slot][i] = *reinterpret_cast<const f32x4*>(asrc[i] + (size_t)tt * kFK);
        };
        auto put_a = [&](int slot, char* stage) {
#pragma unroll
            for (int i = 0; i < NP; ++i) *reinterpret_cast<f32x4*>(stage + adst[i]) = ar[slot][i];
        };
        f32x4 x[2][NJ];  // token fragments of the two halves of a step
        auto get_x = [&](int q, const char* stage) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) x[q][j] = *reinterpret_cast<const f32x4*>(stage + fsrc[q] + j * 2048);
        };
        auto mma = [&](int slot, int q) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int w = 0; w < NW; ++w)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[j][w] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[slot][w][q][c], x[q][j][c], acc[j][w], 0, 0, 0);
        };
        load_a(0, 0);
        load_w(0, 0);
        load_a(1, 1);
        load_w(1, 1);
        put_a(0, lds);
        load_a(0, 2);
        __syncthreads();
        get_x(0, lds);
        int cur = 0, nxt = kStage;  // stages of this step and of the next
        for (int t0 = 0; t0 < steps; t0 += kFRing) {
#pragma unroll
            for (int u = 0; u < kFRing; ++u) {
                const int t = t0 + u;
                // Stage `nxt` was last read in step t-2, which every wavefront has left (barrier of step t-1).
                put_a((u + 1) & 1, lds + nxt);  // step t+1's tokens, loaded during step t-1
                get_x(1, lds + cur);
                load_a((u + 1) & 1, t + 3);
                load_w((u + 2) % kFRing, t + 2);
                __builtin_amdgcn_sched_barrier(0);  // fetches stay in front of the matrix instructions that hide them
                mma(u, 0);
                __builtin_amdgcn_sched_barrier(0);
                __syncthreads();  // step t+1's tokens are in stage `nxt`
                get_x(0, lds + nxt);
                __builtin_amdgcn_sched_barrier(0);
                mma(u, 1);
                __builtin_amdgcn_sched_barrier(0);
                cur = nxt;
                nxt = nxt == 2 * kStage ? 0 : nxt + kStage;
            }
            if ((t0 + kFRing) * kFK % kChain == 0) {  // uniform: a chain ends
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        tot[j][w] += acc[j][w];
                        acc[j][w] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
        }

        // accumulator element i of lane (li, g): feature n0 + 4 g + i of token row li of the fragment
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int row = j * 16 + li;
            if (row >= cnt) continue;
            int orow = r0 + row;
            float gw = 0.0f;
            if (MODE == kModeGatedY) {
                orow = sink_perm[orow];
                gw = sink_w[orow];
            }
            f32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = tot[j][0][i];
                if (MODE == kModeSwigluH) o[i] = v / (1.0f + __expf(-v)) * tot[j][NW - 1][i];
                else if (MODE == kModeReluH) o[i] = fmaxf(v, 0.0f);
                else if (MODE == kModeGeluH) o[i] = 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f));
                else if (MODE == kModeGatedY) o[i] = __builtin_fmaf(gw, v, 0.0f);
                else o[i] = v;
            }
            *reinterpret_cast<f32x4*>(out + (size_t)orow * N + n0 + 4 * g) = o;
        }
    };
    switch ((cnt + 15) / 16) {  // uniform over the workgroup
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        default: run(std::integral_constant<int, 1>{}); break;
    }
}

template <int MODE>
static void launch_product(const TiledPlan& p, int prod, const void* A, const int32_t* perm, int kdiv, const int32_t* tab,
                           const void* W0, const void* W1, void* out, int K, int N, hipStream_t st,
                           GateSink sink = GateSink())
{
    hipLaunchKernelGGL((tiled_f32_kernel<MODE>), dim3(p.L.len[prod] * kXcds), dim3(kFThreads), 0, st, (const float*)A, perm,
                       kdiv, tab, kXcds * prod, p.L.list[prod], p.L.lists[prod] == 1 ? 0 : p.L.len[prod], (const float*)W0,
                       (const float*)W1, (float*)out, K, N, sink.perm, sink.w);
}

void launch_up_f32(const mmoe_shape& s, const TiledPlan& p, const void* rows, const int32_t* perm, const int32_t* tab,
                   const void* W1p, const void* W3p, void* H, hipStream_t st)
{
    const int d = s.d_model, f = s.d_ff;
    if (s.act == MMOE_SWIGLU) launch_product<kModeSwigluH>(p, 0, rows, perm, s.top_k, tab, W1p, W3p, H, d, f, st);
    else if (s.act == MMOE_GELU) launch_product<kModeGeluH>(p, 0, rows, perm, s.top_k, tab, W1p, nullptr, H, d, f, st);
    else launch_product<kModeReluH>(p, 0, rows, perm, s.top_k, tab, W1p, nullptr, H, d, f, st);
}

void launch_down_f32(const mmoe_shape& s, const TiledPlan& p, const int32_t* tab, const void* W2p, const void* H, float* Yg,
                     hipStream_t st, GateSink sink)
{
    const int d = s.d_model, f = s.d_ff;
    if (sink.w) launch_product<kModeGatedY>(p, 1, H, nullptr, 1, tab, W2p, nullptr, sink.Y, f, d, st, sink);
    else launch_product<kModePlainF32>(p, 1, H, nullptr, 1, tab, W2p, nullptr, Yg, f, d, st);
}

}  // namespace mmoe
