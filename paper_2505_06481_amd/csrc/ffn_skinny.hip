// Step F, weight-streaming variant: the grouped expert FFN when a slot sees only a few
// rows (decode-shaped batches) -- Algorithm 2, "expert[iL][iE](act)".  Each expert's
// weights are then read from HBM exactly once and that read is the whole cost, so the
// kernel is built around keeping many 16-byte loads of weights in flight per wavefront.
//
// Both products are of the form  out[r, n] = sum_k A[r, k] * W[s][n][k]  over the packed
// pool.  A workgroup owns a block of output features n of one slot and all rows of that
// slot; its four wavefronts split the reduction dimension and meet in LDS.  The weight rows
// are the row operand of a matrix-core instruction and the tokens its columns, so the
// weights pass through registers once however many tokens (up to 32 per pass) the slot holds.
// In the fused layer the token rows of the first product are read through the grouping
// permutation (row perm[r] / top_k of X) instead of from a gathered copy.
//
// Self-grouping mode (decode-sized batches of the fused layer): no grouping kernel runs at
// all.  The router has written slot[p] for every pair; a workgroup collects the pairs of its
// slot itself, in ascending pair id (which is the stable order of the grouped form), and the
// intermediates H and Yg are indexed by pair id instead of by grouped row.  Every row is still
// summed in the same order, so the layer's output is bit-identical to the staged path's.
//
// fp32 kernel (skinny_kernel): transposed pool [S, N, K], 16 features per wavefront,
// 16x16x4 matrix instructions, one or two 16-row token blocks per pass; see its own comment.
//
// bf16 kernel (skinny_frag_kernel): fragment-packed pool, 32 features per workgroup,
// 32x32x16 matrix instructions, up to 32 rows per pass; see its own comment.
#include <type_traits>

#include "mmoe_internal.h"

namespace mmoe {

// What a product writes: H = act(.) in the storage type (up product), plain fp32 rows of Yg (down
// product), or, for layers with top_k = 1, the layer's output rows themselves: 0 + w[token] * y in the
// storage type at row token (GateSink).
enum { kModeReluH = 0, kModeSwigluH = 1, kModePlainF32 = 2, kModeGeluH = 3, kModeGatedY = 4 };

constexpr int kSkThreads = 256;
constexpr int kSkWaves = 4;
constexpr int kSkMB = 2;  // 16-row token blocks per pass

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }
__device__ __forceinline__ float gelu(float a) { return 0.5f * a * (1.0f + erff(a * 0.70710678118654752440f)); }

constexpr int kSelfMaxP = 1024;  // most pairs for which the expert kernels group by themselves

// Rows of one slot.  Grouped form: rows [r0, r0 + cnt) of the grouped order; input row of grouped
// row r is r itself, or perm[r] / kdiv (gather folded into the loads).  Self-grouping form: the
// pairs p with slot_of_pair[p] == s, ascending, collected into `mine` by the first
// wavefront (ballot + popcount ranks); input row p / kdiv, output row p.
struct RowSet {
    int r0, cnt;
    const int32_t* perm;
    int kdiv;
    const int* mine;  // LDS list of pair ids, or null in the grouped form
    __device__ __forceinline__ int in_row(int rr) const
    {
        if (mine) return mine[rr] / kdiv;
        return perm ? perm[r0 + rr] / kdiv : r0 + rr;
    }
    __device__ __forceinline__ int out_row(int rr) const { return mine ? mine[rr] : r0 + rr; }
};

// The slot of this workgroup: blockIdx.y, or, where the batch has fewer pairs than the pool has slots (`by_pair`), the
// slot of pair blockIdx.y (the workgroups of a pair that is not the first of its slot then find no rows).
__device__ __forceinline__ int slot_of_block(const int32_t* __restrict__ slot_of_pair, bool by_pair)
{
    return by_pair ? slot_of_pair[blockIdx.y] : (int)blockIdx.y;
}

// Called by the whole workgroup.
__device__ __forceinline__ RowSet slot_rows(const int32_t* __restrict__ offsets, const int32_t* __restrict__ perm,
                                            int kdiv, const int32_t* __restrict__ slot_of_pair, int P, int s,
                                            bool by_pair, int* mine, SlotFilter filt)
{
    RowSet rs;
    rs.perm = perm;
    rs.kdiv = kdiv;
    rs.mine = nullptr;
    if (filt.skips(s)) {  // uniform over the workgroup: this launch leaves the slot to another one
        rs.r0 = 0;
        rs.cnt = 0;
        return rs;
    }
    if (!slot_of_pair) {
        rs.r0 = offsets[s];
        rs.cnt = offsets[s + 1] - rs.r0;
        return rs;
    }
    __shared__ int hits;
    if (threadIdx.x < kWave) {
        constexpr int kAtOnce = 4;  // loads of 64 pairs
        int n = 0;
        for (int p0 = threadIdx.x; p0 < P + (int)threadIdx.x; p0 += kAtOnce * kWave) {  // uniform over the wavefront
            int got[kAtOnce];
#pragma unroll
            for (int j = 0; j < kAtOnce; ++j) got[j] = p0 + j * kWave < P ? slot_of_pair[p0 + j * kWave] : -1;
#pragma unroll
            for (int j = 0; j < kAtOnce; ++j) {
                const unsigned long long m = __ballot(got[j] == s);
                if (got[j] == s) mine[n + __popcll(m & ((1ull << threadIdx.x) - 1ull))] = p0 + j * kWave;
                n += __popcll(m);
            }
        }
        if (threadIdx.x == 0) hits = n;
    }
    __syncthreads();
    rs.r0 = 0;
    rs.cnt = by_pair && mine[0] != (int)blockIdx.y ? 0 : hits;
    rs.mine = mine;
    return rs;
}

// NT: the weights of a slot with one pass are read past the caches, at 6.5 to 6.9 TB/s instead of 5.9 (4096 x 14336, 13
// slots: 64 tokens 768 -> 698 us, one token 135 -> 121; 2048 x 1280, 90 slots, 60 tokens 200 -> 179; fp32 768 x 3072, 13 slots,
// 128 tokens 62.7 -> 59.1).  A slot with more rows than a pass takes has its weights read again by every pass, from L2 if
// they came through it (unequal slots: 2048 x 2048 SwiGLU, 13 slots, 200 tokens 109.4 us past the caches in every pass, 92.5
// with several passes through them; 4096 x 14336, 100 tokens 865 : 798; fp32 768 x 3072, 150 tokens 117 : 100).
template <bool NT, typename T>
__device__ __forceinline__ T load_weights(const T* p)
{
    return NT ? __builtin_nontemporal_load(p) : *p;
}

// Unless the batch is expected to touch so little of the pool that the 256 MB last-level cache may still hold it from an
// earlier step: 768 x 3072, 16 slots of 9.4 MB, three pools in turn, cached : past the caches, us: 18.1 : 20.0 with 5 tokens,
// 21.4 : 23.8 with 10, 27.9 : 31.2 with 16, 36.8 : 34.9 with 40; slots of 101 MB, 8 of them, one pick 35.6 : 34.9, two picks
// 48.4 : 42.9; of 235 MB, 9 of them, one pick 59.6 : 52.5.  (P S / (P + S), fractions and all, is a little below the number
// of slots that P picks touch.)
constexpr int64_t kCachedBytes = (int64_t)96 << 20;
bool past_the_caches(const mmoe_shape& s)
{
    const double P = (double)s.T * s.top_k;
    return P * s.S / (P + s.S) * (double)slot_bytes(s) > (double)kCachedBytes;
}

constexpr int skinny_threads(int split) { return split == 8 ? 8 * kWave : kSkThreads; }

// SPLIT 4, 8: so many wavefronts split the reduction dimension of one 16-feature block and meet in
// LDS (long reductions).  1: every wavefront of four owns a 16-feature block of its own and walks the
// whole reduction dimension (K = 256, of which a quarter is a single run: see whole_k): 64 features per workgroup, no
// LDS reduction.
//
// What bounds it is the memory pipeline of a compute unit.  A 1 KB load instruction takes 18 to 20 of its cycles
// where four neighbouring lanes read 64 contiguous bytes and 65 where neighbouring lanes are in different rows, as
// in the order of a matrix operand (measured on data in L2).  So weight and token rows are read along the row, 16
// lanes to the 256 bytes of a run of 64 k, and pass through LDS of the wavefront's own to get into operand order.
// One run is in flight per wavefront, twelve wavefronts on a compute unit (eight of the gated product): with two
// runs in flight the registers (over 168) leave eight, or spill.
// Measured against reading both operands in operand order (768 x 3072 top-1, 13 slots, layer): 4 tokens 36.0 -> 25.6 us
// (21.9 with eight wavefronts in the down product), 24 tokens 66.9 -> 49.2, 128 tokens 79.2 -> 60.5 (246 MB of weights);
// 1024 x 2048 SwiGLU top-2, 64 tokens 97.3 -> 86.
constexpr int kRun = 64;              // k per run
constexpr int kRunRow = kRun * 4;     // bytes of a row per run
constexpr int kRunBlock = 16 * kRunRow;  // bytes of 16 rows
constexpr int kRunLoads = 4;          // load instructions per 16 rows; pieces of an operand per run
constexpr int kChainRuns = 4;         // runs per chain of matrix instructions: rounding errors do not build up over all of K

template <int NW, int MODE, int SPLIT, bool NT>
__global__ __launch_bounds__(skinny_threads(SPLIT), SPLIT == 8 ? 1 : NW == 1 ? 3 : 2) void skinny_kernel(const float* __restrict__ A,
                                                            const int32_t* __restrict__ perm, int kdiv,
                                                            const int32_t* __restrict__ offsets,
                                                            const int32_t* __restrict__ slot_of_pair, int P, int by_pair,
                                                            const float* __restrict__ W0, const float* __restrict__ W1,
                                                            float* __restrict__ out, int K, int N, SlotFilter filt,
                                                            const int32_t* __restrict__ sink_perm,
                                                            const float* __restrict__ sink_w)
{
    constexpr int kWaves = skinny_threads(SPLIT) / kWave;
    __shared__ __attribute__((aligned(256))) char rows[kWaves][(NW + kSkMB) * kRunBlock];  // of a run: weights, tokens
    static_assert(sizeof(rows) >= sizeof(float) * kWaves * kSkMB * NW * kWave * 4, "one array for the partial sums too");
    float(*red)[kSkMB][NW][kWave][4] = reinterpret_cast<float(*)[kSkMB][NW][kWave][4]>(&rows[0][0]);
    __shared__ int mine[kSelfMaxP];

    const int s = slot_of_block(slot_of_pair, by_pair);
    const RowSet rs = slot_rows(offsets, perm, kdiv, slot_of_pair, P, s, by_pair, mine, filt);
    const int cnt = rs.cnt;
    if (cnt <= 0) return;  // uniform over the workgroup

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int n0 = SPLIT > 1 ? blockIdx.x * 16 : (blockIdx.x * kWaves + wave) * 16;
    const int li = lane & 15, g = lane >> 4;
    constexpr int kStride = SPLIT;  // runs between two of one wavefront
    const int first = SPLIT > 1 ? wave : 0;
    const int nrun = K / kRun;

    // Load i of a 16-row block: row 4 i + g, 16 bytes (li) of its 256.  In LDS piece q of row r stands at q ^ r: the
    // 16 lanes that share a cycle of a read or write have 16 different columns of 256 bytes.
    const float* wrow[NW][kRunLoads];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int i = 0; i < kRunLoads; ++i)
            wrow[w][i] = (w == 0 ? W0 : W1) + ((size_t)s * N + n0 + 4 * i + g) * K + 4 * li;
    char* const myrows = rows[wave];
    int dst[kRunLoads], src[kRunLoads];  // of load i; of piece q of an operand: lane (li, g) holds the four k from 16 q + 4 g on of row li
#pragma unroll
    for (int i = 0; i < kRunLoads; ++i) {
        dst[i] = (4 * i + g) * kRunRow + ((li ^ (4 * i + g)) << 4);
        src[i] = li * kRunRow + (((4 * i + g) ^ li) << 4);
    }

    f32x4 wraw[NW][kRunLoads];  // a run's weights as loaded
    auto load_w = [&](int run, auto ntc) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int i = 0; i < kRunLoads; ++i) wraw[w][i] = load_weights<decltype(ntc)::value>(reinterpret_cast<const f32x4*>(wrow[w][i] + (size_t)run * kRun));
    };

    auto pass = [&](int pass0, auto mbc, auto ntc) {
        constexpr int MB = decltype(mbc)::value;  // 16-row blocks of this pass that hold rows
        const float* arow[MB][kRunLoads];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < kRunLoads; ++i) {  // rows past the end re-read the last one; never stored
                const int rr = min(pass0 + mb * 16 + 4 * i + g, cnt - 1);
                arow[mb][i] = A + (size_t)rs.in_row(rr) * K + 4 * li;
            }
        f32x4 tot[MB][NW], acc[MB][NW];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int w = 0; w < NW; ++w) tot[mb][w] = acc[mb][w] = f32x4{0.f, 0.f, 0.f, 0.f};

        f32x4 traw[MB][kRunLoads];  // a run's tokens as loaded
        auto load_t = [&](int run) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < kRunLoads; ++i) traw[mb][i] = *reinterpret_cast<const f32x4*>(arow[mb][i] + (size_t)run * kRun);
        };
        // A wavefront's LDS operations execute in program order; the fences keep the compiler from moving them.
        auto fence = [] {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        auto step = [&](int next) {  // the run in the registers; `next` is fetched during its arithmetic if there is one
            fence();
#pragma unroll
            for (int i = 0; i < kRunLoads; ++i) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4*>(myrows + (NW + mb) * kRunBlock + dst[i]) = traw[mb][i];
#pragma unroll
                for (int w = 0; w < NW; ++w) *reinterpret_cast<f32x4*>(myrows + w * kRunBlock + dst[i]) = wraw[w][i];
            }
            fence();
            if (next >= 0) {
                load_t(next);
                load_w(next, ntc);
            }
#pragma unroll
            for (int q = 0; q < kRunLoads; ++q) {
                f32x4 x[MB], wf[NW];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) x[mb] = *reinterpret_cast<const f32x4*>(myrows + (NW + mb) * kRunBlock + src[q]);
#pragma unroll
                for (int w = 0; w < NW; ++w) wf[w] = *reinterpret_cast<const f32x4*>(myrows + w * kRunBlock + src[q]);
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int w = 0; w < NW; ++w)
                            acc[mb][w] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[w][c], x[mb][c], acc[mb][w], 0, 0, 0);
            }
        };
        // a chain of matrix instructions runs over kChainRuns runs from zero and is then added to the total
        auto end_chain = [&] {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    tot[mb][w] += acc[mb][w];
                    acc[mb][w] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        };
        int run = first, chain = 0;  // a wavefront has at least one run: K >= 256, or 512 with eight of them
        load_t(run);
        load_w(run, ntc);
        for (; run + kStride < nrun; run += kStride) {
            step(run + kStride);
            if (++chain % kChainRuns == 0) end_chain();  // uniform
        }
        step(-1);
        end_chain();

        // accumulator element i of lane l is output feature n0 + 4*(l/16) + i of token column l%16
        auto finish = [&](int row, int l, const float (&v)[NW][4]) {
            float o[4];
            int orow = rs.out_row(row);
            float gw = 0.0f;
            if (MODE == kModeGatedY) {
                if (sink_perm) orow = sink_perm[orow];
                gw = sink_w[orow];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (MODE == kModeSwigluH) o[i] = silu_mul(v[0][i], v[NW - 1][i]);
                else if (MODE == kModeReluH) o[i] = fmaxf(v[0][i], 0.0f);
                else if (MODE == kModeGeluH) o[i] = gelu(v[0][i]);
                else if (MODE == kModeGatedY) o[i] = __builtin_fmaf(gw, v[0][i], 0.0f);
                else o[i] = v[0][i];
            }
            *reinterpret_cast<f32x4*>(out + (size_t)orow * N + n0 + 4 * (l >> 4)) = f32x4{o[0], o[1], o[2], o[3]};
        };
        if (SPLIT == 1) {  // every wavefront finishes its own 16 features straight from its accumulators
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const int row = pass0 + mb * 16 + (lane & 15);
                if (row < cnt) {
                    float v[NW][4];
#pragma unroll
                    for (int w = 0; w < NW; ++w)
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[w][i] = tot[mb][w][i];
                    finish(row, lane, v);
                }
            }
            return;
        }
        __syncthreads();  // the partial sums take the place of the tokens
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[wave][mb][w][lane][i] = tot[mb][w][i];
        __syncthreads();
        for (int idx = threadIdx.x; idx < MB * kWave; idx += skinny_threads(SPLIT)) {
            const int mb = idx / kWave, l = idx % kWave;
            const int row = pass0 + mb * 16 + (l & 15);
            if (row < cnt) {
                float v[NW][4];
#pragma unroll
                for (int w = 0; w < NW; ++w)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                    {
                        v[w][i] = (red[0][mb][w][l][i] + red[1][mb][w][l][i]) + (red[2][mb][w][l][i] + red[3][mb][w][l][i]);
                        if constexpr (SPLIT == 8)
                            v[w][i] += (red[4][mb][w][l][i] + red[5][mb][w][l][i]) + (red[6][mb][w][l][i] + red[7][mb][w][l][i]);
                    }
                finish(row, l, v);
            }
        }
        __syncthreads();
    };
    auto passes = [&](auto ntc) {
        for (int pass0 = 0; pass0 < cnt; pass0 += 16 * kSkMB) {  // uniform over the workgroup
            if (cnt - pass0 > 16) pass(pass0, std::integral_constant<int, 2>{}, ntc);
            else pass(pass0, std::integral_constant<int, 1>{}, ntc);
        }
    };
    if (NT && cnt <= 16 * kSkMB) passes(std::true_type{});  // uniform
    else passes(std::false_type{});
}

// ---- bf16 on the fragment-packed pool ----------------------------------------------------
// Workgroup = one 32-row block of weights (32 output features) of one slot, all rows of the
// slot.  The block's fragments lie one after the other in memory (1 KB each, 16 k per
// fragment), so the four wavefronts take runs of 4 fragments (64 k) in turn and every
// weight load is a fully contiguous 1 KB read that goes straight into the matrix-core
// operand registers.  Tokens are the 32-column operand: lane (token l%32, half h = l/32)
// reads the 64 contiguous bytes of its activation row that the run's permutation assigns
// to it.  Partial sums of the four wavefronts meet in LDS.
template <int NW, int KU, int MODE, bool NT>
__global__ __launch_bounds__(kSkThreads) void skinny_frag_kernel(const uint16_t* __restrict__ A,
                                                                 const int32_t* __restrict__ perm, int kdiv,
                                                                 const int32_t* __restrict__ offsets,
                                                                 const int32_t* __restrict__ slot_of_pair, int P, int by_pair,
                                                                 const uint16_t* __restrict__ W0,
                                                                 const uint16_t* __restrict__ W1,
                                                                 void* __restrict__ out, int K, int N,
                                                                 SlotFilter filt,
                                                                 const int32_t* __restrict__ sink_perm,
                                                                 const float* __restrict__ sink_w)
{
    __shared__ float red[kSkWaves][NW][kWave][16];  // 16 KB per matrix
    __shared__ int mine[kSelfMaxP];

    const int s = slot_of_block(slot_of_pair, by_pair);
    const int nb = blockIdx.x;
    const RowSet rs = slot_rows(offsets, perm, kdiv, slot_of_pair, P, s, by_pair, mine, filt);
    const int cnt = rs.cnt;
    if (cnt <= 0) return;  // uniform over the workgroup

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int tok = lane & 31, h = lane >> 5;
    const int nit = K / (64 * KU);  // iterations of KU runs of 64 k

    // fragment ks of this block: element offset ((s*(N/32) + nb)*(K/16) + ks)*512 + lane*8
    const size_t blk = ((size_t)s * (N / 32) + nb) * (size_t)(K / 16) * 512 + (size_t)lane * 8;
    const uint16_t* wrow[NW];
    wrow[0] = W0 + blk;
    if (NW == 2) wrow[NW - 1] = W1 + blk;

    u32x4 wcur[NW][KU][4], wnxt[NW][KU][4];
    auto load_w = [&](u32x4 (&to)[NW][KU][4], int it, auto ntc) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int u = 0; u < KU; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    to[w][u][q] = load_weights<decltype(ntc)::value>(reinterpret_cast<const u32x4*>(wrow[w] + ((size_t)(it * KU + u) * 4 + q) * 512));
    };

    auto pass = [&](int pass0, auto ntc) {
        const int rr = min(pass0 + tok, cnt - 1);  // tokens past the end re-read the last one; never stored
        const uint16_t* arow = A + (size_t)rs.in_row(rr) * K + h * 32;
        f32x16 acc[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[w][e] = 0.0f;

        // The last step stands alone, so that the waits of the others leave the next weights in flight (a load that may not
        // be there is waited for): down product of 768 x 3072, 4 slots of 32 rows 18.7 -> 17.0 us; 13 slots, 200 tokens
        // spread unequally, layer 88.4 -> 79.1.  Not past the caches (4096 x 14336, 9 slots, 16 tokens spread unequally 326 -> 343),
        // and not for the gated product, whose accumulators then move between registers (4096 x 14336, one token 76.1 -> 83.0).
        constexpr bool kPeel = NW == 1 && !decltype(ntc)::value;
        auto step = [&](int it, bool more) {
            u32x4 xa[KU][4];
#pragma unroll
            for (int u = 0; u < KU; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    xa[u][q] = *reinterpret_cast<const u32x4*>(arow + (size_t)(it * KU + u) * 64 + q * 8);
            if (more) load_w(wnxt, it + kSkWaves, ntc);  // the youngest loads, still in flight during the math below
            if (kPeel) __builtin_amdgcn_sched_barrier(0);  // all loads stay in front of the matrix instructions
#pragma unroll
            for (int u = 0; u < KU; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int w = 0; w < NW; ++w)
                        acc[w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wcur[w][u][q]),
                                                                         __builtin_bit_cast(bf16x8, xa[u][q]), acc[w],
                                                                         0, 0, 0);
            if (!more) return;
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int u = 0; u < KU; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) wcur[w][u][q] = wnxt[w][u][q];
        };
        int it = wave;
        if (it < nit) load_w(wcur, it, ntc);
        if (kPeel) {
            for (; it + kSkWaves < nit; it += kSkWaves) step(it, true);
            if (it < nit) step(it, false);
        } else {
            for (; it < nit; it += kSkWaves) step(it, it + kSkWaves < nit);
        }

#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int e = 0; e < 16; ++e) red[wave][w][lane][e] = acc[w][e];
        __syncthreads();
        // accumulator element e of lane l: feature 8*(e/4) + 4*(l/32) + e%4 of token column l%32.
        // Thread (l = tid%64, q = tid/64) finishes elements 4q .. 4q+3 of lane l: 4 consecutive features.
        {
            const int l = threadIdx.x & 63, q = threadIdx.x >> 6;
            const int row = pass0 + (l & 31);
            if (row < cnt) {
                float o[4];
                int orow = rs.out_row(row);
                float gw = 0.0f;
                if (MODE == kModeGatedY) {
                    if (sink_perm) orow = sink_perm[orow];
                    gw = sink_w[orow];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = 4 * q + i;
                    float v[NW];
#pragma unroll
                    for (int w = 0; w < NW; ++w)
                        v[w] = (red[0][w][l][e] + red[1][w][l][e]) + (red[2][w][l][e] + red[3][w][l][e]);
                    if (MODE == kModeSwigluH) o[i] = silu_mul(v[0], v[NW - 1]);
                    else if (MODE == kModeReluH) o[i] = fmaxf(v[0], 0.0f);
                    else if (MODE == kModeGeluH) o[i] = gelu(v[0]);
                    else if (MODE == kModeGatedY) o[i] = __builtin_fmaf(gw, v[0], 0.0f);
                    else o[i] = v[0];
                }
                const size_t at = (size_t)orow * N + nb * 32 + 8 * q + 4 * (l >> 5);
                if (MODE == kModePlainF32) {
                    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + at) = f32x4{o[0], o[1], o[2], o[3]};
                } else {
                    u32x2 pk;
                    pk[0] = (uint32_t)f32_to_bf16_bits(o[0]) | ((uint32_t)f32_to_bf16_bits(o[1]) << 16);
                    pk[1] = (uint32_t)f32_to_bf16_bits(o[2]) | ((uint32_t)f32_to_bf16_bits(o[3]) << 16);
                    *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(out) + at) = pk;
                }
            }
        }
        __syncthreads();
    };
    if (NT && cnt <= 32) {  // uniform
        pass(0, std::true_type{});
    } else {
        for (int pass0 = 0; pass0 < cnt; pass0 += 32) pass(pass0, std::false_type{});  // uniform over the workgroup
    }
}

template <bool NT>
static int run_skinny_bf16(const mmoe_shape& s, const void* rows, const int32_t* perm, const int32_t* offsets,
                           const int32_t* slot_of_pair, const void* W1p, const void* W3p, const void* W2p, void* H,
                           float* Yg, hipStream_t st, hipEvent_t mid, SlotFilter filt, GateSink sink)
{
    const int32_t* nosink = nullptr;
    const float* now = nullptr;
    const int32_t* noperm = nullptr;
    const int d = s.d_model, f = s.d_ff, P = s.T * s.top_k;
    dim3 block(kSkThreads);
    const int by_pair = slot_of_pair && P < s.S;  // a workgroup row per pair, not per slot
    const int ny = by_pair ? P : s.S;
    dim3 g1(f / 32, ny), g2(d / 32, ny);
    const uint16_t* nul = nullptr;
    if (s.act == MMOE_SWIGLU)
        hipLaunchKernelGGL((skinny_frag_kernel<2, 1, kModeSwigluH, NT>), g1, block, 0, st, (const uint16_t*)rows, perm,
                           s.top_k, offsets, slot_of_pair, P, by_pair, (const uint16_t*)W1p, (const uint16_t*)W3p, H, d, f, filt,
                           nosink, now);
    else if (s.act == MMOE_GELU)
        hipLaunchKernelGGL((skinny_frag_kernel<1, 2, kModeGeluH, NT>), g1, block, 0, st, (const uint16_t*)rows, perm,
                           s.top_k, offsets, slot_of_pair, P, by_pair, (const uint16_t*)W1p, nul, H, d, f, filt, nosink, now);
    else
        hipLaunchKernelGGL((skinny_frag_kernel<1, 2, kModeReluH, NT>), g1, block, 0, st, (const uint16_t*)rows, perm,
                           s.top_k, offsets, slot_of_pair, P, by_pair, (const uint16_t*)W1p, nul, H, d, f, filt, nosink, now);
    if (mid && hipEventRecord(mid, st) != hipSuccess) return MMOE_ERR_LAUNCH;
    if (sink.w)
        hipLaunchKernelGGL((skinny_frag_kernel<1, 2, kModeGatedY, NT>), g2, block, 0, st, (const uint16_t*)H, noperm, 1,
                           offsets, slot_of_pair, P, by_pair, (const uint16_t*)W2p, nul, sink.Y, f, d, filt, sink.perm, sink.w);
    else
        hipLaunchKernelGGL((skinny_frag_kernel<1, 2, kModePlainF32, NT>), g2, block, 0, st, (const uint16_t*)H, noperm, 1,
                           offsets, slot_of_pair, P, by_pair, (const uint16_t*)W2p, nul, (void*)Yg, f, d, filt, nosink, now);
    return launch_status();
}

template <int SPLIT, bool NT>
static void launch_skinny_products(const mmoe_shape& s, const void* rows, const int32_t* perm, const int32_t* offsets,
                                   const int32_t* slot_of_pair, const void* W1p, const void* W3p, const void* W2p,
                                   void* H, float* Yg, hipStream_t st, hipEvent_t mid, SlotFilter filt, bool up,
                                   bool down, GateSink sink)
{
    const int32_t* nosink = nullptr;
    const float* now = nullptr;
    const int32_t* noperm = nullptr;
    const int d = s.d_model, f = s.d_ff, P = s.T * s.top_k;
    constexpr int kFeat = SPLIT > 1 ? 16 : 16 * kSkWaves;  // output features per workgroup
    dim3 block(skinny_threads(SPLIT));
    const int by_pair = slot_of_pair && P < s.S;  // a workgroup row per pair, not per slot
    const int ny = by_pair ? P : s.S;
    dim3 g1(f / kFeat, ny), g2(d / kFeat, ny);
    const float* nul = nullptr;
    if (up) {
        if (s.act == MMOE_SWIGLU)
            hipLaunchKernelGGL((skinny_kernel<2, kModeSwigluH, SPLIT, NT>), g1, block, 0, st, (const float*)rows, perm,
                               s.top_k, offsets, slot_of_pair, P, by_pair, (const float*)W1p, (const float*)W3p, (float*)H, d, f, filt,
                               nosink, now);
        else if (s.act == MMOE_GELU)
            hipLaunchKernelGGL((skinny_kernel<1, kModeGeluH, SPLIT, NT>), g1, block, 0, st, (const float*)rows, perm,
                               s.top_k, offsets, slot_of_pair, P, by_pair, (const float*)W1p, nul, (float*)H, d, f, filt, nosink, now);
        else
            hipLaunchKernelGGL((skinny_kernel<1, kModeReluH, SPLIT, NT>), g1, block, 0, st, (const float*)rows, perm,
                               s.top_k, offsets, slot_of_pair, P, by_pair, (const float*)W1p, nul, (float*)H, d, f, filt, nosink, now);
    }
    if (down && sink.w)
        hipLaunchKernelGGL((skinny_kernel<1, kModeGatedY, SPLIT, NT>), g2, block, 0, st, (const float*)H, noperm, 1,
                           offsets, slot_of_pair, P, by_pair, (const float*)W2p, nul, (float*)sink.Y, f, d, filt, sink.perm, sink.w);
    else if (down)
        hipLaunchKernelGGL((skinny_kernel<1, kModePlainF32, SPLIT, NT>), g2, block, 0, st, (const float*)H, noperm, 1,
                           offsets, slot_of_pair, P, by_pair, (const float*)W2p, nul, Yg, f, d, filt, nosink, now);
    (void)mid;
}

// Split four ways a product has four times the workgroups, so slots with many rows (passes of 32 that one workgroup
// does one after the other) and the last round leave less of the chip idle.  Whole : split, us, rows spread evenly / unequally
// (router bias 1): 1024 x 1024, 8 slots, 12 tokens 35.1 : 24.1 / 34.9 : 19.3; 768 x 3072, 13 slots, 4 tokens 26.3 : 21.9, 64 tokens
// 52.7 : 55.4 / 70.6 : 58.0, 128 tokens 59.3 : 60.4 / 111 : 82; 32 slots, 200 tokens 113 : 121 / 125 : 103; 512 x 512, 110 slots,
// 802 tokens 75.8 : 81.9 / 429 : 166; SwiGLU 512 x 4864, 9 slots 71.8 : 70.7, 1024 x 1024, 24 slots, 160 pairs 68.1 : 83.3 /
// 145 : 66.  Evenly spread rows are up to a fifth faster whole, unequal ones up to 2.6 times as fast split; the host does not know
// the counts.  K = 256 split is one run per wavefront, all latency: 256 x 4096, 30 tokens 27.5 : 33.1 / 29.6 : 28.7; 256 x 1024,
// 60 slots, 240 pairs 46.4 : 51.0 / 38.7 : 36.0.
static bool whole_k(int K) { return K <= 256; }

// With at most one workgroup for each of the 256 compute units, eight wavefronts instead of four: each has one run of 4 KB
// of weights in flight, and four of them do not cover the latency of memory.  Four : eight, us, workgroups of up, down: one
// token, top-1, 4096 x 14336 (896, 256) 123 : 98; 4096 x 4096 (256, 256) 48.2 : 42.3; 256 x 4096 (up whole, 16) 24.9 : 19.9; 768 x
// 3072 (192, 48) 22.3 : 17.3.  With more of them a compute unit has its wavefronts anyway: top-2, 4096 x 4096 (512, 512)
// 69.4 : 76.9; two tokens 2048 x 8192 (2048, 512) 99.5 : 111.1; 4 tokens 768 x 3072 (1536, 384) 41.7 : 48.1.
bool eight_waves(const mmoe_shape& s, int N)
{
    const int64_t P = (int64_t)s.T * s.top_k;
    return (P < s.S ? P : s.S) * (N / 16) <= 256;
}

template <bool NT>
static int run_skinny_f32(const mmoe_shape& s, const void* rows, const int32_t* perm, const int32_t* offsets,
                      const int32_t* slot_of_pair, const void* W1p, const void* W3p, const void* W2p, void* H, float* Yg,
                      hipStream_t st, hipEvent_t mid, SlotFilter filt, GateSink sink)
{
    const auto product = [&](int K, int N, bool up) {
        const auto go = whole_k(K) ? launch_skinny_products<1, NT> : eight_waves(s, N) ? launch_skinny_products<8, NT> : launch_skinny_products<4, NT>;
        go(s, rows, perm, offsets, slot_of_pair, W1p, W3p, W2p, H, Yg, st, mid, filt, up, !up, sink);
    };
    product(s.d_model, s.d_ff, true);
    if (mid && hipEventRecord(mid, st) != hipSuccess) return MMOE_ERR_LAUNCH;
    product(s.d_ff, s.d_model, false);
    return launch_status();
}

bool self_grouping(const mmoe_shape& s)
{
    return use_skinny(s) && (int64_t)s.T * s.top_k <= kSelfMaxP;
}

int launch_ffn_skinny(const mmoe_shape& s, const void* rows, const int32_t* perm, const int32_t* offsets,
                      const int32_t* slot_of_pair, const void* W1p, const void* W3p, const void* W2p, void* H,
                      float* Yg, hipStream_t st, hipEvent_t mid, SlotFilter filt, GateSink sink)
{
    if (slot_of_pair && (int64_t)s.T * s.top_k > kSelfMaxP) return MMOE_ERR_LIMIT;
    // gated output rows: one pick per token; the grouped form needs the permutation, the self-grouping form must not have one
    if (sink.w && (s.top_k != 1 || !sink.Y || (slot_of_pair != nullptr) != (sink.perm == nullptr))) return MMOE_ERR_DIM;
    const auto run = s.dtype == MMOE_BF16 ? (past_the_caches(s) ? run_skinny_bf16<true> : run_skinny_bf16<false>)
                                          : (past_the_caches(s) ? run_skinny_f32<true> : run_skinny_f32<false>);
    return run(s, rows, perm, offsets, slot_of_pair, W1p, W3p, W2p, H, Yg, st, mid, filt, sink);
}

}  // namespace mmoe
