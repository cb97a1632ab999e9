// Step F in fp32 where slots hold many rows: the grouped expert FFN (Algorithm 2, "expert[iL][iE](act)") on the bf16
// matrix instruction v_mfma_f32_16x16x32_bf16.
//
// Both products are  out[r, n] = sum_k A[r, k] * W[s][n][k]  over the transposed pool [S, N, K], fp32 in memory.
//
// Arithmetic.  The fp32 matrix instruction runs at a sixteenth of the bf16 one's rate.  An fp32 number is the
// sum of three bf16 numbers (x0 = x rounded, x1 = x - x0 rounded, x2 = x - x0 - x1: 24 significant bits in all),
// products of bf16 numbers are exact in fp32, and of the nine products of two split numbers three are below
// 2^-24 of the largest: six instructions instead of eight fp32 ones that take 2.7 times as long.
//   Error: what counts is the rounding of the running sum, once per instruction instead of once per k.  The sum
//   starts again every kChain k and is then added to a total.  Relative error against float64 sums (2-norm, 256
//   tiles of 16 x 16; normal inputs / inputs after a ReLU) of the fp32 instruction in chains of 256 k and of this:
//   K = 256 2.9e-7 / 2.0e-7 and 1.5e-7 / 1.5e-7; 768 2.9 / 2.1 and 1.6 / 1.6; 3072 3.0 / 2.1 and 1.8 / 1.8; 8192
//   3.1 / 2.3 and 2.2 / 2.2.  (Chains of 256 k: 2.3 to 2.6, not below the fp32 instruction's after a ReLU.)
//   Range: bf16 has fp32's exponents, but parts and products below 2^-126 may be lost (2-norm error with operands around
//   2^-110 2.7e-6, around 2^-118 1.4e-3).  So both operands are multiplied by 2^24 before they are split: the last bit of
//   the smallest fp32 number is then 2^-125, no part of any number is subnormal, and a product that fp32 can hold is
//   at least 2^-101.  The total is multiplied by 2^-48.  At the other end the scaled numbers overflow: operands above 2^103,
//   sums above 2^80 and what was not finite before make the scaled total infinite or NaN, and such results are
//   computed again on the fp32 instruction in the epilogue, so that they are what fp32 gives.
//   Few terms: where less than some 64 of a sum's terms are not zero, the rounding of the six products shows.
//   2-norm error, parts against fp32 instruction: 2.6e-8 : 2.5e-8 with one term, 5.2e-8 : 4.3e-8 with four, 9.0e-8 : 8.9e-8
//   with 64, 9.3e-8 : 13.5e-8 with 256 (of K = 768, simulated).
//
// What bounds it: matrix instructions, the splitting of the operands (13 vector instructions for two numbers) and the
// loads of the weights in operand order (65 cycles of a compute unit's memory pipeline for each KB, 1040 a step; the
// step's matrix instructions take 1152).  Reading them along the rows and rearranging them in LDS costs less of the
// memory pipeline but fills LDS (2000 tokens of 768 x 3072: 172 -> 185 us).  Tile: up to 96 token rows x 128 output
// features (64 of the gated product) x 32 k per step; four wavefronts, each with all rows and 32 weight rows (for the
// gated product 16 of W1 and the same 16 of W3, so that SiLU(gate)*up is lane-local); two workgroups per compute
// unit, so that one's splitting runs beside the other's matrix instructions.
//   weights   global -> registers two steps ahead, split in registers one step ahead (a weight is one wavefront's only);
//   tokens    global -> registers two steps ahead, split once for the workgroup one step ahead, three bf16 planes -> LDS
//             (two stages, 16-byte pieces swizzled, f32_piece) -> fragments.  The one barrier of a step stands before
//             its last fragment, so the next step's first fragment is fetched while matrix instructions run.
// AHEAD: products of about one tile for each compute unit.  One wavefront on a SIMD does its loads, its splitting and
// its matrix instructions one behind the other, so the tile goes to eight wavefronts of 16 features each, and what they split is
// requested three steps ahead, global -> LDS along the rows (20 cycles per KB), a part of LDS for each wavefront, which alone reads it.
// The waits are written out: nothing else in the loop goes through the vector memory, and what else there were would only make a
// wait longer, since a wait names how many requests younger than the one it wants may be in flight.  The layer of 2000
// tokens, 768 x 3072, 13 slots: 171 -> 164 us; other layers and the line: f32_ahead.  (Four wavefronts with requests ahead: 178 us for the
// layer, 172 without.)
// Measured against the fp32 instruction (ffn_tiled_f32.hip), layer: 768 x 3072 top-1, 13 slots, 2000 tokens 234 -> 176 us,
// 4096 tokens 437 -> 346; 1024 x 2048 SwiGLU top-2, 13 slots, 1200 tokens 357 -> 232, 3000 tokens 780 -> 489 (of which the
// multiplication by 2^24 is 2 to 4 %).  Error of those layers against float64: 3.6e-7 -> 2.4e-7 and 5.1e-7 -> 2.8e-7.
#include <type_traits>

#include "mmoe_internal.h"
#include "tile_table.h"

namespace mmoe {

// What a product writes: as in ffn_tiled.hip, with H in fp32.
enum { kModeReluH = 0, kModeSwigluH = 1, kModePlainF32 = 2, kModeGeluH = 3, kModeGatedY = 4 };

constexpr int kAheadWaves = 8;
constexpr int kFK = 32;            // k per step
constexpr int kChain = 128;        // k per chain of matrix instructions
constexpr int kChainF32 = 64;      // and on the fp32 instruction
constexpr int kFUnroll = kChain / kFK;
static_assert(256 % kChain == 0 && kFUnroll % 2 == 0, "K is a multiple of 256; two sets of registers in turn");

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

constexpr float kUp = 0x1p24f, kBack = 0x1p-48f;  // of an operand, of a result: powers of two, exact

// Three bf16 parts of each of four numbers times kUp, part 0 the largest: 26 vector instructions.
__device__ __forceinline__ void split4(f32x4 v, u32x2 (&part)[3])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float x = v[2 * i] * kUp, y = v[2 * i + 1] * kUp;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const uint32_t h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));  // to nearest even
            part[p][i] = h;
            if (p < 2) {
                x -= __uint_as_float(h << 16);
                y -= __uint_as_float(h & 0xFFFF0000u);
            }
        }
    }
}

// Byte offset of piece g (the 8 k of lane group g) of a row in a plane of 64-byte rows.  The 16 lanes that share
// a cycle of ds_read_b128 hold rows {0-3, 12-15} of one group and {4-11} of its neighbour (or the other way round):
// 16 different columns of 256 bytes.
__device__ __forceinline__ int f32_piece(int row, int g) { return row * 64 + ((g ^ (-(row >> 2) & 3)) << 4); }

template <int MODE, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, 2) void split_f32_kernel(
    const float* __restrict__ A, const int32_t* __restrict__ perm, int kdiv, const int32_t* __restrict__ tab, int hdr,
    int list_at, int list_stride, const float* __restrict__ W0, const float* __restrict__ W1, float* __restrict__ out,
    int K, int N, const int32_t* __restrict__ sink_perm, const float* __restrict__ sink_w)
{
    constexpr bool AHEAD = WAVES == kAheadWaves;
    constexpr int kFThreads = WAVES * kWave;
    constexpr int kNB = AHEAD ? 1 : 2;        // 16-row weight blocks per wavefront
    static_assert(!AHEAD || MODE != kModeSwigluH, "a gated wavefront has a block of each matrix");
    constexpr int kPlane = kFRows * kFK * 2;  // bytes of one part of a token tile
    constexpr int kStage = 3 * kPlane;
    // AHEAD: what the wavefronts have requested, each in a part of its own: weights, then tokens, kRing steps
    constexpr int kPieceRows = kFThreads / 8;  // token rows that the workgroup brings in with one instruction each
    constexpr int kRing = 3, kWRaw = kNB * 16 * kFK * 4, kTRaw = 1024;  // bytes of a wavefront's weights of a step; of a token piece
    constexpr int kPieces = (kFRows + kPieceRows - 1) / kPieceRows, kMine = kRing * (kWRaw + kPieces * kTRaw);
    __shared__ __attribute__((aligned(1024))) char lds[2 * kStage + (AHEAD ? WAVES * kMine : 0)];
    typedef __attribute__((address_space(3))) void* lptr_t;

    // workgroup id -> tile: entry blockIdx.x / 8 of this XCD's list
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const int4* list = reinterpret_cast<const int4*>(tab) + list_at + xcd * list_stride;
    const int n_mine = tab[hdr + xcd];
    const int4 ent = list[local];  // in bounds for every workgroup of the grid
    if (local >= n_mine) return;   // uniform over the workgroup
    const int s = ent.x & kSlotMask;
    const int nt = list_stride ? ent.y : ent.y * kXcds + xcd;
    const int r0 = ent.z, cnt = ent.w;  // first row, rows (1..96)

    constexpr bool kGated = MODE == kModeSwigluH;
    constexpr int kOut = kGated ? 1 : kNB;  // 16-feature blocks of the output per wavefront
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 15, g = lane >> 4;
    const int n0 = nt * (16 * kOut * WAVES) + wave * (16 * kOut);

    // Lane (li, g) of an operand holds, of a step's 32 k, the four from 4 g on and the four from 16 + 4 g on.
    auto token_row = [&](int row) {  // input row of the tile's row
        const int r = r0 + row;
        return A + (size_t)(perm ? perm[r] / kdiv : r) * K;
    };
    const float* wrow[kNB];
#pragma unroll
    for (int i = 0; i < kNB; ++i)
        wrow[i] = (kGated && i == 1 ? W1 : W0) + ((size_t)s * N + n0 + (kGated ? 0 : 16 * i) + li) * K + 4 * g;

    auto run = [&](auto njc) {
        constexpr int NJ = decltype(njc)::value;  // 16-row fragments of the tile that hold rows
        constexpr int NP = (16 * NJ + kPieceRows - 1) / kPieceRows;  // pieces of four k that a thread brings in per step
        // piece i * kFThreads + tid: row (i * kFThreads + tid) / 8, four k from 4 (tid % 8) on; rows past the end re-read the last
        // one (never stored)
        const float* asrc[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) asrc[i] = token_row(min(i * kPieceRows + (tid >> 3), cnt - 1)) + 4 * (tid & 7);
        const int adst = f32_piece(tid >> 3, tid & 3) + 8 * ((tid >> 2) & 1);  // + 64 bytes a row for later pieces
        const int fsrc = f32_piece(li, g);                                     // + 1024 per fragment
        // where the fragments do not fill the last pieces, those are the first wavefronts': two of four, or two, four or six of eight
        auto brings = [&](int i) { return (i + 1) * kPieceRows <= 16 * NJ || i * kPieceRows + 8 * wave < 16 * NJ; };

        f32x4 tot[NJ][kNB], acc[NJ][kNB];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < kNB; ++i) {
                tot[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
                acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        const int steps = K / kFK, last = steps - 1;  // a multiple of 8
        // AHEAD: requests of step t, into its place of the ring; kReq instructions
        constexpr int kReq = 2 * kNB + NP;
        char* const mine = lds + 2 * kStage + wave * kMine;
        uint32_t woff[2 * kNB];
        const char* wsrc = reinterpret_cast<const char*>(W0 + ((size_t)s * N + n0) * K);
#pragma unroll
        for (int i = 0; i < 2 * kNB; ++i) {
            const int r = 8 * i + (lane >> 3);  // of the wavefront's weight rows
            woff[i] = (uint32_t)r * (uint32_t)K * 4u + (((lane & 7) ^ (r & 7)) << 4);
        }
        auto request = [&](int t, int at) {
            const size_t ko = (size_t)min(t, last) * (kFK * 4);
#pragma unroll
            for (int i = 0; i < NP; ++i) {  // token rows may lie more than 4 GB apart
                const uint32_t dst = (uint32_t)(uintptr_t)(lptr_t)(mine + kRing * kWRaw + (at * kPieces + i) * kTRaw);
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(reinterpret_cast<const char*>(asrc[i]) + ko), "s"(dst) : "m0", "memory");
            }
#pragma unroll
            for (int i = 0; i < 2 * kNB; ++i) {
                const uint32_t dst = (uint32_t)(uintptr_t)(lptr_t)(mine + at * kWRaw + i * 1024);
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(woff[i]), "s"(wsrc + ko), "s"(dst) : "m0", "memory");
            }
        };
        f32x4 wr[kNB][2], ar[NP];   // weights and tokens of a step, as loaded
        // the requests of the kRing - 1 steps after step t may be in flight
        auto fetch = [&](int at) {
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kRing - 1) * kReq) : "memory");
            const char* w = mine + at * kWRaw;
#pragma unroll
            for (int i = 0; i < NP; ++i) ar[i] = *reinterpret_cast<const f32x4*>(mine + kRing * kWRaw + (at * kPieces + i) * kTRaw + lane * 16);
#pragma unroll
            for (int i = 0; i < kNB; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    wr[i][h] = *reinterpret_cast<const f32x4*>(w + (16 * i + li) * 128 + (((g + 4 * h) ^ (li & 7)) << 4));
        };
        u32x2 wp[2][kNB][2][3];     // weights split: [step][block][half][part]
        auto load_w = [&](int t, int i, int h) {  // past the end: a harmless reload
            if (AHEAD) return;
            wr[i][h] = *reinterpret_cast<const f32x4*>(wrow[i] + (size_t)min(t, last) * kFK + 16 * h);
        };
        auto load_a = [&](int t, int i) {
            if (AHEAD) return;
            if (brings(i)) ar[i] = *reinterpret_cast<const f32x4*>(asrc[i] + (size_t)min(t, last) * kFK);
        };
        auto put_a = [&](char* stage, int i) {
            if (!brings(i)) return;
            u32x2 x[3];
            split4(ar[i], x);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x2*>(stage + p * kPlane + i * (kPieceRows * 64) + adst) = x[p];
        };
        u32x4 x[2][3];  // parts of this fragment and of the next
        auto get_x = [&](int set, int j, const char* stage) {
#pragma unroll
            for (int p = 0; p < 3; ++p) x[set][p] = *reinterpret_cast<const u32x4*>(stage + p * kPlane + fsrc + j * 1024);
        };
        auto mma = [&](int set, int j, const u32x2 (&w)[kNB][2][3]) {
            constexpr int wpart[6] = {2, 0, 1, 1, 0, 0}, xpart[6] = {0, 2, 1, 0, 1, 0};  // smallest products first
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < kNB; ++i) {
                    const u32x2 lo = w[i][0][wpart[q]], hi = w[i][1][wpart[q]];
                    acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]}),
                                                                        __builtin_bit_cast(bf16x8, x[set][xpart[q]]), acc[j][i], 0, 0, 0);
                }
        };
        if constexpr (AHEAD) {
#pragma unroll
            for (int t = 0; t < kRing; ++t) request(t, t);
            fetch(0);
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) load_a(0, i);
#pragma unroll
        for (int i = 0; i < 2 * kNB; ++i) load_w(0, i / 2, i % 2);
#pragma unroll
        for (int i = 0; i < 2 * kNB; ++i) {
            split4(wr[i / 2][i % 2], wp[0][i / 2][i % 2]);
            load_w(1, i / 2, i % 2);
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            put_a(lds, i);
            load_a(1, i);
        }
        __syncthreads();
        get_x(0, 0, lds);
        int cur = 0, nxt = kStage;  // stages of this step and of the next
        int at = 0;                 // place of this step in the ring
        for (int t0 = 0; t0 < steps; t0 += kFUnroll) {
#pragma unroll
            for (int u = 0; u < kFUnroll; ++u) {
                const int t = t0 + u;
                if constexpr (AHEAD) {
                    // what was fetched of step t has been split (and is waited for here), so its place takes step t + kRing
#pragma unroll
                    for (int i = 0; i < 2 * kNB; ++i) asm volatile("" ::"v"(wr[i / 2][i % 2]));
#pragma unroll
                    for (int i = 0; i < NP; ++i) asm volatile("" ::"v"(ar[i]));
                    request(t + kRing, at);
                    at = at == kRing - 1 ? 0 : at + 1;
                    fetch(at);
                }
#pragma unroll
                for (int n = 0; n < NJ; ++n) {
                    const int set = (u * NJ + n) & 1;  // NJ * kFUnroll is even
                    if (n < NJ - 1) get_x(set ^ 1, n + 1, lds + cur);
                    if (n == NJ - 1 && NJ > 1) {
                        __syncthreads();  // step t+1's tokens are in stage `nxt`
                        get_x(set ^ 1, 0, lds + nxt);
                    }
                    __builtin_amdgcn_sched_barrier(0);  // fetches stay in front of the matrix instructions that hide them
                    // A chain ends: its sum goes to the total (at the start of the next one, when it is long there).
                    if (u == 0) {
#pragma unroll
                        for (int i = 0; i < kNB; ++i) {
                            tot[n][i] += acc[n][i];
                            acc[n][i] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
                    }
                    // The step's other work, shared out to the fragments: the tokens of step t+1 into stage `nxt` (whose last
                    // reads, in step t-1, every wavefront had back before that step's barrier), in front of this step's
                    // barrier; the weights of step t+1 split; and the loads that refill the registers.
                    constexpr int kItems = NP + 2 * kNB, kFront = NJ > 1 ? NJ - 1 : 1;
#pragma unroll
                    for (int w = 0; w < kItems; ++w) {
                        const int at = w < NP && w * NJ / kItems > kFront - 1 ? kFront - 1 : w * NJ / kItems;
                        if (at != n) continue;
                        if (w < NP) {
                            put_a(lds + nxt, w);
                            load_a(t + 2, w);
                        } else {
                            const int i = (w - NP) / 2, h = (w - NP) % 2;
                            split4(wr[i][h], wp[(u + 1) & 1][i][h]);
                            load_w(t + 2, i, h);
                        }
                    }
                    mma(set, n, wp[u & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (NJ == 1) {
                        __syncthreads();
                        get_x(set ^ 1, 0, lds + nxt);
                    }
                }
                cur = nxt;
                nxt = kStage - cur;
            }
        }
        if (AHEAD) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing on its way into LDS when the workgroup ends
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < kNB; ++i) tot[j][i] += acc[j][i];

        // Scaled results that are not finite: again in fp32.  (Never taken where operands are below 2^103 and sums below 2^80.)
        bool odd = false;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < kNB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) odd |= !(fabsf(tot[j][i][e]) < INFINITY);
        if (__any(odd)) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float* a = token_row(min(j * 16 + li, cnt - 1)) + 4 * g;
                f32x4 sum[kNB];
#pragma unroll
                for (int i = 0; i < kNB; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                for (int k0 = 0; k0 < K; k0 += kChainF32) {
                    f32x4 c[kNB];
#pragma unroll
                    for (int i = 0; i < kNB; ++i) c[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                    for (int k = k0; k < k0 + kChainF32; k += 16) {
                        const f32x4 xv = *reinterpret_cast<const f32x4*>(a + k);
#pragma unroll
                        for (int i = 0; i < kNB; ++i) {
                            const f32x4 wv = *reinterpret_cast<const f32x4*>(wrow[i] + k);
#pragma unroll
                            for (int e = 0; e < 4; ++e) c[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[e], xv[e], c[i], 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < kNB; ++i) sum[i] += c[i];
                }
#pragma unroll
                for (int i = 0; i < kNB; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        tot[j][i][e] = fabsf(tot[j][i][e]) < INFINITY ? tot[j][i][e] * kBack : sum[i][e];
            }
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int i = 0; i < kNB; ++i) tot[j][i] *= kBack;
        }

        // accumulator element e of lane (li, g): feature 4 g + e of the block, token row li of the fragment
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
#pragma unroll
            for (int i = 0; i < kOut; ++i) {
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = tot[j][i][e];
                    if (MODE == kModeSwigluH) o[e] = v / (1.0f + __expf(-v)) * tot[j][kNB - 1][e];
                    else if (MODE == kModeReluH) o[e] = fmaxf(v, 0.0f);
                    else if (MODE == kModeGeluH) o[e] = 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f));
                    else if (MODE == kModeGatedY) o[e] = __builtin_fmaf(gw, v, 0.0f);
                    else o[e] = v;
                }
                *reinterpret_cast<f32x4*>(out + (size_t)orow * N + n0 + 16 * i + 4 * g) = o;
            }
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
    auto kernel = split_f32_kernel<MODE, 4>;
    int waves = 4;
    if constexpr (MODE != kModeSwigluH)
        if (p.ahead[prod]) {
            kernel = split_f32_kernel<MODE, kAheadWaves>;
            waves = kAheadWaves;
        }
    hipLaunchKernelGGL(kernel, dim3(p.L.len[prod] * kXcds), dim3(waves * kWave), 0, st, (const float*)A, perm,
                       kdiv, tab, kXcds * prod, p.L.list[prod], p.L.lists[prod] == 1 ? 0 : p.L.len[prod], (const float*)W0,
                       (const float*)W1, (float*)out, K, N, sink.perm, sink.w);
}

void launch_up_split(const mmoe_shape& s, const TiledPlan& p, const void* rows, const int32_t* perm, const int32_t* tab,
                     const void* W1p, const void* W3p, void* H, hipStream_t st)
{
    const int d = s.d_model, f = s.d_ff;
    if (s.act == MMOE_SWIGLU) launch_product<kModeSwigluH>(p, 0, rows, perm, s.top_k, tab, W1p, W3p, H, d, f, st);
    else if (s.act == MMOE_GELU) launch_product<kModeGeluH>(p, 0, rows, perm, s.top_k, tab, W1p, nullptr, H, d, f, st);
    else launch_product<kModeReluH>(p, 0, rows, perm, s.top_k, tab, W1p, nullptr, H, d, f, st);
}

void launch_down_split(const mmoe_shape& s, const TiledPlan& p, const int32_t* tab, const void* W2p, const void* H, float* Yg,
                       hipStream_t st, GateSink sink)
{
    const int d = s.d_model, f = s.d_ff;
    if (sink.w) launch_product<kModeGatedY>(p, 1, H, nullptr, 1, tab, W2p, nullptr, sink.Y, f, d, st, sink);
    else launch_product<kModePlainF32>(p, 1, H, nullptr, 1, tab, W2p, nullptr, Yg, f, d, st);
}

}  // namespace mmoe
