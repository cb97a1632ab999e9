// Step F, matrix-core-bound variant: the grouped expert FFN when slots hold many rows
// (prefill-shaped batches) -- Algorithm 2, "expert[iL][iE](act)"; the expert block is
// where the layer's time goes (section 5.1).
//
// Both products are  out[r, n] = sum_k A[r, k] * W[s][n][k]  over the packed pool, bf16
// inputs, fp32 accumulation on v_mfma_f32_16x16x32_bf16.
//
// Tile: 256 token rows x 256 weight rows x 64 k per step, one workgroup of four
// wavefronts per compute unit.  Each wavefront owns all 256 token rows and 64 weight rows
// (for the gated product: 32 rows of W1 and the same 32 rows of W3, so that SiLU(gate)*up
// is lane-local): 16 x 4 accumulator tiles of 16x16, 256 accumulator registers.  Weights are
// the row operand of the matrix instruction and tokens the column one, hence a lane owns, for one
// token, groups of 4 consecutive output features and stores 16 bytes at a time.
//
// Memory pipeline: the pool is stored as fragments of 32 rows x 16 k, two of which hold, for each
// half of their rows, a 16 x 32 operand: a wavefront loads its weight operands straight from global
// memory into registers (16 bytes per lane, 256-byte runs), three 32-k slices ahead of their use (seven where the tile leaves the registers).
// Token rows are copied global -> LDS without passing registers (global_load_lds, 16 bytes per lane)
// into a ring of LDS tiles (four stages of full tiles, up to eleven of short ones), [row][64 k] bf16 (128 bytes a row)
// with the 16-byte pieces xor-swizzled (piece_swizzle), and are read back as fragments; one barrier per step.
//
// Ragged groups: row ranges come from the device array `offsets`.  A small
// preparation step turns them into lists of tiles; the product kernels map their
// workgroup id to (slot, row tile, feature tile) through those lists, so the host never
// waits for the histogram.  Workgroup ids are dealt round-robin to the 8 XCDs by the
// hardware; every XCD has a list of its own share of the tiles, ordered so that the workgroups
// resident on it share weight and activation panels in that XCD's L2.
#include <type_traits>

#include "mmoe_internal.h"
#include "tile_table.h"

namespace mmoe {

// What a product writes: H = act(.) in bf16 (up product), plain fp32 rows of Yg (down product), or,
// for layers with top_k = 1, the layer's output rows: 0 + w[token] * y in bf16 at row token (GateSink).
enum { kTModeReluH = 0, kTModeSwigluH = 1, kTModePlainF32 = 2, kTModeGeluH = 3, kTModeGatedY = 4 };

constexpr int kBN = 256;  // weight rows per tile: four wavefronts of two 32-row blocks (128 with one block each)
constexpr int kBK = 64;
constexpr int kStagesA = 4;    // LDS ring of token tiles

typedef __attribute__((address_space(3))) void* lptr_t;

// silu(g) * u with the hardware exponential and reciprocal (about 1 ulp each; the result is
// rounded to bf16 right after).  A full-precision division here costs more matrix-core idle
// time at the end of every tile than it is worth.
__device__ __forceinline__ float silu_mul_t(float g, float u)
{
    return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

// Where the 16-byte pieces of a token row stand in LDS: logical piece c of a row is physical piece
// c ^ piece_swizzle(row).  A ds_read_b128 works through its lanes in four cycles of 16: {0-3, 12-15, 20-27},
// {4-11, 16-19, 28-31} and the same from 32 on (measured by timing lane pairs), each free of conflicts if its
// lanes read 16 different 16-byte columns of 256 bytes.  Lane (row lr, group lg) of a fragment read wants
// piece 4 (lg % 2) + const, so a cycle holds rows {0-3, 12-15} of one group and {4-11} of its neighbour: the
// rows of the first set need columns that are closed under xor 4, which plain (row >> 1) & 7 does not give
// (two lanes to a column, half of the LDS's active cycles lost) and this does.
__device__ __forceinline__ constexpr int piece_swizzle(int row) { return ((row >> 1) & 7) ^ ((row >> 2) & 2); }

// The lists of product blockIdx.x, for callers that bring the offsets.
__global__ __launch_bounds__(kListThreads) void tile_table_kernel(const int32_t* __restrict__ offsets,
                                                                  int32_t* __restrict__ tab, int S, int nt_up,
                                                                  int nt_down, TileLists L, SlotFilter filt)
{
    __shared__ int off[kMaxS + 1];
    __shared__ int first[kXcds * kMaxS];
    for (int s = threadIdx.x; s <= S; s += kListThreads) off[s] = offsets[s];
    __syncthreads();
    const int p = blockIdx.x;
    build_tile_lists(off, tab, S, p, p == 0 ? nt_up : nt_down, L, first, filt);
}

// LONE: a tile that holds all rows of its slot is the only reader of its weight panels and reads them past the caches,
// which streams faster where the pool is large (lone_tiles; 4096 x 14336, 18 slots, 777 tokens 1227 -> 1200 us; 4096 x
// 2048, 64 slots, 4800 pairs 737 -> 717; 2560 x 2560 GELU, 20 slots, 2000 pairs 179 -> 171).  A panel with several readers
// has to stay in L2 (8192 tokens 4486 -> 5087 us with every panel past the caches).
template <int MODE, int BM, int NB, bool LONE>
__device__ __forceinline__ void tiled_body(const uint16_t* __restrict__ A, const int32_t* __restrict__ perm, int kdiv,
                                           const int32_t* __restrict__ tab, int hdr, int list_at, int list_stride,
                                           const uint16_t* __restrict__ W0, const uint16_t* __restrict__ W1,
                                           void* __restrict__ out, int K, int N, const int32_t* __restrict__ sink_perm,
                                           const float* __restrict__ sink_w)
{
    constexpr int kTileBytes = BM * kBK * 2;  // one step of the token operand (32 KB for 256 rows)
    __shared__ __attribute__((aligned(1024))) char lds_a[kStagesA * kTileBytes];

    // ---- workgroup id -> tile ------------------------------------------------------------
    // XCD x (= workgroup id mod 8) works through its list of tiles (tile_table.h): all row tiles that
    // share a weight panel run on the XCD whose L2 holds it, and every XCD has the same share of the
    // work.  One 16-byte entry of the list says which tile this workgroup computes.
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
    const int4* list = reinterpret_cast<const int4*>(tab) + list_at + xcd * list_stride;
    const int n_mine = tab[hdr + xcd];
    const int4 ent = list[local];                     // in bounds for every workgroup of the grid
    if (local >= n_mine) return;                      // uniform over the workgroup
    const int s = ent.x & kSlotMask;
    const int nt = list_stride ? ent.y : ent.y * kXcds + xcd;
    const int r0 = ent.z;                             // first row of the tile
    const int cnt = ent.w;                            // rows of the tile that exist (1..256)

    // NB = 32-row weight blocks per wavefront: 2 (256 weight rows per tile), or 1 (128: twice as many
    // tiles for a product that would otherwise leave compute units without work; not for the gated
    // product, whose wavefronts pair a gate block with an up block)
    static_assert(NB == 2 || (NB == 1 && MODE != kTModeSwigluH), "weight blocks per wavefront");
    constexpr int kFeat = MODE == kTModeSwigluH ? kBN / 2 : 128 * NB;  // output features per tile
    const int n0 = nt * kFeat;

    constexpr int kWaves = 4;         // one per SIMD
    constexpr int kThreads = kWaves * 64;
    constexpr int kNF = BM / 16;      // 16-row token fragments of a full tile (a wavefront takes all of them)
    constexpr int kNW = 2 * NB;       // 16-row weight blocks per wavefront
    constexpr int kNP = BM * 8 / kThreads;  // 16-byte pieces of a token tile per thread
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: keeps bases in scalar registers
    const int lr = lane & 15, lg = lane >> 4;  // row of a 16-row fragment, one of its four groups of 8 k
    const int wn = wave;              // which 32 NB weight rows of the tile

    // ---- token operand: global -> LDS ------------------------------------------------------------
    // Piece id = i*kThreads + tid (i < kNP) of a [BM rows][8 pieces of 16 bytes] tile: 8
    // consecutive threads read one row's 128 contiguous bytes.  Rows past the end of the group
    // re-read its last row (they are multiplied but never stored).
    // Grouped row r is row r of A, or, when a permutation is given, row perm[r] / kdiv of A (the
    // gather of the token rows folded into this product's loads).
    // Copy instruction i of a wavefront writes its 64 pieces to 1 KB of consecutive LDS addresses
    // (M0 + 16*lane), 8 rows of 128 bytes, so the swizzle is applied on the global side: the lane
    // that fills physical piece q of a row fetches logical piece q ^ piece_swizzle(row).
    const char* a_base = reinterpret_cast<const char*>(A);
    uint32_t a_goff[kNP];  // byte offset of the piece
#pragma unroll
    for (int i = 0; i < kNP; ++i) {
        const int row = i * (kThreads / 8) + (tid >> 3);
        const int r = r0 + min(row, cnt - 1);
        a_goff[i] = (uint32_t)(perm ? perm[r] / kdiv : r) * (uint32_t)K * 2u + (((tid & 7) ^ piece_swizzle(tid >> 3)) << 4);
    }
    // The copies are written in assembly so that the compiler's wait-count bookkeeping does not
    // see them (it would drain every load in flight before each LDS read); the waits that order
    // them are written out next to the barriers.  M0 is only used here.
    auto copy_a = [&](int stage, int kt, int i) {  // stage: byte offset in lds_a
        const char* ab = a_base + (size_t)kt * (kBK * 2);
        const uint32_t dst =
            (uint32_t)(uintptr_t)(lptr_t)(lds_a + stage + (i * kThreads + wave * 64) * 16);
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :
                     : "v"(a_goff[i]), "s"(ab), "s"(dst)
                     : "m0", "memory");
    };
    // ---- weight operand: fragment-packed pool -> registers ------------------------------------------
    // A wavefront owns 32 NB weight rows of the tile: NB packed 32-row blocks, each two 16-row blocks of
    // the matrix instruction.  For the gated product they are block (n0 + 32 wn)/32 of W1 (gate) and the
    // same block of W3 (up), so that a lane holds matching gate and up values.  Packed fragment ks (16 k)
    // of a 32-row block is 1 KB at ks*1024; slice g of the matrix instruction (32 k) is fragments 2g and
    // 2g + 1: lane group lg takes half lg%2 of fragment 2g + lg/2, 256 contiguous bytes per group.
    const size_t frag_bytes_per_block = (size_t)(K / 16) * 1024;
    const char* wb[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const uint16_t* w = (MODE == kTModeSwigluH && i == 1) ? W1 : W0;
        const int nb = MODE == kTModeSwigluH ? (n0 + wn * 32) / 32 : (n0 + wn * (32 * NB) + i * 32) / 32;
        wb[i] = reinterpret_cast<const char*>(w) + ((size_t)s * (N / 32) + nb) * frag_bytes_per_block;
    }
    const uint32_t w_off = (lg >> 1) * 1024 + (lg & 1) * 512 + lr * 16;

    // ---- token fragments from LDS ------------------------------------------------------------------
    // Slice q (32 k) of a step: lane (row lr, group lg) reads logical piece 4 (lg%2) + 2q + lg/2, the
    // 8 k values that its weight fragment holds.
    int frag_off[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        frag_off[q] = lr * 128 + (((4 * (lg & 1) + 2 * q + (lg >> 1)) ^ piece_swizzle(lr)) << 4);

    // Gated output rows (GateSink): output row (token) and coefficient of this lane's token of every
    // fragment.  Two dependent loads each; tiles of 128 x 128 (short-lived, with registers to spare)
    // start them here, in front of the main loop's own loads, the others when the main loop is over.
    constexpr bool kEarlySink = BM == kBMSmall && NB == 1;
    float gate_w[kNF];
    int sink_row[kNF];
    auto fetch_sink = [&]() {
#pragma unroll
        for (int j = 0; j < kNF; ++j) {
            sink_row[j] = sink_perm[r0 + min(j * 16 + lr, cnt - 1)];
            gate_w[j] = sink_w[sink_row[j]];
        }
    };
    if (MODE == kTModeGatedY && kEarlySink) fetch_sink();

    f32x4 acc[kNF][kNW];  // [token fragment][16-row weight block]
#pragma unroll
    for (int j = 0; j < kNF; ++j)
#pragma unroll
        for (int i = 0; i < kNW; ++i) acc[j][i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // Main loop, instantiated for NJ = number of the tile's 32-row token sub-tiles that hold rows.
    //
    // What bounds it: power.  Under matrix load on real data the chip lowers its clock (1.6 to 1.9 GHz
    // of 2.4), so what counts is energy per flop first and idle matrix cycles second.
    //   - 16x16x32 instructions instead of 32x32x16: a register-only loop on random operands runs at
    //     2.04 against 1.84 PFLOP/s (half the accumulator traffic per flop).
    //   - One vector-memory instruction at a time between groups of matrix instructions, never a burst:
    //     the memory pipeline takes 16 cycles for each 1 KB instruction of each of the four wavefronts, and a
    //     wavefront that issues eight in a row stands still for several hundred cycles.
    // (16384 x 28672 x 4096, uniform tiles, random data: 1.26 -> 1.34 -> 1.41 PFLOP/s.)
    //
    // The matrix instructions are written in assembly with the accumulators tied to AGPRs: from 64
    // small accumulators the compiler's own choice of destination registers moves them around in
    // the loop.  Hazards it can then not see: nothing in the loop writes a matrix operand with a
    // vector instruction (fragments come from LDS and memory reads, whose waits the compiler
    // inserts), and the accumulators are read behind the s_nops that follow the loop.
    //
    // Short tiles (small NJ) are bound by the latency of memory instead: a step is over long before a load
    // issued in it has come back.  They copy only the 32 NJ rows they have (NJ instructions per wavefront and
    // step, not BM / 32), use the LDS and the registers that this leaves for more steps in flight, and so have as
    // many bytes on the way as a full tile.  (4096 x 14336, 777 tokens, tiles of 1 to 4 sub-tiles: 1259 -> 1235 us; 768 x
    // 3072 top-1, 543 tokens: 59.4 -> 55.9 us.)
    //
    // Pipeline (k step t = 64 k = two 32-k slices; step t's tokens live in LDS stage t mod kStages):
    //   weights   slice g is loaded straight into registers kSlices - 1 slices ahead of its use; these
    //             are ordinary loads and the compiler inserts their waits;
    //   tokens    the copies of step t + kStages - 1 are issued during step t, into the stage that step
    //             t-1 has left, and must have landed kDeep steps later; token fragments roll through a
    //             ring of RF register sets: as soon as the kNW matrix instructions that use a fragment
    //             have been issued, the fragment RF further on is fetched into its registers;
    //   barrier   one per step, RF/2 groups before its end: by then every wavefront's reads of the
    //             step's stage have returned (only the first RF/2 fetches of the next stage may be in
    //             flight), so nobody waits for LDS.
    // The loop is unrolled by kUnroll steps so that the rings of registers are indexed statically.
    //
    // What orders the copies.  The compiler does not see them, so the wait that makes them
    // land is written out next to every barrier: s_waitcnt vmcnt(N) returns when at most N of
    // this wavefront's vector-memory instructions are outstanding, and they complete in issue
    // order.  Rule at every such wait: only the most recent kDeep steps' copies (NJ each, kNP at most
    // together) may still be in flight, every older one has landed.  That holds if at least N
    // vector-memory instructions were issued after the last of the older ones: the kDeep NJ copies
    // plus weight-fragment loads, whose place in the instruction stream the compiler
    // chooses.  Their count is therefore not taken on trust: tests/test_tiled_wait_counts.py
    // reads the compiler's assembly output for this file, where each such wait says how many copies may
    // still be in flight at it, and checks the rule at every one of them, in every instantiation and along
    // every path that reaches it.
    // What orders the LDS reads.  Before a stage is handed back to the copies, the fragments
    // of that stage that are still to be used are made operands of an (empty) asm statement in
    // front of the barrier, so the compiler itself waits for exactly those reads and for nothing
    // younger (the RF/2 fetches of the next stage stay in flight across the barrier).
    const int nkt = K / kBK;         // a multiple of 4: K is a multiple of 256
    const int last = nkt - 1;
    const int last_slice = K / 32 - 1;
    constexpr int kUnroll = (BM == kBMBig || NB == 1) ? 4 : 2;
    auto run = [&](auto njc, auto ntc) {
        constexpr int NJ = decltype(njc)::value;
        constexpr bool NT = decltype(ntc)::value;  // weights past the caches
        // ring of weight slices in registers (four steps, two steps): what the accumulators leave room for
        constexpr int kSlices = NB == 1 || (BM == kBMBig && NJ <= 4) ? 8 : 4;
        constexpr int kDeep = kNP / NJ;
        constexpr int kStages = kDeep + 3;
        constexpr int kStageBytes = NJ * 32 * kBK * 2;
        static_assert(kStages * kStageBytes <= kStagesA * kTileBytes && kDeep * NJ <= kNP, "LDS; copies in flight");
        constexpr int NF = 2 * NJ;              // token fragments per slice
        constexpr int G = 2 * NF;               // groups (one fragment against kNW weight blocks) per step
        // fragments in flight: the lead stays within the next step, and 128 x 256 tiles have 256 registers
        constexpr int RF = (NJ == 1 || (BM == kBMSmall && NB == 2)) ? 4 : 8;
        static_assert(G >= RF && (kUnroll * G) % RF == 0, "the fragment ring is indexed statically");
        struct BFrags {
            u32x4 b[kNW];
        };
        bf16x8 fa[RF];
        BFrags bq[kSlices];
        auto load_bf = [&](BFrags& fr, int g, int i) {
            const size_t o = (size_t)min(g, last_slice) * 2048;  // past the end: a harmless reload
            const u32x4* src = reinterpret_cast<const u32x4*>(wb[i >> 1] + o + (w_off + (i & 1) * 256));
            fr.b[i] = NT ? __builtin_nontemporal_load(src) : *src;
        };
        // prologue: copies of steps 0 .. kStages-2, then the first weight slices; the wait leaves at most
        // the copies of the last kDeep of those steps in flight
#pragma unroll
        for (int t = 0; t < kStages - 1; ++t)
#pragma unroll
            for (int i = 0; i < NJ; ++i) copy_a(t * kStageBytes, min(t, last), i);
#pragma unroll
        for (int g = 0; g < kSlices - 1; ++g)
#pragma unroll
            for (int i = 0; i < kNW; ++i) load_bf(bq[g], g, i);
        static_assert(kDeep * NJ + kNW * (kSlices - 1) <= 63, "vmcnt is a 6-bit counter");
        __builtin_amdgcn_sched_barrier(0);  // the weight loads are issued before the wait, not after it
        asm volatile("s_waitcnt vmcnt(%0) ; copies in flight: %1\n\ts_barrier" ::"n"(kDeep * NJ + kNW * (kSlices - 1)),
                     "n"(kDeep * NJ)
                     : "memory");
#pragma unroll
        for (int j = 0; j < RF; ++j)
            fa[j] = *reinterpret_cast<const bf16x8*>(lds_a + (j < NF ? frag_off[0] + j * 2048 : frag_off[1] + (j - NF) * 2048));

        int st = 0;  // LDS stage of step kt (byte offset)
        constexpr int kLastStage = (kStages - 1) * kStageBytes;
        int kt = 0;
        do {  // at least one trip (K >= 256): the prologue's loads have nowhere to sink to
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int t = kt + u;
                const int stn = st == kLastStage ? 0 : st + kStageBytes, stp = st == 0 ? kLastStage : st - kStageBytes;
                const char* cur = lds_a + st;
                const char* nxt = lds_a + stn;
                BFrags& f0 = bq[(2 * u) % kSlices];
                BFrags& f1 = bq[(2 * u + 1) % kSlices];
                BFrags& fp = bq[(2 * u + kSlices - 1) % kSlices];  // the slice in front of this step's
                // Vector-memory instructions of one half of the step, op = 0 .. ops(half)-1: half of the copies
                // (the first half the larger one) and kNW weight loads in turn.  First half: the slice used last
                // in the step before; second half: this step's first slice, used up by then.
                auto copies = [](int half) { return half ? NJ / 2 : (NJ + 1) / 2; };
                auto ops = [&](int half) { return copies(half) + kNW; };
                auto vmem = [&](int half, int op) {
                    const int nc = copies(half), two = 2 * (nc < kNW ? nc : kNW);  // ops that alternate
                    const bool copy = op < two ? op % 2 == 0 : nc > kNW;
                    const int n = op < two ? op / 2 : op - two / 2;
                    if (copy) copy_a(stp, min(t + kStages - 1, last), half * ((NJ + 1) / 2) + n);
                    else if (half == 0) load_bf(fp, 2 * t + kSlices - 1, n);
                    else load_bf(f0, 2 * t + kSlices, n);
                };
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    constexpr int kBar = G - RF / 2;  // the barrier stands in front of this group
                    if (gi == kBar) {
                        // Stage st goes back to the copies after this barrier.  Its fragments that are still
                        // to be used become operands here, so the compiler waits for those reads; every other
                        // read of the stage has been consumed by a matrix instruction above.
#pragma unroll
                        for (int j = kBar; j < G; ++j) asm volatile("" ::"v"(fa[(u * G + j) % RF]));
                        // All vector-memory instructions of step t stand in front of its barrier: NJ copies
                        // (step t + kStages - 1's) and 2 kNW weight loads.  The copies of step t+2 were issued
                        // during step t - kDeep, and the instructions of the kDeep steps since stand behind
                        // them; or in the prologue, and then kDeep NJ copies, the prologue's weight loads and step
                        // t's do.  A wait that leaves the lesser of the two outstanding leaves the copies of
                        // step t+2 landed, and after the barrier every wavefront may read that step, whose
                        // first fragments are fetched before the next barrier.
                        constexpr int kWaitN = kDeep * NJ + kNW * (2 * kDeep < kSlices + 1 ? 2 * kDeep : kSlices + 1);
                        static_assert(kWaitN <= 63, "vmcnt is a 6-bit counter");
                        asm volatile("s_waitcnt vmcnt(%0) ; copies in flight: %1\n\ts_barrier" ::"n"(kWaitN),
                                     "n"(kDeep * NJ)
                                     : "memory");
                    }
                    const int q = gi / NF, j = gi % NF, slot = (u * G + gi) % RF;
                    const BFrags& fb = q ? f1 : f0;
#pragma unroll
                    for (int i = 0; i < kNW; ++i)
                        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                                     : "+a"(acc[j][i])
                                     : "v"(fb.b[i]), "v"(fa[slot]));
                    const int n = gi + RF;  // the fragment that takes this one's registers
                    const char* src = n < NF  ? cur + frag_off[0] + n * 2048
                                      : n < G ? cur + frag_off[1] + (n - NF) * 2048
                                      : n < G + NF ? nxt + frag_off[0] + (n - G) * 2048
                                                   : nxt + frag_off[1] + (n - G - NF) * 2048;
                    fa[slot] = *reinterpret_cast<const bf16x8*>(src);
                    __builtin_amdgcn_sched_barrier(0);
                    // groups of this half that memory instructions may follow: all before the barrier
                    const int half = gi / NF, ng = half ? kBar - NF : NF, at = gi - half * NF;
                    // where few groups put the barrier in front of the second half, its instructions join the first
                    if (kBar > NF) {
#pragma unroll
                        for (int op = 0; op < kNP + kNW; ++op)
                            if (op < ops(half) && gi < kBar && op * ng / ops(half) == at) vmem(half, op);
                    } else if (gi == NF - 1) {
#pragma unroll
                        for (int op = 0; op < ops(0) + ops(1); ++op) vmem(op >= ops(0), op < ops(0) ? op : op - ops(0));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                st = stn;
            }
            kt += kUnroll;
        } while (kt < nkt);
        // no copy may still be on its way into LDS when the workgroup ends; and the matrix pipeline's last
        // results are there before the accumulators are read
        asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    };
    auto sized = [&](auto ntc) {
        switch (min(BM / 32, (cnt + 31) / 32)) {  // uniform over the workgroup
            case 8: if constexpr (BM == kBMBig) run(std::integral_constant<int, 8>{}, ntc); break;
            case 7: if constexpr (BM == kBMBig) run(std::integral_constant<int, 7>{}, ntc); break;
            case 6: if constexpr (BM == kBMBig) run(std::integral_constant<int, 6>{}, ntc); break;
            case 5: if constexpr (BM == kBMBig) run(std::integral_constant<int, 5>{}, ntc); break;
            case 4: run(std::integral_constant<int, 4>{}, ntc); break;
            case 3: run(std::integral_constant<int, 3>{}, ntc); break;
            case 2: run(std::integral_constant<int, 2>{}, ntc); break;
            default: run(std::integral_constant<int, 1>{}, ntc); break;
        }
    };
    if constexpr (LONE) {
        if (ent.x & kOnlyTile) sized(std::true_type{});  // uniform over the workgroup
        else sized(std::false_type{});
    } else {
        sized(std::false_type{});
    }
    // the accumulators stay where the matrix instructions left them until the epilogue reads them
#pragma unroll
    for (int j = 0; j < kNF; ++j)
#pragma unroll
        for (int i = 0; i < kNW; ++i) asm volatile("" : "+a"(acc[j][i]));

    // ---- epilogue -------------------------------------------------------------------------------
    // Accumulator element e of lane (lr, lg) is weight row 4 lg + e of the block, token lr of the
    // fragment.  fp32 output: a lane's four values of a block are 16 consecutive bytes of the token's
    // row, stored as they are.  bf16 output: two blocks are packed to 8 bytes per lane each, and one
    // exchange between neighbouring lane groups (v_permlane16_swap) gives every lane 8 consecutive
    // features of one block: lane group lg holds features 8 (lg/2) .. +7 of block lg%2, 16 bytes,
    // and the four groups of a token cover 64 contiguous bytes.  No LDS, no barrier.
    constexpr int kEsz = MODE == kTModePlainF32 ? 4 : 2;
    constexpr int kOutBlocks = MODE == kTModeSwigluH ? kNW / 2 : kNW;  // 16-feature blocks this wavefront stores
    const int wfeat = wn * 16 * kOutBlocks;
    if (MODE == kTModeGatedY && !kEarlySink) fetch_sink();
    char* const obase = reinterpret_cast<char*>(out) + (size_t)(n0 + wfeat) * kEsz +
                        (kEsz == 4 ? lg * 16 : ((lg & 1) * 16 + (lg >> 1) * 8) * 2);
#pragma unroll
    for (int j = 0; j < kNF; ++j) {
        if (j * 16 >= cnt) break;  // uniform over the workgroup
        const int row = MODE == kTModeGatedY ? sink_row[j] : r0 + j * 16 + lr;
        char* const dst = obase + (size_t)row * N * kEsz;
        f32x4 o[kOutBlocks];
#pragma unroll
        for (int i = 0; i < kOutBlocks; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = acc[j][i][e];
                if (MODE == kTModeSwigluH) o[i][e] = silu_mul_t(v, acc[j][i + kNW / 2][e]);
                else if (MODE == kTModeReluH) o[i][e] = fmaxf(v, 0.0f);
                else if (MODE == kTModeGeluH) o[i][e] = 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f));
                else if (MODE == kTModeGatedY) o[i][e] = __builtin_fmaf(gate_w[j], v, 0.0f);
                else o[i][e] = v;
            }
        if constexpr (kEsz == 4) {
            if (j * 16 + lr < cnt) {
#pragma unroll
                for (int i = 0; i < kOutBlocks; ++i) *reinterpret_cast<f32x4*>(dst + i * 64) = o[i];
            }
        } else {
            u32x4 pk[kOutBlocks / 2];
#pragma unroll
            for (int p = 0; p < kOutBlocks / 2; ++p) {
                u32x2 lo, hi;  // features 4 lg .. +3 of block 2p, of block 2p + 1
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    lo[h] = (uint32_t)f32_to_bf16_bits(o[2 * p][2 * h]) |
                            ((uint32_t)f32_to_bf16_bits(o[2 * p][2 * h + 1]) << 16);
                    hi[h] = (uint32_t)f32_to_bf16_bits(o[2 * p + 1][2 * h]) |
                            ((uint32_t)f32_to_bf16_bits(o[2 * p + 1][2 * h + 1]) << 16);
                }
                const u32x2 s0 = __builtin_amdgcn_permlane16_swap(lo[0], hi[0], false, false);
                const u32x2 s1 = __builtin_amdgcn_permlane16_swap(lo[1], hi[1], false, false);
                pk[p] = u32x4{s0[0], s1[0], s0[1], s1[1]};
            }
            if (j * 16 + lr < cnt) {
#pragma unroll
                for (int p = 0; p < kOutBlocks / 2; ++p) *reinterpret_cast<u32x4*>(dst + p * 64) = pk[p];
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // one fragment at a time: few registers
    }
}

template <int MODE, int BM, int NB>
__global__ __launch_bounds__(256, BM == kBMBig ? 1 : 2) void tiled_kernel(
    const uint16_t* __restrict__ A, const int32_t* __restrict__ perm, int kdiv, const int32_t* __restrict__ tab, int hdr,
    int list_at, int list_stride, const uint16_t* __restrict__ W0, const uint16_t* __restrict__ W1, void* __restrict__ out,
    int K, int N, const int32_t* __restrict__ sink_perm, const float* __restrict__ sink_w)
{
    tiled_body<MODE, BM, NB, false>(A, perm, kdiv, tab, hdr, list_at, list_stride, W0, W1, out, K, N, sink_perm, sink_w);
}

// A batch in which slots may be one tile (lone_tiles): 256-row tiles.
template <int MODE>
__global__ __launch_bounds__(256, 1) void tiled_lone_kernel(
    const uint16_t* __restrict__ A, const int32_t* __restrict__ perm, int kdiv, const int32_t* __restrict__ tab, int hdr,
    int list_at, int list_stride, const uint16_t* __restrict__ W0, const uint16_t* __restrict__ W1, void* __restrict__ out,
    int K, int N, const int32_t* __restrict__ sink_perm, const float* __restrict__ sink_w)
{
    tiled_body<MODE, kBMBig, 2, true>(A, perm, kdiv, tab, hdr, list_at, list_stride, W0, W1, out, K, N, sink_perm, sink_w);
}

// 256-row tiles of 128 features (few_wide_tiles, tile_share).
template <int MODE, bool LONE>
__global__ __launch_bounds__(256, 1) void tiled_narrow_kernel(
    const uint16_t* __restrict__ A, const int32_t* __restrict__ perm, int kdiv, const int32_t* __restrict__ tab, int hdr,
    int list_at, int list_stride, const uint16_t* __restrict__ W0, const uint16_t* __restrict__ W1, void* __restrict__ out,
    int K, int N, const int32_t* __restrict__ sink_perm, const float* __restrict__ sink_w)
{
    tiled_body<MODE, kBMBig, 1, LONE>(A, perm, kdiv, tab, hdr, list_at, list_stride, W0, W1, out, K, N, sink_perm, sink_w);
}

// And 128-row tiles.
template <int MODE, int NB>
__global__ __launch_bounds__(256, 2) void tiled_lone_small_kernel(
    const uint16_t* __restrict__ A, const int32_t* __restrict__ perm, int kdiv, const int32_t* __restrict__ tab, int hdr,
    int list_at, int list_stride, const uint16_t* __restrict__ W0, const uint16_t* __restrict__ W1, void* __restrict__ out,
    int K, int N, const int32_t* __restrict__ sink_perm, const float* __restrict__ sink_w)
{
    tiled_body<MODE, kBMSmall, NB, true>(A, perm, kdiv, tab, hdr, list_at, list_stride, W0, W1, out, K, N, sink_perm, sink_w);
}

constexpr int kCus = 256;  // compute units

// Does an ungated product with N output features take 128 of them to a 256-row tile, not 256?  Twice the tiles, each with
// half of the weights, pay
//   - where the wide ones leave half of the compute units without work: fewer than 128 of them;
//   - where weights are most of the traffic, up to 100 rows per slot, and wide tiles are a little over one round: 257 to 336.
// Tiles counted as if every slot held rows and its last tile were half full.
// Wide : narrow down products, layer, us, three pools in turn, equally used slots / router bias 1, by that count:
//   60   4096 x 8192, 4 slots       248 : 211 / 309 : 271      72   2048 x 2048, 9 slots       96 : 87 / 96 : 89
//   80   2048 x 8192, 10 slots      238 : 205 / 239 : 212      96   4096 x 512                 73.7 : 69.9 / 72.0 : 67.9
//   112  4096 x 14336, 7 slots      576 : 512 / 592 : 532      120  2560 x 7680, 12 slots      257 : 220 / 257 : 245
//   128  4096 x 14336, 8 slots      660 : 593 / 665 : 706      144  4096 x 14336, 9 slots      676 : 679 / 712 : 709
//   192  2048 x 4096, 24 slots      217 : 229 / 222 : 238      280  2560 x 4096, 28 slots      406 : 397 / 420 : 417
//   288  4096 x 14336, 18 slots     1202 : 1188 / 1289 : 1280  304  4096 x 1024, 19 slots      148 : 143 / 141 : 136
//   320  4096 x 8192, 19 slots      754 : 738 / 801 : 788      288  4096 x 4096, 133 rows      441 : 448 / -
// (the down products of 280 to 320 themselves 146 : 136 / 141 : 138, 452 : 440 / 478 : 469, 49 : 45 / 48 : 44, 283 : 265 / 292 : 280).
// Of 260 layers below the first line, random in width, depth, slots and use, narrow tiles take 14 % less from 70 to 90, 9 %
// from 90 to 120, 5 % from there on, where unequal ones of which a few tiles are a second round lose up to 6 %.  From 120 on
// with over 256 rows per slot 20 layers are level on average, from 2048 x 5888, 8 slots of 375 rows 276 : 253 to 2048 x 9984, 9
// of 320 386 : 426; a line at 120 for those changed 9 % both ways.  Past two rounds the narrow tiles' second reading of the
// tokens costs more: 2200 tokens of 4096 x 14336 1818 : 1957.
bool few_wide_tiles(const mmoe_shape& s, int N)
{
    if (s.dtype == MMOE_F32 || planned_tile_rows(s) != kBMBig) return false;
    const int64_t P = (int64_t)s.T * s.top_k, rows2 = s.S + P / 128;  // twice the row tiles
    const int64_t narrow = (rows2 > 2 * s.S ? rows2 : 2 * s.S) * (N / kBN);
    return narrow < kCus || (narrow > 2 * kCus && narrow <= 2 * kCus + 160 && P <= (int64_t)100 * s.S);
}

// Ungated products of 128-row tiles have one weight block per wavefront (128 features) where tiles of two would be fewer
// than the chip holds workgroups, kNb1Room, and two from there on.  Counted as full row tiles of all pairs.
constexpr int kNb1Room = 2 * kCus;
// Two already from kNb1RoomTall on where slots have at least kTallRows rows on average, for more than a tile each: one round
// of wide tiles reads the tokens once where a round and a half of narrow ones reads them twice.  With GELU, whose epilogue
// is long, only if the tiles are one round with another half tile per slot.
// Narrow : wide (up in runs where that is for fewer rounds), layer, us, three pools in turn, equally used slots / router
// bias 0.5 / 1:
//   ReLU  768 x 3072, 4096 tokens   9 slots   87 : 85 / 89 : 86 / 98 : 98         13 slots  93 : 92 / 103 : 101 / 99 : 96
//                                   18 slots  102 : 99 / 103 : 101 / 105 : 104
//         768 x 3072, 5000 tokens   18 slots  111 : 110 / 116 : 116 / 115 : 118
//         1280 x 3328, 4700 tokens  13 slots  157 : 150 / 160 : 159 / 161 : 160
//         1024 x 1536, 9000 tokens  13 slots  112 : 104 / 116 : 108 / 118 : 110
//         1536 x 1536, 8000 tokens  13 slots  136 : 122 / 144 : 124 / 148 : 128 (both products wide)
//   GELU  768 x 3072, 4096 tokens   13 slots  102 : 101 / 112 : 111 / 108 : 104
//         past the round: 5000 tokens, 18 slots 121 : 126 / 124 : 129 / 126 : 131; 1280 x 3328 169 : 170 / 172 : 176 / 176 : 178
// Unequal slots that take a round more than the host can see lose up to 5 % (GELU, 4096 tokens, 18 slots, bias 1 113 : 117).
// Neither line is where both sides are level: 768 x 3072, equally used / bias 1, 210 tiles, 267 rows 62 : 66 / 63 : 67, 178
// rows 68 : 69 / 71 : 73; but 250 tiles, 180 rows 73 : 71 / 76 : 75, 140 rows 80 : 79 / 77 : 75; 384 tiles, 140 rows are equal.
constexpr int kNb1RoomTall = 300, kTallRows = 160;
bool wide_below_a_round(const mmoe_shape& s, int N, bool up)
{
    const int64_t P = (int64_t)s.T * s.top_k, nt = N / kBN, tiles = (P + kBMSmall - 1) / kBMSmall * nt;
    if (P < (int64_t)kTallRows * s.S || tiles < kNb1RoomTall || tiles >= kNb1Room) return false;
    return !up || s.act != MMOE_GELU || (2 * P / kBMSmall + s.S) * nt <= 2 * kNb1Room;
}

// Weight blocks per wavefront of a product with N output features: 2 (256 weight rows to a tile), or 1 (128).  Shape only.
static int planned_nb(const mmoe_shape& s, int bm, int N, bool up)
{
    if (up && s.act == MMOE_SWIGLU) return 2;  // one block of each matrix
    if (bm != kBMSmall) return few_wide_tiles(s, N) ? 1 : 2;
    const int64_t P = (int64_t)s.T * s.top_k;
    return (P + bm - 1) / bm * (N / kBN) >= kNb1Room || wide_below_a_round(s, N, up) ? 2 : 1;
}

// fp32: does a product with N outputs (of each matrix) run on bf16 parts (ffn_split_f32.hip)?  Its tiles have twice the
// features, so it needs rows that fill tiles and tiles that fill the chip: about as many as half the compute units,
// counted as if every slot had one tile more than its share of full ones.  Measured for both products on the fp32
// instruction : on parts : with this rule, us: 768 x 3072, 13 slots 117 : 125 : 108 at 54 rows per slot, 122 : 129 : 113 at 65,
// 169 : 132 : 151 at 77, 172 : 149 : 147 at 90, 229 : 169 : 169 at 154; 256 x 8192 (2 wide tiles down) 238 : 260 : 221 at 115,
// 286 : 289 : 252 at 192; 4096 x 512, 6 slots 80 : 110 : 78 at 62, 155 : 153 : 134 at 192; 768 x 768, 4 slots 50 : 60 : 50 at 250,
// 129 : 90 : 89 at 1000; SwiGLU 1024 x 2048 123 : 123 : 123 at 46, 2048 x 4096 219 : 206 : 192 at 43.  It loses where slots of less than a
// tile count as two: 2048 x 1024, 12 slots 95 : 101 : 102 at 60; 512 x 2048, 32 slots 99 : 110 : 109 at 40.  (With a line of 200
// tiles below 64 rows per slot both take 89, but 768 x 3072, 16 slots of unequal use, at 59 rows 157 instead of 135.)
constexpr int kPartsRows = 40, kPartsTiles = 150;
bool f32_in_parts(const mmoe_shape& s, int N, bool gated)
{
    const int64_t P = (int64_t)s.T * s.top_k;
    if (P < (int64_t)kPartsRows * s.S) return false;
    return gated || (P / kFRows + s.S) * (N / (2 * kFeatF32)) >= kPartsTiles;
}

static void tiled_nts(const mmoe_shape& s, int bm, int& nt_up, int& nt_down, int& nb_up, int& nb_down)
{
    if (s.dtype == MMOE_F32) {
        nb_up = f32_in_parts(s, s.d_ff, s.act == MMOE_SWIGLU) ? 2 : 1;
        nb_down = f32_in_parts(s, s.d_model, false) ? 2 : 1;
        nt_up = s.d_ff / (kFeatF32 * (s.act == MMOE_SWIGLU ? 1 : nb_up));
        nt_down = s.d_model / (kFeatF32 * nb_down);
        return;
    }
    nb_up = planned_nb(s, bm, s.d_ff, true);
    nb_down = planned_nb(s, bm, s.d_model, false);
    nt_up = s.act == MMOE_SWIGLU ? s.d_ff / (kBN / 2) : s.d_ff / (128 * nb_up);
    nt_down = s.d_model / (128 * nb_down);
}

// Tile height: 128 rows (two workgroups per compute unit, so one's prologue and epilogue hide
// behind the other's main loop) when a tile is short-lived -- a short reduction in the up
// product, or slots with few rows -- and 256 rows (deeper weight prefetch, half the weight
// traffic per row) otherwise.  The host knows P and S, not the counts.  Measured with each
// height forced, 128 against 256 rows, us: d = 768 62 : 78 at 154 rows per slot, 223 : 243 at 1231; d = 1280 75 : 94 at
// 125, 373 : 453 at 1000; d = 1536 99 : 128 at 67, 367 : 383 at 1000; d = 1792 109 : 139 at 67, 442 : 428 at 1000;
// d = 2048 134 : 146 (f = 3072) and 200 : 206 (5120) at 67, 231 : 218 at 133, 473 : 449 at 1000; d = 4096 833 : 831 at
// 46, 965 : 851 at 65, 1418 : 969 at 139.
int planned_tile_rows(const mmoe_shape& s)
{
    if (s.dtype == MMOE_F32) return kFRows;  // the fp32 kernel has one height
    if (s.tile_rows) return s.tile_rows;  // forced for this call (checked by check_shape: 128 or 256)
    const int64_t P = (int64_t)s.T * s.top_k;
    if (s.d_model <= 1536) return kBMSmall;
    return P < (int64_t)(s.d_model <= 2048 ? 100 : 64) * s.S ? kBMSmall : kBMBig;
}

// How a product with N output features and 128-row tiles of one weight block per wavefront shares its rows out.
//
// Two tiles on one compute unit take nearly twice the time of one (768 x 3072 down, 128 rows: 17 us of main loop alone on a
// compute unit, 30 beside another; the matrix pipe bounds both), and a tile more than there are compute units puts two on
// one: 258 tiles took 37 us where 252 take 24.  So up to kFillRounds rounds of kCus tiles, counted as a full tile and a part of
// one for every slot, a target height is chosen that just fills whole rounds of one tile for each compute unit, down to one
// sub-tile (kFill); and where 128 rows to a tile do not do, but 256 do, tiles are 256 rows by 128 features and one round
// (kTall: tiled_narrow_kernel, one workgroup to a compute unit).  kPlain: rounds of two tiles for each compute unit.
// The figures are of 35000 layers, random in widths, tokens, picks, slots and router bias: time of the layer with the product so shared
// out in the time with it plain, mean (largest; share over 1.02).
//
// Down products, in runs of tiles.  kFill over up to two rounds, from 32 rows per slot on 0.96 (1.20; 0.01); with fewer, slots of a little
// more than 32 rows become two short tiles, which what they move bounds, and two to a compute unit hide each other's waits: up to
// kFewTiles full tiles of rows, within a round 0.95 (1.25; 0.00), more 0.99 (1.29; 0.12: 512 x 6656, 80 slots, 622 tokens, two
// picks), but 0.98 (1.03; 0.00) of reductions from 2048 on whose panels divide among the XCDs (4096 x 14336, 9 slots, 124 tokens, two picks, bias
// 2.5 550 : 477, 447 layers of those widths 0.99).
// kTall, where kFill is more than a round: reductions of 2048 and more, 64 rows per slot and more 0.93 (1.07; 0.02) where kFill has 0.96
// (1.14; 0.04); shorter reductions 0.98 (1.10; 0.12) where kFill has 0.98 (1.06; 0.01): few steps, and nothing else on the compute unit
// while the prologue waits; fewer rows 0.99 (1.24; 0.10).
//
// Up products, panel by panel: XCDs whose panels are of larger slots have more tiles than compute units, which one tile to each
// does not even out.  Where panels divide among the XCDs, kFill 0.98 (1.10; 0.03) over up to two rounds; otherwise with up to kFewTiles
// full tiles of rows, within a round 0.93 (1.06; 0.00), and within half a round up to 128 rows per slot 0.93 (1.14; 0.01); more 0.99
// (1.19; 0.17).  kTall, of 2100 such layers, 1.05 (1.35).
//
// Layers, us, three pools in turn, plain : so, equally used slots unless a router bias is given:
//   down, kTall  768 x 3072, 18 slots  4096 tokens 99.1 : 90.4, bias 0.5 100.9 : 90.2   8000 132.7 : 128.2
//                24 slots, 4096 tokens, bias 1 111.9 : 103.2, GELU bias 2.5 99.0 : 87.6
//   down, kFill  768 x 3072   8 slots  4096 tokens 84.7 : 75.3   18 slots  1000 63.4 : 61.8   2000 76.7 : 72.7
//                11 slots, 1500 63.3 : 56.7   12 slots, 3000 77.3 : 71.6   512 x 2048, 32 slots, 3000 62.3 : 62.4
//   past the lines, with kFill and with kTall  1024 x 4096, 30 slots, 5000 (560 tiles) 183.2 : 187.5 : 193.4
//          768 x 3072, 14 slots, 12000 (648) 180.3 : 176.4 : 169.8
// (More than a round of 256-row tiles is faster in one of these two layers and slower in the other; two are no line.)
enum TileShare { kPlain, kFill, kTall };
constexpr int kFillRounds = 2, kFewTiles = 32;
int tile_share(const mmoe_shape& s, int N, bool up)
{
    if (s.dtype == MMOE_F32 || planned_tile_rows(s) != kBMSmall || planned_nb(s, kBMSmall, N, up) != 1) return kPlain;
    const int64_t P = (int64_t)s.T * s.top_k, nt = N / 128, most = ((P + kBMSmall - 1) / kBMSmall + s.S) * nt;
    const bool fills = most <= kFillRounds * kCus, few = most <= kCus && P * nt <= kFewTiles * kBMSmall;
    if (up) return (nt % kXcds == 0 ? fills : few || (most <= kCus / 2 && P <= (int64_t)128 * s.S)) ? kFill : kPlain;
    if (P < (int64_t)32 * s.S && !few && (nt % kXcds != 0 || s.d_ff < 2048)) return kPlain;
    // (slots of 256-row tiles counted as five eighths of a tile more than their rows fill)
    const bool tall = most > kCus && (8 * P / kBMBig + 5 * s.S) * nt <= 8 * kCus;
    if (tall && !s.tile_rows && s.d_ff >= 2048 && P >= (int64_t)64 * s.S) return kTall;
    return fills ? kFill : kPlain;
}

// Heights of a product's row tiles.  Shorter ones than five eighths of a full tile are bound by what they move, unless they
// fill a round that would be partly idle.  fp32: down to one sub-tile (the matrix rate bounds tiles of any height, and short
// ones share out a product of few tiles evenly); the workgroups of a compute unit (three, two of the gated product) share
// its matrix pipes, which bound them, so it counts as working on one tile at a time.
static TileRows tile_rows_of(const mmoe_shape& s, int bm, int share)
{
    if (s.dtype == MMOE_F32) return {kFRows / 32, 4, 1, 5, share == kFill};
    if (bm == kBMBig) return {8, 20, 1, 5, false};
    if (share == kTall) return {8, 4, 2, 5, true};
    if (share == kFill) return {4, 4, 1, 5, true};
    return {4, 10, 1, 6, false};
}

// Are panels read past the caches where a tile is the only one of its slot?  Where slots of one tile are likely, and
// the pool is larger than the last-level cache: a smaller one may still be there from an earlier call, and the few
// tiles of a small layer wait longer for each load.  Through the caches : past them, us, one pool again and again / three in
// turn.  256-row tiles: 2304 x 768 SwiGLU, 6 slots (64 MB), 180 rows per slot 72.2 : 82.9 / 72.3 : 83.2; 4096 x 512, 5 slots (42
// MB) 80.9 : 95.4 / 80.0 : 95.4; 4096 x 1024 SwiGLU, 8 slots (201 MB), 110 rows 88.3 : 109.0 / 111.6 : 109.1; 2560 x 2560, 20 slots
// (524 MB) 182.7 : 172.3 / 183.2 : 174.1; 4096 x 2048 SwiGLU, 13 slots (654 MB) 178.9 : 161.1 / 180.0 : 166.2; at 244 and 306
// rows per slot on average both are within 1 %.  128-row tiles: 2048 x 1280 SwiGLU, 90 slots, 46 rows 339 : 314 / 346 : 334;
// 1024 x 1024 SwiGLU, 200 slots, 16 rows 271 : 260 / 272 : 260; 1024 x 4096 SwiGLU, 60 slots, 20 rows 300 : 286 / 305 : 287; 768 x 3072
// SwiGLU, 40 slots, 50 rows 148 : 144 / 149 : 143, 110 rows 145 : 141, 200 rows 204 : 205; pools below the line 2048 x 2048 GELU, 12
// slots (201 MB), 67 rows 72.6 : 81.5 / -; 768 x 3072, 18 slots (170 MB) 95.8 : 101.7 / 106.3 : 107.0.
bool lone_tiles(const mmoe_shape& s)
{
    return (int64_t)s.T * s.top_k <= (int64_t)kBMBig * s.S && s.S * slot_bytes(s) > kLastLevelCache;
}

// Of a large pool a batch may use few slots, which stay cached.  The list builder knows them: panels are read past the
// caches from this many bytes on (the streaming kernels' line, past_the_caches).  Through : past, us, one pool again and
// again / three in turn, by what is used:
//   57 MB   512 x 2048 SwiGLU, 150 slots, 800 tokens  57 : 59 / 56 : 58   63 MB  57 : 60 / 56 : 60   82 MB  57 : 61 / 60 : 60
// and above the line, where one pool alone would rather stay cached and several lose by it:
//   126 MB  the same                       63 : 65 / 66 : 63    157 MB  2560 x 1024, 24 slots, 379 tokens    64 : 73 / 78 : 74
//   182 MB  1024 x 1024, 200 slots, 800    81 : 83 / 87 : 85    184 MB  1536 x 1536, 40 slots, 600 tokens    77 : 88 / 94 : 92
//   195 MB  1024 x 1024, 200 slots, 400    70 : 77 / 81 : 77    267 MB  2048 x 1280, 90 slots, 1037 tokens   149 : 144 / 162 : 163
constexpr int64_t kLoneBytes = (int64_t)96 << 20;

// Do the XCDs take runs of neighbouring tiles of product `prod` (0 up, 1 down; RunsRule, tile_table.h)?
//
// Down products.  What reaches an XCD's L2 from beyond it bounds them (5.7 TB/s; 768 x 3072, 18 slots, 4096 tokens: 251 MB,
// of which 151 token rows, each read by six XCDs).  Panel by panel a slot's rows are read by min(8, NT) XCDs, a weight
// panel by one; in runs the rows by one or two, but the panels at the ends by two.  So runs pay where token rows are a good
// part of the traffic, min(8, NT) P against S N rows: from a quarter on, 128-row tiles with NT a multiple of 8 from half on.
// Panels : runs, layer, us, three pools in turn, equally used slots / router bias 1 / 2.5, 128-row tiles:
//   768 x 3072    13 slots of 300 rows  127 : 116 / 127 : 120 / 118 : 114    24 of 80  106 : 105 / 115 : 105 / 84 : 82
//   1280 x 5120   13 of 300  246 : 243 / 271 : 247 / 275 : 240   1536 x 6144  13 of 300  323 : 325 / 342 : 319 / 335 : 312
//   512 x 2048    13 of 300  68 : 68 / 78 : 74 / 66 : 64         1024 x 4096  13 of 300  172 : 170 / 179 : 178 / 171 : 166
//   below the lines 2048 x 1280, 90 of 46  324 : 329; 2048 x 3072 (NT 8, 16) 13 of 80  138 : 141 / 137 : 139 / 128 : 131
// 256-row tiles of up to 512 rows per slot: always in short reductions with fewer than 16 wide panels, else for fewer
// rounds, and not where panels divide among the XCDs.  Long runs drift apart.  Panels : always in runs, as above:
//   4096 x 14336, 18 slots  130 rows  1311 : 1410 / 1318 : 1407 / 1440 : 1486   250  1856 : 1870 / 1816 : 1869 / 1850 : 1918
//                           450 rows  2729 : 2815 / - / 2802 : 2845
//   3584 x 7680, 12 of 420  842 : 879 / 886 : 897                               3072 x 7680  747 : 777 / 769 : 793
//   short: 2048 x 1536, 19 of 170  123 : 117   1792 x 1536, 13 of 290  105 : 100   means of 10 to 17 layers of each width
//   from 1792 to 3584 K = 1024 1 % less, K = 1536 0.3 % less, but 4096 x 1536 0.9 % more
// Panels : for fewer rounds, equally used / bias 1:
//   2304 x 7680   12 of 420  644 : 563 / 659 : 571    12 of 240  412 : 411 / 468 : 424
//   2304 x 2304   28 of 220  325 : 325 / 386 : 359    2560 x 5120  28 of 220  718 : 685 / 745 : 709
//   3072 x 3072   16 of 350  384 : 381 / 401 : 388
// Over 512 rows the matrix cores bound them (4096 x 14336, 1260 rows, always in runs 4624 : 4690).
//
// Up products read a few short rows of tokens for each of their panels (1024 x 4096 in runs 210 : 219).  Only for fewer
// rounds, and where wide tiles were taken for being one (wide_below_a_round): 12 panels of unequal slots do not divide
// among the XCDs as 24 narrow ones do.  Panels : for fewer rounds, equally used / bias 0.5 / 1 / 2.5:
//   768 x 3072, 4096 tokens   9 slots   84 : 84 / 96 : 88 / 97 : 92 / 82 : 76    13  86 : 86 / 102 : 97 / 100 : 95 / 81 : 75
//                             18 slots  99 : 99 / 106 : 101 / 103 : 104 / 91 : 84
//   1536 x 1536, 8000 tokens  13 slots  133 : 122 / 139 : 124 / 142 : 128 / 133 : 118
constexpr int kShortReduction = 1536;
int xcd_runs(const mmoe_shape& s, int prod)
{
    if (s.dtype == MMOE_F32) return kRunsNever;
    const int bm = planned_tile_rows(s);
    if (prod == 0) {
        const bool few = bm == kBMSmall && s.act != MMOE_SWIGLU && wide_below_a_round(s, s.d_ff, true);
        return few && s.d_ff / kBN % kXcds != 0 ? kRunsForFewerRounds : kRunsNever;
    }
    int nt_up, nt, nb_up, nb_down;
    tiled_nts(s, bm, nt_up, nt, nb_up, nb_down);
    const bool even = nt % kXcds == 0;  // panels divide among the XCDs
    const int64_t P = (int64_t)s.T * s.top_k, rows = P * (nt < kXcds ? nt : kXcds), weights = (int64_t)s.S * s.d_model;
    if (bm == kBMBig) {
        if (P > (int64_t)512 * s.S || 4 * rows < weights) return kRunsNever;
        if (nb_down == 2 && nt < 2 * kXcds && s.d_ff <= kShortReduction) return kRunsAlways;
        return even ? kRunsNever : kRunsForFewerRounds;
    }
    return (even ? 2 : 4) * rows >= weights ? kRunsAlways : kRunsNever;
}

// The same for the down products in fp32, where token rows are twice as much of the traffic: 768 x 3072, 13 slots, 2000 tokens read
// 264 MB in turn, of which 148 token rows.  The time of 10900 layers with runs in the time with panels in turn, random in widths, rows,
// slots, picks and router bias, mean (largest; share over 1.02), from a quarter of the traffic in token rows on:
//   fewer panels than XCDs   0.90 (1.06; 0.01) on bf16 parts, 0.96 (1.03; 0.00) on the fp32 instruction
//   more, not dividing among the XCDs   0.97 (1.12; 0.01) up to 700 tiles of 64 rows, counted with one more for every slot, unequally
//                            used slots down to 0.70; over it 0.99 (1.09; 0.11): an XCD's panels even out by themselves
//   dividing among the XCDs  1.00 (1.15; 0.06): nothing to even out
// Below that share of token rows up to 1.28.  Panels : runs, layer, us:
//   768 x 3072   13 slots  2000 tokens 175 : 172   4096 311 : 282   GELU, bias 2.5 330 : 270   1000, bias 0.5 156.6 : 154.0   200 83.7 : 82.7
//                24 slots  3000, bias 0.5 309 : 262   500 134.2 : 133.3
//   1536 x 4096, 12 slots, 1000 tokens 252 : 231   256 x 2048 GELU, 12 slots, 2000 pairs, bias 0.5 86.4 : 79.6
// (The up product in runs too: 768 x 3072, 13 slots, 2000 tokens 172 : 179.)
constexpr int kF32RunTiles = 700;
bool f32_down_in_runs(const mmoe_shape& s)
{
    int nt_up, nt, nb_up, nb_down;
    tiled_nts(s, kFRows, nt_up, nt, nb_up, nb_down);
    const int64_t P = (int64_t)s.T * s.top_k, rows = P * (nt < kXcds ? nt : kXcds), weights = (int64_t)s.S * s.d_model;
    if (nt % kXcds == 0 || 4 * rows < weights) return false;
    return nt < kXcds || ((P + 63) / 64 + s.S) * nt <= kF32RunTiles;
}

// fp32 on bf16 parts: eight wavefronts to a tile, one tile for each compute unit and heights that fill the round (ffn_split_f32.hip)?
// Where tiles of 64 rows, counted with three quarters of one more for every slot, are a round: taller ones are bound by LDS, where
// eight wavefronts read every token fragment; and in reductions long enough for the prologue.  The time of layers with the product so
// in the time with four wavefronts, random as for f32_down_in_runs, mean (largest; share over 1.02):
//   down products, in runs where the rule says so  0.97 (1.03; 0.01) of 2350   from there up to a count of 288 with a whole tile for
//                              every slot 0.99 (1.08): 768 x 3072, 8 slots, 2500 tokens 188 : 201, 5 slots of 512 x 2816, 4020 178 : 189
//   up products, panel by panel, so that XCDs with more tiles than compute units take another round, which two and three smaller
//   workgroups on a compute unit even out:
//     panels dividing among the XCDs  0.95 (1.02; 0.01) of 80     four panels and more, up to 56 rows per slot 0.94 (1.10; 0.03) of 86
//     others  1.01 (1.16; 0.33): 3072 x 768, 16 slots, 1084 tokens, bias 2.5 137 : 161, 1280 x 512, 12 slots, 2653 87 : 96
// Four : eight wavefronts, layer, us, three pools in turn, with the down products in runs either way:
//   2048 x 1024 GELU, 12 slots, 700 tokens (up) 107.0 : 90.6           768 x 3072, 8 slots, 2000 GELU 171.7 : 167.6
//   768 x 3072, 13 slots, 1000, bias 0.5 153.8 : 153.4   2000 171.3 : 164.2
//   past the line  13 slots, 2500, bias 0.5 199 : 210    4096 290 : 306    24 slots, 3000 261 : 277
//   K = 512  512 x 512, 12 slots, 3000 56.0 : 57.4       K = 1024  768 x 1024, 12 slots, 900 62.6 : 62.7
constexpr int kAheadReduction = 1024, kAheadPanels = 4, kAheadRows = 56;
bool f32_ahead(const mmoe_shape& s, int N, bool up)
{
    if (s.dtype != MMOE_F32 || (up && s.act == MMOE_SWIGLU) || !f32_in_parts(s, N, false)) return false;
    const int64_t P = (int64_t)s.T * s.top_k, nt = N / (2 * kFeatF32);
    if ((up ? s.d_model : s.d_ff) < kAheadReduction || (P + 48 * (int64_t)s.S) * nt > 64 * kCus) return false;
    return !up || nt % kXcds == 0 || (nt >= kAheadPanels && P <= (int64_t)kAheadRows * s.S);
}

static TiledPlan tiled_plan(const mmoe_shape& s)
{
    TiledPlan p;
    p.bm = planned_tile_rows(s);
    p.lone = lone_tiles(s);
    tiled_nts(s, p.bm, p.nt_up, p.nt_down, p.nb_up, p.nb_down);
    p.ahead[0] = f32_ahead(s, s.d_ff, true);
    p.ahead[1] = f32_ahead(s, s.d_model, false);
    const int up = p.ahead[0] ? kFill : tile_share(s, s.d_ff, true), down = p.ahead[1] ? kFill : tile_share(s, s.d_model, false);
    p.tall_down = down == kTall;
    p.L = tile_lists(s.T * s.top_k, s.S, p.nt_up, p.nt_down, tile_rows_of(s, p.bm, up), tile_rows_of(s, p.bm, down),
                     s.dtype == MMOE_F32, xcd_runs(s, 0), s.dtype == MMOE_F32 && f32_down_in_runs(s) ? kRunsAlways : xcd_runs(s, 1),
                     (int)(kLoneBytes / slot_bytes(s)) + 1);
    return p;
}

size_t planned_table_bytes(const mmoe_shape& s) { return align256(tiled_plan(s).L.bytes); }

size_t tiled_table_bytes(const mmoe_shape& s)
{
    if (use_skinny(s)) return 0;
    size_t most = 0;
    for (int rows : {0, kBMSmall, kBMBig}) {  // tile_rows is a field of the call, not of the workspace; 0 has plans of its own
        mmoe_shape call = s;
        call.tile_rows = rows;
        const size_t b = planned_table_bytes(call);
        most = b > most ? b : most;
    }
    return most;
}

size_t tiled_table_most(const mmoe_shape& s)
{
    const int P = s.T * s.top_k;
    // Fewer pairs may get the other height and narrower feature tiles (planned_tile_rows, planned_nb, f32_in_parts,
    // tile_share); with each of them fixed the lists only grow with P.  (Wider feature tiles can make the longer lists: a
    // number of them that is no multiple of 8 takes a list per XCD.)
    const bool f32 = s.dtype == MMOE_F32;
    const int wide = f32 ? kFeatF32 : 128;  // features of a tile with one weight block per wavefront
    size_t at = kListHeader;
    for (int prod = 0; prod < 2; ++prod) {
        int64_t most = 0;
        for (int bm : {kBMSmall, kBMBig})
            for (int nb : {1, 2})
                for (int share : {kPlain, kFill, kTall}) {
                    if (prod == 0 && share == kTall) continue;
                    const int NT = prod == 0 ? (s.act == MMOE_SWIGLU ? s.d_ff / wide : s.d_ff / (wide * nb)) : s.d_model / (wide * nb);
                    const int cap = row_tiles_cap(P, s.S, NT, tile_rows_of(s, bm, share), f32);
                    const int64_t n = (int64_t)list_count(NT, prod == 0 ? kRunsNever : kRunsAlways) * list_len(cap, NT);
                    most = n > most ? n : most;
                }
        at += most;
    }
    return align256(at * 16);
}

template <int MODE, int BM, int NB>
static void launch_product(const TiledPlan& p, int prod, const void* A, const int32_t* perm, int kdiv, const int32_t* tab,
                           const void* W0, const void* W1, void* out, int K, int N, hipStream_t st,
                           GateSink sink = GateSink())
{
    const dim3 grid(p.L.len[prod] * kXcds), block(256);
    const int stride = p.L.lists[prod] == 1 ? 0 : p.L.len[prod];
    void (*kernel)(const uint16_t*, const int32_t*, int, const int32_t*, int, int, int, const uint16_t*, const uint16_t*, void*, int, int,
                   const int32_t*, const float*);
    if constexpr (BM == kBMBig && NB == 1) kernel = p.lone ? tiled_narrow_kernel<MODE, true> : tiled_narrow_kernel<MODE, false>;
    else if constexpr (BM == kBMBig) kernel = p.lone ? tiled_lone_kernel<MODE> : tiled_kernel<MODE, BM, NB>;
    else kernel = p.lone ? tiled_lone_small_kernel<MODE, NB> : tiled_kernel<MODE, BM, NB>;
    hipLaunchKernelGGL(kernel, grid, block, 0, st, (const uint16_t*)A, perm, kdiv, tab, kXcds * prod,
                       p.L.list[prod], stride, (const uint16_t*)W0, (const uint16_t*)W1, out, K, N, sink.perm, sink.w);
}

template <int MODE>
static void launch_plain_product(const TiledPlan& p, int prod, const void* A, const int32_t* perm, int kdiv,
                                 const int32_t* tab, const void* W0, void* out, int K, int N, hipStream_t st,
                                 GateSink sink = GateSink())
{
    const int nb = prod == 0 ? p.nb_up : p.nb_down;
    if ((p.bm == kBMBig || (prod == 1 && p.tall_down)) && nb == 1) launch_product<MODE, kBMBig, 1>(p, prod, A, perm, kdiv, tab, W0, nullptr, out, K, N, st, sink);
    else if (p.bm == kBMBig) launch_product<MODE, kBMBig, 2>(p, prod, A, perm, kdiv, tab, W0, nullptr, out, K, N, st, sink);
    else if (nb == 2) launch_product<MODE, kBMSmall, 2>(p, prod, A, perm, kdiv, tab, W0, nullptr, out, K, N, st, sink);
    else launch_product<MODE, kBMSmall, 1>(p, prod, A, perm, kdiv, tab, W0, nullptr, out, K, N, st, sink);
}

void launch_tile_lists(const mmoe_shape& s, const int32_t* offsets, int32_t* tab, hipStream_t st, SlotFilter filt)
{
    const TiledPlan p = tiled_plan(s);
    hipLaunchKernelGGL(tile_table_kernel, dim3(2), dim3(kListThreads), 0, st, offsets, tab, s.S, p.nt_up, p.nt_down,
                       p.L, filt);
}

TileJob tile_job(const mmoe_shape& s, int32_t* tab)
{
    const TiledPlan p = tiled_plan(s);
    TileJob j;
    j.tab = tab;
    j.nt_up = p.nt_up;
    j.nt_down = p.nt_down;
    j.L = p.L;
    return j;
}

int launch_ffn_tiled(const mmoe_shape& s, const void* rows, const int32_t* perm, const int32_t* offsets,
                     const void* W1p, const void* W3p, const void* W2p, void* H, float* Yg, int32_t* tab,
                     hipStream_t st, hipEvent_t mid, bool tab_ready, SlotFilter filt, GateSink sink)
{
    const int P = s.T * s.top_k, d = s.d_model, f = s.d_ff;
    if ((int64_t)P * (d > f ? d : f) >= ((int64_t)1 << 31)) return MMOE_ERR_LIMIT;  // 32-bit byte offsets inside a panel
    if (sink.w && (s.top_k != 1 || !sink.perm || !sink.Y)) return MMOE_ERR_DIM;
    const TiledPlan p = tiled_plan(s);
    if (!tab_ready) launch_tile_lists(s, offsets, tab, st, filt);
    if (s.dtype == MMOE_F32) {
        (p.nb_up == 2 ? launch_up_split : launch_up_f32)(s, p, rows, perm, tab, W1p, W3p, H, st);
        if (mid && hipEventRecord(mid, st) != hipSuccess) return MMOE_ERR_LAUNCH;
        (p.nb_down == 2 ? launch_down_split : launch_down_f32)(s, p, tab, W2p, H, Yg, st, sink);
        return launch_status();
    }
    if (s.act == MMOE_SWIGLU) {
        if (p.bm == kBMBig)
            launch_product<kTModeSwigluH, kBMBig, 2>(p, 0, rows, perm, s.top_k, tab, W1p, W3p, H, d, f, st);
        else
            launch_product<kTModeSwigluH, kBMSmall, 2>(p, 0, rows, perm, s.top_k, tab, W1p, W3p, H, d, f, st);
    } else if (s.act == MMOE_GELU) {
        launch_plain_product<kTModeGeluH>(p, 0, rows, perm, s.top_k, tab, W1p, H, d, f, st);
    } else {
        launch_plain_product<kTModeReluH>(p, 0, rows, perm, s.top_k, tab, W1p, H, d, f, st);
    }
    if (mid && hipEventRecord(mid, st) != hipSuccess) return MMOE_ERR_LAUNCH;
    if (sink.w) {
        launch_plain_product<kTModeGatedY>(p, 1, H, nullptr, 1, tab, W2p, sink.Y, f, d, st, sink);
    } else {
        launch_plain_product<kTModePlainF32>(p, 1, H, nullptr, 1, tab, W2p, Yg, f, d, st);
    }
    return launch_status();
}

}  // namespace mmoe
