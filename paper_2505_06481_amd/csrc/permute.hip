// Steps M and G: expert-map lookup, slot histogram, exclusive scan, stable grouping of
// the (token, pick) pairs by pool slot, and the row gather (Algorithm 2, the map lookup
// that precedes the expert call; grouping is what lets one resident expert serve every
// token that hit it, whichever variant the token belongs to).
//
// Deterministic by construction: the rank of pair p inside its slot is the number of
// lower pair ids with the same slot, computed from wavefront ballots and integer
// prefix sums.  There are no cursors bumped by atomics and no waiting between
// workgroups.  Up to kGroupMaxP pairs one kernel does it all (group_kernel); larger batches take
// two or three short ones (histogram, scan, scatter; two when the scatter workgroups can afford to sum
// the histograms themselves).
//
// Work split of the large form: workgroup b owns pairs [b*2048, (b+1)*2048); inside it wavefront w
// owns a contiguous quarter, walked 64 pairs at a time in ascending order.
#include "mmoe_internal.h"
#include "tile_table.h"

namespace mmoe {

constexpr int kPermThreads = 256;
constexpr int kPermWaves = kPermThreads / kWave;
constexpr int kPairsPerWave = kPermChunk / kPermWaves;  // 512
constexpr int kOwnScanMax = 1 << 14;  // most per-workgroup counts (workgroups x slots) a scatter workgroup sums by itself
static_assert(kMaxS % kPermThreads == 0, "slots per thread");

// slot[p] = M[vid[p / k]][topk_idx[p]]; per-workgroup histogram of the slots.
__global__ __launch_bounds__(kPermThreads) void slot_hist_kernel(
    const int32_t* __restrict__ vid, const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ M,
    int32_t* __restrict__ slot, int32_t* __restrict__ blk_counts, int P, int k, int V, int E, int S)
{
    __shared__ int hist[kMaxS];
    for (int s = threadIdx.x; s < S; s += kPermThreads) hist[s] = 0;
    __syncthreads();
    const int base = blockIdx.x * kPermChunk;
    for (int i = threadIdx.x; i < kPermChunk; i += kPermThreads) {
        int p = base + i;
        if (p < P) {
            // clamps keep every later index in range even for invalid ids (results then undefined)
            int v = min(max(vid[p / k], 0), V - 1);
            int e = min(max(topk_idx[p], 0), E - 1);
            int s = min(max(M[v * E + e], 0), S - 1);
            slot[p] = s;
            atomicAdd(&hist[s], 1);  // integer LDS atomic: the sum does not depend on order
        }
    }
    __syncthreads();
    for (int s = threadIdx.x; s < S; s += kPermThreads) blk_counts[(size_t)blockIdx.x * S + s] = hist[s];
}

// counts, offsets, and for every (workgroup, slot) the first output row of that workgroup's pairs.
__global__ __launch_bounds__(kPermThreads) void slot_scan_kernel(const int32_t* __restrict__ blk_counts,
                                                                 int32_t* __restrict__ blk_base,
                                                                 int32_t* __restrict__ counts,
                                                                 int32_t* __restrict__ offsets, int nblk, int S)
{
    __shared__ int tot[kMaxS];
    __shared__ int off[kMaxS + 1];
    for (int s = threadIdx.x; s < S; s += kPermThreads) {
        int run = 0;
        for (int b = 0; b < nblk; ++b) {
            int c = blk_counts[(size_t)b * S + s];
            blk_base[(size_t)b * S + s] = run;
            run += c;
        }
        tot[s] = run;
        counts[s] = run;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {  // one wavefront scans the S totals, 64 at a time
        int carry = 0;
        for (int s0 = 0; s0 < S; s0 += kWave) {
            int s = s0 + threadIdx.x;
            int c = s < S ? tot[s] : 0;
            const int incl = wave_scan(c);
            if (s < S) off[s] = carry + incl - c;
            carry += last_lane(incl);
        }
        if (threadIdx.x == 0) off[S] = carry;
    }
    __syncthreads();
    for (int s = threadIdx.x; s <= S; s += kPermThreads) offsets[s] = off[s];
    for (int s = threadIdx.x; s < S; s += kPermThreads) {
        int o = off[s];
        for (int b = 0; b < nblk; ++b) blk_base[(size_t)b * S + s] += o;
    }
}

// Lanes of the wavefront whose pair has this lane's slot: one ballot per bit of the slot id.
__device__ __forceinline__ unsigned long long same_slot(int s, bool valid, int sbits)
{
    unsigned long long m = __ballot(valid);
    for (int b = 0; b < sbits; ++b) {
        const bool bit = (s >> b) & 1;
        const unsigned long long bal = __ballot(bit);
        m &= bit ? bal : ~bal;
    }
    return m;
}

// Stable placement of up to 64 pairs, one per lane, behind the pairs placed before them:
// a lane's row is the slot's cursor plus the number of peers in lower lanes; the lowest
// peer then advances the cursor.  `cur` is this wavefront's private cursor row in LDS, and
// LDS operations of one wavefront execute in program order.
__device__ __forceinline__ void place_pairs(volatile int* cur, int s, bool valid, int lane, int sbits, int p,
                                            int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm)
{
    const unsigned long long m = same_slot(s, valid, sbits);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    int base = 0;
    if (valid) {
        base = cur[s];
        const int r = base + rank;
        perm[r] = p;
        inv_perm[p] = r;
    }
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) cur[s] = base + __popcll(m);
    __builtin_amdgcn_wave_barrier();
}

// perm / inv_perm: stable ranks from ballots.  Where the first output row of this workgroup's pairs of
// every slot comes from:
//   kFromScan    `blk_base`, written by slot_scan_kernel;
//   kOwnScan     few workgroups, few slots, so the table of per-workgroup counts is small: every
//                workgroup sums that table itself, and the scan kernel and its launch are not needed;
// With kOwnScan the grid has one more workgroup, which places no pairs and writes counts and offsets
// instead.
enum { kFromScan = 0, kOwnScan = 1 };
template <int SRC>
__global__ __launch_bounds__(kPermThreads) void slot_scatter_kernel(const int32_t* __restrict__ slot,
                                                                    const int32_t* __restrict__ blk_base,
                                                                    const int32_t* __restrict__ blk_counts, int nblk,
                                                                    int32_t* __restrict__ counts,
                                                                    int32_t* __restrict__ offsets,
                                                                    int32_t* __restrict__ perm,
                                                                    int32_t* __restrict__ inv_perm, int P, int S)
{
    __shared__ int wtot[kPermWaves][kMaxS];  // pairs of each slot owned by each wavefront
    __shared__ int cursor[kPermWaves][kMaxS];
    constexpr bool SCAN = SRC == kOwnScan;
    __shared__ int tot[SCAN ? kMaxS : 1];    // pairs of each slot in the whole batch, then its first row
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int sbits = 32 - __clz(max(S - 1, 1));  // bits of a slot id
    int before[kMaxS / kPermThreads];             // this workgroup's first row of slot threadIdx.x + 256 i
    if (SCAN) {
        const int b = blockIdx.x;  // nblk: the workgroup that writes the tables
#pragma unroll
        for (int i = 0; i < kMaxS / kPermThreads; ++i) {
            const int sl = threadIdx.x + i * kPermThreads;
            int run = 0, mine = 0;
            if (sl < S)
                for (int bb = 0; bb < nblk; ++bb) {
                    if (bb == b) mine = run;
                    run += blk_counts[(size_t)bb * S + sl];
                }
            before[i] = mine;
            if (sl < S) tot[sl] = run;
        }
        __syncthreads();
        if (b == nblk)
            for (int sl = threadIdx.x; sl < S; sl += kPermThreads) counts[sl] = tot[sl];
        __syncthreads();
        if (threadIdx.x < kWave) {  // exclusive scan of the S totals, 64 at a time; tot[s] becomes offsets[s]
            int carry = 0;
            for (int s0 = 0; s0 < S; s0 += kWave) {
                const int sl = s0 + threadIdx.x;
                const int c = sl < S ? tot[sl] : 0;
                const int incl = wave_scan(c);
                if (sl < S) {
                    tot[sl] = carry + incl - c;
                    if (b == nblk) offsets[sl] = carry + incl - c;
                }
                carry += last_lane(incl);
            }
            if (b == nblk && threadIdx.x == 0) offsets[S] = carry;
        }
        __syncthreads();
        if (b == nblk) return;  // uniform over the workgroup
    }
    for (int i = threadIdx.x; i < kPermWaves * S; i += kPermThreads) wtot[i / S][i % S] = 0;
    __syncthreads();
    const int wbase = blockIdx.x * kPermChunk + wave * kPairsPerWave;
    for (int i = lane; i < kPairsPerWave; i += kWave) {
        int p = wbase + i;
        if (p < P) atomicAdd(&wtot[wave][slot[p]], 1);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kMaxS / kPermThreads; ++i) {
        const int s = threadIdx.x + i * kPermThreads;
        if (s < S) {
            int run = SCAN ? tot[s] + before[i] : blk_base[(size_t)blockIdx.x * S + s];
#pragma unroll
            for (int w = 0; w < kPermWaves; ++w) {
                cursor[w][s] = run;
                run += wtot[w][s];
            }
        }
    }
    __syncthreads();
    // From here on a wavefront touches only its own cursor row; LDS operations of one
    // wavefront execute in program order.
    volatile int* cur = cursor[wave];
    for (int i0 = 0; i0 < kPairsPerWave; i0 += kWave) {
        int p = wbase + i0 + lane;
        bool valid = p < P;
        int s = valid ? slot[p] : 0;
        place_pairs(cur, s, valid, lane, sbits, p, perm, inv_perm);
    }
}

// Grouping in one launch.  It stands between the router and the expert kernels with nothing to
// overlap it, so its cost is the length of its dependency chain: every workgroup counts the whole
// batch by itself (sixteen wavefronts, each a contiguous sixteenth of the pairs, ranks from ballots, the
// wavefront's running counts in LDS), so that nothing is handed from one workgroup or launch to the
// next, and workgroup b < nblk then places the pairs of its own four steps.  The last two workgroups
// write the tile lists of the up and of the down product instead.  Ranks and rows are the large
// form's.
// Measured against one workgroup of 256 threads that walked 512 pairs per wavefront, or three to nine
// workgroups that counted with atomics, list building included: 543 pairs 16.4 -> 7.3 us, 4096 pairs
// 16.3 -> 9.6 us, 4148 pairs in 90 slots 25.3 -> 12.5 us, 16384 pairs 24 -> 17 us.  Beyond that every
// workgroup's count of the whole batch outgrows the launches it saves (about 0.5 us per 1024 pairs).
constexpr int kGroupThreads = kListThreads;
constexpr int kGroupWaves = kGroupThreads / kWave;
constexpr int kGroupSteps = 4;                                 // steps of 1024 pairs whose pairs one workgroup places
constexpr int kGroupChunk = kGroupThreads * kGroupSteps;
constexpr int kGroupMaxP = 4 * kGroupChunk;
static_assert(kGroupMaxP <= 65535, "running counts are 16 bits wide");

// LOOKUP: slot[p] is looked up here and written; otherwise the router has written it.
template <bool LOOKUP>
__global__ __launch_bounds__(kGroupThreads) void group_kernel(
    const int32_t* __restrict__ vid, const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ M,
    int32_t* __restrict__ slot, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
    int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, int P, int k, int V, int E, int S, int nblk,
    TileJob tiles)
{
    // running counts of every wavefront, then the rows of the slot in front of the wavefront's; the list
    // builder's scratch at the end
    __shared__ __align__(16) int scratch[kXcds * kMaxS];
    static_assert(sizeof(scratch) >= sizeof(uint16_t) * kGroupWaves * kMaxS, "one array for both");
    __shared__ int off[kMaxS + 1];
    __shared__ int part[kGroupWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int b = blockIdx.x;
    const int sbits = 32 - __clz(max(S - 1, 1));  // bits of a slot id
    const int steps = (P + kGroupThreads - 1) / kGroupThreads;  // of 64 pairs, per wavefront
    const int wbase = wave * steps * kWave;
    volatile uint16_t* row = reinterpret_cast<uint16_t*>(scratch) + wave * kMaxS;
    for (int s = lane; s < S; s += kWave) row[s] = 0;

    auto slot_of = [&](int step) {
        const int p = wbase + step * kWave + lane;
        if (step >= steps || p >= P) return -1;
        if (!LOOKUP) return slot[p];
        // clamps keep every later index in range even for invalid ids (results then undefined)
        const int v = min(max(vid[p / k], 0), V - 1);
        const int e = min(max(topk_idx[p], 0), E - 1);
        return min(max(M[v * E + e], 0), S - 1);
    };
    int cur[kGroupSteps], nxt[kGroupSteps];
    int my_slot[kGroupSteps], my_rank[kGroupSteps];  // of the pairs this workgroup places
#pragma unroll
    for (int u = 0; u < kGroupSteps; ++u) {
        nxt[u] = slot_of(u);
        my_slot[u] = -1;
    }
    for (int blk = 0; blk < nblk; ++blk) {
#pragma unroll
        for (int u = 0; u < kGroupSteps; ++u) {
            cur[u] = nxt[u];
            nxt[u] = slot_of((blk + 1) * kGroupSteps + u);
        }
#pragma unroll
        for (int u = 0; u < kGroupSteps; ++u) {
            if (blk * kGroupSteps + u >= steps) break;  // uniform over the workgroup
            const int s = cur[u];
            const bool valid = s >= 0;
            const unsigned long long m = same_slot(valid ? s : 0, valid, sbits);
            const int rank = __popcll(m & ((1ull << lane) - 1ull));
            int prev = 0;
            if (valid) prev = row[s];
            __builtin_amdgcn_wave_barrier();
            if (valid && rank == 0) row[s] = (uint16_t)(prev + __popcll(m));
            __builtin_amdgcn_wave_barrier();
            if (blk == b) {
                my_slot[u] = s;
                my_rank[u] = prev + rank;
            }
        }
    }
    __syncthreads();
    uint16_t* const all = reinterpret_cast<uint16_t*>(scratch);
    int tot = 0;
    if (tid < S) {  // a slot to a thread (S <= 1024)
#pragma unroll
        for (int w = 0; w < kGroupWaves; ++w) {
            const int c = all[w * kMaxS + tid];
            all[w * kMaxS + tid] = (uint16_t)tot;
            tot += c;
        }
    }
    const int incl = wave_scan(tot);
    if (lane == kWave - 1) part[wave] = incl;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int w = 0; w < kGroupWaves; ++w)
        if (w < wave) before += part[w];
    if (tid < S) {
        off[tid] = before + incl - tot;
        if (b == 0) {
            counts[tid] = tot;
            offsets[tid] = before + incl - tot;
        }
    }
    if (tid == 0) {
        off[S] = P;
        if (b == 0) offsets[S] = P;
    }
    __syncthreads();
    if (b >= nblk) {  // uniform over the workgroup; these two exist only when lists are wanted
        const int prod = b - nblk;
        build_tile_lists(off, tiles.tab, S, prod, prod == 0 ? tiles.nt_up : tiles.nt_down, tiles.L, scratch);
        return;
    }
#pragma unroll
    for (int u = 0; u < kGroupSteps; ++u) {
        if (my_slot[u] < 0) continue;
        const int p = wbase + (b * kGroupSteps + u) * kWave + lane;
        const int r = off[my_slot[u]] + all[wave * kMaxS + my_slot[u]] + my_rank[u];
        if (LOOKUP) slot[p] = my_slot[u];
        perm[r] = p;
        inv_perm[p] = r;
    }
}

// Xg[r,:] = X[perm[r] / k, :], one wavefront per row, 16 bytes per lane per step.
__global__ __launch_bounds__(kPermThreads) void gather_rows_kernel(const u32x4* __restrict__ X,
                                                                   const int32_t* __restrict__ perm,
                                                                   u32x4* __restrict__ Xg, int P, int k,
                                                                   int row_vec)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int r = blockIdx.x * kPermWaves + threadIdx.x / kWave;
    if (r >= P) return;
    const int t = perm[r] / k;
    const u32x4* src = X + (size_t)t * row_vec;
    u32x4* dst = Xg + (size_t)r * row_vec;
    for (int i = lane; i < row_vec; i += kWave) dst[i] = src[i];
}

__global__ void validate_kernel(const int32_t* __restrict__ vid, const int32_t* __restrict__ M,
                                int32_t* __restrict__ flag, int T, int V, int E, int S)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    if (i < T) bad = vid[i] < 0 || vid[i] >= V;
    if (i < V * E) bad = bad || M[i] < 0 || M[i] >= S;
    if (bad) atomicOr(flag, 1);
}

__global__ void clear_flag_kernel(int32_t* flag) { *flag = 0; }

int launch_validate(const mmoe_shape& s, const int32_t* vid, const int32_t* M, int32_t* flag, hipStream_t st)
{
    int n = s.T > s.V * s.E ? s.T : s.V * s.E;
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(1), 0, st, flag);
    hipLaunchKernelGGL(validate_kernel, dim3((n + 255) / 256), dim3(256), 0, st, vid, M, flag, s.T, s.V, s.E,
                       s.S);
    return launch_status();
}

int launch_permute(const mmoe_shape& s, const void* X, const int32_t* vid, const int32_t* topk_idx,
                   const int32_t* M, int32_t* slot, int32_t* counts, int32_t* offsets, int32_t* perm,
                   int32_t* inv_perm, void* Xg, int32_t* blk_counts, int32_t* blk_base, int nblk, hipStream_t st,
                   int32_t* tile_tab, bool slot_ready)
{
    const int P = s.T * s.top_k;
    const TileJob tiles = tile_job(s, tile_tab);
    if (P <= kGroupMaxP) {
        const int n = (P + kGroupChunk - 1) / kGroupChunk;
        const dim3 grid(n + (tiles.tab ? 2 : 0)), block(kGroupThreads);
        if (slot_ready)
            hipLaunchKernelGGL(group_kernel<false>, grid, block, 0, st, vid, topk_idx, M, slot, counts, offsets, perm,
                               inv_perm, P, s.top_k, s.V, s.E, s.S, n, tiles);
        else
            hipLaunchKernelGGL(group_kernel<true>, grid, block, 0, st, vid, topk_idx, M, slot, counts, offsets, perm,
                               inv_perm, P, s.top_k, s.V, s.E, s.S, n, tiles);
    } else {
        hipLaunchKernelGGL(slot_hist_kernel, dim3(nblk), dim3(kPermThreads), 0, st, vid, topk_idx, M, slot,
                           blk_counts, P, s.top_k, s.V, s.E, s.S);
        if ((int64_t)nblk * s.S <= kOwnScanMax) {
            hipLaunchKernelGGL(slot_scatter_kernel<kOwnScan>, dim3(nblk + 1), dim3(kPermThreads), 0, st, slot, blk_base,
                               blk_counts, nblk, counts, offsets, perm, inv_perm, P, s.S);
        } else {
            hipLaunchKernelGGL(slot_scan_kernel, dim3(1), dim3(kPermThreads), 0, st, blk_counts, blk_base, counts,
                               offsets, nblk, s.S);
            hipLaunchKernelGGL(slot_scatter_kernel<kFromScan>, dim3(nblk), dim3(kPermThreads), 0, st, slot, blk_base,
                               blk_counts, nblk, counts, offsets, perm, inv_perm, P, s.S);
        }
        if (tiles.tab) launch_tile_lists(s, offsets, tiles.tab, st);
    }
    if (!Xg) return launch_status();
    const int row_vec = (int)((size_t)s.d_model * elem_size(s.dtype) / 16);
    hipLaunchKernelGGL(gather_rows_kernel, dim3((P + kPermWaves - 1) / kPermWaves), dim3(kPermThreads), 0, st,
                       (const u32x4*)X, perm, (u32x4*)Xg, P, s.top_k, row_vec);
    return launch_status();
}

}  // namespace mmoe
