// Tile lists of the matrix-core expert kernels: layout, sizes, and the device code that writes
// them from the slots' first rows (one workgroup per product: of the kernel that groups the pairs, or
// of a kernel of its own when the caller brings the offsets).
#pragma once

#include "mmoe_internal.h"

namespace mmoe {

constexpr int kBMBig = 256;    // token rows per tile: large batches (one workgroup per compute unit)
constexpr int kBMSmall = 128;  // token rows per tile: batches with few tiles (two workgroups per compute unit)
constexpr int kXcds = 8;
constexpr int kNtGroup = 4;  // least number of feature tiles whose workgroups start back to back on the same token panel

// Tile lists, written by one workgroup from the device-side `offsets`.
//
// Row tiles.  A slot with c rows is u = ceil(c / 32) sub-tiles of 32 rows.  It is cut into
// mt = max(ceil(u / upt), ceil(u / h)) tiles whose heights differ by at most one sub-tile (upt = most
// sub-tiles of a tile, given per product by the host: a full tile's 8 or 4; h <= upt = the target height
// that the builder chooses per product from the counts, see build_tile_lists): the first u mod mt
// tiles have floor(u / mt) + 1 sub-tiles, the others floor(u / mt).  No slot has a short last tile (a tile of one sub-tile streams its weight panel
// for an eighth of the arithmetic), and no matrix instruction is spent on padding beyond the last
// partial sub-tile.
//
// Order.  The tiles of a product are listed by (slot, group of feature tiles, row tile, feature tile
// within the group): workgroups start in id order, so the ones that share a token panel and the ones
// that share a weight panel run close enough in time to find the panel in L2.  The group is sized so
// that the workgroups resident on an XCD at one time form a block of row tiles x feature tiles that is
// as square as the slot allows (8 x 4 for a slot of 8 row tiles, 4 x 8 for one of 4).
//
// XCDs.  Workgroup id 8*local + x runs on XCD x and computes entry `local` of the XCD's list, an int4
// {slot (and kOnlyTile), feature tile, first row, rows}; tab[8 p + x] = number of entries of product p's list for XCD x.
// The weight panels of the batch -- the feature tiles of the slots that hold rows, slot after slot -- are
// dealt to the XCDs in turn: panel c to XCD c mod 8, with all its row tiles, so a weight panel is read
// by one XCD and every XCD has the same number of panels to within one.  Where NT is a multiple of 8 this
// gives XCD x the feature tiles nt with nt mod 8 == x of every slot, and the XCDs share one list whose
// feature tiles count within the XCD (nt = 8*entry + x).  Dealing by nt mod 8 alone whatever NT gave 10
// feature tiles to the XCDs as 2,2,1,1,1,1,1,1 (1.6 times an even share) and 6 as 1,1,1,1,1,1,0,0.
// (64 experts of 2048 x 1280, 1037 tokens, 10 up panels a slot: up product 226 -> 179 us; 768 x 3072,
// 4096 tokens, 6 down panels: 53 -> 47 us.)
// In runs (RunsRule) the list of all tiles is cut into eight contiguous runs of as many tiles each instead: a slot's
// token rows are read by one or two XCDs and not by min(8, NT) of them, and no XCD has more tiles than another
// (xcd_runs says where that pays).  kRunsForFewerRounds: where panels in turn bring some XCD into a further round of
// `conc` tiles and runs do not.  The target height is chosen so that the tiles just fill a round; the panels of unequal
// slots, NT no multiple of 8, then put more than a round on some XCD.
// Neighbouring tiles are of one height, so runs of tiles that differ in cost keep the XCDs busy for unequal times: the
// up product of 4096 x 14336, 777 tokens, 1310 us by panels, 1629 in runs.  Runs of equal cost (half a sub-tile and the
// height for each tile) are worse than runs of equal count: an XCD with more tiles than compute units begins another
// round (layer, us, 2560 x 7680, 3200 pairs, 12 slots 496 : 561; 768 x 3072, 8000 tokens, 16 unequal slots 136 : 152).
//
// Target heights of a row tile that the table builder may choose from, in quarters of a 32-row
// sub-tile: from a full tile (4 upt) down to hq_lo, which the host gives with the tile kernels (tile_rows_of).
constexpr int kMaxHeightCands = 16;

// In an entry's first word: the slot, and whether the tile holds all rows of the slot (not set where few slots hold rows).
constexpr int kSlotMask = 0xFFFF, kOnlyTile = 1 << 16;
static_assert(kMaxS <= kSlotMask, "slot ids");

enum RunsRule { kRunsNever = 0, kRunsAlways = 1, kRunsForFewerRounds = 2 };

// Heights of a product's row tiles, and how many of its tiles a compute unit works on at a time.
struct TileRows {
    int upt;      // most 32-row sub-tiles of a row tile
    int hq_lo;    // least target height, in quarters of a sub-tile
    int hq_step;  // quarters between two target heights
    int conc_log2;  // log2 of the tiles that an XCD works on in the time of one (`conc`), for the choice of the height
    bool fill;    // the lists have room for as many row tiles as fill whole rounds of the chip
};

struct TileLists {
    int list[2];    // [product: up, down] -> int4 index into tab of XCD 0's list
    int lists[2];   // 1: the XCDs share one list; kXcds: one list each, `len` entries apart
    int len[2];     // entries reserved per list of each product: workgroups per XCD
    int runs[2];    // RunsRule
    TileRows rows[2];
    int rows_cap[2]; // most row tiles of each product
    int lone_slots; // least number of slots with rows for which kOnlyTile is set (lone_tiles)
    size_t bytes;
};

// Row tiles the lists have room for: an eighth more than full tiles can need (fp32: than tiles of two
// sub-tiles), which is sum_s ceil(ceil(c_s / 32) / upt) <= P / (32 upt) + S.  The grid of a product is
// sized by this bound (the host does not know the counts), and a workgroup without a tile still waits
// for a compute unit before it can leave, so the room for lower target heights is kept small; with `fill` it
// reaches to the end of the last round that full tiles can need.
inline int row_tiles_cap(int P, int S, int NT, const TileRows& r, bool f32)
{
    const int u = f32 ? 2 : r.upt;
    const int full = (P + 32 * u - 1) / (32 * u) + S, cap = full + (full + 7) / 8;
    if (!r.fill) return cap;
    const int round = kXcds << r.conc_log2;  // tiles
    const int64_t filled = ((int64_t)full * NT + round - 1) / round * round / NT;
    return filled > cap ? (int)filled : cap;
}

// Lists of a product with NT feature tiles, and entries of each: a slot has at most ceil(NT / 8) panels on one XCD.
inline int list_count(int NT, int runs) { return NT % kXcds == 0 && runs == kRunsNever ? 1 : kXcds; }
inline int list_len(int cap, int NT) { return cap * ((NT + kXcds - 1) / kXcds); }
constexpr int kListHeader = 16;  // int4 units: the first 256 bytes

inline TileLists tile_lists(int P, int S, int nt_up, int nt_down, const TileRows& up, const TileRows& down, bool f32,
                            int runs_up, int runs_down, int lone_slots)
{
    TileLists L;
    L.lone_slots = lone_slots;
    L.rows[0] = up;
    L.rows[1] = down;
    L.runs[0] = runs_up;
    L.runs[1] = runs_down;
    int at = kListHeader;
    for (int p = 0; p < 2; ++p) {
        const int NT = p == 0 ? nt_up : nt_down;
        L.rows_cap[p] = row_tiles_cap(P, S, NT, L.rows[p], f32);
        L.lists[p] = list_count(NT, L.runs[p]);
        L.len[p] = list_len(L.rows_cap[p], NT);
        L.list[p] = at;
        at += L.lists[p] * L.len[p];
    }
    L.bytes = (size_t)at * 16;
    return L;
}

// x / d for 0 <= x < 2^24, d > 0: the hardware reciprocal is within one unit in the last place, so the
// truncated product is off by at most one (an integer division in full is some forty instructions, and
// the list builder is one serial chain in front of the expert kernels).
__device__ __forceinline__ int div24(int x, int d)
{
    const int q = (int)((float)x * __builtin_amdgcn_rcpf((float)d));
    const int r = x - q * d;
    return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}

// Inclusive sum over the lanes of a wavefront, all of them taking part: within rows of 16 lanes, then the sums of the rows
// before, in vector instructions (__shfl_up goes through the LDS pipe six times, one behind the other: with it, an exchange
// through LDS for the best height and a division in 64 bits, grouping 4148 pairs in 90 slots and listing their tiles took
// 10.8 us from the first instruction to the last, now 9.7; 4096 pairs in 18 slots 8.8, now 8.2).
__device__ __forceinline__ int wave_scan(int v)
{
    constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    v += __builtin_amdgcn_update_dpp(0, v, kRowShr + 1, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, kRowShr + 2, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, kRowShr + 4, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, kRowShr + 8, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, kRowBcast15, 0xA, 0xF, false);  // rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, kRowBcast31, 0xC, 0xF, false);  // rows 2 and 3
    return v;
}

// The value of the wavefront's last lane.
__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, kWave - 1); }

// Writes the lists of product p.  One workgroup of kListThreads threads, a slot to a thread; every thread
// must call.  LDS, both visible to the whole workgroup: `off` holds the first row of every slot and, at S,
// the number of rows; `first` is kXcds * kMaxS ints of scratch.  Slots that `filt` skips get no tiles.
constexpr int kListThreads = 1024;
constexpr int kListWaves = kListThreads / kWave;
static_assert(kMaxS <= kListThreads && kXcds <= kListWaves, "a slot to a thread, an XCD to a wavefront");

__device__ __forceinline__ void build_tile_lists(const int* off, int32_t* __restrict__ tab, int S, int p, int NT,
                                                 const TileLists& L, int* first, SlotFilter filt = SlotFilter())
{
    __shared__ int base[kMaxS + 1];    // row tiles of the slots before each slot
    __shared__ int pbase[kMaxS];       // slots that hold rows before each slot
    __shared__ int cand[kMaxHeightCands];  // row tiles of the whole batch at every candidate height
    __shared__ int part[kListWaves];
    __shared__ int total[kXcds];       // entries of every XCD's list
    __shared__ int units_all, chosen_hq;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int conc_log2 = L.rows[p].conc_log2, conc = 1 << conc_log2, upt = L.rows[p].upt, hq_step = L.rows[p].hq_step;
    int4* lists = reinterpret_cast<int4*>(tab);
    auto units_of = [&](int s) { return s >= S || filt.skips(s) ? 0 : (off[s + 1] - off[s] + 31) >> 5; };
    auto tiles_at = [&](int u, int hq) { return max(div24(u + upt - 1, upt), div24(4 * u + hq - 1, hq)); };
    // Target height.  A slot of u sub-tiles is cut into max(ceil(u / upt), ceil(u / h)) tiles, h the
    // target height, the same for all slots.  h is chosen here, from the counts, so that the product's
    // tiles fill whole rounds of the chip: with `conc` workgroups resident per XCD a product of M row
    // tiles takes about ceil(M NT / (8 conc)) rounds of one tile each, a tile costing a fixed part
    // (half a sub-tile's worth of time: prologue and epilogue) plus its height.  Lower targets also
    // bring the slots' tile heights closer together.  The cut decides where tiles begin, not what a
    // row's result is.
    const int hq_hi = 4 * upt, ncand = (hq_hi - L.rows[p].hq_lo) / hq_step + 1;  // <= kMaxHeightCands
    if (tid < kMaxHeightCands) cand[tid] = 0;
    if (tid == 0) units_all = 0;
    __syncthreads();
    {   // thread = (candidate c, one of 64 groups of slots): integer sums, so their order does not matter
        const int c = tid % kMaxHeightCands;
        int tiles = 0, units = 0;
        for (int s = tid / kMaxHeightCands; s < S; s += kListThreads / kMaxHeightCands) {
            const int u = units_of(s);
            units += u;
            if (c < ncand) tiles += tiles_at(u, hq_hi - hq_step * c);
        }
        static_assert(kMaxHeightCands == 16, "four groups of slots to a wavefront");
        tiles += lane_xor<16>(tiles);
        tiles += lane_xor<32>(tiles);
        units += lane_xor<16>(units);
        units += lane_xor<32>(units);
        if (lane < kMaxHeightCands && tiles) atomicAdd(&cand[c], tiles);
        if (lane == 0 && units) atomicAdd(&units_all, units);
    }
    __syncthreads();
    if (wave == 0) {  // a candidate to a lane of sixteen; of equal costs the tallest
        const int U = units_all, M = lane < kMaxHeightCands ? cand[lane] : 0;
        float cost = INFINITY;
        // no rows at all, or more tiles than the lists hold (the tallest candidate always fits)
        if (lane < ncand && M > 0 && M <= L.rows_cap[p]) {
            static_assert(kXcds == 8, "rounds are shifts");
            const int rounds = (int)(((int64_t)M * NT + kXcds * conc - 1) >> (3 + conc_log2));
            cost = (float)rounds * (0.5f + (float)U / (float)M);
        }
        int best = lane;
        auto better = [&](auto off) {
            const float oc = __uint_as_float(lane_xor<decltype(off)::value>(__float_as_uint(cost)));
            const int ob = lane_xor<decltype(off)::value>(best);
            const bool take = oc < cost || (oc == cost && ob < best);
            cost = take ? oc : cost;
            best = take ? ob : best;
        };
        better(std::integral_constant<int, 8>{});
        better(std::integral_constant<int, 4>{});
        better(std::integral_constant<int, 2>{});
        better(std::integral_constant<int, 1>{});
        if (lane == 0) chosen_hq = hq_hi - hq_step * best;
    }
    __syncthreads();
    // exclusive prefix sums of the row tiles and of the slots that hold rows, a slot to a thread
    const int u_mine = units_of(tid);
    const int mine = tiles_at(u_mine, chosen_hq), pmine = u_mine > 0 ? 1 : 0;
    // (both sums in one word: up to 1024 slots, and up to 2^18 row tiles of 32 rows, and one a slot, of under 2^31 / 256 rows)
    constexpr int kSlotBits = 11;
    static_assert(kMaxS < 1 << kSlotBits, "slots that hold rows");
    const int both = mine << kSlotBits | pmine, incl = wave_scan(both);
    if (lane == kWave - 1) part[wave] = incl;
    __syncthreads();
    int before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < kListWaves; ++w) {
        const int x = part[w];
        if (w < wave) before += x;
        sum += x;
    }
    const int total_m = sum >> kSlotBits, touched = sum & ((1 << kSlotBits) - 1);
    const bool lone = touched >= L.lone_slots;
    if (tid < S) {
        const int excl = before + incl - both;
        base[tid] = excl >> kSlotBits;
        pbase[tid] = excl & ((1 << kSlotBits) - 1);
    }
    if (tid == 0) base[S] = total_m;
    __syncthreads();
    const bool shared_list = L.lists[p] == 1;
    bool runs = L.runs[p] == kRunsAlways;
    const int share = (total_m * NT + kXcds - 1) / kXcds;  // tiles of an XCD's run
    // Panels of slot s (the r-th that holds rows) on XCD x: the c = r NT + nt with c mod 8 == x.
    // panels_before(x, c) of them lie before panel c.
    auto panels_before = [](int x, int c) { return (c + kXcds - 1 - x) / kXcds; };
    if (!runs && !shared_list) {
        // first entry of every slot in every XCD's list: an XCD to a wavefront, 64 slots at a time
        if (wave < kXcds) {
            const int x = wave;
            int carry = 0;
            for (int s0 = 0; s0 < S; s0 += kWave) {
                const int s = s0 + lane;
                int c = 0;
                if (s < S) {
                    const int c0 = pbase[s] * NT;
                    c = (base[s + 1] - base[s]) * (panels_before(x, c0 + NT) - panels_before(x, c0));
                }
                const int inc = wave_scan(c);
                if (s < S) first[x * kMaxS + s] = carry + inc - c;
                carry += last_lane(inc);
            }
            if (lane == 0) total[x] = carry;
        }
        __syncthreads();
        if (L.runs[p] == kRunsForFewerRounds) {
            int most = 0;
#pragma unroll
            for (int x = 0; x < kXcds; ++x) most = max(most, total[x]);
            runs = div24(most + conc - 1, conc) > div24(share + conc - 1, conc);
        }
    }
    if (tid < kXcds)
        tab[kXcds * p + tid] = shared_list ? total_m * (NT / kXcds) : runs ? min(share, max(total_m * NT - tid * share, 0)) : total[tid];
    // the lists: all threads on the shared one (with runs: on the tiles of all XCDs in order), an eighth of them on each
    // XCD's own
    constexpr int kPerXcd = kListThreads / kXcds;
    const bool all = shared_list || runs;
    const int x = all ? 0 : tid / kPerXcd, nt_all = runs ? NT : NT / kXcds;  // panels of a slot in a list that all work on
    const int n = all ? total_m * nt_all : total[x];
    for (int e = all ? tid : tid % kPerXcd; e < n; e += all ? kListThreads : kPerXcd) {
        auto first_of = [&](int s) { return all ? base[s] * nt_all : first[x * kMaxS + s]; };
        int lo = 0, hi = S;  // largest s with first_of(s) <= e (slots without entries have equal bounds)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first_of(mid) <= e) lo = mid; else hi = mid;
        }
        const int s = lo, mt = base[s + 1] - base[s];
        const int rem = e - first_of(s);
        const int c0 = pbase[s] * NT, j0 = panels_before(x, c0);
        const int nt_x = all ? nt_all : panels_before(x, c0 + NT) - j0;  // the slot's panels on this XCD
        // groups of g feature tiles; inside a group the feature tile runs fastest
        const int g = min(nt_x, max(kNtGroup, div24(conc, mt)));
        const int grp = div24(rem, g * mt), within = rem - grp * (g * mt);
        const int g_sz = min(g, nt_x - grp * g);
        const int i = div24(within, g_sz), j = grp * g + within - i * g_sz;  // j-th panel of the slot here
        const int ntl = all ? j : (j0 + j) * kXcds + x - c0;
        // row tile i of the slot: the first `extra` tiles are one sub-tile taller
        const int u = units_of(s), h = div24(u, mt), extra = u - h * mt;
        const int row0 = 32 * (i * h + min(i, extra));
        const int rows = 32 * (h + (i < extra ? 1 : 0));
        const int to = runs ? div24(e, share) : x;
        lists[L.list[p] + to * L.len[p] + e - (runs ? to * share : 0)] =
            make_int4(lone && mt == 1 ? s | kOnlyTile : s, ntl, off[s] + row0, min(rows, off[s + 1] - off[s] - row0));
    }
}


// Everything the launches of one shape share: tile height, weight blocks per wavefront and feature
// tiles of both products, and the tile lists' layout.
bool lone_tiles(const mmoe_shape& s);
struct TiledPlan {
    int bm, nt_up, nt_down, nb_up, nb_down;
    bool tall_down;  // 256-row tiles of the down product beside a height of 128 (tile_share)
    bool ahead[2];  // fp32 parts: eight wavefronts to a tile (f32_ahead), per product
    bool lone;  // the kernels that read the panels of one-tile slots past the caches (lone_tiles)
    TileLists L;
};

// fp32: tiles of up to 96 rows; 64 features on the fp32 instruction (ffn_tiled_f32.hip: plan with one weight block per
// wavefront), 128 (gated: 64) on bf16 parts (ffn_split_f32.hip: two weight blocks).
constexpr int kFRows = 96, kFeatF32 = 64;
void launch_up_f32(const mmoe_shape& s, const TiledPlan& p, const void* rows, const int32_t* perm, const int32_t* tab,
                   const void* W1p, const void* W3p, void* H, hipStream_t st);
void launch_down_f32(const mmoe_shape& s, const TiledPlan& p, const int32_t* tab, const void* W2p, const void* H, float* Yg,
                     hipStream_t st, GateSink sink);
void launch_up_split(const mmoe_shape& s, const TiledPlan& p, const void* rows, const int32_t* perm, const int32_t* tab,
                     const void* W1p, const void* W3p, void* H, hipStream_t st);
void launch_down_split(const mmoe_shape& s, const TiledPlan& p, const int32_t* tab, const void* W2p, const void* H, float* Yg,
                       hipStream_t st, GateSink sink);

// What the grouping kernels need to write the lists themselves (null `tab`: they do not).
struct TileJob {
    int32_t* tab;
    int nt_up, nt_down;
    TileLists L;
};

// The job for this shape (host side; defined beside the matrix-core kernels).  Null `tab`: no job.
TileJob tile_job(const mmoe_shape& s, int32_t* tab);

// The lists of both products from the device-side `offsets`, in a launch of their own.
void launch_tile_lists(const mmoe_shape& s, const int32_t* offsets, int32_t* tab, hipStream_t st,
                       SlotFilter filt = SlotFilter());

}  // namespace mmoe
