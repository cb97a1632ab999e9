// Step R: per-variant gate, top-k selection and coefficients (Algorithm 2, "gate(act)";
// section 3.2).  Four launch shapes with the same arithmetic: small batches give a token to a
// workgroup whose wavefronts share out the experts (latency); large batches give a token to
// one wavefront that keeps the token row in registers and walks the experts, or four tokens to a workgroup, or, with
// much to score, four tokens of a variant to a wavefront (throughput).
//
// The logit is an fp32 sum in the fixed order the header states: lane l owns the
// elements i with (i div 4) mod 64 == l, which is exactly what a coalesced 4-element
// vector load per lane delivers; each lane folds its elements in ascending i with one
// fused multiply-add each; the 64 partial sums meet in an xor butterfly 32,16,...,1.
// fp32 addition is commutative, so both partners of an exchange compute the same sum and
// every lane ends with the same value.
//
// Logits are parked in LDS, then the k winners are found by wavefront arg-max
// reductions: lane l looks after experts l, l+64, ...; ties go to the lower index.
// Coefficients: softmax over the selected logits, or (gate over all experts) each selected
// expert's entry of the softmax over all E logits, whose normaliser is one more wavefront
// reduction over the parked logits.
#include <type_traits>

#include "mmoe_internal.h"

namespace mmoe {

constexpr int kRouteWaves = 8;   // wavefronts per token: they share out the experts

// Four consecutive elements as loaded (bf16 stays packed until it is used, which halves the
// registers a pending load occupies).
template <typename T> struct Raw4;
template <> struct Raw4<float> {
    typedef f32x4 type;
    static __device__ __forceinline__ float get(const type& r, int q) { return r[q]; }
};
template <> struct Raw4<uint16_t> {
    typedef u32x2 type;
    static __device__ __forceinline__ float get(const type& r, int q)
    {
        return (q & 1) ? __uint_as_float(r[q >> 1] & 0xFFFF0000u) : __uint_as_float(r[q >> 1] << 16);
    }
};

constexpr int kNoExpert = 0x7FFFFFFF;  // a lane with no expert left to offer

// f(offset) for the offsets 32, 16, ..., 1 that are below n.
template <typename F>
__device__ __forceinline__ void for_offsets_below(int n, F f)
{
    if (32 < n) f(std::integral_constant<int, 32>{});
    if (16 < n) f(std::integral_constant<int, 16>{});
    if (8 < n) f(std::integral_constant<int, 8>{});
    if (4 < n) f(std::integral_constant<int, 4>{});
    if (2 < n) f(std::integral_constant<int, 2>{});
    if (1 < n) f(std::integral_constant<int, 1>{});
}

// The butterfly of one sum: every lane has it.
__device__ __forceinline__ float butterfly(float p)
{
    for_offsets_below(kWave, [&](auto off) { p = p + lane_xor<decltype(off)::value>(p); });
    return p;
}

// Two levels of four butterflies at once (one exchange and one addition for two sums), then the other four levels of all of
// them: what a lane adds is its partner's partial sum either way, so every sum is the contract's.  Lanes 0-15 have the sum of
// a, 16-31 of b, 32-47 of c, 48-63 of d.
__device__ __forceinline__ float butterfly4(float a, float b, float c, float d)
{
    auto swap32 = [](float x, float y) {  // x in lanes 0-31, y in lanes 32-63
        const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    const float ac = swap32(a, c), bd = swap32(b, d);
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(ac), __float_as_uint(bd), false, false);
    float p = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    for_offsets_below(16, [&](auto off) { p = p + lane_xor<decltype(off)::value>(p); });
    return p;
}

// Expert e's bit among those of `lane`, which looks after experts lane, lane + 64, ...; 0 if it is another lane's.
// kNoExpert is lane 63's by its low bits and has no bit: its shift count would be out of range.
constexpr uint32_t expert_bit(int e, int lane)
{
    return e < kMaxE && (e & (kWave - 1)) == lane ? 1u << (e / kWave) : 0u;
}
// an out-of-range shift does not compile here
static_assert(expert_bit(kNoExpert, kWave - 1) == 0 && expert_bit(kMaxE - 1, kWave - 1) == 1u << (kMaxE / kWave - 1) &&
                  expert_bit(kWave, 0) == 2 && expert_bit(kWave, 1) == 0,
              "bits of the experts a lane looks after");

// The k winners among E logits in LDS, found by one wavefront: lane l looks after experts
// l, l+64, l+128, l+192; k arg-max reductions, ties to the lower index; coefficients =
// softmax over the selected logits.
// Lanes from the next power of two above E on hold no expert, so the reductions stop there.
// With a table row `map_row` (= M[vid[t]] in LDS, or null) the picks are also looked up in the expert
// map and slot[t*k + j] is written: step M folded into the router for batches whose expert stage
// groups the pairs itself.
__device__ __forceinline__ void select_topk(const float* __restrict__ lds_logit, int lane, int E, int k, int t,
                                            int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                            const int32_t* map_row, int32_t* __restrict__ slot, int S, int gate)
{
    constexpr int kPerLane = kMaxE / kWave;
    float mine[kPerLane];
#pragma unroll
    for (int q = 0; q < kPerLane; ++q) {
        int e = lane + q * kWave;
        mine[q] = e < E ? lds_logit[e] : -INFINITY;
    }
    uint32_t taken = 0;
    float sel[kMaxTopK];
    int seli[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        if (j < k) {
            float bv = -INFINITY;
            int be = kNoExpert;
#pragma unroll
            for (int q = 0; q < kPerLane; ++q) {  // ascending index: strict > keeps the lower one
                int e = lane + q * kWave;
                if (e < E && !(taken & (1u << q)) && (be == kNoExpert || mine[q] > bv)) {
                    bv = mine[q];
                    be = e;
                }
            }
            for_offsets_below(E, [&](auto off) {
                const float ov = lane_xor<decltype(off)::value>(bv);
                const int oe = lane_xor<decltype(off)::value>(be);
                const bool other_valid = oe != kNoExpert, self_valid = be != kNoExpert;
                const bool take = other_valid && (!self_valid || ov > bv || (ov == bv && oe < be));
                bv = take ? ov : bv;
                be = take ? oe : be;
            });
            sel[j] = bv;
            seli[j] = be;
            taken |= expert_bit(be, lane);
        }
    }
    // gate over all experts: the normaliser is the sum of exp(logit - largest logit) over every expert
    // (sel[0] is the largest); fp32, lane-local in ascending expert index, then an xor butterfly
    float all = 0.0f;
    if (gate == MMOE_GATE_ALL) {
#pragma unroll
        for (int q = 0; q < kPerLane; ++q)
            if (lane + q * kWave < E) all += expf(mine[q] - sel[0]);
        for_offsets_below(E, [&](auto off) { all += lane_xor<decltype(off)::value>(all); });
    }
    if (lane == 0) {
        float z[kMaxTopK];
        float tot = 0.0f;
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k) {
                z[j] = expf(sel[j] - sel[0]);
                tot += z[j];
            }
        if (gate == MMOE_GATE_ALL) tot = all;
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k) {
                topk_idx[(size_t)t * k + j] = seli[j];
                topk_w[(size_t)t * k + j] = z[j] / tot;
                // the clamp keeps every later index in range even for an invalid table (results then undefined)
                if (map_row) slot[(size_t)t * k + j] = min(max(map_row[seli[j]], 0), S - 1);
            }
    }
}

// The same for four tokens of a wavefront at once, E <= 16: lanes 16 i .. 16 i + 15 look after token i's experts (its
// logits at lds_logit + i * kMaxE, its number in `t`, `map` the table's entry for this lane's expert if `look_up`; `write`: not
// for the repeats that fill a group).
__device__ __forceinline__ void select_topk4(const float* __restrict__ lds_logit, int lane, int E, int k, int t, bool write,
                                             int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                             bool look_up, int map, int32_t* __restrict__ slot, int S, int gate)
{
    const int e = lane & 15;
    const float mine = e < E ? lds_logit[(lane >> 4) * kMaxE + e] : -INFINITY;
    bool taken = e >= E;
    float sel[kMaxTopK];
    int seli[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        if (j < k) {
            float bv = taken ? -INFINITY : mine;
            int be = taken ? kNoExpert : e;
            for_offsets_below(E, [&](auto off) {  // within 16 lanes
                const float ov = lane_xor<decltype(off)::value>(bv);
                const int oe = lane_xor<decltype(off)::value>(be);
                const bool take = oe != kNoExpert && (be == kNoExpert || ov > bv || (ov == bv && oe < be));
                bv = take ? ov : bv;
                be = take ? oe : be;
            });
            sel[j] = bv;
            seli[j] = be;
            taken = taken || be == e;
        }
    }
    float tot = 0.0f;
    if (gate == MMOE_GATE_ALL) {
        if (e < E) tot += expf(mine - sel[0]);
        for_offsets_below(E, [&](auto off) { tot += lane_xor<decltype(off)::value>(tot); });
    }
    int place[kMaxTopK];
    if (look_up) {
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k) place[j] = __shfl(map, (lane & 48) | (seli[j] & 15), kWave);
    }
    if (e != 0 || !write) return;
    float z[kMaxTopK];
    float picked = 0.0f;
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j)
        if (j < k) {
            z[j] = expf(sel[j] - sel[0]);
            picked += z[j];
        }
    if (gate != MMOE_GATE_ALL) tot = picked;
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j)
        if (j < k) {
            topk_idx[(size_t)t * k + j] = seli[j];
            topk_w[(size_t)t * k + j] = z[j] / tot;
            if (look_up) slot[(size_t)t * k + j] = min(max(place[j], 0), S - 1);  // the clamp as in select_topk
        }
}

// One workgroup per token; wavefront w scores experts w, w+8, ...  A token's dot product
// with one expert is never split between wavefronts, so the summation order is the
// contract's whatever the launch shape.  What bounds it is the chain of dependent memory reads, so there
// are two: the variant id, and then everything else at once -- KU chunks of 256 elements of both rows,
// bias, table row (chunks past the end re-read the last one and are not summed).  With four chunks at a
// time, the remainder one by one and the table read behind the selection one token of 4096 elements took 7.5 us
// (now 6.6), three of 768 5.0 us (4.6), and a layer of 1037 tokens and 64 experts 361 us (346).
template <typename T, int KU>
__global__ __launch_bounds__(kRouteWaves* kWave) void route_kernel(
    const T* __restrict__ X, const int32_t* __restrict__ vid, const T* __restrict__ Wr,
    const float* __restrict__ br, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int Tn, int d,
    int V, int E, int k, const int32_t* __restrict__ M, int32_t* __restrict__ slot, int S, int gate)
{
    __shared__ float lds_logit[kMaxE];
    __shared__ int32_t lds_map[kMaxE];
    static_assert(kMaxE <= kRouteWaves * kWave, "a table entry to a thread");
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int t = blockIdx.x;
    typedef typename Raw4<T>::type raw_t;

    const T* x = X + (size_t)t * d + 4 * lane;
    const int nc = d / 256, last = nc - 1;  // chunks: d is a multiple of 256
    raw_t xv[KU], wv[KU];
#pragma unroll
    for (int u = 0; u < KU; ++u) xv[u] = *reinterpret_cast<const raw_t*>(x + 256 * min(u, last));
    const int v = min(max(vid[t], 0), V - 1);  // out-of-range ids are the caller's error; stay in bounds
    if (M && threadIdx.x < E) lds_map[threadIdx.x] = M[(size_t)v * E + threadIdx.x];

    for (int e = wave; e < E; e += kRouteWaves) {
        const T* w = Wr + ((size_t)v * E + e) * d + 4 * lane;
        const float bias = br ? br[(size_t)v * E + e] : 0.0f;
        float acc = 0.0f;
        for (int c0 = 0; c0 < nc; c0 += KU) {  // ascending i within the lane
#pragma unroll
            for (int u = 0; u < KU; ++u) wv[u] = *reinterpret_cast<const raw_t*>(w + 256 * min(c0 + u, last));
            if (nc > KU) {  // the token row does not fit the registers: its chunks are read again for every expert
#pragma unroll
                for (int u = 0; u < KU; ++u) xv[u] = *reinterpret_cast<const raw_t*>(x + 256 * min(c0 + u, last));
            }
#pragma unroll
            for (int u = 0; u < KU; ++u)
                if (c0 + u < nc) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc = __builtin_fmaf(Raw4<T>::get(xv[u], c), Raw4<T>::get(wv[u], c), acc);
                }
        }
        float p = butterfly(acc);
        if (br) p = p + bias;
        if (lane == 0) lds_logit[e] = p;
    }
    __syncthreads();
    if (wave != 0) return;

    select_topk(lds_logit, lane, E, k, t, topk_idx, topk_w, M ? lds_map : nullptr, slot, S, gate);
}

// Batches with much to score: a workgroup takes kRouteGroup tokens, so a router row is read once for
// those of them that share a variant instead of once per token, and unpacked once.  Token rows in LDS as
// stored; wavefront w of sixteen scores experts w, w+16, ... for all of the group's tokens, whose sums share a
// butterfly.  (Tried: rows in LDS in fp32, pairs of experts, the next rows requested a step ahead, with 4, 8 or 16
// wavefronts: equal to a quarter slower, 6000 tokens of 2048, 32 experts 46 -> 48 to 57 us.)  Bound by the chain of reads per
// expert at the small end, by vector issue at the large.
// 1024 tokens of 3072 elements, 64 experts, bf16: 39.1 (workgroup per token) -> 27.5 us, fp32 62.7 -> 25.5;
// 8192 tokens of 4096, 64 experts: 237 (wavefront per token) -> 158 us; of 2304, 8 experts: 76.6 -> 35.7 us.
constexpr int kRouteGroup = 4;
constexpr int kGroupRound = 256 * kRouteGroup;  // tokens of a workgroup for each compute unit
constexpr int kRouteGroupWaves = 16;

template <typename T>
__global__ __launch_bounds__(kRouteGroupWaves* kWave) void route_group_kernel(
    const T* __restrict__ X, const int32_t* __restrict__ vid, const T* __restrict__ Wr,
    const float* __restrict__ br, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int Tn, int d,
    int V, int E, int k, const int32_t* __restrict__ M, int32_t* __restrict__ slot, int S, int gate)
{
    constexpr int TB = kRouteGroup, KU = 8;
    static_assert(TB == 4, "two levels of the butterfly");
    extern __shared__ __align__(16) char rows[];  // [TB][d] as stored
    __shared__ float lds_logit[TB][kMaxE];
    __shared__ int32_t lds_map[TB][kMaxE];
    typedef typename Raw4<T>::type raw_t;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int t0 = blockIdx.x * TB;
    const int nc = d / 256, last = nc - 1;

    int v[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) v[i] = min(max(vid[min(t0 + i, Tn - 1)], 0), V - 1);
    const int pieces = d * (int)sizeof(T) / 16;  // per row
#pragma unroll
    for (int i = 0; i < TB; ++i) {
        const u32x4* src = reinterpret_cast<const u32x4*>(X + (size_t)min(t0 + i, Tn - 1) * d);
        for (int q = threadIdx.x; q < pieces; q += kRouteGroupWaves * kWave) reinterpret_cast<u32x4*>(rows)[i * pieces + q] = src[q];
        if (M)
            for (int e = threadIdx.x; e < E; e += kRouteGroupWaves * kWave) lds_map[i][e] = M[(size_t)v[i] * E + e];
    }
    __syncthreads();

    const T* xrow = reinterpret_cast<const T*>(rows) + 4 * lane;
    for (int e = wave; e < E; e += kRouteGroupWaves) {
        float acc[TB];
#pragma unroll
        for (int i = 0; i < TB; ++i) acc[i] = 0.0f;
        unsigned todo = (1u << TB) - 1;
        while (todo) {  // uniform: the tokens of one variant at a time
            const int first = __builtin_ctz(todo);
            int ve = v[0];
#pragma unroll
            for (int i = 1; i < TB; ++i) ve = first == i ? v[i] : ve;
            unsigned set = 0;
#pragma unroll
            for (int i = 0; i < TB; ++i) set |= v[i] == ve ? 1u << i : 0u;
            todo &= ~set;
            const T* w = Wr + ((size_t)ve * E + e) * d + 4 * lane;
            for (int c0 = 0; c0 < nc; c0 += KU) {  // ascending i within the lane
                raw_t wv[KU];
#pragma unroll
                for (int u = 0; u < KU; ++u) wv[u] = *reinterpret_cast<const raw_t*>(w + 256 * min(c0 + u, last));
#pragma unroll
                for (int i = 0; i < TB; ++i)
                    if (set & (1u << i)) {
#pragma unroll
                        for (int u = 0; u < KU; ++u)
                            if (c0 + u < nc) {
                                const raw_t xv = *reinterpret_cast<const raw_t*>(xrow + (size_t)i * d + 256 * (c0 + u));
#pragma unroll
                                for (int c = 0; c < 4; ++c)
                                    acc[i] = __builtin_fmaf(Raw4<T>::get(xv, c), Raw4<T>::get(wv[u], c), acc[i]);
                            }
                    }
            }
        }
        const float p = butterfly4(acc[0], acc[1], acc[2], acc[3]);
        const int tok = lane / 16;
        if ((lane & 15) == 0) {
            const int vt = tok == 0 ? v[0] : tok == 1 ? v[1] : tok == 2 ? v[2] : v[3];
            lds_logit[tok][e] = br ? p + br[(size_t)vt * E + e] : p;
        }
    }
    __syncthreads();
    if (wave >= TB || t0 + wave >= Tn) return;
    select_topk(lds_logit[wave], lane, E, k, t0 + wave, topk_idx, topk_w, M ? lds_map[wave] : nullptr, slot, S, gate);
}

// Throughput variant for large batches: one wavefront per token.  The token's elements
// stay in registers (NC chunks of 256, d = 256*NC exactly, so that every load of a pass is
// issued before the first one is waited for) and the wavefront walks the experts
// four at a time, so that the token row crosses the memory pipeline once instead of once
// per expert and four sums share a butterfly (two experts at a time and a butterfly for each: 16000 tokens of 256
// elements, 64 experts 79 -> 39 us; 4000 of 1024, 32 experts 22.8 -> 19.6; 4096 of 768, 8 experts 7.6 -> 6.9; 16384 of 4096, 8 experts 76.6 ->
// 74.6).  Each (token, expert) sum is formed by one wavefront in the contract's order:
// the results are bit-identical to route_kernel's.
constexpr int kRouteTokWaves = 4;
// batches at least this large use the wavefront-per-token kernel (measured crossover: between
// 1024 and 2048 tokens at d = 4096 and at d = 768)
constexpr int kRouteTokMinT = 2048;

template <typename T, int NC>
__global__ __launch_bounds__(kRouteTokWaves* kWave) void route_token_kernel(
    const T* __restrict__ X, const int32_t* __restrict__ vid, const T* __restrict__ Wr,
    const float* __restrict__ br, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int Tn, int d,
    int V, int E, int k, const int32_t* __restrict__ M, int32_t* __restrict__ slot, int S, int gate)
{
    __shared__ float lds_logit[kRouteTokWaves][kMaxE];
    __shared__ int32_t lds_map[kRouteTokWaves][kMaxE];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int t = blockIdx.x * kRouteTokWaves + wave;
    if (t >= Tn) return;  // uniform over the wavefront; no workgroup barrier below

    const int v = min(max(vid[t], 0), V - 1);
    const T* x = X + (size_t)t * d + 4 * lane;
    typedef typename Raw4<T>::type raw_t;
    raw_t xv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) xv[c] = *reinterpret_cast<const raw_t*>(x + 256 * c);

    const T* wv0 = Wr + (size_t)v * E * d + 4 * lane;
    float* mylogit = lds_logit[wave];
    if (M)
        for (int e = lane; e < E; e += kWave) lds_map[wave][e] = M[(size_t)v * E + e];
    constexpr int EB = 4;  // experts at a time
    for (int e = 0; e < E; e += EB) {
        float a[EB];
        constexpr int NB = NC * (int)sizeof(raw_t) > 64 ? 2 : EB;  // router rows in registers
#pragma unroll
        for (int b0 = 0; b0 < EB; b0 += NB) {
            raw_t p[NB][NC];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    p[b][c] = *reinterpret_cast<const raw_t*>(wv0 + (size_t)min(e + b0 + b, E - 1) * d + 256 * c);
#pragma unroll
            for (int b = 0; b < NB; ++b) a[b0 + b] = 0.0f;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {  // ascending i within the lane
                    const float xq = Raw4<T>::get(xv[c], q);
#pragma unroll
                    for (int b = 0; b < NB; ++b) a[b0 + b] = __builtin_fmaf(xq, Raw4<T>::get(p[b][c], q), a[b0 + b]);
                }
        }
        float p = butterfly4(a[0], a[1], a[2], a[3]);
        const int mine = e + lane / 16;
        if ((lane & 15) == 0 && mine < E) mylogit[mine] = br ? p + br[(size_t)v * E + mine] : p;
    }
    // the LDS writes of this wavefront's lanes before its reads: one wavefront's LDS operations execute in
    // program order, the fence keeps the compiler from moving them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    select_topk(mylogit, lane, E, k, t, topk_idx, topk_w, M ? lds_map[wave] : nullptr, slot, S, gate);
}

// bf16 batches with much to score: four tokens of one variant against four or eight experts to a wavefront, straight from
// memory.  A router row is then read and unpacked once for four tokens, a token row once for as many experts, where the
// other kernels unpack one or both for every product; bound by vector issue and, at the small end, by the latency of the
// loads, which only other wavefronts hide: chunks requested ahead cost the registers of those (1037 tokens of 2048, 64 experts, four
// chunks in flight 30.2 us, two 20.1, one 19.9).  Time against the other kernels: route_in_tiles.
//
// Groups: a chunk of 64 tokens is cut, variant by variant in the order of their first tokens, into groups of four of a
// variant (the last one of a variant filled up with repeats, which are not written); workgroup or wavefront j of a chunk
// finds group j from the 64 ids by ballots, and leaves if there are fewer.
constexpr int kTileChunk = 64, kTileTokens = 4;
inline int tile_groups(int V) { return kTileChunk / kTileTokens + (3 * V + 3) / 4 < kTileChunk ? kTileChunk / kTileTokens + (3 * V + 3) / 4 : kTileChunk; }

// SOLO: every wavefront of four has a group of its own and scores all experts (E <= EB); otherwise the W wavefronts of a
// workgroup share a group, EB experts at a time each.
template <int EB, int W, bool SOLO>
__global__ __launch_bounds__(W* kWave) void route_tile_kernel(
    const uint16_t* __restrict__ X, const int32_t* __restrict__ vid, const uint16_t* __restrict__ Wr,
    const float* __restrict__ br, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w, int Tn, int d,
    int V, int E, int k, const int32_t* __restrict__ M, int32_t* __restrict__ slot, int S, int gate, int groups)
{
    constexpr int TB = kTileTokens;
    static_assert(EB % 4 == 0 && TB == 4 && W >= TB, "sums of four experts share a butterfly; a wavefront selects for a token");
    __shared__ float lds_logit[SOLO ? W : 1][TB][kMaxE];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int unit = SOLO ? blockIdx.x * W + wave : blockIdx.x;
    const int chunk = unit / groups, base = chunk * kTileChunk;
    if (base >= Tn) return;  // uniform over the wavefront, and over the workgroup where it shares a group
    int j = unit - chunk * groups;

    const bool there = base + lane < Tn;
    const int mv = there ? min(max(vid[base + lane], 0), V - 1) : -1;  // out-of-range ids are the caller's error; stay in bounds
    unsigned long long todo = __ballot(there), members = 0;
    int v = 0, n = 0;
    while (todo) {
        v = __builtin_amdgcn_readlane(mv, (int)__builtin_ctzll(todo));
        members = __ballot(mv == v);
        n = __popcll(members);
        const int g = (n + TB - 1) / TB;
        if (j < g) break;
        j -= g;
        todo &= ~members;
    }
    if (!todo) return;  // the chunk has fewer groups; uniform as above
    const int rank = __popcll(members & ((1ull << lane) - 1ull));
    int tok[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i)
        tok[i] = base + (int)__builtin_ctzll(__ballot(mv == v && rank == min(TB * j + i, n - 1)));
    const int have = min(TB, n - TB * j);

    __shared__ int32_t lds_map[SOLO ? 1 : kMaxE];
    int map = 0;
    if (M && SOLO) map = M[(size_t)v * E + min(lane & 15, E - 1)];
    if (M && !SOLO)
        for (int e = threadIdx.x; e < E; e += W * kWave) lds_map[e] = M[(size_t)v * E + e];

    const uint16_t* xrow[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) xrow[i] = X + (size_t)tok[i] * d;
    const uint16_t* wbase = Wr + (size_t)v * E * d;
    const int nc = d / 256;
    float* const logit = &lds_logit[SOLO ? wave : 0][0][0];
    for (int e0 = SOLO ? 0 : wave * EB; e0 < E; e0 += W * EB) {
        const uint16_t* wrow[EB];
#pragma unroll
        for (int b = 0; b < EB; ++b) wrow[b] = wbase + (size_t)min(e0 + b, E - 1) * d;
        float acc[TB][EB];
#pragma unroll
        for (int i = 0; i < TB; ++i)
#pragma unroll
            for (int b = 0; b < EB; ++b) acc[i][b] = 0.0f;
        for (int c = 0; c < nc; ++c) {
            const int o = 256 * c + 4 * lane;
            u32x2 xv[TB], wv[EB];
#pragma unroll
            for (int i = 0; i < TB; ++i) xv[i] = *reinterpret_cast<const u32x2*>(xrow[i] + o);
#pragma unroll
            for (int b = 0; b < EB; ++b) wv[b] = *reinterpret_cast<const u32x2*>(wrow[b] + o);
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // ascending i within the lane
                float x[TB];
#pragma unroll
                for (int i = 0; i < TB; ++i) x[i] = Raw4<uint16_t>::get(xv[i], q);
#pragma unroll
                for (int b = 0; b < EB; ++b) {
                    const float w = Raw4<uint16_t>::get(wv[b], q);
#pragma unroll
                    for (int i = 0; i < TB; ++i) acc[i][b] = __builtin_fmaf(x[i], w, acc[i][b]);
                }
            }
        }
#pragma unroll
        for (int b0 = 0; b0 < EB; b0 += 4) {
            const int e = e0 + b0 + lane / 16;
            const bool mine = (lane & 15) == 0 && e < E;
            const float bias = br && mine ? br[(size_t)v * E + e] : 0.0f;
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                const float p = butterfly4(acc[i][b0], acc[i][b0 + 1], acc[i][b0 + 2], acc[i][b0 + 3]);
                if (mine) logit[i * kMaxE + e] = br ? p + bias : p;
            }
        }
    }
    if (SOLO) {
        // one wavefront's LDS operations execute in program order, the fence keeps the compiler from moving them
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int i = lane >> 4, t = i == 0 ? tok[0] : i == 1 ? tok[1] : i == 2 ? tok[2] : tok[3];
        select_topk4(logit, lane, E, k, t, i < have, topk_idx, topk_w, M != nullptr, map, slot, S, gate);
        return;
    }
    __syncthreads();
    if (wave >= have) return;
    const int t = wave == 0 ? tok[0] : wave == 1 ? tok[1] : wave == 2 ? tok[2] : tok[3];
    select_topk(logit + wave * kMaxE, lane, E, k, t, topk_idx, topk_w, M ? lds_map : nullptr, slot, S, gate);
}

template <int EB, int W, bool SOLO>
static void launch_tiles(const mmoe_shape& s, const void* X, const int32_t* vid, const void* Wr, const float* br,
                         int32_t* topk_idx, float* topk_w, hipStream_t st, const int32_t* M, int32_t* slot)
{
    const int groups = tile_groups(s.V);
    const int64_t units = (int64_t)((s.T + kTileChunk - 1) / kTileChunk) * groups;
    const dim3 grid((unsigned)(SOLO ? (units + W - 1) / W : units));
    hipLaunchKernelGGL((route_tile_kernel<EB, W, SOLO>), grid, dim3(W * kWave), 0, st, (const uint16_t*)X, vid, (const uint16_t*)Wr,
                       br, topk_idx, topk_w, s.T, s.d_model, s.V, s.E, s.top_k, M, slot, s.S, s.gate, groups);
}

// Most LDS for the token rows of a group: fp32 rows of 4096.  Over kRouteGroupLarge the rows, which have to arrive before the
// first score, take long enough that there has to be something to score.  fp32 rows of 3584 and 4096, two variants, us,
// caches warm / cold, the other kernel : groups, by tokens and experts:
//   768   1  9.5 : 9.5 / 10.0 : 13.1     4  9.5 : 9.5 / 12.6 : 13.7    8  10.6 : 9.4 / 16.2 : 14.9   64  48 : 26 / 59 : 32
//   1024  1  9.5 : 9.5 / 12.5 : 14.3     3  9.5 : 9.4 / 13.9 : 14.6    4  9.5 : 9.5 / 14.9 : 14.8    8  12.7 : 10.6 / 19.4 : 16.3
//   1536  2  9.7 : 9.6 / 17.2 : 17.5     3  10.5 : 9.8 / 18.3 : 17.7   8  17.2 : 12.3 / 25.8 : 20.2
//   2000  1  11.0 : 9.6 / 19.2 : 19.3    2  12.2 : 9.9 / 20.4 : 19.6
//   against a wavefront per token  2500 tokens of 4096  16  37 : 25 / 60 : 36   64  122 : 69 / 186 : 76
constexpr size_t kRouteGroupBytes = 64 << 10, kRouteGroupLarge = 48 << 10;
constexpr int64_t kRouteLargeScores = 3500;  // tokens x experts

// A wavefront per token, unless four tokens go to a workgroup?  Large batches of a common hidden size.
static bool wavefront_per_token(const mmoe_shape& s)
{
    const int nc = s.d_model / 256;
    return s.T >= kRouteTokMinT && (nc == 1 || nc == 2 || nc == 3 || nc == 4 || nc == 6 || nc == 8 || nc == 12 || nc == 16);
}

// Four tokens to a workgroup?  Measured against the other two, bf16, us, two variants:
//   workgroup per token (under 2048 tokens, or an uncommon hidden size): 8 experts, 768 elements 8.2 : 8.6 at 1900 tokens;
//   1536 9.4 : 9.3 at 1500; 2048 7.8 : 8.0 at 1024; 3072 7.8 : 9.1 at 512, 12.1 : 9.2 at 768; 64 experts 2048 22.6 : 19.4 at
//   1024, 14.2 : 18.3 at 512;
//   wavefront per token: 4096 tokens, 64 experts 768 27.5 : 42.4, 1536 51.0 : 43.9, 4096 123 : 84; 16 experts 2048 19.9 : 20.1,
//   3072 28.1 : 26.6, 4096 35.7 : 29.5; 8 experts 4096 20.9 : 22.5.
bool route_in_groups(const mmoe_shape& s)
{
    const size_t bytes = (size_t)kRouteGroup * s.d_model * elem_size(s.dtype);
    if (bytes > kRouteGroupBytes || (bytes > kRouteGroupLarge && (int64_t)s.T * s.E < kRouteLargeScores)) return false;
    if (wavefront_per_token(s)) return s.d_model >= 1536 && (int64_t)s.E * s.d_model >= 49152;
    // (inside a layer, whose weights push the router out of the L2s, 1037 tokens of 2048 and 64 experts take 348 : 350 us and
    // 1900 of 2048 and 8 154 : 155; 1900 of 2304 and 8 131 : 121, 1200 of 3072 and 64 243 : 237)
    return (s.d_model >= 2304 || s.T >= kRouteTokMinT) && s.T >= 768 && (int64_t)s.T * s.d_model >= ((int64_t)1 << 21);
}

// Four tokens of a variant to a wavefront?  Measured against the other kernels, other : tiles, us.  Caches warm / cold, two to
// four variants:
//   8 experts   2500 tokens of 4096 18.2 : 16.4 / 27.8 : 24.2   8192 of 4096 41.4 : 24.5 / 59.0 : 44.5   16384 of 4096 82 : 49 / 105 : 70
//               8000 of 768 10.6 : 9.1 / 15.4 : 14.2   16000 of 2048 38 : 22 / 53 : 38   1500 of 4096 14.9 : 16.1 / 18.8 : 23.1
//               4096 of 768 6.8 : 7.4 / 11.0 : 11.6   2049 of 3072 10.4 : 12.6 / -   3000 of 2048 10.2 : 11.2 / -
//   16          9000 of 2048 40 : 26 / 49 : 39   600 of 1024 5.7 : 6.2 / 8.4 : 10.7
//   32          700 of 3072 19.7 : 11.4 / 23.0 : 20.4   8000 of 1024 35.8 : 27.0 / 41.4 : 33.7   600 of 1024 8.3 : 7.4 / 11.1 : 12.2
//   64          1037 of 2048 28.6 : 19.8 / 32.3 : 24.0   4000 of 2048 54 : 39 / 59 : 47   512 of 2048 16.4 : 13.6 / 19.0 : 20.6
// Wavefronts of eight experts with fewer than seven to score would idle.
//
// kTileVariants: in any order, the tokens of many variants leave more of the groups partly filled, and there may be more groups.
// Mixed tokens, 8 / 16 / 32 / 64 variants:
//   32 experts  8000 of 1024  34.0 : 29.4 / 34.2 : 36.9 / 34.8 : 56.7 / 35.8 : 105.6
//   8           8192 of 4096  40.3 : 23.8 / 40.5 : 30.1 / 40.9 : 34.1 / 42.2 : 54.2    8000 of 768 10.5 : 9.5 / 10.5 : 10.7 / 10.7 : 13.7 / 11.4 : 25.5
//   64          4000 of 2048  67.1 : 36.9 / 67.8 : 48.7 / 69.8 : 62.7 / 83.2 : 106.5
// Rows of up to 1024 elements, where there is less to share: 12 experts, 4096 of 1024, 8 variants 9.8 : 10.8.
//
// Batches of a few rounds of route_group_kernel (a round: a workgroup to every compute unit): where neighbouring tokens are of one
// variant, its groups read a router row once for four tokens too, with eight chunks in flight.  They win with few experts, and
// with more where they fill their rounds: the line for one variant.  Variants that take turns are the ordinary batch, where tiles win
// from 16 experts on.  Tiles in their time, one variant / four, mixed / four, one after the other:
//   12 experts  1024 of 4096 1.13 / 1.30 / 1.12   2040 of 4096 1.29 / 0.92 / 1.25   13, 3072 of 8192, eight, one after the other 1.28
//   16          1024 of 3072 1.12 / 0.83 / 1.09   1200 of 5120 1.15 / 0.75 / 1.16   1500 of 2304 0.81 / 0.51 / 0.80
//   32          1024 of 4096 1.28 / 0.87 / 1.17   1200 of 4096 0.86 / 0.59 / 0.83   1800 of 4096 0.84 / 0.77 / 1.14   2040 1.16 / 0.77 / 1.15
//   64          900 of 4096 0.71 / 0.71 / 0.98    1024 1.13 / 0.72 / 1.00           1500 0.72 / 0.45 / 0.68   2040 1.03 / 0.73 / 1.01
// Layers with variants in turn or at random, other : tiles: 32 experts, 1733 tokens of 2816 141 : 123, 3184 of 3584 309 : 288, 808 of 3328 453 : 448;
// 16, 4275 of 3840 134 : 124, 1425 of 2304 405 : 399, 1825 of 3840 502 : 504; 64, 982 of 2560 170 : 159.
// (Left over, variants one after the other: the last figures of the table; 48 experts, 900 of 8192 1.07; 65, 6144 of 4096 1.13.)
//
// Short rows: few chunks to a sum and its butterfly, so wavefronts with fewer experts than they have room for cost more than
// the tokens' shared rows save.  12000 tokens of 512, four variants: 9 experts 1.13, 16 1.02, 17 1.21, 32 0.96, 48 0.84; of 768 0.99,
// 0.88, 1.05, 0.78, 0.68; of 256, 64 experts 3000 tokens 1.05, 5000 0.92.  And a second pass over the experts that has few of them:
// 33 experts, 2048 tokens of 2048 1.22 / 0.89 / 1.18, 5000 0.87 / 0.89 / 1.11, 8000 1.00 / 0.76 / 1.00.
// With several variants, layers: 64 experts, 3319 tokens of 768 78 : 67, 2085 184 : 176, 2116 of 512 304 : 300.
constexpr int64_t kTileScores = 45 << 20;  // elements multiplied
constexpr int kTileVariants = 8;
bool route_in_tiles(const mmoe_shape& s)
{
    if (s.dtype != MMOE_BF16 || s.E < 7 || s.V > kTileVariants || (int64_t)s.T * s.d_model * s.E < kTileScores) return false;
    const bool groups = route_in_groups(s), short_rows = s.d_model < 1024 && s.T >= kRouteTokMinT, mixed = s.V > 1;
    if (s.E <= 8) return s.T >= (groups || s.d_model >= 2304 ? 2304 : 4096);
    if (s.T < 640) return false;
    const int past = s.T % kGroupRound;  // tokens of the groups' last round, 0 if it is full
    if (s.E >= 48) {
        if (groups && !mixed && s.T <= 3 * kGroupRound) return past != 0 && past <= kGroupRound * 15 / 16;
        return !short_rows || (mixed && s.d_model > 256) || (s.T >= 3584 && (s.d_model > 256 || s.E >= 64));
    }
    if ((s.d_model <= 1024 && s.V > 4) || (s.E < 12 && s.d_model > 4096)) return false;
    if (groups && mixed && s.E >= 16 && s.E <= 32) return s.E >= 24 || s.d_model < 3584 || s.T > 2 * kGroupRound;
    if (groups && s.T <= 2 * kGroupRound) return s.E >= 24 && s.T > kGroupRound && past != 0 && past <= kGroupRound * 3 / 8;
    if (groups && s.T < 6 * kGroupRound && s.d_model >= 3584) return false;
    if (s.E > 32 && s.T > 2 * kGroupRound * 15 / 16) return s.T >= 8192 && s.d_model >= 1024;
    return !short_rows || (s.d_model == 768 && s.E % 16 == 0);
}

enum RouteKernel { kRoutePerToken, kRouteTokens, kRouteGroups, kRouteTiles };
int route_kernel_for(const mmoe_shape& s)
{
    if (route_in_tiles(s)) return kRouteTiles;
    if (route_in_groups(s)) return kRouteGroups;
    return wavefront_per_token(s) ? kRouteTokens : kRoutePerToken;
}

int launch_route(const mmoe_shape& s, const void* X, const int32_t* vid, const void* Wr, const float* br,
                 int32_t* topk_idx, float* topk_w, hipStream_t st, const int32_t* M, int32_t* slot)
{
    const int which = route_kernel_for(s);
    if (which == kRouteTiles) {
        // (with one workgroup of eight wavefronts to a group the few tokens of small batches occupy more of the chip)
        if (s.E <= 8) launch_tiles<8, 4, true>(s, X, vid, Wr, br, topk_idx, topk_w, st, M, slot);
        else if (s.E <= 16) launch_tiles<4, 4, false>(s, X, vid, Wr, br, topk_idx, topk_w, st, M, slot);
        else if (s.E <= 32) launch_tiles<4, 8, false>(s, X, vid, Wr, br, topk_idx, topk_w, st, M, slot);
        else if (s.T < kRouteTokMinT) launch_tiles<8, 8, false>(s, X, vid, Wr, br, topk_idx, topk_w, st, M, slot);
        else launch_tiles<8, 4, false>(s, X, vid, Wr, br, topk_idx, topk_w, st, M, slot);
        return launch_status();
    }
    // Large batches of a common hidden size: a wavefront per token (the token row is read
    // once); with more to score, a workgroup per four tokens; otherwise a workgroup per token (lower
    // latency, any d).
    const int nc = s.d_model / 256;
    if (which == kRouteTokens) {
        dim3 grid((s.T + kRouteTokWaves - 1) / kRouteTokWaves), block(kRouteTokWaves * kWave);
#define MMOE_ROUTE_TOK(NC)                                                                                          \
    case NC:                                                                                                        \
        if (s.dtype == MMOE_BF16)                                                                                   \
            hipLaunchKernelGGL((route_token_kernel<uint16_t, NC>), grid, block, 0, st, (const uint16_t*)X, vid,     \
                               (const uint16_t*)Wr, br, topk_idx, topk_w, s.T, s.d_model, s.V, s.E, s.top_k, M, slot, s.S, s.gate);       \
        else                                                                                                        \
            hipLaunchKernelGGL((route_token_kernel<float, NC>), grid, block, 0, st, (const float*)X, vid,           \
                               (const float*)Wr, br, topk_idx, topk_w, s.T, s.d_model, s.V, s.E, s.top_k, M, slot, s.S, s.gate);          \
        break
        switch (nc) {
            MMOE_ROUTE_TOK(1);
            MMOE_ROUTE_TOK(2);
            MMOE_ROUTE_TOK(3);
            MMOE_ROUTE_TOK(4);
            MMOE_ROUTE_TOK(6);
            MMOE_ROUTE_TOK(8);
            MMOE_ROUTE_TOK(12);
            default: MMOE_ROUTE_TOK(16);
        }
#undef MMOE_ROUTE_TOK
        return launch_status();
    }
    dim3 grid(s.T), block(kRouteWaves * kWave);
    if (which == kRouteGroups) {
        const size_t group_bytes = (size_t)kRouteGroup * s.d_model * elem_size(s.dtype);
        const dim3 g4((s.T + kRouteGroup - 1) / kRouteGroup);
        const dim3 b16(kRouteGroupWaves * kWave);
        if (s.dtype == MMOE_BF16)
            hipLaunchKernelGGL(route_group_kernel<uint16_t>, g4, b16, group_bytes, st, (const uint16_t*)X, vid,
                               (const uint16_t*)Wr, br, topk_idx, topk_w, s.T, s.d_model, s.V, s.E, s.top_k, M, slot, s.S,
                               s.gate);
        else
            hipLaunchKernelGGL(route_group_kernel<float>, g4, b16, group_bytes, st, (const float*)X, vid,
                               (const float*)Wr, br, topk_idx, topk_w, s.T, s.d_model, s.V, s.E, s.top_k, M, slot, s.S,
                               s.gate);
        return launch_status();
    }
#define MMOE_ROUTE(TT, KU)                                                                                          \
    hipLaunchKernelGGL((route_kernel<TT, KU>), grid, block, 0, st, (const TT*)X, vid, (const TT*)Wr, br, topk_idx,     \
                       topk_w, s.T, s.d_model, s.V, s.E, s.top_k, M, slot, s.S, s.gate)
    // chunks in flight: the whole row where the registers hold it (64 for both rows)
    if (s.dtype == MMOE_BF16) {
        if (nc <= 4) MMOE_ROUTE(uint16_t, 4);
        else if (nc <= 8) MMOE_ROUTE(uint16_t, 8);
        else MMOE_ROUTE(uint16_t, 16);
    } else {
        if (nc <= 4) MMOE_ROUTE(float, 4);
        else MMOE_ROUTE(float, 8);
    }
#undef MMOE_ROUTE
    return launch_status();
}

}  // namespace mmoe
