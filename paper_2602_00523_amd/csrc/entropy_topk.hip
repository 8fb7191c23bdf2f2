// sage_entropy_topk: softmax statistics, top-k and confidence over vocabulary-sized logits
// (Sec. 3.1: Eq. 7 renormalised top-k, Eq. 8 its entropy, Eq. 9 confidence; Eq. 1 softmax) and, with k = 1,
// the target's greedy token per tree node (Sec. 2.2 / Def. 4.1).
//
// Every logit is read exactly once with 16-byte loads.  Candidates are ordered by a 64-bit composite key (value
// descending, index ascending).  Pass 1 cuts a row into slices of UNIT logits, which a WAVE owns up to k = 48: with k = 1 it takes
// the maximum (DPP row rotations and the 16/32-lane swaps, no LDS, no workgroup barrier), with more it finds what its k best
// logits reach and ranks by counting what reaches that; longer lists are found by a workgroup per slice.  Either reduces the
// slice's softmax statistics
//   Z = sum exp(x - m),  T = sum exp(x - m) (m - x)   so that   H = ln Z + T / Z   (both terms >= 0).
// Pass 2 combines the slice statistics by log-sum-exp, finds the k winners of the sorted per-slice lists (k = 1: a wave per
// row; k > 1: a workgroup per row, merge_row in topk_device.h) and evaluates Eq. 7-9 on them.
#include "sage_internal.h"
#include "topk_common.h"
#include "topk_device.h"

using namespace sage::topk;

namespace {

constexpr int THREADS = 256;
constexpr int EPT = 16;                  // logits per lane
// The greedy first pass over rows that are more than this, live or not, reads them with loads that leave nothing in the memory-side cache (256 MB):
// nobody reads the logits again.  Whole call, 152064 logits, us, plain / so: 512 live rows in groups of 64 38.6 / 36.5 (with the 156 MB
// written just before, copy included, 92.6 / 86.9), 512 rows 33.0 / 31.8 (86.7 / 80.1), fp32 58.9 / 54.3, fp32 30 rows in each of eight groups 29.9 / 27.8, 1024
// rows 60.3 / 59.6.  What has stayed in that cache from a call before is read faster from there: 384 rows (117 MB), three buffers in turn, 24.5 /
// 25.0; past the line, of groups mostly dead: 30 live in each of eight, two buffers in turn, 19.4 / 20.1, 12 live 11.15 / 11.2, fp32 14.1 / 14.5.  (To
// decide by the live rows of a group, in the kernel, cost 12 live rows 0.4 us.)
constexpr long READ_ONCE_BYTES = 128L << 20;
constexpr int UNIT = 64 * EPT;           // logits per wave
constexpr int WAVES = THREADS / 64;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <typename Raw>
__device__ __forceinline__ Raw load_once(const void* p) { return __builtin_bit_cast(Raw, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p))); }
template <typename T> struct Loader;
template <> struct Loader<float> {
    static constexpr int VEC = 4;   // elements per 16-byte load
    using Raw = float4;
    template <bool ONCE>
    __device__ static Raw fetch(const float* p) {
        if constexpr (ONCE) return load_once<Raw>(p);
        else return *reinterpret_cast<const Raw*>(p);
    }
    __device__ static void unpack(Raw v, float* out) { out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w; }
    __device__ static float one(const float* p) { return *p; }
};
template <> struct Loader<uint16_t> {
    static constexpr int VEC = 8;
    using Raw = uint4;
    template <bool ONCE>
    __device__ static Raw fetch(const uint16_t* p) {
        if constexpr (ONCE) return load_once<Raw>(p);
        else return *reinterpret_cast<const Raw*>(p);
    }
    __device__ static void unpack(Raw v, float* out) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    __device__ static float one(const uint16_t* p) { return sage::bf16_bits_to_float(*p); }
};

// Pass 1 for k = 1 (many rows, one candidate per slice): one wave per (slice, row), 16 logits per lane.  With many rows the stream
// bounds it (512 rows, all valid: 156 MB in 30.4 us, 5.1 TB/s, where a copy reaches 5.15; in full groups, three rows a workgroup one after
// the other, 35.7), and what a wave executes takes nearly as long, so that is kept short: the maximum by three-operand maxima, its place by ballots once it is known (a compare and two selects per logit before),
// both sums through one chain of lane exchanges, and no look at the row's end in whole slices.  Whole call, 152064 bf16 logits, groups of
// 64: 512 live rows 39.1 -> 37.9 us on one machine, 38.5 -> 38.4 on another, 256 of 256 23.5 -> 22.9, 192 of 1024 16.5 -> 16.0, up to 64
// rows the same.  The statistics are an exp2 and five operations per logit.  Differences to the maximum are capped at 87, where
// exp is below 2^-125: a -inf logit or a padding slot then adds about 1e-38 instead of 0 to sums that are >= 1.
//
// The 16-byte loads of a (row, slice) are requested by request_unit and consumed by reduce_unit, so that a wave that
// walks several rows can have the next row's loads in flight while it reduces the current one.
template <typename T, int NV, bool ONCE = false>
__device__ __forceinline__ void request_unit(const T* __restrict__ rowp, int base, int lane, int vocab,
                                             typename Loader<T>::Raw (&raw)[NV]) {
    using L = Loader<T>;
    if (base + UNIT <= vocab) {                          // a whole slice (wave-uniform)
#pragma unroll
        for (int j = 0; j < NV; ++j) raw[j] = L::template fetch<ONCE>(rowp + base + (j * 64 + lane) * L::VEC);
        return;
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int e0 = base + (j * 64 + lane) * L::VEC;
        if (e0 + L::VEC <= vocab) raw[j] = L::template fetch<ONCE>(rowp + e0);      // the ragged end is read element by element later
    }
}
// The largest of three numbers, a NaN if one of them is none, so that one compare a slice says whether its maximum is to be taken again
// without them.  (v_max3_f32 passes over quiet NaNs, but a signalling one takes the larger numbers before it along.  To make all logits
// canonical first costs 2-3 % of the pass, 512 rows as above 38.4 -> 39.5 us, 96 of 512 11.0 -> 11.3; this nothing.)
__device__ __forceinline__ float maximum3(float a, float b, float c) {
    float r;
    asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// Sums of two values over the wave, in every lane: the two share a wave from the first exchange on.
__device__ __forceinline__ void wave_sums(float& a, float& b) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);   // a in lanes 0 to 31, b in the others
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    v += sage::f_dpp<0x128>(v); v += sage::f_dpp<0x124>(v); v += sage::f_dpp<0x122>(v); v += sage::f_dpp<0x121>(v);
    a = sage::lane_value(v, 0);
    b = sage::lane_value(v, 32);
}
// The 16 logits of a lane, -inf past the row's end.
template <typename T, int NV>
__device__ __forceinline__ void unpack_unit(const T* __restrict__ rowp, int base, int lane, int vocab,
                                            const typename Loader<T>::Raw (&raw)[NV], float (&v)[EPT]) {
    using L = Loader<T>;
    constexpr int VEC = L::VEC;
    if (base + UNIT <= vocab) {                          // a whole slice (wave-uniform)
#pragma unroll
        for (int j = 0; j < NV; ++j) L::unpack(raw[j], v + j * VEC);
    } else {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int e0 = base + (j * 64 + lane) * VEC;
            if (e0 + VEC <= vocab) {
                L::unpack(raw[j], v + j * VEC);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) v[j * VEC + e] = -INFINITY;
                if (e0 < vocab) {                        // (one lane of the row; where there is none, no questions)
#pragma unroll
                    for (int e = 0; e + 1 < VEC; ++e)
                        if (e0 + e < vocab) v[j * VEC + e] = L::one(rowp + e0 + e);
                }
            }
        }
    }
}
// Softmax statistics of the slice relative to its maximum: a lane's share of the sums.  (EXACT: a -inf logit adds exactly 0, not 1e-38.)
template <bool EXACT>
__device__ __forceinline__ void unit_sums(const float (&v)[EPT], float unit_max, float& Z, float& Tm) {
    Z = 0.f;
    Tm = 0.f;
    if (unit_max > -INFINITY) {
#pragma unroll
        for (int s = 0; s < EPT; ++s) {
            const float dlt = EXACT ? unit_max - v[s] : fminf(unit_max - v[s], 87.0f);
            const float e = __builtin_amdgcn_exp2f(dlt * -1.4426950408889634f);
            Z += e;
            Tm = fmaf(e, EXACT && !(e > 0.f) ? 0.f : dlt, Tm);
        }
    }
}
// (returned in every lane, and stored)
struct Reduced { UnitStats stats; uint64_t key; };
template <typename T, int NV>
__device__ __forceinline__ Reduced reduce_unit(const T* __restrict__ rowp, int base, int lane, int vocab,
                                               const typename Loader<T>::Raw (&raw)[NV], UnitStats* __restrict__ stat_out,
                                               uint64_t* __restrict__ key_out) {
    constexpr int VEC = Loader<T>::VEC;
    float v[EPT];
    unpack_unit<T, NV>(rowp, base, lane, vocab, raw, v);

    // ---- the slice's best candidate: the largest value, at its lowest index.  Indices ascend by load, lane and element: the first load
    // that has the value, its first lane, that lane's first element.
    float most[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        most[j] = v[j * VEC];
#pragma unroll
        for (int e = 1; e + 1 < VEC; e += 2) most[j] = maximum3(most[j], v[j * VEC + e], v[j * VEC + e + 1]);
        most[j] = maximum3(most[j], v[j * VEC + VEC - 1], v[j * VEC + VEC - 1]);
    }
    float unit_max = most[0];
#pragma unroll
    for (int j = 1; j < NV; ++j) unit_max = maximum3(unit_max, most[j], most[j]);
    if (__builtin_expect(__any(unit_max != unit_max), 0)) {   // again, passing over what is no number
        unit_max = -INFINITY;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            most[j] = -INFINITY;
#pragma unroll
            for (int e = 0; e < VEC; ++e) most[j] = v[j * VEC + e] > most[j] ? v[j * VEC + e] : most[j];
            unit_max = most[j] > unit_max ? most[j] : unit_max;
        }
    }
    unit_max = wave_max(unit_max) + 0.f;                 // (-0 is +0, as in the key)
    float Z, Tm;
    unit_sums<false>(v, unit_max, Z, Tm);
    int at = base;                                       // (a slice without a number: a token of the row all the same)
    bool found = false;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        if (found) continue;                             // (wave-uniform)
        const uint64_t holders = __ballot(most[j] == unit_max);
        if (holders == 0) continue;
        found = true;
        const int holder = __builtin_ctzll(holders);
        int element = VEC - 1;
#pragma unroll
        for (int e = VEC - 2; e >= 0; --e)
            if ((__ballot(v[j * VEC + e] == unit_max) >> holder) & 1) element = e;
        at = base + (j * 64 + holder) * VEC + element;
    }
    // (no value is larger than what fills a lane past the end, so that one of those may be the holder only of a value that index `base` has)
    if (at >= vocab) at = base;
    const Key g = make_key(unit_max, at);
    if (lane == 0) *key_out = key_pack(g);
    wave_sums(Z, Tm);
    if (lane == 0) *stat_out = UnitStats{unit_max, Z, Tm, 0.f};
    return Reduced{UnitStats{unit_max, Z, Tm, 0.f}, key_pack(g)};
}

// Every row is valid (n_valid == null): grid (slices / 4, rows).
template <typename T, bool ONCE>
__global__ __launch_bounds__(THREADS) void slice_kernel(const T* __restrict__ logits, int vocab, long row_stride, int nunits,
                                                        UnitStats* __restrict__ stats, uint64_t* __restrict__ keys) {
    constexpr int NV = EPT / Loader<T>::VEC;
    const int row = blockIdx.y;
    const int unit = blockIdx.x * WAVES + (threadIdx.x >> 6);
    if (unit >= nunits) return;
    const int lane = threadIdx.x & 63;
    const T* rowp = logits + static_cast<long>(row) * row_stride;
    typename Loader<T>::Raw raw[NV];
    request_unit<T, NV, ONCE>(rowp, unit * UNIT, lane, vocab, raw);
    const long o = static_cast<long>(row) * nunits + unit;
    reduce_unit<T, NV>(rowp, unit * UNIT, lane, vocab, raw, stats + o, keys + o);
}

// Rows in groups of which only the first n_valid[group] count (the target rows of a tree): grid (slices / 4, phases,
// groups).  A workgroup walks the live rows phase, phase + phases, ... of its group, the next row's loads in flight
// while the current one is reduced, so rows past n_valid cost no workgroup of their own.
// Phases: with one or two groups every live row may have its workgroups at once (64 live rows of 152064 in one group, first
// pass 8.4 -> 6.6 us, 40 in each of two 8.9 -> 7.9; 12 rows 3.1 either way).  With more groups 16 of them fill the chip, and the
// workgroups of dead rows that more would add show (8 x 12 rows 8.5 us at 16, 9.1 at 32, 9.7 at 64).
// By themselves the slice passes of more groups take 22, so that a workgroup walks one or two rows of a group of 20 to 40 and three of a
// full one.  Calls, us, at 16 -> 22: 20 rows in each of eight 15.1 -> 14.0, 30 in each of five 15.5 -> 14.9, 40 in each of eight 25.3 ->
// 24.0, 64 in each of three 20.0 -> 19.2, of four and of eight the same; 12 in each of three, eight, twelve and sixteen the same within 0.1,
// in each of five 8.8 -> 9.1.  Beside a draft row's, in a step, whose trees are seldom full, 16: 12 rows in each of three 5.65 us (22: 5.9),
// of eight 10.6 (10.8), of twelve 14.7 (14.9), 15 in each of eight 11.8 (12.0), though full groups would be faster with 22 (three 17.2
// and 16.3, four 20.6 and 19.8, eight 36.1 and 35.6).
inline int row_phases(int groups, int rows_per_group, bool in_a_step) {
    const int phases = groups == 1 ? 64 : groups == 2 ? 32 : in_a_step ? 16 : 22;
    return rows_per_group < phases ? rows_per_group : phases;
}
template <typename T, bool ONCE>
__device__ __forceinline__ void slice_rows_block(const T* __restrict__ logits, int vocab, long row_stride,
                                                 const int* __restrict__ n_valid, int rows_per_group, int rows, int nunits,
                                                 UnitStats* __restrict__ stats, uint64_t* __restrict__ keys, int block_x,
                                                 int phase, int phases, int group) {
    constexpr int NV = EPT / Loader<T>::VEC;
    const int unit = block_x * WAVES + (threadIdx.x >> 6);
    const int n = min(n_valid[group], min(rows_per_group, rows - group * rows_per_group));   // the last group may be short
    int r = phase;
    if (unit >= nunits || r >= n) return;
    const int lane = threadIdx.x & 63;
    const int base = unit * UNIT;
    const long row0 = static_cast<long>(group) * rows_per_group;
    typename Loader<T>::Raw cur[NV], nxt[NV];
    request_unit<T, NV, ONCE>(logits + (row0 + r) * row_stride, base, lane, vocab, cur);
    while (true) {
        const int rn = r + phases;
        const bool more = rn < n;                            // wave-uniform
        if (more) request_unit<T, NV, ONCE>(logits + (row0 + rn) * row_stride, base, lane, vocab, nxt);
        const long o = (row0 + r) * nunits + unit;
        reduce_unit<T, NV>(logits + (row0 + r) * row_stride, base, lane, vocab, cur, stats + o, keys + o);
        if (!more) break;
        for (int j = 0; j < NV; ++j) cur[j] = nxt[j];
        r = rn;
    }
}
template <typename T, bool ONCE>
__global__ __launch_bounds__(THREADS) void slice_rows_kernel(const T* __restrict__ logits, int vocab, long row_stride,
                                                             const int* __restrict__ n_valid, int rows_per_group, int rows,
                                                             int nunits, UnitStats* __restrict__ stats,
                                                             uint64_t* __restrict__ keys) {
    slice_rows_block<T, ONCE>(logits, vocab, row_stride, n_valid, rows_per_group, rows, nunits, stats, keys, blockIdx.x, blockIdx.y,
                        gridDim.y, blockIdx.z);
}

// Pass 1 for 1 < k <= WAVE_MAX_K (draft rows): a wave per slice, 16 logits per lane, as with k = 1.  The k best of the slice reach what k of the
// lanes' largest logits reach, and few others do: that threshold is found bit by bit, a ballot a bit, from the first bit in which those 64
// differ; what reaches it goes to LDS, a logit of every lane at a time, and a lane per entry counts the entries above its own, which is its place.
// Where that does not hold (more logits reach the threshold than the list has room for, fewer than k lanes have a logit above -inf, or some are
// no numbers) the threshold is settled among all 1024 codes, and of those that equal it the first are taken.
// What bounds it is what is executed: 149 slices of a row are 149 waves on 1024 SIMDs, so that with few rows the chain counts and with many the
// instructions.  Against a workgroup per slice (four waves that each selected k of 256 logits, by k rounds of a maximum for bf16 and k <= 16, by
// ballots over all values otherwise, and a fifth selection among theirs), whole call, 152064 logits: fp32 k = 10, one row 8.95 -> 8.15 us,
// eight 12.0 -> 8.9, a hundred 46 -> 18.5; bf16 k = 10, one row 8.45 -> 8.1, eight 10.9 -> 8.9, forty 21.6 -> 11.6, three hundred 103 -> 35; k = 16, twelve rows 14.4
// -> 9.8; k = 40, eight rows 18.7 -> 14.5.  Beside the rows of trees of 12 nodes, in a step: one sequence 4.7 -> 4.5, three 5.9 -> 5.6, eight 10.9 -> 9.4.
// Of the odd ones, eight rows: all logits equal 15.3 -> 15.7 (fp32 19.5 -> 15.7), bf16 in steps of one 13.5 -> 14.2, all but 1000 logits -inf 11.6 -> 12.3 (fp32
// 15.7 -> 13.2), rising bf16 logits 13.3 -> 16.1 (fp32 15.9 -> 12.9).
// MOST_LANES: with k near 64 a threshold that nearly all lanes reach lets too many logits through (k = 40, eight fp32 rows: 14.4 us with 44 lanes at
// most, 15.3 with 52).  Beyond k = 48 a workgroup per slice is the faster one (one row, k = 56, 15.1 us and 18.0; k = 48, 14.7 and 14.4).
constexpr int WAVE_MAX_K = 48;
constexpr int WAVE_LIST = 128;
constexpr int MOST_LANES = 44;
struct SliceTop { UnitStats stats; uint64_t key[2]; int place[2]; };   // a lane's entries and their places in the slice's list (none: WAVE_LIST)
template <typename T, int NV>
__device__ __forceinline__ SliceTop slice_topk_wave(const T* __restrict__ rowp, int base, int lane, int vocab, int k,
                                                    const typename Loader<T>::Raw (&raw)[NV], uint64_t* list) {
    constexpr int VEC = Loader<T>::VEC;
    // the codes of different bf16 values differ in their upper halves
    constexpr uint32_t LAST_BIT = sizeof(T) == 4 ? 1u : 0x10000u, REST = LAST_BIT - 1;
    float v[EPT];
    unpack_unit<T, NV>(rowp, base, lane, vocab, raw, v);
    auto index = [&](int i) __attribute__((always_inline)) { return base + ((i / VEC) * 64 + lane) * VEC + i % VEC; };
    const int present = vocab - base, want = min(k, present);
    float top = v[0];                                    // (a NaN if the lane has one, see maximum3)
#pragma unroll
    for (int i = 1; i + 1 < EPT; i += 2) top = maximum3(top, v[i], v[i + 1]);
    top = maximum3(top, v[EPT - 1], v[EPT - 1]);
    const uint32_t code = sortable(top);
    uint32_t hi = __builtin_amdgcn_readfirstlane(wave_max_u32(code));
    const uint32_t lo = __builtin_amdgcn_readfirstlane(~wave_max_u32(~code));
    uint32_t bit = hi == lo ? 0u : 0x80000000u >> __builtin_clz(hi ^ lo);
    uint32_t thr = bit ? hi & ~(2u * bit - 1u) : hi;     // what all lanes have in common (2 bit wraps to 0: nothing)
    int got = 64;
    auto search = [&](int most) __attribute__((always_inline)) {       // until at most that many lanes reach it, or it is a lane's value
        while ((bit >= LAST_BIT) & (got > most)) {
            const int n = __builtin_popcountll(__ballot(code >= (thr | bit)));
            thr = n >= want ? thr | bit : thr;
            got = n >= want ? n : got;
            bit >>= 1;
        }
    };
    bool tail = present <= WAVE_LIST && present <= VEC * (want - 1);   // a last slice that fits the list whole, with logits in too few lanes
    if (!tail) search(min(want + want / 2 + 2, max(want, MOST_LANES)));
    const float floor = unsortable(thr);
    const bool nan = __any(top != top);
    const bool clear = !tail && !nan && floor > -INFINITY;   // (a number then: thr lies between two lanes' codes, or is what they share)
    tail = !clear && present <= WAVE_LIST;
    const bool usual = clear || tail;
    uint32_t mine = 0;                                   // which of its logits the lane has yet to put on the list
#pragma unroll
    for (int i = EPT - 1; i >= 0; --i) mine = mine + mine + (v[i] >= floor ? 1u : 0u);
    if (tail) {
        mine = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) mine |= ((1u << min(max(present - (j * 64 + lane) * VEC, 0), VEC)) - 1u) << (j * VEC);
    }
    int n = 0;
    uint64_t b = usual ? __ballot(mine != 0) : 0;
    while (b != 0) {                                     // one by every lane at a time, seldom more than two
        const int i = __builtin_ctz(mine | 0x10000u);
        float x[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) x[e] = v[e];
#pragma unroll
        for (int w = 1; w < EPT; w *= 2) {
            const bool upper = (i & w) != 0;
#pragma unroll
            for (int e = 0; e < EPT; e += 2 * w) {
                const float a = x[e], b = x[e + w];      // (of two array elements the compiler would choose the address)
                x[e] = upper ? b : a;
            }
        }
        const int to = n + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
        const int at = base + ((i / VEC) * 64 + lane) * VEC + i % VEC;
        if (mine != 0 && to < WAVE_LIST) list[to] = key_pack(make_key(x[0], at));
        mine &= mine - 1;
        n += __builtin_popcountll(b);
        b = n <= WAVE_LIST ? __ballot(mine != 0) : 0;
    }
    if (__builtin_expect(!usual || n > WAVE_LIST, 0)) {
        uint32_t all[EPT];
        bool have[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            have[i] = index(i) < vocab;
            all[i] = sortable(v[i]);
        }
        search(want);
        auto count = [&](uint32_t t) __attribute__((always_inline)) {  // how many reach t
            int a = 0;
#pragma unroll
            for (int i = 0; i < EPT; ++i) a += __builtin_popcountll(__ballot(have[i] && all[i] >= t));
            return a;
        };
        auto above = [&]() __attribute__((always_inline)) { return (thr | REST) == 0xFFFFFFFFu ? 0 : count((thr | REST) + 1u); };
        int more = above();
        if (nan || more > WAVE_LIST) {                   // the threshold of all values, which is above that of the lanes'
            hi = 0;
#pragma unroll
            for (int i = 0; i < EPT; ++i) hi = max(hi, have[i] ? all[i] : 0u);
            hi = __builtin_amdgcn_readfirstlane(wave_max_u32(hi));
            const uint32_t low = nan ? 0u : thr;
            bit = hi == low ? 0u : 0x80000000u >> __builtin_clz(hi ^ low);
            thr = bit ? hi & ~(2u * bit - 1u) : hi;
            for (got = EPT * 64; (bit >= LAST_BIT) & (got > WAVE_LIST); bit >>= 1) {
                const int reach = count(thr | bit);
                thr = reach >= want ? thr | bit : thr;
                got = reach >= want ? reach : got;
            }
            more = got > WAVE_LIST ? above() : got;      // (what reaches it fits the list: nothing is left to choose)
            thr = got > WAVE_LIST ? thr : thr - 1;
        }
        int left = max(want - more, 0);                  // so many of those that equal it, by index: by load, lane, element
        n = 0;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            int own = 0, before = 0, all_of = 0;
#pragma unroll
            for (int e = 0; e < VEC; ++e) own += have[j * VEC + e] && (all[j * VEC + e] | REST) == (thr | REST) ? 1 : 0;
#pragma unroll
            for (int w = 1; w <= VEC; w *= 2) {          // (own is at most VEC)
                const uint64_t b = __ballot((own & w) != 0);
                before += w * static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
                all_of += w * __builtin_popcountll(b);
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const int i = j * VEC + e;
                const bool equal = have[i] && (all[i] | REST) == (thr | REST);
                const bool in = have[i] && (all[i] > (thr | REST) || (equal && before < left));
                const uint64_t b = __ballot(in);
                if (b != 0) {
                    const int to = n + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
                    if (in) list[to] = key_pack(Key{all[i], 0xFFFFFFFFu - static_cast<uint32_t>(index(i))});
                    n += __builtin_popcountll(b);
                }
                before += equal ? 1 : 0;
            }
            left -= all_of;
        }
#pragma unroll
        for (int i = 0; i < EPT; ++i) v[i] = have[i] ? unsortable(all[i]) : -INFINITY;   // (so that only one of the two is kept meanwhile)
    }
    if (lane < (-n & 15)) list[n + lane] = 0;
    const float unit_max = unsortable(hi);
    float Z, Tm;
    unit_sums<true>(v, unit_max, Z, Tm);
    wave_sums(Z, Tm);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    SliceTop out;
    out.stats = UnitStats{unit_max, Z, Tm, 0.f};
    const int padded = (n + 15) & ~15;
    out.key[0] = lane < n ? list[lane] : 0;
    out.place[0] = count_above(list, padded, out.key[0]);
    out.place[0] = lane < n ? out.place[0] : WAVE_LIST;
    out.key[1] = 0;
    out.place[1] = WAVE_LIST;
    if (n > 64) {                                        // (uniform)
        out.key[1] = 64 + lane < n ? list[64 + lane] : 0;
        const int above = count_above(list, padded, out.key[1]);
        out.place[1] = 64 + lane < n ? above : WAVE_LIST;
    }
    return out;
}
// One (slice, row) by every wave of a workgroup: the four slices from 4 block_x on.
template <typename T>
__device__ __forceinline__ void slice_topk_wave_block(const T* __restrict__ logits, int vocab, long row_stride, int k,
                                                      const int* __restrict__ n_valid, int rows_per_group, int nunits,
                                                      UnitStats* __restrict__ stats, uint64_t* __restrict__ keys, int block_x, int row) {
    constexpr int NV = EPT / Loader<T>::VEC;
    __shared__ __align__(16) uint64_t s_list[WAVES][WAVE_LIST];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int unit = block_x * WAVES + wave;
    if (unit >= nunits || !row_is_valid(row, n_valid, rows_per_group)) return;
    const int lane = threadIdx.x & 63;
    const T* rowp = logits + static_cast<long>(row) * row_stride;
    typename Loader<T>::Raw raw[NV];
    request_unit<T, NV>(rowp, unit * UNIT, lane, vocab, raw);
    const SliceTop r = slice_topk_wave<T, NV>(rowp, unit * UNIT, lane, vocab, k, raw, s_list[wave]);
    const long o = static_cast<long>(row) * nunits + unit;
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (r.place[e] < k) keys[o * k + r.place[e]] = r.key[e];
    if (lane < k && lane >= vocab - unit * UNIT) keys[o * k + lane] = 0;   // a short last slice has no more candidates than logits
    if (lane == 0) stats[o] = r.stats;
}
template <typename T>
__global__ __launch_bounds__(THREADS) void slice_topk_wave_kernel(const T* __restrict__ logits, int vocab, long row_stride, int k,
                                                                  const int* __restrict__ n_valid, int rows_per_group, int nunits,
                                                                  UnitStats* __restrict__ stats, uint64_t* __restrict__ keys) {
    slice_topk_wave_block<T>(logits, vocab, row_stride, k, n_valid, rows_per_group, nunits, stats, keys, blockIdx.x, blockIdx.y);
}

// Pass 1 for longer lists: one WORKGROUP per slice, 4 logits per lane.  Each wave finds the value that exactly k of its 256 logits reach,
// bit by bit from the top, each bit one ballot per logit (about 20 of the 32 bits on Gaussian logits).  Equal
// values at the threshold are admitted lowest index first.  The survivors of the four waves, in any order, are then ranked
// by counting.  (Selecting by k rounds of a wave-wide maximum of 64-bit keys took one row 36 us at k = 64.)
template <typename T>
__device__ __forceinline__ void slice_topk_block(const T* __restrict__ logits, int vocab, long row_stride, int k,
                                                 const int* __restrict__ n_valid, int rows_per_group, int nunits,
                                                 UnitStats* __restrict__ stats, uint64_t* __restrict__ keys, int unit, int row) {
    __shared__ __align__(16) uint64_t s_list[WAVES * SAGE_MAX_TOPK];
    __shared__ float s_red[3][WAVES];
    if (!row_is_valid(row, n_valid, rows_per_group)) return;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const T* rowp = logits + static_cast<long>(row) * row_stride;
    const int e0 = unit * UNIT + threadIdx.x * 4;

    float v[4];
    if (e0 + 4 <= vocab) {
        if constexpr (sizeof(T) == 4) {
            const float4 q = *reinterpret_cast<const float4*>(rowp + e0);
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else {
            const uint2 q = *reinterpret_cast<const uint2*>(rowp + e0);
            v[0] = __uint_as_float(q.x << 16); v[1] = __uint_as_float(q.x & 0xFFFF0000u);
            v[2] = __uint_as_float(q.y << 16); v[3] = __uint_as_float(q.y & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (e0 + e < vocab) ? Loader<T>::one(rowp + e0 + e) : -INFINITY;
    }
    // What the search runs on: the value's code, which for bf16 leaves 16 bits for the (inverted) position in the slice, so
    // that equal values differ.  0 = no candidate.
    uint32_t code[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        // (NaNs of the extreme codes move by one: 0 marks no candidate, and the rounds below start under 0xFFFFFFFF)
        const uint32_t full = min(max(sortable(v[e]), 1u), 0xFFFFFFFEu);
        code[e] = e0 + e >= vocab ? 0u : sizeof(T) == 4 ? full : ((full & 0xFFFF0000u) | static_cast<uint32_t>(UNIT - (static_cast<int>(threadIdx.x) * 4 + e)));
    }
    auto reach = [&](uint32_t t) __attribute__((always_inline)) {     // how many of the wave's logits reach t (uniform)
        return __builtin_popcountll(__ballot(code[0] >= t)) + __builtin_popcountll(__ballot(code[1] >= t)) +
               __builtin_popcountll(__ballot(code[2] >= t)) + __builtin_popcountll(__ballot(code[3] >= t));
    };
    const int present = reach(1u);
    const int want = min(k, present);
    uint32_t thr = 1u;
    int got = present;
    if (got > want) {                                // the threshold bit by bit (about 170 cycles each, 20 of them)
        thr = 0u;
        for (uint32_t bit = 0x80000000u; bit != 0; bit >>= 1) {
            const int n = reach(thr | bit);
            if (n >= want) {
                thr |= bit;
                got = n;
                if (n == want) break;
            }
        }
    }
    bool in[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) in[e] = code[e] >= thr;
    auto below_me = [&](const bool (&f)[4]) __attribute__((always_inline)) {   // flags set in lower lanes
        int n = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t b = __ballot(f[e]);
            n += static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
        }
        return n;
    };
    if (got > want) {                                // (uniform) several logits equal the threshold: the lowest indices of them
        bool eq[4];
        int above = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            eq[e] = code[e] == thr;
            above += __builtin_popcountll(__ballot(code[e] > thr));
        }
        int nth = below_me(eq);                      // indices ascend with the lane, then with e
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            in[e] = code[e] > thr || (eq[e] && nth < want - above);
            nth += eq[e] ? 1 : 0;
        }
    }
    int at = below_me(in);
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (in[e]) s_list[wave * k + at++] = key_pack(make_key(v[e], e0 + e));
    if (lane >= want && lane < k) s_list[wave * k + lane] = 0;
    if (wave == WAVES - 1 && WAVES * k + lane < ((WAVES * k + 15) & ~15)) s_list[WAVES * k + lane] = 0;
    const uint32_t top = wave_max_u32(max(max(sortable(v[0]), sortable(v[1])), max(sortable(v[2]), sortable(v[3]))));
    // softmax statistics relative to the wave's maximum, combined across the four waves below
    const float wmax = unsortable(top);              // (-inf where the wave has no logit)
    float Z = 0.f, Tm = 0.f;
    if (wmax > -INFINITY) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float dlt = wmax - v[e];
            const float ex = expf(-dlt);
            Z += ex;
            Tm += (ex > 0.f) ? ex * dlt : 0.f;
        }
    }
    Z = wave_sum(Z);
    Tm = wave_sum(Tm);
    if (lane == 0) { s_red[0][wave] = wmax; s_red[1][wave] = Z; s_red[2][wave] = Tm; }
    __syncthreads();
    // ---- a thread per survivor counts the survivors above it: its place in the slice's list
    uint64_t* const kout = keys + (static_cast<long>(row) * nunits + unit) * k;
    const int tid = threadIdx.x;
    if (tid < WAVES * k) {
        const uint64_t mine = s_list[tid];
        const int above = count_above(s_list, (WAVES * k + 15) & ~15, mine);
        if (mine != 0 && above < k) kout[above] = mine;
    }
    if (tid < k && tid >= vocab - unit * UNIT) kout[tid] = 0;    // a short last slice has no more candidates than logits
    if (wave != 0) return;
    if (lane == 0) {
        float m = fmaxf(fmaxf(s_red[0][0], s_red[0][1]), fmaxf(s_red[0][2], s_red[0][3]));
        float z = 0.f, t = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            if (s_red[0][w] > -INFINITY) {
                const float dlt = m - s_red[0][w];
                const float sc = expf(-dlt);
                z += sc * s_red[1][w];
                t += sc * (s_red[2][w] + s_red[1][w] * dlt);
            }
        }
        stats[static_cast<long>(row) * nunits + unit] = UnitStats{m, z, t, 0.f};
    }
}
template <typename T>
__global__ __launch_bounds__(THREADS) void slice_topk_kernel(const T* __restrict__ logits, int vocab, long row_stride, int k,
                                                             const int* __restrict__ n_valid, int rows_per_group, int nunits,
                                                             UnitStats* __restrict__ stats, uint64_t* __restrict__ keys) {
    slice_topk_block<T>(logits, vocab, row_stride, k, n_valid, rows_per_group, nunits, stats, keys, blockIdx.x, blockIdx.y);
}

// Two first passes in one launch (sage_entropy_topk_slices_pair): the k = 1 pass over grouped rows (job A, the grid
// of slice_rows_kernel) with the k > 1 pass over a few rows (job B) in workgroups ahead of it.  A step is a
// chain of dependent launches, each a few microseconds whatever it computes; two passes that do not depend on each
// other share one.  Job B comes first, because its chain is the longer one (behind job A: 0.5 to 1 us more).  BY_WAVES: a wave per slice
// in job B (k <= WAVE_MAX_K).
struct PairJob {
    const void* logits; long row_stride; int rows, k, nunits;
    UnitStats* stats; uint64_t* keys;
};
template <typename T, bool BY_WAVES>
__global__ __launch_bounds__(THREADS) void slice_pair_kernel(const T* __restrict__ logits_a, int vocab, long row_stride_a,
                                                             const int* __restrict__ n_valid_a, int rows_per_group_a,
                                                             int rows_a, int nunits, UnitStats* __restrict__ stats_a,
                                                             uint64_t* __restrict__ keys_a, int slabs_b, const PairJob b) {
    // one group: the rows of job B come ahead of the phases of job A; several: in slabs ahead of theirs
    const int y = blockIdx.y, z = blockIdx.z, ahead = slabs_b == 0 ? b.rows : 0;
    if (z < slabs_b || y < ahead) {                          // workgroup-uniform
        if constexpr (BY_WAVES) {
            const int row = z * static_cast<int>(gridDim.y) + y;
            if (row < b.rows)
                slice_topk_wave_block<T>(static_cast<const T*>(b.logits), vocab, b.row_stride, b.k, nullptr, 1, b.nunits, b.stats, b.keys, blockIdx.x, row);
        } else {
            const int lin = (z * gridDim.y + y) * gridDim.x + blockIdx.x;
            if (lin >= b.nunits * b.rows) return;
            const int row = lin / b.nunits, unit = lin - row * b.nunits;
            slice_topk_block<T>(static_cast<const T*>(b.logits), vocab, b.row_stride, b.k, nullptr, 1, b.nunits, b.stats, b.keys,
                                unit, row);
        }
        return;
    }
    slice_rows_block<T, false>(logits_a, vocab, row_stride_a, n_valid_a, rows_per_group_a, rows_a, nunits, stats_a, keys_a, blockIdx.x,
                        y - ahead, static_cast<int>(gridDim.y) - ahead, z - slabs_b);
}

// Pass 2 for k = 1 (the target rows): a wave per row, no LDS and no barrier.  Statistics and candidates of the row's slices
// are requested together (one memory round trip) and reduced in registers, OWN slices per lane at a time.  units_used (nullable)
// is the number of slices where the device has decided it, at most `nunits`; it is requested together with the row's validity,
// so that it costs no round trip.
template <int OWN>
__global__ __launch_bounds__(MERGE_THREADS) void merge_one_kernel(const int* __restrict__ n_valid, int rows_per_group, int rows, int nunits,
                                                                  const int* __restrict__ units_used,
                                                                  const UnitStats* __restrict__ stats, const uint64_t* __restrict__ keys,
                                                                  float* __restrict__ entropy, int* __restrict__ topk_idx,
                                                                  float* __restrict__ topk_prob, float* __restrict__ topk_renorm,
                                                                  float* __restrict__ topk_entropy, float* __restrict__ alpha) {
    const int row = blockIdx.x * (MERGE_THREADS / 64) + (threadIdx.x >> 6);
    if (row >= rows) return;
    if (units_used) {                                // (with n_valid only)
        int used = *units_used, valid = n_valid[row / rows_per_group];
        asm volatile("" : "+v"(used), "+v"(valid));  // both loads before the branch
        if (row % rows_per_group >= valid) return;
        nunits = min(__builtin_amdgcn_readfirstlane(used), nunits);
    } else if (!row_is_valid(row, n_valid, rows_per_group)) {
        return;
    }
    const int lane = threadIdx.x & 63;
    const UnitStats* st = stats + static_cast<long>(row) * nunits;
    const uint64_t* kk = keys + static_cast<long>(row) * nunits;
    UnitStats u[OWN];
    uint64_t key[OWN];
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        const bool live = lane + 64 * i < nunits;
        u[i] = live ? st[lane + 64 * i] : UnitStats{-INFINITY, 0.f, 0.f, 0.f};
        key[i] = live ? kk[lane + 64 * i] : 0ull;
    }
    float m, Z, Tm;
    combine_unit_stats<OWN>(u, lane, nunits, m, Z, Tm);
    uint64_t best = key[0];
#pragma unroll
    for (int i = 1; i < OWN; ++i) best = max(best, key[i]);
    const Key g = wave_max_key(key_unpack(best));
    if (lane == 0 && entropy) entropy[row] = logf(Z) + Tm / Z;
    MergedRow r;
    finish_row(row, 1, lane, g, m, Z, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, r);
}

// Pass 2 as a launch of its own: one workgroup per row (see merge_row).
template <int OWN>
__global__ __launch_bounds__(MERGE_THREADS) void merge_kernel(int k, const int* __restrict__ n_valid, int rows_per_group, int nunits,
                                                              const UnitStats* __restrict__ stats, const uint64_t* __restrict__ keys,
                                                              float* __restrict__ entropy, int* __restrict__ topk_idx,
                                                              float* __restrict__ topk_prob, float* __restrict__ topk_renorm,
                                                              float* __restrict__ topk_entropy, float* __restrict__ alpha) {
    __shared__ MergeShared<OWN> sh;
    const int row = blockIdx.x;
    if (!row_is_valid(row, n_valid, rows_per_group)) return;
    MergedRow r;
    merge_row<OWN>(row, k, nunits, stats, keys, sh, entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, r);
}

// Both passes in one launch, for vocabularies of a few slices: a second launch costs as much as such a row does (2.5 us on
// the device, 3.5 on the host).  Same device functions, same bits, and the workspace as after the two.
// k = 1: a wave per slice, PER_ROW of them (at least the row's slices) side by side in a workgroup; the first one finishes the
// row.  64 rows of 1024 fp32 logits 5.1 -> 3.2 us, of 4096 4.9 -> 3.3.
constexpr int ONE_LAUNCH_UNITS = WAVES;
template <typename T, int PER_ROW>
__global__ __launch_bounds__(THREADS) void rows_in_one_kernel(const T* __restrict__ logits, int vocab, long row_stride, const int* __restrict__ n_valid,
                                                              int rows_per_group, int rows, int nunits, UnitStats* __restrict__ stats,
                                                              uint64_t* __restrict__ keys, float* __restrict__ entropy, int* __restrict__ topk_idx,
                                                              float* __restrict__ topk_prob, float* __restrict__ topk_renorm,
                                                              float* __restrict__ topk_entropy, float* __restrict__ alpha) {
    constexpr int NV = EPT / Loader<T>::VEC;
    __shared__ Reduced s_unit[WAVES];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = blockIdx.x * (WAVES / PER_ROW) + wave / PER_ROW, unit = wave % PER_ROW;
    const bool live = row < rows && row_is_valid(row, n_valid, rows_per_group);
    const int lane = threadIdx.x & 63;
    Reduced mine = Reduced{UnitStats{-INFINITY, 0.f, 0.f, 0.f}, 0};
    if (live && unit < nunits) {                             // (uniform in a wave)
        const T* rowp = logits + static_cast<long>(row) * row_stride;
        typename Loader<T>::Raw raw[NV];
        request_unit<T, NV>(rowp, unit * UNIT, lane, vocab, raw);
        const long o = static_cast<long>(row) * nunits + unit;
        mine = reduce_unit<T, NV>(rowp, unit * UNIT, lane, vocab, raw, stats + o, keys + o);
    }
    if (PER_ROW > 1) {
        if (lane == 0) s_unit[wave] = mine;
        __syncthreads();
        mine = s_unit[wave + min(lane, PER_ROW - 1 - unit)];   // (of the first wave: lane u gets slice u)
    }
    if (!live || unit != 0) return;
    const UnitStats u[1] = {mine.stats};
    float m, Z, Tm;
    combine_unit_stats<1>(u, lane, nunits, m, Z, Tm);
    const Key g = wave_max_key(key_unpack(lane < nunits ? mine.key : 0));
    if (lane == 0 && entropy) entropy[row] = logf(Z) + Tm / Z;
    MergedRow r;
    finish_row(row, 1, lane, g, m, Z, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, r);
}
// k > 1, one slice: up to WAVE_MAX_K by a wave per row, which finishes the row (fp32, k = 8, 1000 logits: 6.5 -> 4.3 us, k = 33 10.8 -> 4.8;
// the list is the row's, and nothing goes through memory); longer lists by a workgroup per row, which merges the one list (two slices one
// after the other are slower than two launches).
template <typename T>
__global__ __launch_bounds__(THREADS) void row_topk_by_wave_kernel(const T* __restrict__ logits, int vocab, long row_stride, int k,
                                                                   const int* __restrict__ n_valid, int rows_per_group, int rows,
                                                                   UnitStats* __restrict__ stats, uint64_t* __restrict__ keys,
                                                                   float* __restrict__ entropy, int* __restrict__ topk_idx,
                                                                   float* __restrict__ topk_prob, float* __restrict__ topk_renorm,
                                                                   float* __restrict__ topk_entropy, float* __restrict__ alpha) {
    constexpr int NV = EPT / Loader<T>::VEC;
    __shared__ __align__(16) uint64_t s_list[WAVES][WAVE_LIST];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = blockIdx.x * WAVES + wave;
    if (row >= rows || !row_is_valid(row, n_valid, rows_per_group)) return;
    const int lane = threadIdx.x & 63;
    const T* rowp = logits + static_cast<long>(row) * row_stride;
    typename Loader<T>::Raw raw[NV];
    request_unit<T, NV>(rowp, 0, lane, vocab, raw);
    const SliceTop r = slice_topk_wave<T, NV>(rowp, 0, lane, vocab, k, raw, s_list[wave]);
    uint64_t* const kout = keys + static_cast<long>(row) * k;
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (r.place[e] < k) kout[r.place[e]] = r.key[e];
    if (lane == 0) stats[row] = r.stats;
    // the list in order: every lane has read its entry and counted
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (r.place[e] < k) s_list[wave][r.place[e]] = r.key[e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const UnitStats u[1] = {r.stats};
    float m, Z, Tm;
    combine_unit_stats<1>(u, lane, 1, m, Z, Tm);
    if (lane == 0 && entropy) entropy[row] = logf(Z) + Tm / Z;
    MergedRow out;
    finish_row(row, k, lane, lane < k ? key_unpack(s_list[wave][lane]) : Key{0, 0}, m, Z, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, out);
}
template <typename T>
__global__ __launch_bounds__(THREADS) void row_topk_in_one_kernel(const T* __restrict__ logits, int vocab, long row_stride, int k,
                                                                  const int* __restrict__ n_valid, int rows_per_group,
                                                                  UnitStats* __restrict__ stats, uint64_t* __restrict__ keys,
                                                                  float* __restrict__ entropy, int* __restrict__ topk_idx,
                                                                  float* __restrict__ topk_prob, float* __restrict__ topk_renorm,
                                                                  float* __restrict__ topk_entropy, float* __restrict__ alpha) {
    static_assert(THREADS == MERGE_THREADS, "both passes by the same workgroup");
    __shared__ MergeShared<1> sh;
    const int row = blockIdx.x;
    if (!row_is_valid(row, n_valid, rows_per_group)) return;
    slice_topk_block<T>(logits, vocab, row_stride, k, n_valid, rows_per_group, 1, stats, keys, 0, row);
    __syncthreads();                                         // what it stored is there for the workgroup
    MergedRow r;
    merge_row<1>(row, k, 1, stats, keys, sh, entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, r);
}

// The launch of the two kernels above; the caller has checked the arguments.
template <typename T>
void launch_in_one(const T* logits, int rows, int vocab, long row_stride, int k, const int* n_valid, int rows_per_group, int nunits,
                   UnitStats* stats, uint64_t* keys, float* entropy, int* topk_idx, float* topk_prob, float* topk_renorm,
                   float* topk_entropy, float* alpha, hipStream_t s) {
    if (k == 1) {
        const int per_row = nunits <= 2 ? nunits : 4, rows_per_wg = WAVES / per_row;
        const auto kernel = per_row == 1 ? rows_in_one_kernel<T, 1> : per_row == 2 ? rows_in_one_kernel<T, 2> : rows_in_one_kernel<T, 4>;
        hipLaunchKernelGGL(kernel, dim3((rows + rows_per_wg - 1) / rows_per_wg), dim3(THREADS), 0, s, logits, vocab, row_stride, n_valid,
                           rows_per_group, rows, nunits, stats, keys, entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
        return;
    }
    if (k <= WAVE_MAX_K)
        hipLaunchKernelGGL(row_topk_by_wave_kernel<T>, dim3((rows + WAVES - 1) / WAVES), dim3(THREADS), 0, s, logits, vocab, row_stride, k, n_valid,
                           rows_per_group, rows, stats, keys, entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
    else
        hipLaunchKernelGGL(row_topk_in_one_kernel<T>, dim3(rows), dim3(THREADS), 0, s, logits, vocab, row_stride, k, n_valid, rows_per_group, stats,
                           keys, entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
}

inline int num_units(int vocab) { return (vocab + UNIT - 1) / UNIT; }
inline size_t stats_bytes(int rows, int vocab) {
    size_t b = static_cast<size_t>(rows) * num_units(vocab) * sizeof(UnitStats);
    return (b + 255) & ~static_cast<size_t>(255);
}

}  // namespace

namespace sage {

int topk_max_units() { return 64 * MAX_OWN; }
int topk_merge_max_units(int k) { return 64 * (k == 1 ? MERGE_MAX_OWN : MAX_OWN); }

// Pass 2 for `rows` rows whose `nunits` slices each left UnitStats and k sorted keys in stats / keys ([row][unit]).
// units_used (k = 1 only, nullable): the number of slices where the device has decided it; then `nunits` is the most it can be.
void topk_merge(int rows, int k, const int* n_valid, int rows_per_group, int nunits, const UnitStats* stats,
                const uint64_t* keys, float* entropy, int* topk_idx, float* topk_prob, float* topk_renorm,
                float* topk_entropy, float* alpha, hipStream_t s, const int* units_used) {
    if (k == 1) {
        const dim3 grid((rows + MERGE_THREADS / 64 - 1) / (MERGE_THREADS / 64)), block(MERGE_THREADS);
        if (nunits <= 256)
            hipLaunchKernelGGL(merge_one_kernel<4>, grid, block, 0, s, n_valid, rows_per_group, rows, nunits, units_used, stats, keys, entropy, topk_idx,
                               topk_prob, topk_renorm, topk_entropy, alpha);
        else if (nunits <= 64 * MAX_OWN)
            hipLaunchKernelGGL(merge_one_kernel<MAX_OWN>, grid, block, 0, s, n_valid, rows_per_group, rows, nunits, units_used, stats, keys, entropy,
                               topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
        else
            hipLaunchKernelGGL(merge_one_kernel<MERGE_MAX_OWN>, grid, block, 0, s, n_valid, rows_per_group, rows, nunits, units_used, stats, keys,
                               entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
    } else if (nunits <= 64 * 4)
        hipLaunchKernelGGL(merge_kernel<4>, dim3(rows), dim3(MERGE_THREADS), 0, s, k, n_valid, rows_per_group, nunits, stats, keys,
                           entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
    else
        hipLaunchKernelGGL(merge_kernel<MAX_OWN>, dim3(rows), dim3(MERGE_THREADS), 0, s, k, n_valid, rows_per_group, nunits, stats,
                           keys, entropy, topk_idx, topk_prob, topk_renorm, topk_entropy, alpha);
}

}  // namespace sage

extern "C" size_t sage_entropy_topk_workspace_bytes(int rows, int vocab, int k) {
    if (rows < 0 || vocab < 1 || k < 1) return 0;
    return stats_bytes(rows, vocab) + static_cast<size_t>(rows) * num_units(vocab) * k * sizeof(uint64_t) + 256;
}

namespace sage {

// Where the first pass leaves its results inside a workspace of sage_entropy_topk_workspace_bytes(rows, vocab, k).
void topk_workspace_layout(int rows, int vocab, void* workspace, UnitStats** stats, uint64_t** keys, int* nunits) {
    *stats = static_cast<UnitStats*>(workspace);
    *keys = reinterpret_cast<uint64_t*>(static_cast<char*>(workspace) + stats_bytes(rows, vocab));
    *nunits = num_units(vocab);
}

}  // namespace sage

// Argument checks of a first pass; SAGE_OK means it may be launched (rows == 0: there is nothing to launch).
static int check_first_pass(const void* logits, int dtype, int rows, int vocab, long row_stride, int k, const int* n_valid,
                            int rows_per_group, void* workspace, size_t workspace_bytes) {
    if (!logits || !workspace) return SAGE_INVALID_ARG;
    if (rows < 0 || vocab < 1 || k < 1 || k > SAGE_MAX_TOPK || k > vocab || row_stride < vocab) return SAGE_INVALID_ARG;
    if (dtype != SAGE_F32 && dtype != SAGE_BF16) return SAGE_INVALID_ARG;
    if (n_valid && rows_per_group < 1) return SAGE_INVALID_ARG;
    const size_t esz = dtype == SAGE_F32 ? 4 : 2;
    if (!sage::aligned(logits, 16) || (static_cast<size_t>(row_stride) * esz) % 16 != 0 || !sage::aligned(workspace, 16))
        return SAGE_INVALID_ARG;
    const int nunits = num_units(vocab);
    if (nunits > 64 * MAX_OWN) return SAGE_UNSUPPORTED;
    if (rows > 65535) return SAGE_UNSUPPORTED;
    if (workspace_bytes < sage_entropy_topk_workspace_bytes(rows, vocab, k)) return SAGE_WORKSPACE_TOO_SMALL;
    return SAGE_OK;
}

template <typename F>
static void with_loads(const void* logits, int dtype, bool once, F launch) {
    auto of = [&](auto* x) { if (once) launch(x, std::true_type{}); else launch(x, std::false_type{}); };
    if (dtype == SAGE_F32) of(static_cast<const float*>(logits));
    else of(static_cast<const uint16_t*>(logits));
}
// Argument checks and the first pass, common to sage_entropy_topk and sage_entropy_topk_slices.
static int run_first_pass(const void* logits, int dtype, int rows, int vocab, long row_stride, int k, const int* n_valid,
                          int rows_per_group, void* workspace, size_t workspace_bytes, hipStream_t s) {
    const int rc = check_first_pass(logits, dtype, rows, vocab, row_stride, k, n_valid, rows_per_group, workspace, workspace_bytes);
    if (rc != SAGE_OK || rows == 0) return rc;
    const int nunits = num_units(vocab);
    UnitStats* stats = static_cast<UnitStats*>(workspace);
    uint64_t* keys = reinterpret_cast<uint64_t*>(static_cast<char*>(workspace) + stats_bytes(rows, vocab));
    const bool once = static_cast<long>(rows) * vocab * (dtype == SAGE_F32 ? 4 : 2) > READ_ONCE_BYTES;
    if (k == 1 && !n_valid) {                        // many rows, one round: a wave per slice, 16 logits per lane
        const dim3 grid((nunits + WAVES - 1) / WAVES, rows);
        auto launch = [&](auto* x, auto once) {
            using T = std::remove_const_t<std::remove_pointer_t<decltype(x)>>;
            hipLaunchKernelGGL((slice_kernel<T, decltype(once)::value>), grid, dim3(THREADS), 0, s, x, vocab, row_stride, nunits, stats, keys);
        };
        with_loads(logits, dtype, once, launch);
    } else if (k == 1) {                             // grouped rows: workgroups walk the live rows of their group
        const int groups = (rows + rows_per_group - 1) / rows_per_group;
        const dim3 grid((nunits + WAVES - 1) / WAVES, row_phases(groups, rows_per_group, false), groups);
        auto launch = [&](auto* x, auto once) {
            using T = std::remove_const_t<std::remove_pointer_t<decltype(x)>>;
            hipLaunchKernelGGL((slice_rows_kernel<T, decltype(once)::value>), grid, dim3(THREADS), 0, s, x, vocab, row_stride, n_valid, rows_per_group, rows,
                               nunits, stats, keys);
        };
        with_loads(logits, dtype, once, launch);
    } else if (k <= WAVE_MAX_K) {                    // few rows, short lists: a wave per slice
        const dim3 grid((nunits + WAVES - 1) / WAVES, rows);
        if (dtype == SAGE_F32)
            hipLaunchKernelGGL(slice_topk_wave_kernel<float>, grid, dim3(THREADS), 0, s, static_cast<const float*>(logits), vocab,
                               row_stride, k, n_valid, rows_per_group, nunits, stats, keys);
        else
            hipLaunchKernelGGL(slice_topk_wave_kernel<uint16_t>, grid, dim3(THREADS), 0, s, static_cast<const uint16_t*>(logits), vocab,
                               row_stride, k, n_valid, rows_per_group, nunits, stats, keys);
    } else {                                         // a workgroup per slice, 4 logits per lane
        const dim3 grid(nunits, rows);
        if (dtype == SAGE_F32)
            hipLaunchKernelGGL(slice_topk_kernel<float>, grid, dim3(THREADS), 0, s, static_cast<const float*>(logits), vocab,
                               row_stride, k, n_valid, rows_per_group, nunits, stats, keys);
        else
            hipLaunchKernelGGL(slice_topk_kernel<uint16_t>, grid, dim3(THREADS), 0, s, static_cast<const uint16_t*>(logits),
                               vocab, row_stride, k, n_valid, rows_per_group, nunits, stats, keys);
    }
    return sage::launch_status();
}

extern "C" int sage_entropy_topk(const void* logits, int dtype, int rows, int vocab, long row_stride, int k,
                                 const int* n_valid, int rows_per_group, float* entropy, int* topk_idx,
                                 float* topk_prob, float* topk_renorm, float* topk_entropy, float* alpha,
                                 void* workspace, size_t workspace_bytes, void* stream) {
    if (!topk_idx) return SAGE_INVALID_ARG;
    hipStream_t s = sage::as_stream(stream);
    if (vocab >= 1 && num_units(vocab) <= (k == 1 ? ONE_LAUNCH_UNITS : 1)) {
        const int rc = check_first_pass(logits, dtype, rows, vocab, row_stride, k, n_valid, rows_per_group, workspace, workspace_bytes);
        if (rc != SAGE_OK || rows == 0) return rc;
        UnitStats* stats;
        uint64_t* keys;
        int nunits;
        sage::topk_workspace_layout(rows, vocab, workspace, &stats, &keys, &nunits);
        if (dtype == SAGE_F32)
            launch_in_one(static_cast<const float*>(logits), rows, vocab, row_stride, k, n_valid, rows_per_group, nunits, stats, keys, entropy,
                          topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, s);
        else
            launch_in_one(static_cast<const uint16_t*>(logits), rows, vocab, row_stride, k, n_valid, rows_per_group, nunits, stats, keys, entropy,
                          topk_idx, topk_prob, topk_renorm, topk_entropy, alpha, s);
        return sage::launch_status();
    }
    const int rc = run_first_pass(logits, dtype, rows, vocab, row_stride, k, n_valid, rows_per_group, workspace, workspace_bytes, s);
    if (rc != SAGE_OK || rows == 0) return rc;
    UnitStats* stats;
    uint64_t* keys;
    int nunits;
    sage::topk_workspace_layout(rows, vocab, workspace, &stats, &keys, &nunits);
    sage::topk_merge(rows, k, n_valid, rows_per_group, nunits, stats, keys, entropy, topk_idx, topk_prob, topk_renorm,
                     topk_entropy, alpha, s);
    return sage::launch_status();
}

extern "C" int sage_entropy_topk_slices(const void* logits, int dtype, int rows, int vocab, long row_stride, int k,
                                        const int* n_valid, int rows_per_group, void* workspace, size_t workspace_bytes,
                                        void* stream) {
    return run_first_pass(logits, dtype, rows, vocab, row_stride, k, n_valid, rows_per_group, workspace, workspace_bytes,
                          sage::as_stream(stream));
}

extern "C" int sage_entropy_topk_slices_pair(const void* logits_a, int rows_a, long row_stride_a, const int* n_valid_a,
                                             int rows_per_group_a, void* workspace_a, size_t workspace_a_bytes,
                                             const void* logits_b, int rows_b, long row_stride_b, int k_b, void* workspace_b,
                                             size_t workspace_b_bytes, int dtype, int vocab, void* stream) {
    if (!n_valid_a || k_b < 2) return SAGE_INVALID_ARG;      // job A is the grouped k = 1 pass, job B a k > 1 pass
    int rc = check_first_pass(logits_a, dtype, rows_a, vocab, row_stride_a, 1, n_valid_a, rows_per_group_a, workspace_a,
                              workspace_a_bytes);
    if (rc != SAGE_OK) return rc;
    rc = check_first_pass(logits_b, dtype, rows_b, vocab, row_stride_b, k_b, nullptr, 1, workspace_b, workspace_b_bytes);
    if (rc != SAGE_OK) return rc;
    hipStream_t s = sage::as_stream(stream);
    if (rows_a == 0 || rows_b == 0) {                        // one job is empty: the other one's own launch
        if (rows_a) return run_first_pass(logits_a, dtype, rows_a, vocab, row_stride_a, 1, n_valid_a, rows_per_group_a, workspace_a,
                                          workspace_a_bytes, s);
        return run_first_pass(logits_b, dtype, rows_b, vocab, row_stride_b, k_b, nullptr, 1, workspace_b, workspace_b_bytes, s);
    }
    const int nunits = num_units(vocab);
    UnitStats* stats_a = static_cast<UnitStats*>(workspace_a);
    uint64_t* keys_a = reinterpret_cast<uint64_t*>(static_cast<char*>(workspace_a) + stats_bytes(rows_a, vocab));
    PairJob b;
    b.logits = logits_b; b.row_stride = row_stride_b; b.rows = rows_b; b.k = k_b; b.nunits = nunits;
    b.stats = static_cast<UnitStats*>(workspace_b);
    b.keys = reinterpret_cast<uint64_t*>(static_cast<char*>(workspace_b) + stats_bytes(rows_b, vocab));
    const int groups = (rows_a + rows_per_group_a - 1) / rows_per_group_a;
    const int gx = (nunits + WAVES - 1) / WAVES, gy = row_phases(groups, rows_per_group_a, true);
    const bool by_waves = k_b <= WAVE_MAX_K;                 // workgroups of job B, in rows of the grid
    const long rows_of_b = by_waves ? rows_b : (static_cast<long>(nunits) * rows_b + gx - 1) / gx;
    const bool ahead = groups == 1 && by_waves && rows_b + gy <= 65535;
    const long slabs_b = ahead ? 0 : (rows_of_b + gy - 1) / gy;
    if (slabs_b + groups > 65535) return SAGE_UNSUPPORTED;
    const dim3 grid(gx, ahead ? gy + rows_b : gy, static_cast<unsigned>(slabs_b + groups));
    auto launch = [&](auto kernel, auto* logits) {
        hipLaunchKernelGGL(kernel, grid, dim3(THREADS), 0, s, logits, vocab, row_stride_a, n_valid_a, rows_per_group_a, rows_a, nunits, stats_a,
                           keys_a, static_cast<int>(slabs_b), b);
    };
    if (dtype == SAGE_F32)
        launch(by_waves ? slice_pair_kernel<float, true> : slice_pair_kernel<float, false>, static_cast<const float*>(logits_a));
    else
        launch(by_waves ? slice_pair_kernel<uint16_t, true> : slice_pair_kernel<uint16_t, false>, static_cast<const uint16_t*>(logits_a));
    return sage::launch_status();
}
