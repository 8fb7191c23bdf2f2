// Device-side pieces of the top-k second pass, shared by the kernels that run it on its own (entropy_topk.hip) and by
// the kernels that fold it into the step that consumes its result (fused_steps.hip): wave-wide reductions, the per-row
// merge of slice statistics and candidate lists, Eq. 7-9 on the winners.
#pragma once
#include <type_traits>

#include "topk_common.h"

namespace sage {
namespace topk {

constexpr int MERGE_THREADS = 256;
constexpr int MERGE_LDS_KEYS = 6144;     // lists are staged in LDS when they fit (48 KB)
constexpr int MAX_OWN = 16;              // lists per lane in the second pass: up to 1024 slices = 1M logits
// ... in the second pass of k = 1 as a launch of its own: projections of more than 64 rows cut the vocabulary into units of at
// most 256, up to 2635 of them at the 655360 tokens that they take
constexpr int MERGE_MAX_OWN = 42;

// The wave-wide reductions of sage_internal.h, under this namespace's names.
using sage::wave_max;
using sage::wave_max_u32;
using sage::wave_sum;

// A key is reduced in two passes: the value code first, then the index code among the lanes that hold the winning value.
__device__ __forceinline__ Key wave_max_key(Key k) {
    const uint32_t hi = wave_max_u32(k.hi);
    const uint64_t holders = __ballot(k.hi == hi);
    uint32_t lo;
    if (__builtin_popcountll(holders) == 1)          // the usual case: no second reduction, just fetch the winner's index
        lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(k.lo), __builtin_ctzll(holders)));
    else
        lo = wave_max_u32(k.hi == hi ? k.lo : 0u);
    return Key{hi, lo};
}
__device__ __forceinline__ bool row_is_valid(int row, const int* n_valid, int rows_per_group) {
    if (!n_valid) return true;
    return (row % rows_per_group) < n_valid[row / rows_per_group];
}

// Log-sum-exp combination of slice statistics held OWN per lane (lane owns slices lane, lane + 64, ...): the row's
// maximum m and the sums Z, T relative to it, in every lane.  One definition for every kernel that finishes a row, so
// that they agree to the bit.
template <int OWN>
__device__ __forceinline__ void combine_unit_stats(const UnitStats (&u)[OWN], int lane, int nunits, float& m, float& Z, float& Tm) {
    m = -INFINITY;
#pragma unroll
    for (int i = 0; i < OWN; ++i)
        if (lane + 64 * i < nunits) m = fmaxf(m, u[i].m);
    m = wave_max(m);
    Z = 0.f;
    Tm = 0.f;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
        if (lane + 64 * i < nunits && u[i].m > -INFINITY) {
            const float dlt = m - u[i].m;
            const float w = __builtin_amdgcn_exp2f(dlt * -1.4426950408889634f);
            Z += w * u[i].Z;
            Tm += w * (u[i].T + u[i].Z * dlt);
        }
    }
    Z = wave_sum(Z);
    Tm = wave_sum(Tm);
}

// LDS of one merging workgroup.  merge_row takes any type with these members (keys, pick, row_m, row_Z; LDS_KEYS = how many
// keys fit), so a kernel with another LDS budget can bring a smaller one.
constexpr int PICK_CANDS = 512;          // candidates that the counting selection takes
constexpr int PICK_LISTS = 256;          // lists that they may come from
constexpr int STAGED_MAX_K = 16;         // longer lists are not staged in LDS
// Entry number `at` of lists of `width` lies in list (at * reciprocal(width)) >> 16: true of what is asked for here, up to
// PICK_LISTS lists of up to STAGED_MAX_K (it fails at entry 3293 of lists of 27, and at 1448 of lists of 63).
__host__ __device__ constexpr unsigned reciprocal(unsigned width) { return (65536u + width - 1) / width; }
constexpr bool reciprocal_holds(unsigned width) {
    for (unsigned at = 0; at < PICK_LISTS * width; ++at)
        if ((at * reciprocal(width)) >> 16 != at / width) return false;
    return true;
}
static_assert([] { for (unsigned w = 1; w <= STAGED_MAX_K; ++w) if (!reciprocal_holds(w)) return false; return true; }(), "reciprocal");
struct PickShared {
    alignas(16) uint64_t cand[PICK_CANDS];   // candidates for the row's k winners, any order
    uint64_t win[SAGE_MAX_TOPK];             // the winners, in order
    uint16_t lists[PICK_LISTS];              // the lists that hold them
    int nlists, ncand, nkept;
    uint32_t floor;                          // value code below which no candidate lies
};
template <int OWN> struct MergeShared {
    static constexpr int LDS_KEYS = MERGE_LDS_KEYS;
    uint64_t keys[MERGE_LDS_KEYS];
    PickShared pick;
    float row_m, row_Z;                  // the row's maximum and sum, from the wave that combines the statistics
};

// How many of keys[0 .. n) (n a multiple of 16, LDS, 16-byte aligned) are above `mine`: broadcast reads, eight in flight.
__device__ __forceinline__ int count_above(const uint64_t* keys, int n, uint64_t mine) {
    int above = 0;
    for (int o = 0; o < n; o += 16) {
        ulonglong2 h[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = *reinterpret_cast<const ulonglong2*>(keys + o + 2 * u);
#pragma unroll
        for (int u = 0; u < 8; ++u) above += (h[u].x > mine ? 1 : 0) + (h[u].y > mine ? 1 : 0);
    }
    return above;
}

// What wave 0 holds once a row is merged: lane j < k owns winner j (token index, probability, renormalised probability);
// alpha (Eq. 9) is wave-uniform.
struct MergedRow {
    int idx;
    float p, q, alpha;
};

// Eq. 7-9 on the winners that the lanes of one wave hold (lane j < k: winner j), given the row's maximum and sum.  Writes the
// row's outputs (null pointers are skipped).
__device__ __forceinline__ void finish_row(int row, int k, int lane, Key mine, float m, float Z, int* __restrict__ topk_idx,
                                           float* __restrict__ topk_prob, float* __restrict__ topk_renorm,
                                           float* __restrict__ topk_entropy, float* __restrict__ alpha, MergedRow& out) {
    const bool have = lane < k;
    const float x = have ? key_value(mine) : -INFINITY;
    const float p = have ? expf(x - m) / Z : 0.f;
    const float mass = wave_sum(p);
    const float q = have ? p / mass : 0.f;
    const float hk = wave_sum(q > 0.f ? -q * logf(q) : 0.f);
    float a = (k == 1) ? 1.0f : 1.0f - hk / logf(static_cast<float>(k));
    a = fminf(fmaxf(a, 0.0f), 1.0f);
    if (have) {
        const long o = static_cast<long>(row) * k + lane;
        topk_idx[o] = key_index(mine);
        if (topk_prob) topk_prob[o] = p;
        if (topk_renorm) topk_renorm[o] = q;
    }
    if (lane == 0) {
        if (topk_entropy) topk_entropy[row] = hk;
        if (alpha) alpha[row] = a;
    }
    out.idx = have ? key_index(mine) : -1;
    out.p = p;
    out.q = q;
    out.alpha = a;
}

// Of the N values that every lane of a wave holds (those with have[i]), mark in in[i] at least the `want` and at most the
// `most` largest (want <= how many there are, want <= most).  A threshold that at least `want` values reach is built bit by
// bit, a ballot per value and bit, from the first bit in which the largest and the smallest value differ until no more
// than `most` reach it: about six bits of 80 cycles on ordinary values when `most` leaves some room.  Only when too many
// values equal the threshold are those admitted one by one, in order of (i, lane).  Returns the threshold.
template <int N>
__device__ __forceinline__ uint32_t wave_pick(const uint32_t (&code)[N], const bool (&have)[N], int want, int most, bool (&in)[N]) {
    uint32_t hi = 0, lo = 0xFFFFFFFFu;
    int got = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        hi = max(hi, have[i] ? code[i] : 0u);
        lo = min(lo, have[i] ? code[i] : 0xFFFFFFFFu);
        got += __builtin_popcountll(__ballot(have[i]));
    }
    uint32_t thr = 0;
    int above = 0;
    if (got > most) {                                // (uniform)
        hi = __builtin_amdgcn_readfirstlane(wave_max_u32(hi));
        lo = __builtin_amdgcn_readfirstlane(~wave_max_u32(~lo));
        auto reach = [&](uint32_t t) __attribute__((always_inline)) {
            int n = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) n += __builtin_popcountll(__ballot(have[i] && code[i] >= t));
            return n;
        };
        uint32_t bit = hi == lo ? 0u : 0x80000000u >> __builtin_clz(hi ^ lo);
        thr = bit ? hi & ~(2u * bit - 1u) : hi;      // what all values have in common (2 bit wraps to 0: nothing)
        for (; bit != 0 && got > most; bit >>= 1) {
            const int n = reach(thr | bit);
            if (n >= want) {
                thr |= bit;
                got = n;
            }
        }
        if (got > most && thr != 0xFFFFFFFFu) above = reach(thr + 1u);   // (nothing is above the largest code)
    }
    int left = want - above;                         // how many equal ones are admitted
#pragma unroll
    for (int i = 0; i < N; ++i) {
        in[i] = have[i] && code[i] >= thr;
        if (got > most) {
            const bool eq = in[i] && code[i] == thr;
            const uint64_t b = __ballot(eq);
            const int before = static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
            in[i] = in[i] && (!eq || before < left);
            left -= __builtin_popcountll(b);
        }
    }
    return thr;
}

// The same for a `most` well above `want` (up to 64, both), without a ballot per value and bit: the threshold comes from the
// lanes' largest values, one ballot a bit.  What `want` of those reach, at least `want` of all values reach, and seldom many more; should
// too many do (a lane's values are near each other, long runs of equal ones), or fewer than `want` lanes have a value, all values are looked at
// as well: with nothing but equal logits a projection of 8, 16 and 33 rows takes 1.0, 1.8 and 4 us more than with the ballots alone (k = 10 or
// 16; 78, 81 and 98 us), with others 1.5 to 13 less.
template <int N>
__device__ __forceinline__ void wave_pick_roughly(const uint32_t (&code)[N], const bool (&have)[N], int want, int most, bool (&in)[N]) {
    uint32_t top[1] = {0};
    bool some[1] = {false}, reached[1];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        top[0] = max(top[0], have[i] ? code[i] : 0u);
        some[0] = some[0] || have[i];
    }
    if (__builtin_popcountll(__ballot(some[0])) >= want) {
        const uint32_t thr = wave_pick<1>(top, some, want, want + want / 2 + 2, reached);
        int n = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            in[i] = have[i] && code[i] >= thr;
            n += __builtin_popcountll(__ballot(in[i]));
        }
        if (n <= most) return;
    }
    wave_pick<N>(code, have, want, most, in);
}

// Second pass for one row, called by all WG_THREADS threads of a workgroup (at least two waves): combine the slice
// statistics, merge the per-slice sorted key lists, Eq. 7-9.  OWN = lists per lane of one wave (lane owns lists lane,
// lane+64, ...).  Writes the row's outputs (null pointers are skipped) and returns true in wave 0, whose lanes receive `out`;
// the other waves help and return false.  Every thread passes the same workgroup barriers.
//
// This is pure latency (a few KB of data, one workgroup per row), so what counts is the length of its dependent chain, and
// k rounds of a wave-wide maximum and the advance of one list (about 250 ns each; more when the lists do not fit LDS)
// were most of it: 2.5 us at k = 10, 26 us at k = 64.  Instead: (1) wave 0 finds a value that at least k candidates reach
// and not many more: the p-th largest of the lists' entries at depth d, p (d + 1) >= k, d chosen so that p is a small
// part of the lists; (2) the entries that reach it are gathered from the lists whose heads do; (3) a thread per candidate
// counts the candidates above it, which is its place.  A row of few large logits over a level floor has a threshold that
// thousands of entries equal: when there are too many candidates, those strictly above the threshold are gathered instead,
// and do if they are k (64 planted logits over a floor, k = 64, whole call: 35.5 us by the rounds that it took before, 18.4
// now).  What is left takes the k rounds, over the k lists with the largest heads, a lane per list.
template <int OWN, int WG_THREADS = MERGE_THREADS, class Shared>
__device__ __forceinline__ bool merge_row(int row, int k, int nunits, const UnitStats* __restrict__ stats,
                                          const uint64_t* __restrict__ keys, Shared& sh, float* __restrict__ entropy,
                                          int* __restrict__ topk_idx, float* __restrict__ topk_prob,
                                          float* __restrict__ topk_renorm, float* __restrict__ topk_entropy,
                                          float* __restrict__ alpha, MergedRow& out) {
    constexpr int THREADS = WG_THREADS;
    static_assert(THREADS >= 192, "a wave for the pick, one for the statistics, others to stage");
    PickShared& pk = sh.pick;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const uint64_t* kk = keys + static_cast<long>(row) * nunits * k;
    const int total = nunits * k;
    // Short lists are staged in LDS while wave 0 picks; of long ones only the picked lists are fetched, afterwards.
    const bool in_lds = k <= STAGED_MAX_K && total <= Shared::LDS_KEYS;
    auto stage = [&](int t0, int step) __attribute__((always_inline)) {   // eight independent loads per thread at a time
        for (int i0 = t0; i0 < total; i0 += step * 8) {
            uint64_t tmp[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) tmp[j] = (i0 + j * step < total) ? kk[i0 + j * step] : 0;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (i0 + j * step < total) sh.keys[i0 + j * step] = tmp[j];
        }
    };
    if (tid < 64) {
        const int depth = min(k - 1, (4 * k + nunits - 1) / nunits - 1);   // k / (depth + 1) is at most a quarter of the lists
        uint32_t code[OWN], head[OWN];
        bool have[OWN], in[OWN];
        int deep = 0;
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int c = lane + 64 * i;
            const Key h = c < nunits ? key_unpack(kk[static_cast<long>(c) * k]) : Key{0, 0};
            const Key e = c < nunits ? key_unpack(kk[static_cast<long>(c) * k + depth]) : Key{0, 0};
            head[i] = h.hi;
            code[i] = e.hi;
            have[i] = !key_none(e);
        }
        if (lane == 0) pk.ncand = 0;
        pk.win[lane] = 0;
#pragma unroll
        for (int i = 0; i < OWN; ++i) deep += __builtin_popcountll(__ballot(have[i]));
        const int want = (k + depth) / (depth + 1);
        // (too few lists that deep: everything is a candidate)
        const uint32_t thr = deep < want ? 0u : wave_pick<OWN>(code, have, want, want + want / 2 + 2, in);
        int at = 0;
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const bool use = lane + 64 * i < nunits && head[i] >= thr;
            const uint64_t b = __ballot(use);
            const int to = at + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
            if (use && to < PICK_LISTS) pk.lists[to] = static_cast<uint16_t>(lane + 64 * i);
            at += __builtin_popcountll(b);
        }
        if (lane == 0) {
            pk.nlists = at;
            pk.floor = thr;
        }
    } else if (tid < 128) {                          // wave 1 combines the slice statistics (and stores the row's entropy)
        const UnitStats* st = stats + static_cast<long>(row) * nunits;
        UnitStats mine_stats[OWN];
#pragma unroll
        for (int i = 0; i < OWN; ++i)
            mine_stats[i] = lane + 64 * i < nunits ? st[lane + 64 * i] : UnitStats{-INFINITY, 0.f, 0.f, 0.f};
        float m, Z, Tm;
        combine_unit_stats<OWN>(mine_stats, lane, nunits, m, Z, Tm);
        if (lane == 0) {
            sh.row_m = m;
            sh.row_Z = Z;
            if (entropy) entropy[row] = logf(Z) + Tm / Z;
        }
    } else if (in_lds) {
        stage(tid - 128, THREADS - 128);
    }
    __syncthreads();
    auto entry = [&](int list, int j) __attribute__((always_inline)) {
        return in_lds ? sh.keys[list * k + j] : kk[static_cast<long>(list) * k + j];
    };
    // ---- candidates: a thread per entry of the picked lists; of lists that are not staged only the first eight entries, then
    // eight more while some list's last one fetched still is a candidate (lists are sorted)
    const int nl = pk.nlists <= PICK_LISTS ? pk.nlists : 0;
    const uint32_t floor = pk.floor;
    // entries j0 .. j0 + width - 1 of every picked list, BATCH of them per thread requested before the first is looked at;
    // width <= STAGED_MAX_K; returns whether a list's last one fetched was a candidate
    auto gather = [&](auto batch, int j0, int width, bool strictly) __attribute__((always_inline)) {
        constexpr int BATCH = decltype(batch)::value;
        const int entries = nl * width;
        const unsigned inv = reciprocal(width);
        bool more = false;
        for (int at0 = 0; at0 < entries; at0 += BATCH * THREADS) {
            uint64_t e[BATCH];
            bool last[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int at = at0 + u * THREADS + tid;
                const int r = static_cast<int>((static_cast<unsigned>(at) * inv) >> 16), j = j0 + at - r * width;
                e[u] = at < entries && j < k ? entry(pk.lists[r], j) : 0;
                last[u] = at - r * width == width - 1;
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const uint32_t code = static_cast<uint32_t>(e[u] >> 32);
                const bool cand = e[u] != 0 && (strictly ? code > floor : code >= floor);
                more = more || (cand && last[u]);
                const uint64_t b = __ballot(cand);
                if (b != 0) {
                    int base = 0;
                    if (lane == 0) base = atomicAdd(&pk.ncand, static_cast<int>(__builtin_popcountll(b)));
                    base = __builtin_amdgcn_readfirstlane(base);
                    const int to = base + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)));
                    if (cand && to < PICK_CANDS) pk.cand[to] = e[u];
                }
            }
        }
        return more;
    };
    // all candidates of the picked lists; returns how many (or that they are too many), after a barrier
    auto gather_all = [&](bool strictly) __attribute__((always_inline)) {
        if (in_lds) {
            gather(std::integral_constant<int, 1>{}, 0, k, strictly);
            __syncthreads();
            return pk.ncand;
        }
        const bool many = nl * 8 > THREADS;          // more than an entry per thread (of few lists one round trip is enough)
        for (int j0 = 0;; j0 += 8) {
            const bool any = many ? gather(std::integral_constant<int, 4>{}, j0, 8, strictly) : gather(std::integral_constant<int, 1>{}, j0, 8, strictly);
            const bool more = __syncthreads_or(any ? 1 : 0) != 0;
            if (!more || j0 + 8 >= k) return pk.ncand;
            if (many) {                              // stop as soon as they are too many
                const int n = pk.ncand;
                if (n > PICK_CANDS) return n;
                __syncthreads();                     // everyone has read the count before the next round adds to it
            }
        }
    };
    int nc = gather_all(false);
    if (pk.nlists > PICK_LISTS) {                    // (uniform, like what follows)
        nc = PICK_CANDS + 1;
    } else if (nc > PICK_CANDS) {
        __syncthreads();
        if (tid == 0) pk.ncand = 0;
        __syncthreads();
        nc = gather_all(true);
        if (nc < k) nc = PICK_CANDS + 1;
    }
    if (nc <= PICK_CANDS) {                          // (uniform)
        if (nc > 2 * SAGE_MAX_TOPK) {                // wave 0 picks again among them, k or a few more
            if (tid < 64) {
                constexpr int N = PICK_CANDS / 64;
                uint64_t key[N];
                uint32_t code[N];
                bool have[N], in[N];
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    have[i] = lane + 64 * i < nc;
                    key[i] = have[i] ? pk.cand[lane + 64 * i] : 0;
                    code[i] = static_cast<uint32_t>(key[i] >> 32);
                }
                const int want = min(k, nc), most = min(2 * SAGE_MAX_TOPK, k + k / 2 + 2);
                const uint32_t thr = wave_pick<N>(code, have, want, most, in);
                int equal = 0, admitted = 0, at = 0;
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    equal += __builtin_popcountll(__ballot(have[i] && code[i] == thr));
                    admitted += __builtin_popcountll(__ballot(in[i] && code[i] == thr));
                }
                if (admitted != equal) {             // of equal values the lowest indices: the largest lower words
                    bool eq[N], pick[N];
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        eq[i] = have[i] && code[i] == thr;
                        code[i] = eq[i] ? static_cast<uint32_t>(key[i]) : code[i];
                    }
                    wave_pick<N>(code, eq, admitted, admitted, pick);
#pragma unroll
                    for (int i = 0; i < N; ++i) in[i] = eq[i] ? pick[i] : in[i];
                }
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const uint64_t b = __ballot(in[i]);
                    if (in[i]) pk.cand[at + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)))] = key[i];
                    at += __builtin_popcountll(b);
                }
                if (lane == 0) pk.nkept = at;
            }
            __syncthreads();
            nc = pk.nkept;
        }
    }
    if (nc <= PICK_CANDS) {                          // a thread per candidate
        for (int c = tid; c < nc; c += THREADS) {
            const uint64_t mine = pk.cand[c];
            int above = 0;
            for (int o = 0; o < nc; o += 8) {        // broadcast reads, eight keys at a time; entries past nc are not counted
                ulonglong2 h[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) h[u] = *reinterpret_cast<const ulonglong2*>(pk.cand + o + 2 * u);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    above += (o + 2 * u < nc && h[u].x > mine ? 1 : 0) + (o + 2 * u + 1 < nc && h[u].y > mine ? 1 : 0);
            }
            if (above < k) pk.win[above] = mine;
        }
    } else if (tid < 64) {                           // k rounds over the k lists with the largest heads, a lane per list
        uint32_t code[OWN];
        bool have[OWN], in[OWN];
        int nonempty = 0, nl2 = 0;
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const Key h = lane + 64 * i < nunits ? key_unpack(entry(lane + 64 * i, 0)) : Key{0, 0};
            code[i] = h.hi;
            have[i] = !key_none(h);
            nonempty += __builtin_popcountll(__ballot(have[i]));
        }
        wave_pick<OWN>(code, have, min(k, nonempty), min(k, nonempty), in);   // (i, lane) is list order, which is index order
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const uint64_t b = __ballot(in[i]);
            if (in[i]) pk.lists[nl2 + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)))] = static_cast<uint16_t>(lane + 64 * i);
            nl2 += __builtin_popcountll(b);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int list = lane < nl2 ? pk.lists[lane] : 0;
        int cursor = 0;
        Key head = lane < nl2 ? key_unpack(entry(list, 0)) : Key{0, 0};
        for (int round = 0; round < k; ++round) {
            const Key g = wave_max_key(head);
            if (lane == round) pk.win[round] = key_pack(g);
            if (!key_none(g) && key_equal(head, g)) {
                ++cursor;
                head = cursor < k ? key_unpack(entry(list, cursor)) : Key{0, 0};
            }
        }
    }
    __syncthreads();
    if (tid >= 64) return false;                     // wave 0 finishes the row
    finish_row(row, k, lane, lane < k ? key_unpack(pk.win[lane]) : Key{0, 0}, sh.row_m, sh.row_Z, topk_idx, topk_prob, topk_renorm,
               topk_entropy, alpha, out);
    return true;
}

}  // namespace topk
}  // namespace sage
