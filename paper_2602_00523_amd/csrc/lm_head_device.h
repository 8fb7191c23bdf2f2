// What the two projection kernels (lm_head_topk.hip: up to 64 rows; lm_head_rows.hip: more) do alike once a unit's logits
// are in registers: fold them into softmax statistics and the best candidate of a hidden row, and combine the four
// partial results of a row.  One definition, so that a row's result does not depend on which kernel it went through (as
// long as both cut the vocabulary alike).
#pragma once
#include "topk_common.h"

namespace sage {
namespace lmhead {

// A weight matrix of more bytes than the memory-side cache holds (256 MB) is read with loads that leave nothing there: it would have pushed itself out
// before the next call came, and to place it costs memory bandwidth.  Whole call, us, plain / so, k = 10 with 16 rows and greedy with 40 of 64: 389 MB 95.1 /
// 83.7 and 79.2 / 69.5, 623 MB 162 / 147 and 160 / 147, 1.09 GB 210 / 184, 2.49 GB (greedy, 64 rows) 433 / 397; at the line 272 MB 68.9 / 66.6 and 53.1 / 52.0,
// 262 MB 79.9 / 79.5 and 68.5 / 70.0.  A smaller matrix stays there from one call to the next: 246 MB, 48 rows, k = 4, 55 / 70 (though not in a
// program that reads more than the cache holds between two calls).
constexpr long READ_ONCE_BYTES = 256L << 20;
inline bool read_once(int vocab, int dim) { return static_cast<long>(vocab) * dim * 2 > READ_ONCE_BYTES; }

struct Fold { float m, Z, T; uint64_t key; };

// This lane's 16 N logits of one row: logit(a, i, left) is logit i of tile a if fewer than `left` rows precede it and -inf
// otherwise; its vocabulary index is v0 + stride a + 8 (i / 4) + i % 4 (the accumulator layout of a 32 x 32 MFMA), and
// v_end is one past the last row.  Two passes: the maximum first, then one exp2 and two multiply-adds per logit.
template <int N, class Logit>
__device__ __forceinline__ Fold fold_logits(int v0, int stride, int v_end, Logit logit) {
    // (`left` is made opaque, or the compiler keeps one comparison mask per register alive from the first pass to the second)
    auto left_of = [&](int a) __attribute__((always_inline)) {
        int left = v_end - v0 - stride * a;
        asm volatile("" : "+v"(left));
        return left;
    };
    float best = -INFINITY;
    int at = v0;
#pragma unroll
    for (int a = 0; a < N; ++a) {
        const int left = left_of(a);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float x = logit(a, i, left);
            const bool better = x > best;                    // indices ascend: equal values keep the earlier one
            best = better ? x : best;
            at = better ? v0 + stride * a + 8 * (i >> 2) + (i & 3) : at;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    float Z = 0.f, Tm = 0.f;
#pragma unroll
    for (int a = 0; a < N; ++a) {
        const int left = left_of(a);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            // capped where exp is below 2^-125: a masked entry then adds about 1e-38 instead of 0 to a sum that is >= 1
            // (the minimum that keeps a NaN: a NaN or +inf logit makes the row's statistics NaN; the best candidate is the
            // best of the numbers)
            const float dlt = __builtin_elementwise_minimum(best - logit(a, i, left), 87.0f);
            const float e = __builtin_amdgcn_exp2f(dlt * -1.4426950408889634f);
            Z += e;
            Tm = fmaf(e, dlt, Tm);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // (a lane past the end starts past the end: no candidate; its maximum is -inf and its sums are skipped)
    return Fold{best, Z, Tm, at < v_end ? topk::key_pack(topk::make_key(best, at)) : 0ull};
}

// The four partial results of one row (part: 4 x (m, Z, T), key: 4) as one slice of the row.
__device__ __forceinline__ void combine_folds(const float* part, const uint64_t* key, topk::UnitStats* stat_out, uint64_t* key_out) {
    float m = -INFINITY;
    uint64_t k = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        m = fmaxf(m, part[3 * p]);
        k = max(k, key[p]);
    }
    float z = 0.f, t = 0.f;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (part[3 * p] > -INFINITY) {
            const float dlt = m - part[3 * p];
            const float sc = __builtin_amdgcn_exp2f(dlt * -1.4426950408889634f);
            z += sc * part[3 * p + 1];
            t += sc * (part[3 * p + 2] + part[3 * p + 1] * dlt);
        }
    }
    *stat_out = topk::UnitStats{m, z, t, 0.f};
    if (key_out) *key_out = k;
}

}  // namespace lmhead
}  // namespace sage
