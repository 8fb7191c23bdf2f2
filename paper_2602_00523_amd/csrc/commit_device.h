// Device-side pieces of the calls that close a step (Alg. 1 Phase 3: the accepted tokens join the context; Sec. 3.3
// adaptive history tracking), shared by the kernels of commit_history.hip and by the kernel that runs them right after
// the acceptance rule (fused_steps.hip).
#pragma once
#include "sage_internal.h"

namespace sage {
namespace closing {

// Closing a step is latency, a chain of round trips to memory: what decides (lengths, state, path), then the rows, all of them at once.
// Step, before (lengths after the acceptance rule, a row after the other) -> now: one layer over 4096 positions 20.3 -> 19.7 us, over
// 16384 32.7 -> 32.2, three short sequences of four layers 79.4 -> 78.7.  What is executed costs, too:
// copying every piece of all rows in one flat loop, two per thread held, with the divisions that takes, made the steps 0.6 us slower
// than before.
// 2^row_shift threads copy a row of `pieces` 16-byte pieces: one piece each while there are threads, so that a short path costs one round
// trip however wide its rows are, and more rows at a time where they are narrow.  The number of turns of a long path is the same
// either way.  Calls, us, with 256 threads a row and one row at a time in a workgroup (1024 in the acceptance) -> 128 -> this: a row of 512
// pieces, path of one, sage_commit_path 2.20 -> 2.33 -> 2.10, sage_close_step 2.61 -> 2.67 -> 2.19, with the acceptance 7.94 -> 7.99 -> 7.50;
// of three 2.32 -> 2.42 -> 2.24, 3.58 -> 2.89 -> 2.65, 8.87 -> 8.13 -> 7.96; 1024 pieces, path of one 2.51 -> 2.95 -> 2.18, 3.01 -> 3.36 ->
// 2.39, 8.38 -> 8.74 -> 7.76, of eight 2.63 -> 3.16 -> 2.31, 9.23 -> 6.11 -> 6.24, 12.9 -> 11.4 -> 11.6; rows of up to 128 as with 128.
constexpr int MIN_ROW_SHIFT = 7;
inline int row_shift(long pieces, int most) {
    int s = MIN_ROW_SHIFT;
    while ((1 << s) < pieces && (2 << s) <= most) ++s;
    return s;
}
// 2^shift threads, of which this one is `t0`, copy the K row and the V row of `node`, path entry j of sequence b (Hkv heads x d elements
// each), to cache position len_b + j in 16-byte pieces.
__device__ __forceinline__ void commit_row(
    const unsigned char* __restrict__ Kt, const unsigned char* __restrict__ Vt, unsigned char* __restrict__ Kc,
    unsigned char* __restrict__ Vc, int esz, int Hkv, int d, int64_t start, int len_b, int kv_capacity, long kv_token_stride,
    long kv_head_stride, int node, int j, int b, int t0, int shift) {
    const long pos = static_cast<long>(len_b) + j;
    if (node < 0 || node >= SAGE_MAX_NODES || pos >= kv_capacity) return;      // never read or write out of range
    const int pieces = d * esz / 16;                                           // 16-byte pieces of one head's row
    const long src_row = (static_cast<long>(b) * SAGE_MAX_NODES + node) * Hkv * d * esz;
    const long dst_tok = (start + pos) * kv_token_stride * esz;
    for (int t = t0; t < Hkv * pieces; t += 1 << shift) {
        const int g = t / pieces, c = t % pieces;
        const long src = src_row + (static_cast<long>(g) * d * esz) + c * 16;
        const long dst = dst_tok + static_cast<long>(g) * kv_head_stride * esz + c * 16;
        const uint4 k = *reinterpret_cast<const uint4*>(Kt + src), v = *reinterpret_cast<const uint4*>(Vt + src);
        *reinterpret_cast<uint4*>(Kc + dst) = k;
        *reinterpret_cast<uint4*>(Vc + dst) = v;
    }
}

__device__ __forceinline__ int advanced_len(int len_b, int tau, int kv_capacity) {
    const long n = static_cast<long>(len_b) + tau + 1;                        // the root and the tau accepted tokens
    return n > kv_capacity ? kv_capacity : static_cast<int>(n);
}

// One wave for sequence b: lane i holds window slot i.  What the update reads of its own state is asked for by itself, so that a kernel
// that has yet to find tau can have it on the way meanwhile.
struct HistoryState { int count, value, d_max; };
__device__ __forceinline__ HistoryState history_state(int b, int lane, int window, const int* hist, const int* count, const int* d_max_in) {
    return HistoryState{count[b], lane < window ? hist[static_cast<long>(b) * window + lane] : 0, d_max_in[b]};
}
// The new depth limit goes to d_max_out (which may be d_max_in).
__device__ __forceinline__ void history_wave(int b, int lane, int tau, int window, float lo, float hi, int d_floor, int d_cap,
                                             const HistoryState& was, int* __restrict__ hist, int* __restrict__ count, int* d_max_out,
                                             float* __restrict__ avg_out) {
    const int cnt = was.count;
    const int slot = cnt % window;
    const int n = min(cnt + 1, window);
    int v = 0;
    if (lane < n) v = (lane == slot) ? tau : was.value;
    const int sum = static_cast<int>(sage::wave_sum_u32(static_cast<uint32_t>(v)));
    if (lane == 0) {
        hist[static_cast<long>(b) * window + slot] = tau;
        count[b] = cnt + 1;
        const float fs = static_cast<float>(sum), fn = static_cast<float>(n);
        if (avg_out) avg_out[b] = __fdiv_rn(fs, fn);
        int dm = was.d_max;
        if (fs < __fmul_rn(lo, fn)) dm -= 1;                                   // strictly below the lower threshold
        else if (fs > __fmul_rn(hi, fn)) dm += 1;                              // strictly above the upper one
        d_max_out[b] = min(max(dm, d_floor), d_cap);
    }
}

}  // namespace closing
}  // namespace sage
