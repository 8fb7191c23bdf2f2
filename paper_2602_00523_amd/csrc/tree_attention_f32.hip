// sage_tree_attention, fp32 instantiation: tree-masked GQA attention of the verify pass (Sec. 2.2 tree mask;
// Alg. 1 Phase 2) in plain fp32 FMA arithmetic.  Used for small full-precision shapes; the bf16 MFMA kernel
// carries the 72B-shape workloads.
//
// One workgroup per (node, query head, sequence).  The keys are one list, the cache's positions and then the tree's nodes,
// and 16 lanes share a key: a lane holds float4 pieces of its row, 64 dims apart, so that a load instruction reads whole
// rows.  A wave takes four keys at a time and keeps a softmax of its own (reference maximum, sum, weighted values) over all
// the keys it takes; the eight waves meet once, at the end, through LDS.
//
// What bounds it is latency: at 16 nodes x 4 heads x 272 keys of 64 dims a workgroup has 136 KB to read and a chain of
// dependent round trips.  There are two of those to memory, the sequence's sizes and then Q and every key and value of a
// tile of up to 288 keys, all requested before the first is used, and one barrier.  Before (a lane per key, whose loads
// touch 64 rows each, the cache's keys before the tree's, scores before values,
// six barriers a block) -> now, us per call: 8 nodes x 4 heads x 264 keys x 64 dims 8.6 -> 5.4, 16 x 8 x 527 x 128 29.4 -> 15.1,
// 64 x 32 x 2064 x 128 323 -> 157, 16 x 4 x 1016 x 256 80 -> 22.5.  Against 64 bits: 1.5-2.3e-7, 3.0-7.9e-7 before.
#include <utility>

#include "sage_internal.h"

namespace {

constexpr int THREADS = 512;
constexpr int WAVES = THREADS / 64;

// Four floats that need be aligned like one only: rows of Q, K and V may begin anywhere (16-byte loads either way).
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4(const float* p) {
    const float4_any x = *reinterpret_cast<const float4_any*>(p);
    return make_float4(x[0], x[1], x[2], x[3]);
}

// sum / maximum over the 16 lanes of a row, in each of them
__device__ __forceinline__ float row_sum(float v) {
    v += sage::f_dpp<0x128>(v); v += sage::f_dpp<0x124>(v); v += sage::f_dpp<0x122>(v); v += sage::f_dpp<0x121>(v);
    return v;
}
__device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, sage::f_dpp<0x128>(v)); v = fmaxf(v, sage::f_dpp<0x124>(v)); v = fmaxf(v, sage::f_dpp<0x122>(v)); v = fmaxf(v, sage::f_dpp<0x121>(v));
    return v;
}
// lane u of its row of 16, in each of them
template <int U> __device__ __forceinline__ float row_lane(float v) { return sage::f_dpp<0x150 + U>(v); }   // row_newbcast
template <class F, int... U> __device__ __forceinline__ void each(F f, std::integer_sequence<int, U...>) { (f(std::integral_constant<int, U>{}), ...); }
// sum / maximum over the four rows of a wave
__device__ __forceinline__ float rows_sum(float v) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
__device__ __forceinline__ float rows_max(float v) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}

// NC = pieces of 64 dims (the last one may be partly past d); TAKES = times that a tile's keys are taken.
template <int NC, int TAKES>
__global__ __launch_bounds__(THREADS) void tree_attention_f32_kernel(
    const int* __restrict__ n_nodes, const int* __restrict__ kv_len, const int64_t* __restrict__ kv_start,
    const int* __restrict__ first_node, const uint64_t* __restrict__ anc_mask, int Hq, int Hkv, int d,
    const float* __restrict__ Q, const float* __restrict__ Kc, const float* __restrict__ Vc, const float* __restrict__ Kt,
    const float* __restrict__ Vt, float* __restrict__ O, long kv_token_stride, long kv_head_stride, float scale) {
    __shared__ float s_acc[WAVES][NC * 64];
    __shared__ float s_m[WAVES], s_l[WAVES];

    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    int n = n_nodes[b];
    const int len = kv_len[b];
    const int64_t start = kv_start[b];
    const uint64_t mask = anc_mask[static_cast<long>(b) * SAGE_MAX_NODES + i];
    int first = first_node ? first_node[b] : 0;              // rows of earlier nodes are not asked for
    n = n < 1 ? 1 : (n > SAGE_MAX_NODES ? SAGE_MAX_NODES : n);   // a tree always has its root
    first = first < 0 ? 0 : (first > n - 1 ? n - 1 : first);
    if (i >= n || i < first) return;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dim0 = (tid & 15) * 4, row = (tid >> 4) & 3;
    const int g = h / (Hq / Hkv);
    const int L = len > 0 ? len : 0;
    const int cache_fours = (L + 3) / 4, fours = cache_fours + (n + 3) / 4;   // a wave takes four keys, all of the cache or all of the tree
    const long q_at = ((static_cast<long>(b) * SAGE_MAX_NODES + i) * Hq + h) * d;
    const long cache_at = start * kv_token_stride + static_cast<long>(g) * kv_head_stride;
    const long tree_at = (static_cast<long>(b) * SAGE_MAX_NODES * Hkv + g) * d, tree_stride = static_cast<long>(Hkv) * d;

    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    int dims[NC];                                            // (d is a multiple of 4; pieces past d are read inside the row
    float4 acc[NC];                                          // and not counted)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        dims[c] = min(64 * c + dim0, d - 4);
        acc[c] = zero;
    }
    float m = -INFINITY, l = 0.f;                            // of this wave; l of this lane's keys
    for (int tile = 0; tile < fours; tile += TAKES * WAVES) {
        float4 k[TAKES][NC], v[TAKES][NC];
#pragma unroll
        for (int u = 0; u < TAKES; ++u) {                    // what is past the end repeats the last four, or the last key, and is
            const int f = min(tile + u * WAVES + wave, fours - 1);   // not admitted
            const bool tree = f >= cache_fours;              // (uniform, like everything but the lane's row and dims)
            const int j0 = 4 * (tree ? f - cache_fours : f), last = (tree ? n : L) - 1 - j0;
            const long stride = tree ? tree_stride : kv_token_stride;
            const long at = (tree ? tree_at : cache_at) + j0 * stride;
            const long off = min(row, last) * stride;
            const float* kr = (tree ? Kt : Kc) + at;
            const float* vr = (tree ? Vt : Vc) + at;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                k[u][c] = load4(kr + off + dims[c]);
                v[u][c] = load4(vr + off + dims[c]);
            }
        }
        float4 q[NC];                                        // (here, and not ahead of the loop, whose entry would wait for it)
#pragma unroll
        for (int c = 0; c < NC; ++c) q[c] = load4(Q + q_at + dims[c]);
        __builtin_amdgcn_sched_barrier(0);                   // every load is out before the first one is used
        // scores: every lane of a row has all of the row's; lane u keeps the one of take u
        float mine = -INFINITY;
        const int lane16 = tid & 15;
#pragma unroll
        for (int u = 0; u < TAKES; ++u) {
            float a = 0.f;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const bool whole = NC == 1 ? dim0 < d : 64 * c + dim0 < d;
                float t = fmaf(q[c].x, k[u][c].x, a);
                t = fmaf(q[c].y, k[u][c].y, t);
                t = fmaf(q[c].z, k[u][c].z, t);
                t = fmaf(q[c].w, k[u][c].w, t);
                a = whole ? t : a;
            }
            a = row_sum(a);
            mine = lane16 == u ? a * scale : mine;
        }
        const int f = tile + lane16 * WAVES + wave, j = 4 * (f < cache_fours ? f : f - cache_fours) + row;
        const bool admitted = lane16 < TAKES && (f < cache_fours ? j < L : j < n && ((mask >> j) & 1));
        mine = admitted ? mine : -INFINITY;
        // A score that is NaN makes the row NaN; the maximum passes over it, and these four keys may be all that the wave has.
        const float m_new = __any(mine != mine) ? NAN : fmaxf(m, rows_max(row_max(mine)));
        if (m_new == -INFINITY) continue;                    // no score above -inf so far (uniform across the wave)
        const float corr = m == -INFINITY ? 0.f : expf(m - m_new);
        m = m_new;
        const float p = admitted ? expf(mine - m) : 0.f;
        l = l * corr + p;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            acc[c].x *= corr; acc[c].y *= corr; acc[c].z *= corr; acc[c].w *= corr;
        }
        // a value that has no weight does not count, whatever it is
        const bool all = __all(lane16 >= TAKES || p != 0.f);
        each([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            const float pu = row_lane<u>(p);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float4 x = v[u][c];
                if (!all && pu == 0.f) x = zero;
                acc[c].x = fmaf(pu, x.x, acc[c].x);
                acc[c].y = fmaf(pu, x.y, acc[c].y);
                acc[c].z = fmaf(pu, x.z, acc[c].z);
                acc[c].w = fmaf(pu, x.w, acc[c].w);
            }
        }, std::make_integer_sequence<int, TAKES>{});
    }
    l = row_sum(l);
    l = rows_sum(l);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const float4 sum = make_float4(rows_sum(acc[c].x), rows_sum(acc[c].y), rows_sum(acc[c].z), rows_sum(acc[c].w));
        if (row == 0) *reinterpret_cast<float4*>(&s_acc[wave][64 * c + dim0]) = sum;
    }
    if ((tid & 63) == 0) {
        s_m[wave] = m;
        s_l[wave] = l;
    }
    __syncthreads();
    if (wave * 64 >= d) return;
    float m_all = -INFINITY, l_all = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m_all = fmaxf(m_all, s_m[w]);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const float weight = s_m[w] == -INFINITY ? 0.f : expf(s_m[w] - m_all);
        l_all = fmaf(weight, s_l[w], l_all);
        o = fmaf(weight, s_acc[w][tid], o);
    }
    o /= l_all;
    // A value whose weight in the row is zero does not count, whatever it is.  A wave weighs by the maximum of its own keys, so one
    // that is infinite or NaN may have come in with a weight that other waves' keys make zero: where a result is not finite and
    // the weights are, the values are summed again, by the row's maximum.
    const bool again = tid < d && l_all > 0.f && l_all < INFINITY && !(fabsf(o) < INFINITY);
    if (__builtin_expect(__any(again), 0)) {
        float sum = 0.f;
        for (int f = 0; f < fours; ++f) {
            const bool tree = f >= cache_fours;
            const int j0 = 4 * (tree ? f - cache_fours : f), last = (tree ? n : L) - 1 - j0;
            const long stride = tree ? tree_stride : kv_token_stride;
            const long at = (tree ? tree_at : cache_at) + j0 * stride;
            const float* kr = (tree ? Kt : Kc) + at + min(row, last) * stride;
            float a = 0.f;
            for (int c = 0; c < NC; ++c) {
                const int dim = min(64 * c + dim0, d - 4);
                const float4 x = load4(Q + q_at + dim), y = load4(kr + dim);
                const float t = fmaf(x.w, y.w, fmaf(x.z, y.z, fmaf(x.y, y.y, fmaf(x.x, y.x, a))));
                a = 64 * c + dim0 < d ? t : a;
            }
            const bool admitted = row <= last && (!tree || ((mask >> (j0 + row)) & 1));
            const float p = admitted ? expf(row_sum(a) * scale - m_all) : 0.f;
            for (int r = 0; r < 4; ++r) {
                const float pr = sage::lane_value(p, 16 * r);
                if (pr != 0.f) sum = fmaf(pr, (tree ? Vt : Vc)[at + r * stride + min(tid, d - 1)], sum);
            }
        }
        if (again) o = sum / l_all;
    }
    if (tid < d) O[q_at + tid] = o;
}

}  // namespace

namespace sage {

int tree_attention_f32(const void* Q, const void* Kc, const void* Vc, const void* Kt, const void* Vt, void* O, int B,
                       int Hq, int Hkv, int d, const int64_t* kv_start, const int* kv_len, long kv_token_stride,
                       long kv_head_stride, const uint64_t* anc_mask, const int* n_nodes, const int* first_node,
                       float scale, hipStream_t stream) {
    if (d < 4 || d > 256 || (d % 4) != 0) return SAGE_UNSUPPORTED;
    if ((kv_token_stride % 4) != 0 || (kv_head_stride % 4) != 0) return SAGE_INVALID_ARG;
    if (Hq > 65535 || B > 65535) return SAGE_UNSUPPORTED;
    // Keys of a tile: 288, 128, 64.  A tile takes its time however full it is, and a longer context takes more of them; more takes a
    // tile need more registers, which leaves fewer workgroups resident.  us per call at these takes, at about twice and at half of them:
    //   64 dims    72 keys 5.3, 7.2, 4.2     264 keys 5.3, 7.2, 5.6     512 keys 7.9, 7.3, 9.2     1516 keys x 16 nodes 26.7, 16.1, 26.6
    //   128 dims  108 keys 4.6, 6.0, 4.6     527 keys 16.6, 12.8, 16.3     2064 keys x 64 nodes x 32 heads 163, 216, 171
    //   256 dims  216 keys 8.9, 9.3, 12.8   1016 keys x 16 nodes 23.1, 21.5, 31.6
    // The lines lie where contexts of a small model's checks are served best, a few hundred positions of 64 dims.
    const auto kernel = d <= 64 ? tree_attention_f32_kernel<1, 9> : d <= 128 ? tree_attention_f32_kernel<2, 4> : tree_attention_f32_kernel<4, 2>;
    hipLaunchKernelGGL(kernel, dim3(SAGE_MAX_NODES, Hq, B), dim3(THREADS), 0, stream, n_nodes, kv_len, kv_start, first_node, anc_mask, Hq,
                       Hkv, d, static_cast<const float*>(Q), static_cast<const float*>(Kc), static_cast<const float*>(Vc),
                       static_cast<const float*>(Kt), static_cast<const float*>(Vt), static_cast<float*>(O), kv_token_stride,
                       kv_head_stride, scale);
    return launch_status();
}

}  // namespace sage
