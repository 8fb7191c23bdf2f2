// sage_lm_head_topk: the target's greedy token and softmax statistics per row (Sec. 2.2 / Def. 4.1, Eq. 1) taken
// straight from the output projection, logits = hidden . weight^T, so that the rows x vocabulary logits never
// exist in memory.  The weight matrix ([vocab, dim] bf16, 2.5 GB at the 72B shape) is fetched from HBM once per call.  This
// file: up to 64 rows (one block), where that stream is the bound, and the entry point; more rows: lm_head_rows.hip.
// Rows that n_valid marks dead are left out first (the live rows of all groups are packed).  The hidden rows (1 MB per block
// of 64) are read once per workgroup from L2.
//
// A workgroup of 4 waves owns T consecutive 64-row vocabulary tiles and all hidden rows and keeps the
// logits of ALL of them in registers (T accumulators of 32 x 32 per wave; with one wave per SIMD a wave has 512
// registers).  The loop runs over chunks of 128 hidden elements on the outside and the T tiles on the inside, so a
// hidden chunk is fetched once and its MFMA operands stay in registers for T steps, while the weight tiles (64 rows x
// 256 B) stream from global memory straight into LDS through a ring of 8 stages, all but one of
// them ahead of the MFMAs, in the same padded layout as the attention kernel's K tiles (conflict-free 16-byte reads
// with compile-time offsets).  Wave (vt, rt) accumulates logits^T[32 vocabulary rows of half vt][32 hidden rows of
// half rt] with v_mfma_f32_32x32x16_bf16 (A = weight rows, B = hidden rows, both as stored), so a lane
// owns one hidden row and 16 vocabulary entries of it per tile.  After the last chunk every lane folds its
// 16 T logits into statistics of its row (maximum m, Z = sum exp(x - m), T = sum exp(x - m)(m - x), best (value,
// index) key); the four partial statistics of a row are combined through LDS and written as one "slice" per
// (row, unit), in the format of the stored-logits first pass, whose second pass finishes the row.
//
// The launch has at most one workgroup per CU (a workgroup fills a CU's LDS); each stays resident and walks the units id,
// id + grid, ...
#include <type_traits>

#include "lm_head_device.h"
#include "sage_internal.h"
#include "topk_device.h"

using namespace sage::topk;

namespace sage {
int lm_head_rows_units(int vocab, int rows);
int lm_head_rows_slots(int vocab, int rows);
int launch_lm_head_rows(const void*, const void*, int, int, int, long, long, const int*, int, UnitStats*, uint64_t*, int*, hipStream_t);
}  // namespace sage

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_byte;
#define LDS_AS __attribute__((address_space(3)))

constexpr int TILE_V = 64;               // vocabulary rows per tile
constexpr int TILE_R = 64;               // hidden rows per launch block
constexpr int CHUNK = 128;               // hidden elements per stage
constexpr int ROW_B = CHUNK * 2;         // bytes of one row of a stage
constexpr int THREADS = 256;
constexpr int MAX_K = 16;                // largest candidate list per row
constexpr int MAX_VOCAB = 655360;        // 1024 units of 10 tiles
constexpr int CUS = 256;                 // compute units of the MI355X: workgroups of a launch that stay resident
constexpr int STAGES = 8;                // weight ring: all but one stage in flight per workgroup
// stage layout: row t at (t % 16) * GROUP + (t / 16) * ROW_B; a group is the 1 KB one wave-level LDS-direct load
// writes (rows t, t+16, t+32, t+48) plus 16 bytes, which staggers consecutive rows across the banks
constexpr int GROUP = 4 * ROW_B + 16;
constexpr int STAGE_B = 16 * GROUP;
constexpr int LOADS_PER_TILE = TILE_V * ROW_B / (THREADS * 16);       // 16-byte loads per thread and tile

struct Params {
    const unsigned char* hidden; const unsigned char* weight;
    long hidden_stride_b, weight_stride_b;
    int rows, dim, vocab, k, nunits, ntiles;
    const int* n_valid; int rows_per_group;
    UnitStats* stats; uint64_t* keys;    // [rows][nunits]
};

template <int N> __device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// wait until at most `tiles` tiles' worth of this thread's loads are outstanding (0..7)
__device__ __forceinline__ void wait_vm_tiles(int tiles) {
    switch (tiles) {
        case 0: wait_vm<0>(); break;
        case 1: wait_vm<1 * LOADS_PER_TILE>(); break;
        case 2: wait_vm<2 * LOADS_PER_TILE>(); break;
        case 3: wait_vm<3 * LOADS_PER_TILE>(); break;
        case 4: wait_vm<4 * LOADS_PER_TILE>(); break;
        case 5: wait_vm<5 * LOADS_PER_TILE>(); break;
        case 6: wait_vm<6 * LOADS_PER_TILE>(); break;
        default: wait_vm<7 * LOADS_PER_TILE>(); break;
    }
}
// bare barrier with wavefront-scope fences (a workgroup-scope release would wait for every load in flight)
__device__ __forceinline__ void stage_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// TOPK: k candidates per (row, unit) instead of one (the draft side of Sec. 3.1, whose rows are few), after the fold, at the
// end of every workgroup's only unit, when no loads are in flight.  Two ways, by the number of live rows and k:
//   counting: the unit's logits of 32 rows at a time are laid out in the idle ring and a wave per row finds a value that at
//     least k and at most 64 of them reach (the lanes' largest ones give it, a ballot a bit, and rarely too low; a ballot per 64
//     logits and bit, about nine bits, took twice as long), then ranks those by counting, four rows side by side: 0.45 to 0.5 us a live
//     row (T = 10; before 1.0), 0.45 (T = 5), whatever k.  16 rows of 3584, k = 10, T = 10, whole call: 217.2 -> 209.8 us
//     (184.5 since the weights are read past the memory-side cache);
//   rounds: every lane scans its 16 T logits for the best one after the previous winner, the four lanes of a row are combined
//     (lane halves by a swap, vocabulary halves through LDS): 3.1 us each (T = 5: 1.6), whatever the rows.
// LIST_ROWS_PER_K live rows per candidate is about where the two meet (us of the call, counting / rounds; vocabulary 152064, hidden
// 1024, T = 10, at 4, 5 and 6 rows per k: k = 4 74.7 / 79.7, 76.8 / 79.9, 78.4 / 79.5; k = 6 78.9 / 85.6, 82.5 / 85.8, 87.8 / 85.8; k = 8
// 83.1 / 91.4, 90.1 / 91.9, 93.7 / 92.1; k = 12 95.9 / 104.2 and 101.5 / 104.4; 64 rows k = 16 104 / 115.  Vocabulary 32000, hidden 3584,
// T = 5, just below 4 and at 5: k = 4 72.7 / 74.3, 74.2 / 74.3; k = 8 79.0 / 80.3, 83.9 / 80.4; k = 12 88.5 / 86.9 and k = 16 96.0 / 92.9).
// So the rule loses up to 3.4 us (k = 6, 30 rows, T = 10) or 3.1 (k = 16, 63 rows, T = 5) next to the line, and nothing away from it.
template <int T, bool TOPK, bool ONCE>
__global__ __launch_bounds__(THREADS) void lm_head_kernel(const Params prm) {
    // The ring position of a step must be a compile-time constant (every stage is its own LDS object, so that loads
    // in flight into one stage are known not to alias reads of another): step t of chunk kc uses stage
    // (kc T + t) mod STAGES, which is static once the chunk loop is unrolled UNROLL times.
    constexpr int AHEAD = STAGES - 1;
    constexpr int UNROLL = (T % 8 == 0) ? 1 : (T % 4 == 0) ? 2 : (T % 2 == 0) ? 4 : 8;
    static_assert((UNROLL * T) % STAGES == 0, "ring positions must be static");
    constexpr int ROWS = TILE_R;                             // hidden rows of this workgroup
    constexpr int LIST_ROWS_PER_K = T > 5 ? 5 : 4;           // candidate lists: see above
    __shared__ __align__(16) unsigned char sW0[STAGE_B];
    __shared__ __align__(16) unsigned char sW1[STAGE_B];
    __shared__ __align__(16) unsigned char sW2[STAGE_B];
    __shared__ __align__(16) unsigned char sW3[STAGE_B];
    __shared__ __align__(16) unsigned char sW4[STAGE_B];
    __shared__ __align__(16) unsigned char sW5[STAGE_B];
    __shared__ __align__(16) unsigned char sW6[STAGE_B];
    __shared__ __align__(16) unsigned char sW7[STAGE_B];
    __shared__ __align__(16) unsigned char sH0[STAGE_B];    // the current hidden chunk (read into registers in step 0)
    __shared__ float s_part[ROWS][4][3];                     // per hidden row: 4 partial (m, Z, T)
    __shared__ uint64_t s_key[ROWS][4];
    __shared__ int s_row[ROWS];                              // hidden row behind each of this block's slots, -1 = none
    __shared__ int s_cnt[THREADS];
    __shared__ __align__(16) uint64_t s_cand[TOPK ? THREADS / 64 : 1][TOPK ? 64 : 1];   // candidate lists: what a wave ranks
    __shared__ uint64_t s_sel[TOPK ? 2 : 1][TOPK ? TILE_R : 1][2];   // candidate rounds: a row's winner per vocabulary half
#define SW(i) ((i) == 0 ? sW0 : (i) == 1 ? sW1 : (i) == 2 ? sW2 : (i) == 3 ? sW3 : (i) == 4 ? sW4 : (i) == 5 ? sW5 : (i) == 6 ? sW6 : sW7)

    const int tid = threadIdx.x;
    // ---- the rows: slot j is live row number j, counted over the groups in order.  Fills s_row and returns how many
    // are live (the same in every thread).
    auto map_rows = [&]() __attribute__((always_inline)) {
        int live = prm.rows;
        if (prm.n_valid == nullptr) {
            if (tid < ROWS) s_row[tid] = tid < prm.rows ? tid : -1;
        } else {
            const int groups = (prm.rows + prm.rows_per_group - 1) / prm.rows_per_group;   // (at most 64: a row each)
            int before = 0, found = -1;
            s_cnt[tid] = tid < groups ? max(0, min(prm.n_valid[tid], min(prm.rows_per_group, prm.rows - tid * prm.rows_per_group))) : 0;
            __syncthreads();
            for (int j = 0; j < groups; ++j) {
                const int c = s_cnt[j];
                if (found < 0 && tid < before + c) found = j * prm.rows_per_group + (tid - before);
                before += c;
            }
            if (tid < ROWS) s_row[tid] = found;
            live = before;
        }
        __syncthreads();
        return live;
    };
    const int live = __builtin_amdgcn_readfirstlane(map_rows());
    if (live <= 0) return;
    // candidate lists: the codes of one hidden row (of 32) lie in the ring, CODE_ROWS rows per stage; the four words between
    // rows put the 16-byte writes of 16 consecutive rows on all 64 banks once
    constexpr int CODE_PITCH = T * TILE_V + 4, CODE_ROWS = 6;
    static_assert(CODE_ROWS * CODE_PITCH * 4 <= STAGE_B && 6 * CODE_ROWS >= 32, "32 rows of codes fit six stages");
    auto code_row = [&](int q) __attribute__((always_inline)) {
        const int st = q / CODE_ROWS;
        LDS_AS unsigned char* const base = (LDS_AS unsigned char*)(SW(st));
        return (LDS_AS uint32_t*)base + (q - st * CODE_ROWS) * CODE_PITCH;
    };
    for (int unit = blockIdx.x; unit < prm.nunits; unit += gridDim.x) {
    // (the thread index is made opaque per unit: the compiler would otherwise hoist everything that depends on the index alone
    // out of this loop, which seldom runs twice, and keep it alive across the main loop)
    int tid = static_cast<int>(threadIdx.x);
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, half = lane >> 5;
    const int vt = wave & 1, rt = wave >> 1;
    // this unit's tiles: an even share of the vocabulary, at most T; missing ones are phantom steps that re-read one
    // row (an L2 hit) and whose logits are masked, so that every unit runs the same step sequence
    const int tile_begin = static_cast<int>(static_cast<long>(unit) * prm.ntiles / prm.nunits);
    const int tile_end = static_cast<int>(static_cast<long>(unit + 1) * prm.ntiles / prm.nunits);
    const int v_end = min(prm.vocab, tile_end * TILE_V);     // one past this unit's last vocabulary row
    const int nchunk = prm.dim / CHUNK;
    const int nsteps = nchunk * T;

    // ---- loader: instruction i of wave w copies rows r, r+16, r+32, r+48 (r = 4w + i) of a 64-row tile: lane l fills
    // chunk l%16 of row r + 16 (l/16).  Vocabulary rows past the end (the last unit's missing tiles, a partial last
    // tile) re-read the last valid row; their results are masked.
    const int ld_row = (lane >> 4) * 16 + wave * 4;
    const unsigned ld_chunk_b = (lane & 15) * 16;
    // (a slot without a row re-reads the block's first row)
    const unsigned char* w_base = prm.weight + static_cast<long>(tile_begin) * TILE_V * prm.weight_stride_b;
    const int rows_mine = v_end - tile_begin * TILE_V;       // vocabulary rows of this unit (>= 1)
    const int full_tiles = rows_mine / TILE_V;               // tiles that need no clamping
    // per-lane pointers into the first tile / first chunk; a step adds one wave-uniform offset to them.  (The offset is
    // made opaque to the compiler, which would otherwise keep a separate address pair per tile and load alive across
    // the whole loop: 8 registers instead of 8 T.)
    const unsigned char* w_ptr[4];
    const unsigned char* h_ptr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w_ptr[i] = w_base + static_cast<long>(ld_row + i) * prm.weight_stride_b + ld_chunk_b;
        const int hr = s_row[ld_row + i] >= 0 ? s_row[ld_row + i] : s_row[0];
        h_ptr[i] = prm.hidden + static_cast<long>(hr) * prm.hidden_stride_b + ld_chunk_b;
    }

    auto issue_w = [&](int kc, int t, auto stc) __attribute__((always_inline)) {
        constexpr int ST = decltype(stc)::value;
        LDS_AS unsigned char* dst = (LDS_AS unsigned char*)(&SW(ST)[wave * 4 * GROUP]);
        if (t < full_tiles) {
            long off = static_cast<long>(t) * TILE_V * prm.weight_stride_b + static_cast<long>(kc) * ROW_B;
            asm volatile("" : "+s"(off));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (ONCE) sage::lds_direct_load16_once(w_ptr[i] + off, dst + i * GROUP);
                else sage::lds_direct_load16(w_ptr[i] + off, dst + i * GROUP);
            }
        } else {
            const unsigned char* wb = w_base + static_cast<long>(kc) * ROW_B;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long r = min(t * TILE_V + ld_row + i, rows_mine - 1);
                sage::lds_direct_load16(reinterpret_cast<const unsigned char*>(wb + r * prm.weight_stride_b + ld_chunk_b), dst + i * GROUP);
            }
        }
    };
    auto issue_h = [&](int kc) __attribute__((always_inline)) {
        long off = static_cast<long>(kc) * ROW_B;
        asm volatile("" : "+s"(off));
        LDS_AS unsigned char* dst = (LDS_AS unsigned char*)(&sH0[wave * 4 * GROUP]);
#pragma unroll
        for (int i = 0; i < 4; ++i) sage::lds_direct_load16(reinterpret_cast<const unsigned char*>(h_ptr[i] + off), dst + i * GROUP);
    };

    // ---- per-lane read offsets: fragment kk of row r32 of this wave's half: chunk 2kk + half
    const int w_lane = (r32 & 15) * GROUP + (2 * vt + (r32 >> 4)) * ROW_B + half * 16;
    const int h_lane = (r32 & 15) * GROUP + (2 * rt + (r32 >> 4)) * ROW_B + half * 16;

    f32x16 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    bf16x8 hb_frag[8];                                       // this wave's hidden rows of the current chunk (B operands)

    // one hidden chunk: T steps; J = kc mod UNROLL fixes the ring positions
    auto chunk = [&](int kc, auto jc) __attribute__((always_inline)) {
        constexpr int J = decltype(jc)::value;
        auto step = [&](auto tc) __attribute__((always_inline)) {
            constexpr int t = decltype(tc)::value;
            constexpr int ST = (J * T + t) % STAGES;
            const int s = kc * T + t;
            // This thread's loads of step s have landed; younger ones may stay in flight (the counter retires loads in
            // order): the weight tiles of the next AHEAD - 1 steps and, during steps 2..AHEAD of a chunk, the next
            // hidden chunk, requested in step 1.  Step 0 also needs the hidden chunk itself, which only the weight
            // tiles requested after it (steps 2..T-1 of the previous chunk) are younger than.
            int younger = min(AHEAD - 1, nsteps - 1 - s);
            if (t >= 2 && t <= AHEAD && kc + 1 < nchunk) younger += 1;   // (a hidden chunk is a tile's worth of loads)
            if (t == 0 && kc > 0) younger = min(younger, max(0, min(T - 2, nsteps - AHEAD - ((kc - 1) * T + 2))));
            wait_vm_tiles(younger);
            stage_barrier();                                 // ... for every wave, and the stage read last step is free
            if (s + AHEAD < nsteps) {
                constexpr int ta = (t + AHEAD) % T;
                issue_w(kc + (t + AHEAD) / T, ta, std::integral_constant<int, (ST + AHEAD) % STAGES>{});
            }
            if (t == 1 && kc + 1 < nchunk) issue_h(kc + 1);  // every wave has taken its fragments of chunk kc in step 0
            if (t == 0) {
                const lds_byte* hst = (const lds_byte*)sH0 + h_lane;
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) hb_frag[kk] = __builtin_bit_cast(bf16x8, *(const LDS_AS uint4*)(hst + kk * 32));
            }
            const lds_byte* wst = (const lds_byte*)(SW(ST)) + w_lane;
            bf16x8 a[8];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) a[kk] = __builtin_bit_cast(bf16x8, *(const LDS_AS uint4*)(wst + kk * 32));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], hb_frag[kk], acc[t], 0, 0, 0);
        };
        [&]<int... Is>(std::integer_sequence<int, Is...>) __attribute__((always_inline)) {
            (step(std::integral_constant<int, Is>{}), ...);
        }(std::make_integer_sequence<int, T>{});
    };

    static_assert(T >= 2 && AHEAD + 1 <= 8, "prologue below issues the first AHEAD steps; waits count up to seven tiles");
    issue_h(0);
    [&]<int... Is>(std::integer_sequence<int, Is...>) __attribute__((always_inline)) {
        ((Is < nsteps ? issue_w(Is / T, Is % T, std::integral_constant<int, Is % STAGES>{}) : (void)0), ...);
    }(std::make_integer_sequence<int, AHEAD>{});
    for (int kc = 0; kc < nchunk; kc += UNROLL) {
        [&]<int... Js>(std::integer_sequence<int, Js...>) __attribute__((always_inline)) {
            ((kc + Js < nchunk ? chunk(kc + Js, std::integral_constant<int, Js>{}) : (void)0), ...);
        }(std::make_integer_sequence<int, UNROLL>{});
    }

    // ---- fold the logits into softmax statistics and the best candidate of this lane's hidden row, and park the four partial
    // statistics of every hidden row (two lane halves x two vocabulary halves) in LDS
    {
        const int v0 = tile_begin * TILE_V + 32 * vt + 4 * half;
        const sage::lmhead::Fold f = sage::lmhead::fold_logits<T>(v0, TILE_V, v_end, [&](int t, int i, int left) __attribute__((always_inline)) {
            return 8 * (i >> 2) + (i & 3) < left ? acc[t][i] : -INFINITY;
        });
        const int hr = rt * 32 + r32;
        s_part[hr][vt * 2 + half][0] = f.m;
        s_part[hr][vt * 2 + half][1] = f.Z;
        s_part[hr][vt * 2 + half][2] = f.T;
        s_key[hr][vt * 2 + half] = f.key;
    }
    __syncthreads();
    if (tid < ROWS && s_row[tid] >= 0) {
        const long o = static_cast<long>(s_row[tid]) * prm.nunits + unit;
        sage::lmhead::combine_folds(&s_part[tid][0][0], s_key[tid], prm.stats + o, TOPK ? nullptr : prm.keys + o);
    }
    if constexpr (TOPK) {
        if (live >= LIST_ROWS_PER_K * prm.k) {               // (uniform) rounds
            // (made opaque, or what depends on the thread index alone would be kept alive across the main loop)
            int lane = threadIdx.x & 63;
            asm volatile("" : "+v"(lane));
            const int half = lane >> 5;
            const int hr = rt * 32 + (lane & 31);
            const int row = s_row[hr];
            // the statistics are done: the logits give way, in place, to their order-preserving codes (0 = not a candidate: past
            // the unit's end, or -inf), so that a round costs one 64-bit compare pair per logit
#pragma unroll
            for (int t = 0; t < T; ++t) {
                int left = v_end - ((tile_begin + t) * TILE_V + 32 * vt + 4 * half);
                asm volatile("" : "+v"(left));               // (or the fold's comparison masks would be kept for this loop)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float x = acc[t][i];
                    acc[t][i] = __uint_as_float((8 * (i >> 2) + (i & 3) < left && x > -INFINITY) ? sortable(x) : 0u);
                }
            }
            uint64_t prev = ~0ull;                           // the previous winner: candidates come after it in the order
            for (int j = 0; j < prm.k; ++j) {
                uint64_t best = 0xFFFFFFFFull;               // (code 0, lowest index word): below every candidate
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    uint32_t lo0 = 0xFFFFFFFFu - static_cast<uint32_t>((tile_begin + t) * TILE_V + 32 * vt + 4 * half);
                    asm volatile("" : "+v"(lo0));            // (or 16 T index words would be kept for all rounds)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const uint64_t key = (static_cast<uint64_t>(__float_as_uint(acc[t][i])) << 32) | (lo0 - (8 * (i >> 2) + (i & 3)));
                        best = (key < prev && key > best) ? key : best;
                    }
                }
                Key mine = (best >> 32) == 0 ? Key{0, 0} : key_unpack(best);
                {                                            // the other lane half of this row
                    const auto hi = __builtin_amdgcn_permlane32_swap(mine.hi, mine.hi, false, false);
                    const auto lo = __builtin_amdgcn_permlane32_swap(mine.lo, mine.lo, false, false);
                    mine = key_max(Key{hi[0], lo[0]}, Key{hi[1], lo[1]});
                }
                if (half == 0) s_sel[j & 1][hr][vt] = key_pack(mine);
                __syncthreads();                             // (rounds alternate between two buffers: one barrier per round)
                const Key w = key_max(key_unpack(s_sel[j & 1][hr][0]), key_unpack(s_sel[j & 1][hr][1]));
                if (vt == 0 && half == 0 && row >= 0)
                    prm.keys[(static_cast<long>(row) * prm.nunits + unit) * prm.k + j] = key_pack(w);
                prev = key_none(w) ? 0ull : key_pack(w);     // an exhausted unit: nothing comes after
            }
        } else {
            // The statistics are done: the logits' order-preserving codes (0 = not a candidate: past the unit's end, or -inf) of 32
            // hidden rows go into the idle ring, row by row in vocabulary order, and a wave selects from one row at a time.
#pragma unroll 1
            for (int batch = 0; batch < TILE_R / 32; ++batch) {
                if (s_row[batch * 32] < 0) break;                // (live rows come first)
                // (made opaque, or what depends on the thread index alone would be kept alive across the main loop)
                int lane = threadIdx.x & 63;
                asm volatile("" : "+v"(lane));
                if (rt == batch) {
                    const int half = lane >> 5;
                    LDS_AS uint32_t* const mine = code_row(lane & 31) + 32 * vt + 4 * half;
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        int left = v_end - ((tile_begin + t) * TILE_V + 32 * vt + 4 * half);
                        asm volatile("" : "+v"(left));           // (or the fold's comparison masks would be kept for this loop)
#pragma unroll
                        for (int i0 = 0; i0 < 16; i0 += 4) {
                            uint32_t code[4];
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const float x = acc[t][i0 + i];
                                code[i] = (2 * i0 + i < left && x > -INFINITY) ? sortable(x) : 0u;
                            }
                            *(LDS_AS u32x4*)(mine + t * TILE_V + 2 * i0) = u32x4{code[0], code[1], code[2], code[3]};
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __syncthreads();
#pragma unroll 1
                for (int q = wave; q < 32; q += THREADS / 64) {
                    const int row = __builtin_amdgcn_readfirstlane(s_row[batch * 32 + q]);
                    if (row < 0) break;
                    const LDS_AS uint32_t* const codes = code_row(q);
                    uint32_t code[T];
                    bool have[T], in[T];
                    int present = 0;
#pragma unroll
                    for (int i = 0; i < T; ++i) code[i] = codes[i * 64 + lane];
#pragma unroll
                    for (int i = 0; i < T; ++i) {
                        have[i] = code[i] != 0;
                        present += __builtin_popcountll(__ballot(have[i]));
                    }
                    // at least k candidates and no more than a lane can take each; of equal values the lowest indices
                    wave_pick_roughly<T>(code, have, min(prm.k, present), 64, in);
                    int n = 0;
#pragma unroll
                    for (int i = 0; i < T; ++i) {
                        const uint64_t b = __ballot(in[i]);
                        if (in[i])
                            s_cand[wave][n + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(b >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(b), 0u)))] =
                                key_pack(Key{code[i], 0xFFFFFFFFu - static_cast<uint32_t>(tile_begin * TILE_V + i * 64 + lane)});
                        n += __builtin_popcountll(b);
                    }
                    if (lane >= n && lane < ((n + 15) & ~15)) s_cand[wave][lane] = 0;   // whole pieces of 16 to count in
                    // (a wave's LDS operations complete in order; the fence keeps the compiler from reading ahead of the writes)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    uint64_t* const out = prm.keys + (static_cast<long>(row) * prm.nunits + unit) * prm.k;
                    const uint64_t key = lane < n ? s_cand[wave][lane] : 0;
                    const int above = count_above(s_cand[wave], (n + 15) & ~15, key);
                    if (lane < n && above < prm.k) out[above] = key;
                    if (lane >= n && lane < prm.k) out[lane] = 0;   // fewer candidates than k
                }
                __syncthreads();                                 // the next batch's codes go over these
            }
        }
    }
    __syncthreads();                                         // the next unit rewrites s_part
    }   // units
#undef SW
}

inline size_t align256(size_t b) { return (b + 255) & ~static_cast<size_t>(255); }

// Launch shape for up to 64 rows: T <= 10 accumulators per wave (more do not fit the register file without spills), T = 5 or
// 10 tiles per workgroup and about one workgroup per CU, each with an even share of the tiles; a vocabulary too large for
// that takes more units (several rounds).
struct Shape { int nunits, tiles_per_unit, ntiles; };
inline Shape launch_shape(int vocab) {
    Shape sh;
    sh.ntiles = (vocab + TILE_V - 1) / TILE_V;
    sh.tiles_per_unit = sh.ntiles <= 5 * 256 ? 5 : 10;
    const int need = (sh.ntiles + sh.tiles_per_unit - 1) / sh.tiles_per_unit;
    sh.nunits = need > 256 ? need : (sh.ntiles < 256 ? sh.ntiles : 256);
    return sh;
}
// slices ("units") that a row has room for, whichever kernel fills them; never fewer than for a smaller number of rows, so that
// a workspace for the largest batch does for every batch
inline int slices_of(int vocab, int rows) { return rows > TILE_R ? sage::lm_head_rows_slots(vocab, rows) : launch_shape(vocab).nunits; }

}  // namespace

extern "C" size_t sage_lm_head_topk_workspace_bytes(int rows, int vocab, int k) {
    if (rows < 0 || vocab < 1 || k < 1) return 0;
    const int n = slices_of(vocab, rows);
    return align256(static_cast<size_t>(rows) * n * sizeof(UnitStats)) + static_cast<size_t>(rows) * n * k * sizeof(uint64_t) + 256;
}

extern "C" int sage_lm_head_topk(const void* hidden, const void* weight, int dtype, int rows, int dim, int vocab,
                                 long hidden_stride, long weight_stride, int k, const int* n_valid, int rows_per_group,
                                 float* entropy, int* topk_idx, float* topk_prob, float* topk_renorm,
                                 float* topk_entropy, float* alpha, void* workspace, size_t workspace_bytes, void* stream) {
    if (!hidden || !weight || !topk_idx || !workspace) return SAGE_INVALID_ARG;
    if (rows < 0 || dim < 1 || vocab < 1 || k < 1 || hidden_stride < dim || weight_stride < dim) return SAGE_INVALID_ARG;
    if (dtype != SAGE_F32 && dtype != SAGE_BF16) return SAGE_INVALID_ARG;
    if (n_valid && rows_per_group < 1) return SAGE_INVALID_ARG;
    if (k > SAGE_MAX_TOPK || k > vocab) return SAGE_INVALID_ARG;
    if (dtype != SAGE_BF16 || dim % CHUNK != 0) return SAGE_UNSUPPORTED;
    if (k > MAX_K || (k > 1 && rows > TILE_R)) return SAGE_UNSUPPORTED;   // candidate lists: the draft side, few rows
    if ((hidden_stride % 8) != 0 || (weight_stride % 8) != 0 || !sage::aligned(hidden, 16) || !sage::aligned(weight, 16) ||
        !sage::aligned(workspace, 16))
        return SAGE_INVALID_ARG;
    if (weight_stride > (1L << 24) || hidden_stride > (1L << 24)) return SAGE_UNSUPPORTED;
    if (rows > (1 << 20)) return SAGE_UNSUPPORTED;                                            // grid size
    if (workspace_bytes < sage_lm_head_topk_workspace_bytes(rows, vocab, k)) return SAGE_WORKSPACE_TOO_SMALL;
    if (rows == 0) return SAGE_OK;
    int nunits = slices_of(vocab, rows);
    // (one limit for every number of rows; the second pass takes what either kernel cuts such a vocabulary into)
    if (vocab > MAX_VOCAB || nunits > sage::topk_merge_max_units(k)) return SAGE_UNSUPPORTED;
    UnitStats* stats = static_cast<UnitStats*>(workspace);
    uint64_t* keys = reinterpret_cast<uint64_t*>(static_cast<char*>(workspace) +
                                                 align256(static_cast<size_t>(rows) * nunits * sizeof(UnitStats)));
    int* units_used = nullptr;
    hipStream_t s = sage::as_stream(stream);
    if (rows > TILE_R) {
        // with n_valid there are one of two numbers of slices, and the device says which behind the keys, in the last 256
        // bytes of the size; without, or when the two are the same, it is known here
        if (n_valid && sage::lm_head_rows_units(vocab, 1) != sage::lm_head_rows_units(vocab, rows))
            units_used = reinterpret_cast<int*>(keys + static_cast<size_t>(rows) * nunits * k);
        else
            nunits = sage::lm_head_rows_units(vocab, rows);
        const int rc = sage::launch_lm_head_rows(hidden, weight, rows, dim, vocab, hidden_stride, weight_stride, n_valid, rows_per_group,
                                                 stats, keys, units_used, s);
        if (rc != SAGE_OK) return rc;
    } else {
        const Shape sh = launch_shape(vocab);
        Params p;
        p.hidden = static_cast<const unsigned char*>(hidden);
        p.weight = static_cast<const unsigned char*>(weight);
        p.hidden_stride_b = hidden_stride * 2;
        p.weight_stride_b = weight_stride * 2;
        p.rows = rows; p.dim = dim; p.vocab = vocab; p.k = k; p.nunits = nunits; p.ntiles = sh.ntiles;
        p.n_valid = n_valid; p.rows_per_group = rows_per_group;
        p.stats = stats; p.keys = keys;
        const dim3 grid(nunits < CUS ? nunits : CUS);        // a workgroup fills a CU's LDS: one resident workgroup per CU
        auto launch = [&](auto once) {
            constexpr bool ONCE = decltype(once)::value;
            const auto kernel = k > 1 ? (sh.tiles_per_unit == 5 ? lm_head_kernel<5, true, ONCE> : lm_head_kernel<10, true, ONCE>)
                                      : (sh.tiles_per_unit == 5 ? lm_head_kernel<5, false, ONCE> : lm_head_kernel<10, false, ONCE>);
            hipLaunchKernelGGL(kernel, grid, dim3(THREADS), 0, s, p);
        };
        if (sage::lmhead::read_once(vocab, dim)) launch(std::true_type{});
        else launch(std::false_type{});
        if (hipGetLastError() != hipSuccess) return SAGE_LAUNCH_FAILED;
    }
    sage::topk_merge(rows, k, n_valid, rows_per_group, nunits, stats, keys, entropy, topk_idx, topk_prob, topk_renorm,
                     topk_entropy, alpha, s, units_used);
    return sage::launch_status();
}
