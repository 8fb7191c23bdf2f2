// sage_lm_head_topk for more than 64 rows (the node rows of a batch of trees; Sec. 2.2 / Def. 4.1, Eq. 1): greedy token and
// softmax statistics per row of hidden . weight^T, the logits kept in registers.
//
// What bounds it: with 512 live rows the contraction (512 flops per weight byte against a ridge of about 260 at the rates
// this chip reaches), with up to about 128 the stream of the weight matrix.  Between the two stands the rate at which a CU
// can pull operands in through L2, so a workgroup's tile is as square as the register file allows: up to 256 vocabulary
// rows x 256 hidden rows on 4 waves, one per SIMD with all 512 registers, each wave 128 x 128 as 4 x 4 accumulators of
// v_mfma_f32_32x32x16_bf16 (A = weight rows, B = hidden rows, both as stored).  A step covers 64 elements of the hidden
// dimension: 64 KB of operands for 8.4 MFLOP, against 92 KB for a tile of 128 rows x 320 (the layout this one replaced).
//
// Data movement.  Operands go from global memory straight into LDS (16-byte LDS-direct loads, 8 rows x 128 bytes per
// wave-level load) through two rings, of WR weight stages and of HR hidden stages.  Weights are requested WR - 1 steps ahead,
// into the stage that the step before has left, hidden rows HR steps ahead, into the stage that the step itself leaves.  Both
// rings have as many stages as fit, up to eight; with a unit and block of NV + NR >= 7 only WR = 3 and HR = 2 fit (the
// weights come from HBM, the hidden rows from L2).  The counted waits follow from these numbers.  A row of a stage is 128
// bytes; its 16-byte chunk c sits at position c ^ ((row / 2) % 8), which a loading lane achieves by fetching another chunk
// of its row, and which makes the 16-byte fragment reads of 16 consecutive rows hit all 64 banks once.
// The fragments of a 16-element block are read while the MFMAs of the block before it run, so a wave that has its SIMD
// to itself never waits for LDS; the one barrier of a step comes before the step's last block of MFMAs, whose fragments
// are in registers by then.  No load returns into a register: all waits on the vector-memory counter are counted ones
// (and the kernel must not spill; the build checks that).
//
// Decomposition.  The vocabulary is cut into `ranges` (one per workgroup that a row block leaves: 256 CUs / row blocks), a
// range into units of up to 4 tiles of 64 vocabulary rows, as even as can be; units are numbered first units of all ranges
// first, so that the workgroups go through units of one size at a time and the chip finishes together (152064 x 512 rows:
// 18-19 tiles per pair of CUs = 5 units of 3 or 4, 4.75 rounds of work in place of the 5 that equal units of 4 would
// need).  Only blocks of live rows are items; a block is 64, 128, 192 or 256 rows deep.  Row blocks of one unit are
// consecutive items of one XCD and share the unit's weights through that XCD's L2 as far as they stay together (1.21 fetches
// of the matrix at 512 rows).  Up to 128 live rows the weight stream is the bound, and what counts is that every CU has the same
// share of it: the cut for one block, three units of at most 4 tiles on each of 256 CUs (152064 tokens), whatever the number of
// rows; cut for the blocks of 1024 rows, 64 live ones take 459 us instead of 446, 128 of 512 470 instead of 456 (before READ_ONCE_BYTES).  With more
// live rows the larger units of the rows' own cut are as good or better (256 of 512: 622 us, 645 with the cut for one block).
//
// Measured (hidden 8192, vocabulary 152064; before = 4 waves on 320 vocabulary rows x 128 hidden rows): 512 live rows
// 1690 -> 1045 us (1.22 PFLOP/s), 256 live 880 -> 620, 160 live 920 -> 500, 128 live 505 -> 453, 1024 live 3140 -> 1975; 64 live
// of 512 443 -> 442; since then calls of one block with weights past the memory-side cache, 64 live rows 431 -> 397, 160 535 -> 516,
// 240 (hidden 5120) 426 -> 413 (see READ_ONCE_BYTES).  At 512 rows the matrix pipe is busy 74 % of the cycles and the chip clocks down to 1.48 GHz (2.19 in the
// 64-row call): what is left is power, so bytes moved per flop are what counts.
#include <type_traits>

#include "lm_head_device.h"
#include "sage_internal.h"

using namespace sage::topk;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) unsigned char lds_byte;
#define LDS_AS __attribute__((address_space(3)))

constexpr int THREADS = 256;
constexpr int CUS = 256;                 // workgroups that stay resident: one per CU
constexpr int STRIP = 32;                // vocabulary rows of one accumulator
constexpr int TILE_V = 64;               // vocabulary rows of a tile: a strip for each of the two vocabulary waves
constexpr int MAX_TILES = 4;             // tiles of a unit
constexpr int BLOCK_ROWS = 256;          // hidden rows of a full block
constexpr int STEP_B = 128;              // bytes of one row per step (64 elements)
constexpr int FEW_LIVE = 128;            // up to so many live rows of any number: the vocabulary is cut as for one block
constexpr int LDS_B = 160 * 1024;

// How the vocabulary is cut; see the top of the file.
struct Cut { int ranges, units_per_range; };

struct Params {
    const unsigned char* hidden; const unsigned char* weight;
    long hidden_stride_b, weight_stride_b;
    int rows, vocab, nsteps, ntiles;
    int read_once;                       // the weights are more than stays in memory-side cache (see lm_head_device.h)
    Cut few, all;                        // for up to FEW_LIVE live rows; for more
    const int* n_valid; int rows_per_group;
    UnitStats* stats; uint64_t* keys;    // [rows][units]
    int* units_used;                     // receives the number of units, which follows from the live rows
};

template <int N> __device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// bare barrier with wavefront-scope fences (a workgroup-scope release would wait for every load in flight)
__device__ __forceinline__ void bare_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One unit x row block: NV tiles = 2 NV strips of vocabulary rows (those at or past v_end repeat the last one and are masked) times
// 64 NR hidden rows.  s_row[0 .. 64 NR) at the start of LDS holds the hidden row behind each slot (-1 = none).
template <int NV, int NR, bool ONCE>
__device__ __forceinline__ void pass(const Params& prm, unsigned char* lds, int units, int unit, int v_begin, int v_end) {
    // Stages of the weight and of the hidden ring: as many as fit (small units would otherwise have too little in flight),
    // the same number unless only two hidden stages fit beside three weight stages.
    constexpr int FIT = LDS_B / ((NV + NR) * TILE_V * STEP_B);
    constexpr int WR = FIT > 8 ? 8 : FIT < 3 ? 3 : FIT;
    constexpr int HR = FIT > 8 ? 8 : FIT < 3 ? 2 : FIT;
    constexpr int W_STAGE = 2 * NV * STRIP * STEP_B, H_STAGE = 64 * NR * STEP_B;
    constexpr int H_BASE = WR * W_STAGE;
    static_assert(H_BASE + HR * H_STAGE <= LDS_B, "both rings fit");
    constexpr int W_LOADS = 2 * NV, H_LOADS = 2 * NR;        // loads per wave and stage
    // (the thread index is made opaque per pass: a workgroup calls this in a loop, and the compiler would hoist everything
    // that depends on the index alone, for all instantiations at once, and keep it alive)
    int tid = static_cast<int>(threadIdx.x);
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, half = lane >> 5;
    const int vw = wave & 1, rw = wave >> 1;

    const int* s_row = reinterpret_cast<const int*>(lds);
    const int my_row = tid < 64 * NR ? s_row[tid] : -1;      // the row this thread writes at the end
    // ---- loader: load i of this wave brings rows 8 g .. 8 g + 7 (g = wave * loads + i) of a stage, lane l the position l % 8
    // of row 8 g + l / 8
    const unsigned char* w_ptr[W_LOADS];
    const unsigned char* h_ptr[H_LOADS];
    const int v_rows = v_end - v_begin;
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i) {
        const int row = (wave * W_LOADS + i) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        w_ptr[i] = prm.weight + static_cast<long>(v_begin + min(row, v_rows - 1)) * prm.weight_stride_b + chunk * 16;
    }
#pragma unroll
    for (int i = 0; i < H_LOADS; ++i) {
        const int row = (wave * H_LOADS + i) * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        const int hr = s_row[row] >= 0 ? s_row[row] : s_row[0];   // (a slot without a row repeats the block's first one)
        h_ptr[i] = prm.hidden + static_cast<long>(hr) * prm.hidden_stride_b + chunk * 16;
    }
    __syncthreads();                                         // everyone has read the row map: the rings may overwrite it

    LDS_AS unsigned char* const lds3 = (LDS_AS unsigned char*)lds;
    // Load i of a stage; `next` advances the pointer to the next stage's piece afterwards.  Past the last stage the pointers
    // stay and the loads repeat it (an L2 hit, into a stage nobody reads any more), so that every step issues the same
    // number of loads, the waits are fixed counts, and the block of MFMAs around them has no branch.
    auto issue_w1 = [&](int i, unsigned stage_off, int next) __attribute__((always_inline)) {
        if constexpr (ONCE) sage::lds_direct_load16_once(w_ptr[i], lds3 + (stage_off + (wave * W_LOADS + i) * 1024));
        else sage::lds_direct_load16(w_ptr[i], lds3 + (stage_off + (wave * W_LOADS + i) * 1024));
        w_ptr[i] += next;
    };
    auto issue_h1 = [&](int i, unsigned stage_off, int next) __attribute__((always_inline)) {
        sage::lds_direct_load16(h_ptr[i], lds3 + (stage_off + (wave * H_LOADS + i) * 1024));
        h_ptr[i] += next;
    };
    const int n = prm.nsteps;                                // >= 2
    auto more = [&](int stage) __attribute__((always_inline)) { return stage + 1 < n ? STEP_B : 0; };

    // fragment (strip or row tile j, block kk): row r32 of the tile, chunk 2 kk + half
    unsigned frag[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) frag[kk] = r32 * STEP_B + (((2 * kk + half) ^ ((r32 >> 1) & 7)) * 16);

    f32x16 acc[NV][NR];
#pragma unroll
    for (int a = 0; a < NV; ++a)
#pragma unroll
        for (int b = 0; b < NR; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    // ---- prologue: what the loop would have requested before step 0, in its order
#pragma unroll
    for (int t = 0; t < WR - 1; ++t) {
        if (t < HR) {
#pragma unroll
            for (int i = 0; i < H_LOADS; ++i) issue_h1(i, H_BASE + t * H_STAGE, more(t));
        }
#pragma unroll
        for (int i = 0; i < W_LOADS; ++i) issue_w1(i, t * W_STAGE, more(t));
    }
    if (HR > WR - 1) {
#pragma unroll
        for (int i = 0; i < H_LOADS; ++i) issue_h1(i, H_BASE + (HR - 1) * H_STAGE, more(HR - 1));
    }
    wait_vm<(WR - 2) * W_LOADS + (HR - 1) * H_LOADS>();
    bare_barrier();

    bf16x8 fa[2][NV], fb[2][NR];
    auto read_a = [&](int set, int j, unsigned addr) __attribute__((always_inline)) {
        fa[set][j] = __builtin_bit_cast(bf16x8, *(const LDS_AS uint4*)(lds3 + (addr + (vw * NV + j) * STRIP * STEP_B)));
    };
    auto read_b = [&](int set, int j, unsigned addr) __attribute__((always_inline)) {
        fb[set][j] = __builtin_bit_cast(bf16x8, *(const LDS_AS uint4*)(lds3 + (addr + (rw * NR + j) * 32 * STEP_B)));
    };
    unsigned w_off = 0, h_off = H_BASE;                      // the stages of step s
    unsigned w_free = (WR - 1) * W_STAGE;                    // the weight stage the step before has left
    {
        const unsigned wa = w_off + frag[0], ha = h_off + frag[0];
#pragma unroll
        for (int j = 0; j < NV; ++j) read_a(0, j, wa);
#pragma unroll
        for (int j = 0; j < NR; ++j) read_b(0, j, ha);
    }
    // One block of 16 elements: NV NR MFMAs on fragment set SET, with the reads of the next block (into the other set) and
    // COUNT loads from number FIRST on (KIND 1: of a weight stage, 2: of a hidden stage) dealt out between them.  The loads
    // of a step are spread over three blocks: a load occupies the CU's address path for 16 cycles, so the 64 loads of
    // four waves would hold up the MFMAs of a single block.
    auto block = [&](auto setc, auto kindc, auto firstc, auto countc, unsigned wa, unsigned ha, unsigned stage, int next)
                     __attribute__((always_inline)) {
        constexpr int SET = decltype(setc)::value, KIND = decltype(kindc)::value;
        constexpr int FIRST = decltype(firstc)::value, COUNT = decltype(countc)::value;
        constexpr int M = NV * NR, READS = NV + NR;
        constexpr int READ_BY = M > 3 ? M * 3 / 4 : 1;       // reads are out by three quarters of the block
        auto read_nth = [&](int q) __attribute__((always_inline)) {   // what the next block's first MFMAs need comes first
            if (q == 0) read_a(SET ^ 1, 0, wa);
            else if (q <= NR) read_b(SET ^ 1, q - 1, ha);
            else read_a(SET ^ 1, q - NR, wa);
        };
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int a = m / NR, b = (a & 1) ? NR - 1 - m % NR : m % NR;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[SET][a], fb[SET][b], acc[a][b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < READS; ++q)
                if (q >= (m * READS + READ_BY - 1) / READ_BY && q < ((m + 1) * READS + READ_BY - 1) / READ_BY) read_nth(q);
#pragma unroll
            for (int q = 0; q < COUNT; ++q)
                if (q >= (m * COUNT + M - 1) / M && q < ((m + 1) * COUNT + M - 1) / M) {
                    if (KIND == 1) issue_w1(FIRST + q, stage, next); else issue_h1(FIRST + q, stage, next);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    using WHALF = std::integral_constant<int, W_LOADS / 2>;
    using HALL = std::integral_constant<int, H_LOADS>;
    int s = 0;
    do {
        const int next_w = more(s + WR - 1);
        block(C0{}, C1{}, C0{}, WHALF{}, w_off + frag[1], h_off + frag[1], w_free, next_w);
        block(C1{}, C1{}, WHALF{}, WHALF{}, w_off + frag[2], h_off + frag[2], w_free, next_w);
        block(C0{}, C0{}, C0{}, C0{}, w_off + frag[3], h_off + frag[3], 0u, 0);
        // this wave's fragments of the step are all in registers; the next stages have landed when no more than the younger
        // stages' loads are out
        __builtin_amdgcn_s_waitcnt(0xc07f);                  // lgkmcnt(0)
        wait_vm<(WR - 2) * W_LOADS + (HR - 2) * H_LOADS>();
        bare_barrier();                                      // ... for every wave, and this step's stages are free
        const unsigned h_free = h_off;
        w_free = w_off;
        w_off = w_off + W_STAGE == H_BASE ? 0 : w_off + W_STAGE;
        h_off = h_off + H_STAGE == H_BASE + HR * H_STAGE ? H_BASE : h_off + H_STAGE;
        // (the last step reads a stage that holds old data, inside LDS; nothing uses it)
        block(C1{}, C2{}, C0{}, HALL{}, w_off + frag[0], h_off + frag[0], h_free, more(s + HR));
    } while (++s < n);

    // ---- fold: statistics and best candidate of this lane's rows over its 16 NV logits of each, parked in LDS for the four
    // lanes (two lane halves, two vocabulary waves) that share a row
    wait_vm<0>();                                            // the last steps' repeated loads have landed too
    __syncthreads();                                         // the rings are idle
    // the last MFMAs' results may be read (the accumulator reads below are inline assembly, for which the compiler does not
    // count wait states: 18 at most are needed)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    float* s_part = reinterpret_cast<float*>(lds);           // [row][4][3]
    uint64_t* s_key = reinterpret_cast<uint64_t*>(lds + BLOCK_ROWS * 12 * 4);
#pragma unroll
    for (int b = 0; b < NR; ++b) {
        const int v0 = v_begin + vw * NV * STRIP + 4 * half;
        const sage::lmhead::Fold f = sage::lmhead::fold_logits<NV>(v0, STRIP, v_end, [&](int a, int i, int left) __attribute__((always_inline)) {
            // read where it lies: with an ordinary use the compiler moves accumulators to the vector half of the register
            // file ahead of the fold and spills in the main loop for it
            float x;
            asm("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[a][b][i]));
            return 8 * (i >> 2) + (i & 3) < left ? x : -INFINITY;
        });
        const int slot = ((rw * NR + b) * 32 + r32) * 4 + vw * 2 + half;
        s_part[slot * 3] = f.m;
        s_part[slot * 3 + 1] = f.Z;
        s_part[slot * 3 + 2] = f.T;
        s_key[slot] = f.key;
    }
    __syncthreads();
    if (my_row >= 0) {
        const long o = static_cast<long>(my_row) * units + unit;
        sage::lmhead::combine_folds(s_part + tid * 12, s_key + tid * 4, prm.stats + o, prm.keys + o);
    }
}

__global__ __launch_bounds__(THREADS) void lm_head_rows_kernel(const Params prm) {
    __shared__ __align__(1024) unsigned char lds[LDS_B];
    const int tid = threadIdx.x;
    // The rows of block rb: slot j is live row number BLOCK_ROWS rb + j, counted over the groups in order.  Fills the row map
    // at the start of LDS and returns the number of live rows of the whole call (the same in every thread).
    auto map_rows = [&](int rb) __attribute__((always_inline)) {
        int* s_row = reinterpret_cast<int*>(lds);
        int* s_cnt = s_row + BLOCK_ROWS;
        int live = prm.rows;
        const int want = rb * BLOCK_ROWS + tid;
        if (prm.n_valid == nullptr) {
            s_row[tid] = want < prm.rows ? want : -1;
        } else {
            const int groups = (prm.rows + prm.rows_per_group - 1) / prm.rows_per_group;
            int before = 0, found = -1;
            for (int g0 = 0; g0 < groups; g0 += THREADS) {   // uniform trip count
                const int g = g0 + tid;
                s_cnt[tid] = g < groups ? max(0, min(prm.n_valid[g], min(prm.rows_per_group, prm.rows - g * prm.rows_per_group))) : 0;
                __syncthreads();
                const int here = min(THREADS, groups - g0);
                for (int j = 0; j < here; ++j) {
                    const int c = s_cnt[j];
                    if (found < 0 && want < before + c) found = (g0 + j) * prm.rows_per_group + (want - before);
                    before += c;
                }
                __syncthreads();
            }
            s_row[tid] = found;
            live = before;
        }
        __syncthreads();
        return live;
    };
    const int live = __builtin_amdgcn_readfirstlane(map_rows(0));
    if (live <= 0) return;
    const int blocks = (live + BLOCK_ROWS - 1) / BLOCK_ROWS;
    const Cut cut = live <= FEW_LIVE ? prm.few : prm.all;
    const int units = cut.ranges * cut.units_per_range;
    if (prm.units_used && blockIdx.x == 0 && tid == 0) *prm.units_used = units;
    const int items = ((units + 7) / 8) * 8 * blocks;
    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        const int slot = item >> 3;
        const int u = (slot / blocks) * 8 + (item & 7);      // first units of all ranges, then second ones, ...
        const int rb = slot % blocks;
        if (u >= units) continue;                            // (uniform)
        const int range = u % cut.ranges, j = u / cut.ranges;
        const int r_begin = static_cast<int>(static_cast<long>(range) * prm.ntiles / cut.ranges);
        const int r_tiles = static_cast<int>(static_cast<long>(range + 1) * prm.ntiles / cut.ranges) - r_begin;   // >= units_per_range
        const int t_begin = r_begin + j * r_tiles / cut.units_per_range;                // even shares: 1 to MAX_TILES
        const int t_end = r_begin + (j + 1) * r_tiles / cut.units_per_range;
        const int rows_here = min(BLOCK_ROWS, live - rb * BLOCK_ROWS);
        __syncthreads();                                     // the previous item has left LDS
        map_rows(rb);
        const int v_begin = t_begin * TILE_V, v_end = min(prm.vocab, t_end * TILE_V);
        const int nv = t_end - t_begin, nr = (rows_here + 63) / 64;
        auto one = [&](auto once) __attribute__((always_inline)) {
            constexpr bool ONCE = decltype(once)::value;
#define SAGE_PASS(V, R) pass<V, R, ONCE>(prm, lds, units, u, v_begin, v_end)
            if (nv == 4) {
                if (nr == 4) SAGE_PASS(4, 4); else if (nr == 3) SAGE_PASS(4, 3); else if (nr == 2) SAGE_PASS(4, 2); else SAGE_PASS(4, 1);
            } else if (nv == 3) {
                if (nr == 4) SAGE_PASS(3, 4); else if (nr == 3) SAGE_PASS(3, 3); else if (nr == 2) SAGE_PASS(3, 2); else SAGE_PASS(3, 1);
            } else if (nv == 2) {
                if (nr == 4) SAGE_PASS(2, 4); else if (nr == 3) SAGE_PASS(2, 3); else if (nr == 2) SAGE_PASS(2, 2); else SAGE_PASS(2, 1);
            } else {
                if (nr == 4) SAGE_PASS(1, 4); else if (nr == 3) SAGE_PASS(1, 3); else if (nr == 2) SAGE_PASS(1, 2); else SAGE_PASS(1, 1);
            }
#undef SAGE_PASS
        };
        // (the blocks of several share the weights through an L2, and are as fast or faster if these stay there: 512 live rows 1044 us, read so 1053)
        if (blocks == 1 && prm.read_once) one(std::true_type{});
        else one(std::false_type{});
    }
}

}  // namespace

namespace sage {

static Cut cut_vocabulary(int vocab, int rows) {
    const int ntiles = (vocab + TILE_V - 1) / TILE_V, blocks = (rows + BLOCK_ROWS - 1) / BLOCK_ROWS;
    Cut c;
    c.ranges = CUS / blocks > 1 ? CUS / blocks : 1;
    if (c.ranges > ntiles) c.ranges = ntiles;
    const int most = (ntiles + c.ranges - 1) / c.ranges;
    c.units_per_range = (most + MAX_TILES - 1) / MAX_TILES;
    return c;
}

// Slices per row when more than FEW_LIVE of the rows are live.
int lm_head_rows_units(int vocab, int rows) {
    const Cut c = cut_vocabulary(vocab, rows);
    return c.ranges * c.units_per_range;
}

// Slices that a row has room for: the most of any number of rows up to `rows`, since few live rows are cut for as one block and
// a workspace has to do for fewer rows.  More row blocks mean fewer ranges and, by rounding, sometimes fewer units (152064
// tokens: 768 with one block, 640 with two).
int lm_head_rows_slots(int vocab, int rows) {
    int most = 0;
    for (int r = BLOCK_ROWS; ; r += BLOCK_ROWS) {            // past CUS blocks nothing changes
        const int n = lm_head_rows_units(vocab, r);
        most = n > most ? n : most;
        if (r >= rows || r >= CUS * BLOCK_ROWS) return most;
    }
}

// units_used: receives the number of slices per row, which the live rows decide (nullable: nobody needs to know).
int launch_lm_head_rows(const void* hidden, const void* weight, int rows, int dim, int vocab, long hidden_stride,
                        long weight_stride, const int* n_valid, int rows_per_group, UnitStats* stats, uint64_t* keys, int* units_used, hipStream_t s) {
    Params p;
    p.hidden = static_cast<const unsigned char*>(hidden);
    p.weight = static_cast<const unsigned char*>(weight);
    p.hidden_stride_b = hidden_stride * 2;
    p.weight_stride_b = weight_stride * 2;
    p.rows = rows; p.vocab = vocab; p.nsteps = dim / 64;
    p.read_once = sage::lmhead::read_once(vocab, dim) ? 1 : 0;
    p.ntiles = (vocab + TILE_V - 1) / TILE_V;
    p.few = cut_vocabulary(vocab, n_valid ? 1 : rows);
    p.all = cut_vocabulary(vocab, rows);
    p.n_valid = n_valid; p.rows_per_group = rows_per_group;
    p.stats = stats; p.keys = keys; p.units_used = units_used;
    const long most = static_cast<long>((lm_head_rows_slots(vocab, rows) + 7) / 8) * 8 * ((rows + BLOCK_ROWS - 1) / BLOCK_ROWS);
    hipLaunchKernelGGL(lm_head_rows_kernel, dim3(most < CUS ? static_cast<unsigned>(most) : CUS), dim3(THREADS), 0, s, p);
    return launch_status();
}

}  // namespace sage
