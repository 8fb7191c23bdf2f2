// sage_tree_attention, bf16 MFMA instantiation (head_dim 128): tree-masked GQA attention of the target's
// verify pass (Sec. 2.2 tree mask; Alg. 1 Phase 2) against a long KV cache plus the tree's own keys.
//
// Formulation.  All query rows that share a KV head (node i, head-in-group hg -> row m = i*G + hg, up to 512
// rows at G = 8) are processed together so each K/V byte is fetched from HBM once.  Everything is computed transposed:
//   S^T = K Q^T   (tokens x rows):  A operand = K rows as stored in the cache (16-byte LDS reads),
//                                   B operand = Q rows, brought in through LDS once and held in registers
//                                   for the whole kernel;
//   O^T = V^T P^T (dims x rows):    A operand = V^T, read from row-major V in LDS with the transposing
//                                   64-bit LDS read of gfx950, B operand = P^T.
// In the 32x32 MFMA accumulator layout a lane owns ONE query row (column lane%32) and 16 tokens of it per 32-token
// half tile, so the softmax sums are in-register, the rescale factor is a per-lane scalar, and the accumulator
// registers of S^T are, as they stand, the B operand of the PV product (the token order inside a 16-token k-block
// is whatever the accumulator layout says; the V^T reads follow that order).
//
// Decomposition (decided on the device from n_nodes/kv_len, so no host round trip): a workgroup of 8 waves, two per SIMD,
// owns (sequence, KV head, group of up to 256 query rows, KV split); wave w owns one column tile of 32 rows and processes
// every 32-token block of the split for it, so nothing is shared between waves but the K/V blocks, and a wave's partial result
// is complete for its rows.  A block that has been brought into LDS
// serves as many query rows as registers allow: what a CU can pull in (about 24 GB/s from HBM) bounds small trees, and a
// tree of up to 32 nodes (G = 8) is one group.  With 2..64 sequences the splits are equal ranges of one list of all sequences'
// blocks, so ragged lengths leave no CU idle (see the kernel).  The KV head is the fastest grid index, so in launch order the
// workgroups of one KV head are congruent modulo the KV-head count, which with 8 KV heads pins a head to one XCD and its L2: the
// two groups of a 64-node tree re-read K/V from that L2, not from HBM.  Each workgroup writes an un-normalised partial (max, sum
// in fp32, O^T in bf16); a second kernel merges the splits in a fixed order (deterministic, no float atomics) and writes bf16.
//
// Data movement.  K/V blocks of 32 tokens go from global memory straight into LDS (16-byte LDS-direct loads, no staging
// registers; issued through inline assembly, see lds_direct_load16) through two rings of four blocks.  A wave-level load
// writes 1 KB of contiguous LDS; it carries four tokens that are 8 apart, and the 1 KB groups are padded so that the reads
// are free of bank conflicts at compile-time offsets (see the layout constants).  The ancestor masks and the Q rows take
// the same road ahead of the first blocks, so that no load of the kernel returns into a register and every wait on the
// vector-memory counter is a counted one (which is also why these kernels must not spill: the build checks that they use no
// scratch memory).
//
// Softmax.  The reference maximum of a row is only moved by rebase(): the usual block costs one maximum over the scaled
// differences to the reference, which says whether a probability would pass 2^8.  Probabilities are exp2 of the differences,
// rounded to bf16 (the B operand of PV); their sum is taken over the rounded values, in fp32, by small MFMAs.  The final
// normalisation uses the same reference for numerator and denominator, so the result does not depend on it.
//
// What bounds it, and against the kernel before this one (4 waves, one per SIMD, of one or two column tiles each, the second of
// which saved the other's LDS reads; every address and every "is there another block" worked out in every block); whole call, before
// -> now:
//   64 nodes: 32768 positions 78.7-81.5 -> 73.3 us, 0.94 PFLOP/s; 300 positions 13.4 -> 11.9; 24 nodes x 32768 41.9 -> 39.3.  A wave alone on
//   its SIMD issues one instruction at a time: about 600 cycles of a unit's 1016 (below) it issued, 100 of them scalar, and its
//   MFMAs take 577.  Taking out its LDS reads, its loads or its exponentials made a unit 1-3 % shorter, each by itself: the matrix pipe
//   waited for the order of the program.  Two waves, of which each fills what the other leaves open: 832 cycles a unit and SIMD (1663
//   a block); with the scalar work out of the block (the loop once around the rings), 745.  Power then keeps the clock at 1.2-1.9 GHz,
//   by machine and by how long the calls go on (80 layers in a row 82.4 -> 79.0 us a call); these MFMAs with this softmax and these
//   LDS reads, and nothing else, take 610 cycles and reach 1.27 PFLOP/s.
//   small trees: the stream, and at short contexts launch, two round trips, the merge launch, and what is executed once: a call over
//   4096 positions has its sizes after 0.9 us, has requested everything 1.0 us later and has it 0.6 us after that; five blocks take 3.5,
//   the epilogue 1.2, and the merge ends 4.2 us after the last store.  12 nodes, 64/8 heads, 4096 positions 12.5 -> 11.7 us, 32768
//   positions 31.6 -> 31.4; 15 nodes, 8192 positions 16.5 -> 15.4, 16384 22.1 -> 20.8 (1.8 us more in one run, on a machine where the
//   stream was slower the sooner a block was requested; in five later ones not); three sequences of 301 to 1999 positions 15.2 -> 14.5; eight of
//   2205 to 12133 53.8 -> 53.5; 28/4 heads, 3 new rows of 12, 2560 positions 9.2 -> 8.6.
#include <type_traits>

#include "plan_device.h"
#include "sage_internal.h"
#include "split_divisions.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
#define LDS_AS __attribute__((address_space(3)))

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 128;                  // head_dim
constexpr int BLK = 32;                 // tokens per block
constexpr int THREADS = 512;
constexpr int WAVES = THREADS / 64;     // two per SIMD
constexpr int ROWS_PER_WG = 32 * WAVES; // query rows of a group: a column tile of 32 per wave
constexpr int ROW_B = 256;              // bytes of one token row (128 bf16)
// LDS layout of a block: token t of a block sits at (t % 8) * GROUP + (t / 8) * ROW_B, where a group is the 1 KB that one
// wave-level LDS-direct load writes (tokens t, t+8, t+16, t+24) plus padding.  K is read 16 consecutive tokens x one 16-byte
// chunk at a time: 32 bytes of padding put eight consecutive tokens on eight different even chunk positions, and the rows
// with t / 8 odd hold their chunks with the lowest index bit flipped, so that the other eight are on the odd ones.  V is
// read 4 consecutive tokens x 64 bytes at a time: 64 bytes of padding.  Every fragment offset is a per-lane constant plus
// a compile-time one, and the reads are conflict-free.
constexpr int K_GROUP = 4 * ROW_B + 32;
constexpr int V_GROUP = 4 * ROW_B + 64;
constexpr int K_BLOCK_B = 8 * K_GROUP;
constexpr int V_BLOCK_B = 8 * V_GROUP;
// Two rings of four blocks, K and V, K two blocks ahead.  More do not help, they cost: with 4, 5, 6, 7 and 9 blocks (and four waves),
// 32768 positions under 12 nodes took 32.8, 34.4, 34.3, 35.2 and 36.5 us, 4096 positions 12.6, 13.0, 13.2, 13.4 and 13.7 (a call
// that starts by requesting more waits longer for its first block, and workgroups of different KV heads that run further apart
// read the cache's rows in smaller pieces); with 3 blocks 41.1 and 12.8.
constexpr int SLOTS = 4;
constexpr int V_AT = SLOTS * K_BLOCK_B;
constexpr int Q_AT = V_AT + SLOTS * V_BLOCK_B;
constexpr int Q_TILE_B = K_BLOCK_B;     // 32 query rows in the layout of a K block, behind the rings
constexpr int ZERO_AT = Q_AT + WAVES * Q_TILE_B;   // 1 KB of zeros: what the first unit reads as the V of the one before it
constexpr int RING_B = ZERO_AT + 1024;
// A partial: per query row O^T[128] in bf16, then max and sum in fp32.
constexpr int PART_ROW_B = D * 2 + 16;   // (8 bytes of padding keep the rows 16-byte aligned)
constexpr int PART_SLOT_B = ROWS_PER_WG * PART_ROW_B;
// (a slot's number is an int: what memory there is holds a few million of them)
__device__ __forceinline__ size_t slot_at(int slot) { return static_cast<size_t>(static_cast<unsigned>(slot)) * PART_SLOT_B; }
constexpr int EPI_ROW_B = PART_ROW_B;    // a parked row of the epilogue has the layout of a partial row
static_assert(ROWS_PER_WG * EPI_ROW_B <= RING_B, "the rings hold the epilogue's rows");
// A sequence of which B have more keys and values than this is read with loads that leave nothing in the memory-side cache
// (256 MB), if its rows are one group: a decoding step has read other layers and weights by the time they
// come up again, and to place them there costs memory bandwidth.  Whole call, 12 nodes, us, plain / so, over enough buffers in turn that none is still
// there: 32768 positions (134 MB) 30.0 / 27.8, 49152 41.2 / 37.5, 65536 53.1 / 49.3; eight of 4000 33.1 / 30.7, of 7000 53.2 / 48.3, of 12000 78.3 /
// 71.3.  What has stayed there is faster to read from there, so the line lies where few such buffers could: three of 67 MB in turn
// 17.3 / 18.8 (eight in turn 20.1 / 18.3), of 82 MB 19.4 / 21.2, of 101 MB 23.0 / 22.8; one of 134 MB again and again 25.8 / 27.2.
// Two row groups share a block through their L2 and lose it to these loads: 64 nodes, 32768 positions, 2 to 4 % slower.
constexpr long READ_ONCE_BYTES = 96L << 20;
constexpr int TWO_STEP_ROWS = 128;      // groups of more rows take their reference in two steps (see the first two blocks)
constexpr float RAISE_MIN = 4.0f;       // rebase() raises a row's reference maximum only past 2^4;
constexpr float REBASE_PAST = 8.0f;     // it is called when a probability would pass 2^8
constexpr float NO_REFERENCE = 3e38f;   // stands for -(reference * scale) while a row has none: every admitted key passes 2^8 then

// (What the kernels read first stands first, in the fewest cache lines of the argument block.)
struct Params {
    const uint16_t* Q; const uint16_t* Kc; const uint16_t* Vc; const uint16_t* Kt; const uint16_t* Vt;
    const uint64_t* anc_mask;
    unsigned char* part;                 // [B][Hkv][nslot] slots of PART_SLOT_B bytes; batched launches: [Hkv][nslot]
    long kv_token_stride, kv_head_stride;
    int Hq, Hkv, G;
    int inv_G;                           // 65536 / G rounded up: (m * inv_G) >> 16 == m / G for the rows of a KV head
    float scale_log2e;                   // softmax scale times log2(e): probabilities are exp2 of scaled differences
    int once_past;                       // sequences of more positions and one row group are read past the memory-side cache
    int B, nslot, min_blocks_per_split;
    int nrange;                          // batched launches: ranges (workgroups) per KV head
    int merge_phases;                    // merge workgroups per (sequence, KV head)
    uint16_t* O;
    const int64_t* kv_start; const int* kv_len; const int* n_nodes;
    const int* first_node;               // nullable: rows are computed for nodes first_node[b] .. n_nodes[b] - 1 only
};
// Has the arguments of an attention workgroup on their way with the first ones (they come from memory, a round trip for every cache
// line that is first asked for later): the empty statement needs them in registers where it stands.
__device__ __forceinline__ void arguments_here(const Params& p) {
    asm volatile("" : : "s"(p.Q), "s"(p.Kc), "s"(p.Vc), "s"(p.anc_mask), "s"(p.part), "s"(p.kv_token_stride), "s"(p.kv_head_stride),
                 "s"(p.Hq), "s"(p.Hkv), "s"(p.G), "s"(p.inv_G), "s"(p.scale_log2e));
}

// blocks of the cache and of the tree's own keys
__device__ __forceinline__ int blocks_of(int tokens) { return (tokens + BLK - 1) / BLK; }

// The sizes go through a few divisions before a kernel can request anything.  A general one is some 25 dependent
// instructions, and there were five of them in the attention kernel's way to its first load and four in the merge's (whole
// call of 3 new rows over 41 splits 9.3 -> 8.85 us, of 12 nodes over 4096 positions 12.7 -> 12.35, with the merge's first_node
// and reciprocal brought by the host).
__device__ __forceinline__ int div_floor(int x, int y) {
    return sage::div_floor(x, y, [](int a, int b) __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane(sage::by_reciprocal(a, __builtin_amdgcn_rcpf(static_cast<float>(b))));
    });
}
__device__ __forceinline__ int div_ceil(int x, int y) { return div_floor(x + y - 1, y); }
using sage::per_group;

// How one (sequence, KV head) is cut into workgroups; evaluated identically by both kernels.
struct Split {
    int n, first, rows, col_groups, blocks, max_split, blocks_per_split;
    __device__ __forceinline__ int count() const { return __builtin_amdgcn_readfirstlane(div_ceil(blocks, blocks_per_split)); }   // of splits
};
// the first node whose rows are computed: inside [0, n), so that a call always has a row
__device__ __forceinline__ int clamp_first(int first, int n) { return first < 0 ? 0 : (first > n - 1 ? n - 1 : first); }
// inv_nslot: sage::inverse(nslot), or 0 where a division is needed (see the host).
// One or two groups, which is what there is at 8 heads a KV head, then need neither a division nor a branch each.
// (Whole call, by divisions -> so, and with the merge's arguments on their way with the sizes: 12 nodes x 4096 positions 10.83 -> 10.64 us, x 300
// 7.95 -> 7.75, 64 nodes x 2000 15.7 -> 15.5, 28/4 heads, 3 new rows of 12 over 2560, 8.0 -> 7.83.)
__device__ __forceinline__ Split make_split(int n_nodes, int first_node, int kv_len, int G, int nslot, unsigned inv_nslot, int min_bps) {
    Split s;
    s.n = n_nodes < 1 ? 1 : (n_nodes > SAGE_MAX_NODES ? SAGE_MAX_NODES : n_nodes);
    s.first = clamp_first(first_node, s.n);
    s.rows = (s.n - s.first) * G;
    const int L = kv_len > 0 ? kv_len : 0;
    s.blocks = blocks_of(L) + blocks_of(s.n);               // cache blocks, then one or two with the tree's keys
    if (s.rows <= 2 * ROWS_PER_WG && inv_nslot != 0) {       // (uniform)
        const int second = s.rows > ROWS_PER_WG ? 1 : 0;
        s.col_groups = 1 + second;
        s.max_split = nslot >> second;                       // (nslot is even then)
        s.blocks_per_split = max(min_bps, sage::by_product((s.blocks + s.max_split - 1) << second, inv_nslot));
    } else {
        s.col_groups = (s.rows + ROWS_PER_WG - 1) / ROWS_PER_WG;
        s.max_split = max(1, per_group(nslot, s.col_groups));
        s.blocks_per_split = max(min_bps, __builtin_amdgcn_readfirstlane(div_ceil(s.blocks, s.max_split)));   // (or the other branch's is per lane, too)
    }
    return s;
}

// Batched decomposition: lane b of a wave holds the shape of sequence b.  Every (sequence, column group) segment
// occupies SEG_COST + blocks times the cost of a block positions of one line per KV head (the SEG_COST stand for the prologue
// and epilogue a pass costs, about that many block steps); the line of `total` positions is cut into ranges of q, so a
// workgroup whose range starts several segments gets fewer blocks.  A block belongs to the range that its first position lies
// in.  Evaluated identically by both kernels.
// Cost of a block: a group of up to LIGHT_ROWS rows is four waves, one per SIMD, and waits for the stream; with more rows two waves share a SIMD.
// Among seven sequences of 12 nodes over 8192 positions, a workgroup of one with 4, 8, 12 and 16 nodes took 0.50, 0.51, 0.54 and 0.55 us a block,
// with 17, 20, 24, 28 and 32 nodes 0.69, 0.68, 0.69, 0.69 and 0.70: the ranges of that sequence ended at 49 us, the others at 37.5; with 3 and
// 4 positions a block the last ends at 44.7.  A batch of one kind only keeps one position a block.
// In such mixed batches the last range is TAIL_BLOCKS shorter: where ranges fill the CUs, it is the one that waits for the workgroups that plan
// (see tree_attention_plan_kernel).  Whole call, at 0, 8 and 12, planning along: two sequences of 12 and 24 nodes over 16096 and 13000 34.5, 32.3 and 32.7
// us, eight of 9 to 19 nodes over 2800 to 11000 68.9, 65.9 and 66.0; attention alone 32.7, 32.5 and 32.5, 67.8, 67.4 and 67.1.
// Whole call, equal costs before -> now: three sequences of 12, 18 and 12 nodes over 301, 1900 and 1200 positions 15.4 -> 14.3 us, twelve of 9 to 40
// nodes over 400 to 5000 43.3 -> 42.1, five of 9 to 25 over 14000 to 20000 76.2 -> 72.0, the eight 67.7 -> 64.8.  Batches of one kind: forty of 12
// nodes 38.8 -> 37.2 (positions by a scan of the lanes, where every workgroup walked the sequences before its own), twelve 17.0 -> 16.8, three 12.15 ->
// 12.25, two 26.5 -> 26.9.
constexpr int SEG_COST = 6;
constexpr int LIGHT_ROWS = 128, LIGHT_COST = 3, HEAVY_COST = 4;
constexpr int TAIL_BLOCKS = 8;
struct BatchShape {
    int n, first, L, start_lo, start_hi;                     // per lane (sequence)
    int seg, col_groups;                                     // SEG_COST + blocks, and column groups (0 in lanes past the batch)
    int cost, last_cost;                                     // positions of a block: of a full group of rows, of the last one
    int length, at, groups_before;                           // its length on the line; position and segments of the sequences before it
    int total, q;                                            // wave-uniform
};
// how many blocks of `cost` positions begin before position x, counted from the first one's
__device__ __forceinline__ int blocks_until(int x, int cost) {
    static_assert(LIGHT_COST == 3 && HEAVY_COST == 4, "the costs that it divides by");
    return sage::div_up_by_cost(max(x, 0), cost);
}
// Sums over the lanes up to and including a lane's own, of two values at a time (the steps of one fill the wait states of the other's).
__device__ __forceinline__ void wave_scan2(int& a, int& b) {
    auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
        const int x = __builtin_amdgcn_update_dpp(0, a, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
        const int y = __builtin_amdgcn_update_dpp(0, b, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
        a += x;
        b += y;
    };
    using All = std::integral_constant<int, 0xF>;
    step(std::integral_constant<int, 0x111>{}, All{});       // row_shr:1
    step(std::integral_constant<int, 0x112>{}, All{});       // row_shr:2
    step(std::integral_constant<int, 0x114>{}, All{});       // row_shr:4
    step(std::integral_constant<int, 0x118>{}, All{});       // row_shr:8
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});   // row_bcast:15 into rows 1 and 3
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});   // row_bcast:31 into rows 2 and 3
}
// What it needs of the arguments comes in scalars that are preloaded at wave launch, see the kernels, and its loads are the first thing
// that a wave does: from the argument block in memory they were two round trips later, in the attention's workgroups and in the merge's
// (whole call, three sequences of 301 to 1999 positions 12.8 -> 12.4 us, seven of 300 to 1300 16.3 -> 15.6, eight of 2800 to 11000 64.3 ->
// 62.8).  `others_here`: what else is to be on its way before they are waited for.
template <bool WITH_START, class F>
__device__ __forceinline__ BatchShape make_batch_shape(const int* __restrict__ kv_len, const int* __restrict__ n_nodes, const int* __restrict__ first_node,
                                                       const int64_t* __restrict__ kv_start, int B, int nrange, int min_bps, int G, int light_rows, int lane, F others_here) {
    BatchShape bs;
    const int seq = min(lane, B - 1);
    int nn = n_nodes[seq], len = kv_len[seq], f = first_node ? first_node[seq] : 0;
    bs.start_lo = 0; bs.start_hi = 0;
    if (WITH_START) {
        const int64_t st = kv_start[seq];
        bs.start_lo = static_cast<int>(static_cast<uint32_t>(st));
        bs.start_hi = static_cast<int>(st >> 32);
    }
    others_here();
    asm volatile("" : "+v"(nn), "+v"(len), "+v"(f), "+v"(bs.start_lo), "+v"(bs.start_hi));
    bs.n = nn < 1 ? 1 : (nn > SAGE_MAX_NODES ? SAGE_MAX_NODES : nn);
    bs.first = clamp_first(f, bs.n);
    bs.L = len > 0 ? len : 0;
    bs.seg = blocks_of(bs.L) + blocks_of(bs.n) + SEG_COST;   // cache blocks, then one or two with the tree's keys
    const int last = (bs.n - bs.first) * G - 1;              // its last row (there is at least one)
    static_assert(ROWS_PER_WG == 256 && LIGHT_ROWS == 128, "bits of a row's number");
    // (lanes past the batch repeat its last sequence here)
    const bool mixed = __ballot(last >= light_rows) != 0 && __ballot(!(last & 128)) != 0;
    bs.cost = mixed ? HEAVY_COST : 1;
    bs.last_cost = mixed ? LIGHT_COST + (static_cast<unsigned>(last) >> 7 & 1) : 1;
    const int groups_before_last = last >> 8;
    bs.length = lane < B ? bs.seg * (bs.cost * groups_before_last + bs.last_cost) : 0;
    bs.col_groups = lane < B ? groups_before_last + 1 : 0;
    int at = bs.length, groups = bs.col_groups;
    wave_scan2(at, groups);
    bs.total = __builtin_amdgcn_readlane(at, 63);
    bs.at = at - bs.length;
    bs.groups_before = groups - bs.col_groups;
    bs.q = max(mixed ? min_bps * LIGHT_COST : min_bps, div_ceil(bs.total + (mixed ? TAIL_BLOCKS * LIGHT_COST : 0), nrange));
    return bs;
}

// s_waitcnt on the vector-memory counter only (expcnt and lgkmcnt fields left at "no wait")
template <int N> __device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// Workgroup barrier of the rings.  __syncthreads() would also fence, and a workgroup-scope release makes the
// compiler wait for every LDS-direct load still in flight, which is exactly what the ring must not do: each
// thread has already waited for its own share of the block (wait_vm), LDS needs no cache maintenance, so the bare
// barrier is enough; the wavefront-scope fences only pin the order of memory operations around it.
__device__ __forceinline__ void stage_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// After an MFMA whose result is read past a branch.  Twelve wait states lie between a 32x32x16 MFMA and a vector instruction that
// reads its result; the compiler sees to them, but where paths join it has been seen to count along a longer one than the
// shortest (the maximum over the first scores came after nine or ten on the path past the masking).
__device__ __forceinline__ void mfma_results_ready() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 11");
    __builtin_amdgcn_sched_barrier(0);
}

// max / sum of a value with its partner in the other 32-lane half (both halves receive the result)
__device__ __forceinline__ float cross_half_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float cross_half_sum(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS of a workgroup.
struct Lds {
    unsigned char ring[RING_B];
    uint64_t mask[ROWS_PER_WG];          // the rows' ancestor masks
    i32x4 seq[64];                       // batches: nodes and first node, length, start of each sequence
    i32x4 line[64];                      // ... its position on the line, SEG_COST + blocks, costs and column groups, segments before it
};

// What one pass works on; every field is wave-uniform.
struct Segment {
    int b, g, L, n, node0, rows, cg;     // sequence, KV head, cache length, nodes, first node computed, rows, column group
    int begin, count, cache_blocks;      // blocks begin .. begin + count - 1 (count >= 1); those from cache_blocks on are the tree's
    long kv_start;
    int slot;                            // of the partial
};

// One pass: the blocks of a segment for one column group.  Wave w owns column tile w, 32 rows, and processes every block for it
// (the accumulators of two tiles would leave a wave alone on its SIMD).
//
// The loop runs over units, a unit being one block for the wave's column tile.  While the vector pipe turns the scores of unit
// h into probabilities, the matrix pipe computes the scores of unit h + 1 and the PV product of unit h - 1: 16 MFMAs that
// depend on nothing of unit h, one ahead of each of its 16 scores per lane, in program order (scheduling fences).  What one
// wave leaves open (waits, branches, the end of a unit, scalar instructions), the other wave of its SIMD fills, as far as the
// barrier of the block lets it.
// ONCE: the cache is read past the memory-side cache (see READ_ONCE_BYTES).
template <bool KEYS_FIRST, bool ONCE>
__device__ __forceinline__ void attention_pass(const Params& prm, LDS_AS Lds* lds, const Segment& sg, const int inv_G, const int tid) {
    LDS_AS unsigned char* const ring = lds->ring;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, so LDS addresses stay scalar
    const int r32 = lane & 31;           // MFMA row (A) / column (B, C) owned by this lane
    const int half = lane >> 5;
    const int group_rows = min(ROWS_PER_WG, sg.rows - sg.cg * ROWS_PER_WG);
    const int row0 = wave * 32;          // this wave's first row within the group
    const bool active = row0 < group_rows;
    const int H = sg.count;
    const int slot0 = H & 1 ? 1 : 2;     // block h lies in slot (h + slot0) % SLOTS of its ring (see the loop)

    // ---- loader: wave w brings tokens w, w+8, w+16, w+24 of a block, 1 KB of LDS: lane l fills chunk position l % 16 of token
    // w + 8 (l / 16).  Addresses are a wave-uniform block base in scalar registers plus a 32-bit per-lane offset that is the
    // same for every full block.
    const int ld_tok = (lane >> 4) * 8 + wave;
    const unsigned k_chunk_b = ((lane & 15) ^ ((lane >> 4) & 1)) * 16;
    const unsigned v_chunk_b = (lane & 15) * 16;
    const unsigned cache_row_b = static_cast<unsigned>(prm.kv_token_stride) * 2u;   // host: 32 rows fit 32 bits
    const long cache_at = sg.kv_start * prm.kv_token_stride + static_cast<long>(sg.g) * prm.kv_head_stride;
    const unsigned k_off = static_cast<unsigned>(ld_tok) * cache_row_b + k_chunk_b;
    const unsigned v_off = static_cast<unsigned>(ld_tok) * cache_row_b + v_chunk_b;
    const int full = min(H, max(0, sg.L / BLK - sg.begin));  // leading blocks that are whole blocks of the cache
    const unsigned long block_b = static_cast<unsigned long>(BLK) * cache_row_b;
    const unsigned char* const k_cache = reinterpret_cast<const unsigned char*>(prm.Kc + cache_at) + static_cast<long>(sg.begin) * static_cast<long>(block_b);
    const unsigned char* const v_cache = reinterpret_cast<const unsigned char*>(prm.Vc + cache_at) + static_cast<long>(sg.begin) * static_cast<long>(block_b);

    // where block h of K or V lies: a uniform base and this lane's offset
    struct At { const unsigned char* base; unsigned off; };
    auto locate = [&](auto is_v, int h) __attribute__((always_inline)) {
        constexpr bool V = decltype(is_v)::value;
        const int blk = sg.begin + h;
        const bool is_tree = blk >= sg.cache_blocks;
        const int tb = is_tree ? blk - sg.cache_blocks : blk;
        const long tree_at = (static_cast<long>(sg.b) * SAGE_MAX_NODES * prm.Hkv + sg.g) * D;
        const unsigned row_b = is_tree ? static_cast<unsigned>(prm.Hkv) * D * 2u : cache_row_b;
        At l;
        l.base = reinterpret_cast<const unsigned char*>(is_tree ? (V ? prm.Vt : prm.Kt) + tree_at : (V ? prm.Vc : prm.Kc) + cache_at) +
                 static_cast<long>(tb) * BLK * row_b;
        // in a ragged tail and in the tree's keys the rows past the end repeat the last one: they are masked later
        const int last = (is_tree ? sg.n : sg.L) - 1 - tb * BLK;
        l.off = static_cast<unsigned>(min(ld_tok, last)) * row_b + (V ? v_chunk_b : k_chunk_b);
        return l;
    };
    auto slot_of = [&](int h) __attribute__((always_inline)) { return static_cast<unsigned>(h + slot0) % SLOTS; };
    auto issue = [&](auto is_v, int h, const unsigned char* in_cache) __attribute__((always_inline)) {   // in_cache: where it is if a whole block of the cache
        constexpr bool V = decltype(is_v)::value;
        if (h >= H) return;
        At l;
        if (h < full) l = At{in_cache, V ? v_off : k_off};
        else l = locate(is_v, h);
        sage::lds_direct_load16<ONCE>(l.base, l.off, ring + (V ? V_AT + slot_of(h) * V_BLOCK_B + wave * V_GROUP : slot_of(h) * K_BLOCK_B + wave * K_GROUP));
    };
    using IsK = std::false_type;
    using IsV = std::true_type;
    const unsigned char* k_next = k_cache + 4 * block_b;     // block h + 4 of K, block h + 2 of V
    const unsigned char* v_next = v_cache + 2 * block_b;
    // Before unit h: K of block h + 2 and V of block h have landed for every wave, and the slots of K of block h and V of block
    // h - 2 are free (an MFMA of unit h - 1 has used what was read from them).  Loads complete in order, and what was
    // requested after the two, V of block h + 1 and K of block h + 3, is out at most.  This is the way of the first and last blocks;
    // in the middle (see the loop) nothing is left to decide.
    auto arrive = [&](int h) __attribute__((always_inline)) {
        if (h + 3 < H) wait_vm<2>();
        else if (h + 1 < H) wait_vm<1>();
        else wait_vm<0>();
        stage_barrier();
        issue(IsV{}, h + 2, v_next);
        issue(IsK{}, h + 4, k_next);
        v_next += block_b;
        k_next += block_b;
    };

    // Everything the prologue needs from memory goes straight into LDS, requested back to back: the wave's
    // ancestor masks, its Q rows, the first blocks.  No load of the kernel returns into a
    // register, so the compiler never waits on the vector-memory counter here and the only waits are the counted ones.
    // Rows past the group's last one repeat that row (their results are never written).
    auto row_of = [&](int local) __attribute__((always_inline)) {      // row `local` of this group, of the rows of the KV head
        return static_cast<unsigned>(min(sg.cg * ROWS_PER_WG + local, sg.rows - 1));
    };
    auto node_of = [&](unsigned m) __attribute__((always_inline)) { return (m * static_cast<unsigned>(inv_G)) >> 16; };   // exact for m < 64 G, G <= 16
    // Addresses of Q rows take 0.4 us of instructions, those of whole blocks few: where the stream is what a pass waits for, the first two blocks of K go
    // ahead of them (15 nodes x 16384 positions 19.2 -> 18.5 us, 12 x 4096 10.97 -> 10.83, 12 x 32768 27.3 -> 27.0).  With more than 128 rows (64
    // nodes x 2000 15.7 -> 15.8, 32 x 2000 14.3 -> 14.45) and in batches, whose first passes begin later (three sequences 12.45 -> 12.65), they do not.
    const bool keys_first = KEYS_FIRST && group_rows <= LIGHT_ROWS;
    if (keys_first) {
        issue(IsK{}, 0, k_cache);
        issue(IsK{}, 1, k_cache + block_b);
    }
    // Q rows as tiles of 32 in the layout of a K block: row q of a tile sits at (q % 8) * K_GROUP + (q / 8) * ROW_B
    LDS_AS unsigned char* const q_tile = ring + Q_AT + wave * Q_TILE_B;
    if (active) {
        {                                                    // both words of the masks of rows lane / 2
            const unsigned char* masks = reinterpret_cast<const unsigned char*>(prm.anc_mask + static_cast<long>(sg.b) * SAGE_MAX_NODES + sg.node0);
            sage::lds_direct_load4(masks + (node_of(row_of(row0 + (lane >> 1))) * 8u + (lane & 1) * 4u), (LDS_AS unsigned char*)(&lds->mask[row0]));
        }
        const unsigned char* q_rows = reinterpret_cast<const unsigned char*>(prm.Q + ((static_cast<long>(sg.b) * SAGE_MAX_NODES + sg.node0) * prm.Hq + sg.g * prm.G) * D);
        const unsigned node_b = static_cast<unsigned>(prm.Hq - prm.G) * (D * 2u);   // (64 nodes of up to 65535 heads: within 32 bits)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned m = row_of(row0 + i + 8 * (lane >> 4));
            sage::lds_direct_load16(q_rows, node_of(m) * node_b + m * (D * 2u) + k_chunk_b, q_tile + i * K_GROUP);
        }
    }
    if (!keys_first) {
        issue(IsK{}, 0, k_cache);
        issue(IsK{}, 1, k_cache + block_b);
    }
    issue(IsV{}, 0, v_cache);
    issue(IsK{}, 2, k_cache + 2 * block_b);
    issue(IsV{}, 1, v_cache + block_b);
    issue(IsK{}, 3, k_cache + 3 * block_b);
    *(LDS_AS u32x4*)(ring + ZERO_AT + lane * 16) = u32x4{0, 0, 0, 0};   // (by every wave, which reads it after its own write)
    if (H >= 4) wait_vm<4>();                                // masks, Q and the first two blocks of K have landed
    else if (H == 2) wait_vm<2>();
    else wait_vm<0>();
    stage_barrier();                                         // ... everyone's have

    if (!active) {                                           // no rows: this wave only brings its share of the blocks
        for (int h = 0; h < H; ++h) arrive(h);
        wait_vm<0>();
        __syncthreads();
        return;
    }

    f32x16 acc[4];                                           // O^T: 4 tiles of 32 dims x this lane's query row
    float m_ref = -INFINITY;                                 // reference maximum of raw (unscaled) scores
    // ---- per-lane LDS read offsets.  K fragment kk: token r32, chunk 2 kk + half -> k_lane + 32 kk.
    const unsigned k_lane = (r32 & 7) * K_GROUP + (r32 >> 3) * ROW_B + ((half ^ ((r32 >> 3) & 1)) * 16);
    // V^T fragment (dt, jj, u): k-block jj (16 tokens); the 16-lane group q = lane/16 reads tokens 16jj + 8u + 4(q/2) + s/4
    // and dims dt*32 + 16(q%2) + 4(s%4) .. +3  (s = lane%16); after the transposing read lane s holds dim dt*32+16(q%2)+s.
    // Offset: v_lane + (2 jj + u) * ROW_B + dt * 64.
    unsigned v_lane;
    {
        const int q = lane >> 4, s16 = lane & 15;
        v_lane = V_AT + (4 * (q >> 1) + (s16 >> 2)) * V_GROUP + (2 * (q & 1) + ((s16 & 3) >> 1)) * 16 + 8 * (s16 & 1);
    }
    auto read16 = [&](unsigned at) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, *(const LDS_AS u32x4*)(ring + at));
    };
    bf16x8 qf[8];                                        // this lane's query row: the B operand of every score MFMA
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = read16(Q_AT + wave * Q_TILE_B + k_lane + kk * 32);

#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float neg_mc = NO_REFERENCE;                         // -(m_ref * c)
    f32x4 l_run = {0.f, 0.f, 0.f, 0.f};                  // this lane's share of the running sum, four times
    const float c_log2 = prm.scale_log2e;
    f32x16 sc[2];                                        // scores of the current and of the next unit
    bf16x8 pf[2][2];                                     // P^T of the current and of the last unit, B operand of PV
    bf16x8 kf[4], vf[4];                                 // fragments of K (by 16 dims) and V^T (by 32 dims)

    auto read_k = [&](bf16x8& f, unsigned at, int kk) __attribute__((always_inline)) { f = read16(at + kk * 32); };
    auto read_v = [&](bf16x8& f, unsigned at, int dt, int jj) __attribute__((always_inline)) {
        LDS_AS unsigned char* p = ring + (at + 2 * jj * ROW_B + dt * 64);
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)p);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(p + ROW_B));
        f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // admit keys: cache positions below kv_len; tree nodes in this row's ancestor-or-self mask
    auto mask_scores = [&](f32x16& s, int h) __attribute__((always_inline)) {
        const int blk = sg.begin + h;
        uint32_t admit;
        if (blk >= sg.cache_blocks) {
            admit = reinterpret_cast<LDS_AS uint32_t*>(lds->mask)[2 * (row0 + r32) + (blk - sg.cache_blocks)];
        } else {
            admit = (1u << (sg.L - blk * BLK)) - 1u;     // 1..31 valid tokens
        }
        admit >>= 4 * half;
        // token of accumulator register i: 8 (i/4) + 4 half + i%4
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (!((admit >> (8 * (i >> 2) + (i & 3))) & 1u)) s[i] = -INFINITY;
    };
    // Move the reference maximum of the rows that need it to the row maximum of the current unit (both 32-lane halves of
    // a row decide alike) and rescale what has been accumulated so far.
    auto rebase = [&](const f32x16& s, bool nothing_yet, float raise_min) __attribute__((always_inline)) {
        float tmax = fmaxf(s[0], s[1]);
#pragma unroll
        for (int i = 2; i < 16; ++i) tmax = fmaxf(tmax, s[i]);
        tmax = cross_half_max(tmax);
        const bool raise = (m_ref == -INFINITY) ? (tmax > -INFINITY) : ((tmax - m_ref) * c_log2 > raise_min);
        const float m_new = raise ? tmax : m_ref;
        const float corr = !raise ? 1.f : (m_ref == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((m_ref - m_new) * c_log2);
        m_ref = m_new;
        neg_mc = m_new == -INFINITY ? NO_REFERENCE : -m_new * c_log2;
        if (!nothing_yet) {
            l_run[0] *= corr;                            // (the other three are not read)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[dt][i] *= corr;
        }
    };
    // (the compiler does not move the computation of x past this point)
#define PIN(x) asm volatile("" : "+v"(x))
#define FENCE() __builtin_amdgcn_sched_barrier(0)
    // two probabilities to bf16 in place i, i + 1 of f
    auto pack2 = [&](bf16x8& f, int i, float p0, float p1) __attribute__((always_inline)) {
        const f32x2 pp = {p0, p1};
        uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
        PIN(u);                                          // (or it would be computed after the branch that follows)
        const bf16x2 pb = __builtin_bit_cast(bf16x2, u);
        f[i] = pb[0];
        f[i + 1] = pb[1];
    };
    // The running sums of the rounded probabilities, four of a lane's 16 at a time: of the 16 products of 4 x 4 matrices that
    // this MFMA does, a lane's four values are one column, and a matrix of ones adds it up.  16 cycles of the matrix pipe
    // (a loop of a unit's MFMAs takes 513 cycles without its four and 577 with them; the counter of busy cycles advances by 8 for each);
    // two two-element dot products block it for 16 each, and unpacking and adding are eight instructions of a full vector pipe.
    auto add_up = [&](const bf16x8 (&before)[2], int j) __attribute__((always_inline)) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        const s16x4 ones = {0x3F80, 0x3F80, 0x3F80, 0x3F80};
        const bf16x8& p = before[j >> 1];
        const bf16x4 four = (j & 1) == 0 ? __builtin_shufflevector(p, p, 0, 1, 2, 3) : __builtin_shufflevector(p, p, 4, 5, 6, 7);
        l_run = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, four), l_run, 0, 0, 0);
    };
    // Unit h; CUR = which of the two score and probability sets, its parity counted from the end of the pass.  `usual`: the
    // blocks in SLOT and around it are whole blocks of the cache, and so are those that are requested.
    const unsigned k_dst = wave * K_GROUP, v_dst = V_AT + wave * V_GROUP;
    auto unit = [&](auto is_usual, auto slot, auto cur, const int h) __attribute__((always_inline)) {
        constexpr bool USUAL = decltype(is_usual)::value;
        constexpr int SLOT = decltype(slot)::value, CUR = decltype(cur)::value;
        f32x16& s = sc[CUR];
        f32x16& next = sc[1 - CUR];
        float most = -INFINITY;                              // the largest exponent of a probability
        // where this lane reads K of blocks h + 1 (second half) and h + 2 (first half), V of blocks h - 1 (second half) and h
        unsigned k1, k2, v0, v1;
        if (USUAL) {
            k1 = k_lane + (SLOT + 1) % SLOTS * K_BLOCK_B;
            k2 = k_lane + (SLOT + 2) % SLOTS * K_BLOCK_B;
            v0 = v_lane + (SLOT + 3) % SLOTS * V_BLOCK_B;
            v1 = v_lane + SLOT * V_BLOCK_B;
        } else {
            k1 = k_lane + slot_of(h + 1) * K_BLOCK_B;
            k2 = k_lane + slot_of(h + 2) * K_BLOCK_B;
            v0 = h == 0 ? ZERO_AT : v_lane + slot_of(h + 3) * V_BLOCK_B;
            v1 = v_lane + slot_of(h) * V_BLOCK_B;
            if (__builtin_expect(h >= full || h <= 1, 0)) {
                if (h >= full) mask_scores(s, h);
                // The reference of a pass is the maximum of its first two blocks (64 tokens), so that the largest probability of a short
                // pass is exactly one in bf16.  Error against 64 bits, 28/4 heads over 2560 positions: 2.61-2.65e-3 (2.69-2.75e-3 with the
                // first block's maximum).  In larger groups block 0 keeps its probabilities, and its products are rescaled: 0.2-0.6 % smaller
                // errors, but 64 instructions more, 0.2 us of a short call.
                if (h == 0) rebase(s, true, RAISE_MIN);
                if (h == 1) {
                    if (group_rows > TWO_STEP_ROWS) {
                        most = INFINITY;                     // (the reference moves after this unit's MFMAs, below)
                    } else {                                 // (block 0 has not been multiplied yet: its probabilities again)
                        rebase(s, true, 0.f);
                        float neg_mc_now = neg_mc;
                        PIN(neg_mc_now);
#pragma unroll
                        for (int i = 0; i < 16; i += 2)
                            pack2(pf[1 - CUR][i >> 3], i & 7, __builtin_amdgcn_exp2f(fmaf(next[i], c_log2, neg_mc_now)),
                                  __builtin_amdgcn_exp2f(fmaf(next[i + 1], c_log2, neg_mc_now)));
                    }
                }
            }
        }
        bf16x8 (&p)[2] = pf[CUR];
        bf16x8 (&before)[2] = pf[1 - CUR];                   // the last unit's
        // The softmax of score m takes three steps, each in a later MFMA's shadow than the one before, so that no instruction
        // waits for the result of the one ahead of it.
        float x[2], e[4];
        bool over = false;
        FENCE();
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            // alternately a score MFMA and a PV MFMA, the last score MFMA third from the end; a fragment's registers take the next
            // one that they are for as soon as its MFMA has been issued
            const int mm = m == 13 ? 14 : m == 14 ? 13 : m, i = mm >> 1;
            if (mm & 1) {
                acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i & 3], before[i >> 2], acc[i & 3], 0, 0, 0);
                if (i < 4) read_v(vf[i], v0, i, 1);
                else read_v(vf[i & 3], v1, i & 3, 0);
            } else {
                if (i == 0) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) next[r] = 0.f;
                }
                next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i & 3], qf[i], next, 0, 0, 0);
                if (i < 4) read_k(kf[i], k1, i + 4);
                else read_k(kf[i & 3], k2, i - 4);
            }
            if ((m & 3) == 2) add_up(before, m >> 2);
            // (requested late in the unit: 15 nodes x 16384 positions 23.3, 22.9 and 22.3 us with the two at m = 0, at 1 and 5, at 7 and 11 on
            // a machine where the kernel before took 22.4; on others the place makes no difference)
            if (USUAL && m == 13) {
                sage::lds_direct_load16<ONCE>(v_next, v_off, ring + (v_dst + (SLOT + 2) % SLOTS * V_BLOCK_B));
                v_next += block_b;
            }
            if (USUAL && m == 15) {
                sage::lds_direct_load16<ONCE>(k_next, k_off, ring + (k_dst + SLOT * K_BLOCK_B));
                k_next += block_b;
            }
            if (m == 0) {
                x[0] = fmaf(s[0], c_log2, neg_mc);
                x[1] = fmaf(s[1], c_log2, neg_mc);
                PIN(x[0]);
                PIN(x[1]);
                e[0] = __builtin_amdgcn_exp2f(x[0]);
                PIN(e[0]);
            }
            if (!(m & 1)) {
                if (m > 0) pack2(p[(m - 2) >> 3], (m - 2) & 7, e[(m - 2) & 3], e[(m - 1) & 3]);
                most = fmaxf(fmaxf(most, x[0]), x[1]);       // scores m, m + 1
                PIN(most);
            }
            if (m < 15) {
                e[(m + 1) & 3] = __builtin_amdgcn_exp2f(x[(m + 1) & 1]);
                PIN(e[(m + 1) & 3]);
            } else {
                pack2(p[1], 6, e[2], e[3]);
            }
            if (m < 14) {
                x[m & 1] = fmaf(s[m + 2], c_log2, neg_mc);
                PIN(x[m & 1]);
            }
            if (m == 14) over = __any(most > REBASE_PAST);
            FENCE();
        }
        // A probability that may have overflowed, a row's first admitted key, or (said by `most`) the pass's second block.
        if (__builtin_expect(over, 0)) {
            rebase(s, false, !USUAL && h == 1 ? 0.f : RAISE_MIN);
            float neg_mc_now = neg_mc;
            PIN(neg_mc_now);                                 // (or the differences above would be kept for the rows that did not move)
#pragma unroll
            for (int i = 0; i < 16; i += 2)
                pack2(p[i >> 3], i & 7, __builtin_amdgcn_exp2f(fmaf(s[i], c_log2, neg_mc_now)),
                      __builtin_amdgcn_exp2f(fmaf(s[i + 1], c_log2, neg_mc_now)));
        }
        FENCE();
    };
#undef PIN
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;

    // The scores of the first unit; what the first unit multiplies as "the last one's" is zero.  Units go in pairs, for the two sets of
    // scores; of an odd number the first one goes ahead.
    {
        const unsigned k0 = k_lane + slot_of(0) * K_BLOCK_B;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) read_k(kf[kk], k0, kk);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            vf[i][e] = static_cast<__bf16>(0.0f);
            pf[i & 1][i >> 1][e] = static_cast<__bf16>(0.0f);
        }
    auto first_scores = [&](f32x16& s) __attribute__((always_inline)) {
        const unsigned k0 = k_lane + slot_of(0) * K_BLOCK_B, k1 = k_lane + slot_of(1) * K_BLOCK_B;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk & 3], qf[kk], s, 0, 0, 0);
            if (kk < 4) read_k(kf[kk], k0, kk + 4);
            else read_k(kf[kk & 3], k1, kk - 4);
        }
        mfma_results_ready();
    };
    using Usual = std::true_type;
    using Any = std::false_type;
    int h = 0;
    if (H & 1) {
        first_scores(sc[1]);
        arrive(0);
        unit(Any{}, I0{}, I1{}, 0);
        h = 1;
    } else {
        first_scores(sc[0]);
    }
    while (h < H) {
        arrive(h);
        unit(Any{}, I0{}, I0{}, h);
        arrive(h + 1);
        unit(Any{}, I0{}, I1{}, h + 1);
        h += 2;
        // Four units at a time, once around the rings: every address is a compile-time offset.  Block h is in slot 0 now (2 or 3 blocks
        // are done, and what slot0 is comes from that); past the last of these units this is not reached again with enough blocks left.
        while (h + 7 < full) {
            wait_vm<2>();
            stage_barrier();
            unit(Usual{}, I0{}, I0{}, h);
            wait_vm<2>();
            stage_barrier();
            unit(Usual{}, I1{}, I1{}, h);
            wait_vm<2>();
            stage_barrier();
            unit(Usual{}, I2{}, I0{}, h);
            wait_vm<2>();
            stage_barrier();
            unit(Usual{}, I3{}, I1{}, h);
            h += 4;
        }
    }
    // PV of the last unit
    const unsigned v_last = v_lane + slot_of(H - 1) * V_BLOCK_B;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i & 3], pf[1][i >> 2], acc[i & 3], 0, 0, 0);
        if (i < 4) read_v(vf[i], v_last, i, 1);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) add_up(pf[1], j);
#undef FENCE
    const float l_tot = cross_half_sum(l_run[0]);
    wait_vm<0>();

    // ---- epilogue: a wave's rows (O^T in bf16, max, sum) are complete.  They go through the wave's own piece of the ring as
    // rows of EPI_ROW_B bytes, transposed on the way: written 8 bytes (4 dims) at a time from the accumulator layout, read
    // back and stored to the partial in row order, for the second kernel to merge.
    __syncthreads();                                         // the rings are idle now
    LDS_AS unsigned char* const mine = ring + row0 * EPI_ROW_B;
    LDS_AS unsigned char* const row = mine + r32 * EPI_ROW_B;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 v = {acc[dt][4 * q], acc[dt][4 * q + 1], acc[dt][4 * q + 2], acc[dt][4 * q + 3]};
            *reinterpret_cast<LDS_AS bf16x4*>(row + (dt * 32 + 8 * q + 4 * half) * 2) = __builtin_convertvector(v, bf16x4);
        }
    if (half == 0) *reinterpret_cast<LDS_AS f32x2*>(row + D * 2) = f32x2{m_ref, l_tot};
    // (a wave's LDS operations complete in order, and the reads below wait for them: no barrier inside a wave)
    // Parked rows and partial rows have the same pitch, so the wave's rows go out as one contiguous copy of 17 chunks of 16
    // bytes a row (16 of O^T, one of max and sum), 64 chunks per store instruction
    const int last_chunk = min(32, group_rows - row0) * (PART_ROW_B / 16);
    // They are written through the L2 (see store_through16): what a kernel leaves in an L2 is written back at its end, before the merge
    // may start, and 64 nodes leave 17 MB.
    unsigned char* const out = prm.part + slot_at(sg.slot) + row0 * PART_ROW_B + lane * 16;
    constexpr int COPIES = (32 * (PART_ROW_B / 16) + 63) / 64;
    u32x4 chunk[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; ++i) chunk[i] = *reinterpret_cast<LDS_AS u32x4*>(mine + (lane + 64 * i) * 16);
    __builtin_amdgcn_sched_barrier(0);
    sage::unrolled<COPIES>([&](auto i) __attribute__((always_inline)) {
        constexpr int I = decltype(i)::value;
        if (lane + 64 * I < last_chunk) sage::store_through16<I % 4 * 1024>(out + I / 4 * 4096, chunk[I]);
    });
}

// BATCH = false: one sequence per launch slot, every (sequence, KV head) cut into equal splits (see make_split).
// BATCH = true (2..64 sequences): the blocks of all sequences form one list per KV head (sequence-major, then column
// group), cut into prm.nrange equal ranges; a workgroup owns one range and runs one pass (prologue, block loop,
// epilogue) per (sequence, column group) segment its range touches, so ragged lengths cannot unbalance the launch.
// The leading arguments repeat fields of prm: explicit scalar arguments are preloaded into registers at wave launch
// (the library is built with kernel-argument preloading), so the first thing a workgroup does, fetching its sequence's
// length and node count, does not wait for a fetch of the argument block first.
template <bool BATCH, bool ONCE>
__device__ __forceinline__ void attention_workgroup(const int* __restrict__ kv_len_arg, const int* __restrict__ n_nodes_arg,
                                                    const int* __restrict__ first_node_arg,
                                                    const int64_t* __restrict__ kv_start_arg, int nslot_arg, int min_bps_arg,
                                                    int G_arg, int B_arg, int cut_arg, int light_rows_arg, const Params& prm, const int first_slab, LDS_AS Lds* lds) {
    // grid = (KV head, slot or range, sequence): the KV head is the fastest index of the launch order, and no index
    // costs a division
    const int g = blockIdx.x;
    const int id = static_cast<int>(blockIdx.y) - first_slab;   // slabs before first_slab belong to somebody else
    const int inv_G = prm.inv_G;

    auto run_segment = [&](const Segment& v) __attribute__((always_inline)) {
        // every field is wave-uniform; said to the compiler (the batched walk derives them through lane reads), so that
        // everything computed from them stays in scalar registers
        auto uni = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
        auto uni64 = [&](uint64_t x) __attribute__((always_inline)) {
            return (static_cast<uint64_t>(static_cast<uint32_t>(uni(static_cast<int>(x >> 32)))) << 32) |
                   static_cast<uint32_t>(uni(static_cast<int>(static_cast<uint32_t>(x))));
        };
        Segment sg;
        sg.b = uni(v.b); sg.g = g; sg.L = uni(v.L); sg.n = uni(v.n); sg.node0 = uni(v.node0); sg.rows = uni(v.rows); sg.cg = uni(v.cg);
        sg.begin = uni(v.begin); sg.count = uni(v.count); sg.cache_blocks = uni(v.cache_blocks);
        sg.kv_start = static_cast<long>(uni64(static_cast<uint64_t>(v.kv_start)));
        sg.slot = uni(v.slot);
        if (BATCH) __syncthreads();                          // the previous segment's epilogue has left the ring
        // A batched workgroup calls this in a loop.  Everything that depends only on the thread index would be
        // loop-invariant, and the compiler hoists all of it out of the loop and keeps it alive across the whole pass.
        // The thread index is therefore made opaque per pass, and its derived values are recomputed.
        int tid = static_cast<int>(threadIdx.x);
        if (BATCH) asm volatile("" : "+v"(tid));
        // (a kernel without ONCE has one pass only: both behind a flag cost 0.15 us of 10.6 at 4096 positions, 3 % of the short batches)
        if (ONCE && sg.L > prm.once_past && sg.rows <= ROWS_PER_WG) attention_pass<!BATCH, true>(prm, lds, sg, inv_G, tid);
        else attention_pass<!BATCH, false>(prm, lds, sg, inv_G, tid);
    };

    if (!BATCH) {
        const int slot = id;
        const int b = blockIdx.z;
        // the three per-sequence words are requested together and waited for once: the empty statement needs all of
        // them in scalar registers at one point (readfirstlane: uniform values, wherever the compiler loaded them)
        int len_b = __builtin_amdgcn_readfirstlane(kv_len_arg[b]);
        int n_b = __builtin_amdgcn_readfirstlane(n_nodes_arg[b]);
        const int64_t start_w = kv_start_arg[b];
        int start_lo = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(start_w)));
        int start_hi = __builtin_amdgcn_readfirstlane(static_cast<int>(start_w >> 32));
        int f_b = first_node_arg ? __builtin_amdgcn_readfirstlane(first_node_arg[b]) : 0;   // (a uniform branch on an argument)
        arguments_here(prm);
        asm("" : "+s"(len_b), "+s"(n_b), "+s"(start_lo), "+s"(start_hi), "+s"(f_b));
        const long start_b = (static_cast<long>(start_hi) << 32) | static_cast<uint32_t>(start_lo);
        const int L = len_b > 0 ? len_b : 0;
        const Split sp = make_split(n_b, f_b, L, G_arg, nslot_arg, static_cast<unsigned>(cut_arg), min_bps_arg);
        int split = slot >> 1, cg = slot & 1;
        if (sp.col_groups == 1) {
            split = slot;
            cg = 0;
        } else if (sp.col_groups != 2) {
            split = per_group(slot, sp.col_groups);
            cg = slot - split * sp.col_groups;
        }
        if (sp.col_groups > nslot_arg) return;              // host guarantees nslot >= the largest group count
        const int begin = split * sp.blocks_per_split;
        if (begin >= sp.blocks) return;
        run_segment(Segment{b, g, L, sp.n, sp.first, sp.rows, cg, begin, min(sp.blocks - begin, sp.blocks_per_split), blocks_of(L),
                            start_b, (b * prm.Hkv + g) * nslot_arg + cg * sp.max_split + split});
    } else {
        const int lane = threadIdx.x & 63;
        int r0, r1;                                          // this workgroup's range of the line
        uint64_t todo;                                       // the sequences that it touches
        struct { int nodes, L, start_lo, start_hi, at, seg, costs, groups_before; } now;
        {
            const BatchShape bs = make_batch_shape<true>(kv_len_arg, n_nodes_arg, first_node_arg, kv_start_arg, B_arg, cut_arg, min_bps_arg, G_arg,
                                                         light_rows_arg, lane, [&]() __attribute__((always_inline)) { arguments_here(prm); });
            r0 = id * bs.q;
            r1 = min(bs.total, r0 + bs.q);
            if (r0 >= r1) return;
            todo = __ballot(bs.at < r1 && bs.at + bs.length > r0);
            // What a pass needs of its sequence waits in LDS, not in registers, which the passes take all of.  (Every wave writes
            // all of it and reads what it wrote itself: no barrier.)
            const int nodes = bs.n << 8 | bs.first, costs = bs.cost << 8 | bs.last_cost << 4 | bs.col_groups;
            lds->seq[lane] = i32x4{nodes, bs.L, bs.start_lo, bs.start_hi};
            lds->line[lane] = i32x4{bs.at, bs.seg, costs, bs.groups_before};
            const int b = __builtin_ctzll(todo);             // (the first pass does not wait for LDS)
            auto of = [b](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(x, b); };
            now = {of(nodes), of(bs.L), of(bs.start_lo), of(bs.start_hi), of(bs.at), of(bs.seg), of(costs), of(bs.groups_before)};
        }
        while (true) {                                       // (todo is not empty: a range has positions)
            const int b = __builtin_ctzll(todo);
            const int n_b = now.nodes >> 8, f_b = now.nodes & 255, L_b = now.L, seg = now.seg, cgs_b = now.costs & 15;
            const long start_b = (static_cast<long>(now.start_hi) << 32) | static_cast<uint32_t>(now.start_lo);
            int at = now.at, slot_b = g * nslot_arg + id + now.groups_before;
            for (int cg = 0; cg < cgs_b; ++cg) {
                const int cost = cg + 1 == cgs_b ? now.costs >> 4 & 15 : now.costs >> 8;
                const int block0 = at + SEG_COST * cost;     // position of the segment's first block
                const int lo = blocks_until(r0 - block0, cost), hi = min(seg - SEG_COST, blocks_until(r1 - block0, cost));
                if (lo < hi)
                    run_segment(Segment{b, g, L_b, n_b, f_b, (n_b - f_b) * G_arg, cg, lo, hi - lo, blocks_of(L_b), start_b, slot_b + cg});
                at += seg * cost;
            }
            todo &= todo - 1;
            if (todo == 0) break;
            const i32x4 s = lds->seq[__builtin_ctzll(todo)], l = lds->line[__builtin_ctzll(todo)];
            auto uni = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
            now = {uni(s.x), uni(s.y), uni(s.z), uni(s.w), uni(l.x), uni(l.y), uni(l.z), uni(l.w)};
        }
    }
}

template <bool BATCH, bool ONCE>
__global__ __launch_bounds__(THREADS) void tree_attention_bf16_kernel(const int* __restrict__ kv_len_arg,
                                                                      const int* __restrict__ n_nodes_arg,
                                                                      const int* __restrict__ first_node_arg,
                                                                      const int64_t* __restrict__ kv_start_arg, int nslot_arg,
                                                                      int min_bps_arg, int G_arg, int B_arg, int cut_arg, int light_rows_arg, const Params prm) {
    __shared__ __align__(256) Lds lds;
    attention_workgroup<BATCH, ONCE>(kv_len_arg, n_nodes_arg, first_node_arg, kv_start_arg, nslot_arg, min_bps_arg, G_arg, B_arg, cut_arg, light_rows_arg, prm, 0,
                               (LDS_AS Lds*)&lds);
}

// The same launch carrying the planning of the next tree along (sage_tree_attention_with_plan): the grid has extra
// slabs of workgroups ahead of the attention's own (blockIdx.y < plan_slabs), one workgroup of which per sequence runs
// sage_build_tree_from_slices' work for that sequence, with LDS of its own, while the attention workgroups stream the
// cache.  The two halves share nothing: the tree being planned is the next step's, not the one whose mask the
// attention reads.  A step is a chain of dependent launches and planning is two of them; inside this launch it costs
// no launch and, as long as it is shorter than the attention, no time.  The planning slabs come first in launch order:
// when the attention's own workgroups fill every CU, the one that has to wait for a free CU is then the attention's
// last (a sequence's final split, seldom a full one), and it waits for the short planning workgroup, not the other
// way round.
constexpr int PLAN_LDS_KEYS = 2400;     // short lists staged in LDS (k = 16 at 152064 tokens: 2384)
constexpr int PLAN_OWN = 4;              // slices per lane: up to 256 slices per draft row
struct PlanLds {                         // (a planning workgroup uses the same LDS as an attention workgroup)
    uint64_t keys[PLAN_LDS_KEYS];
    sage::topk::PickShared pick;
    float row[2];
};
struct PlanShared {
    static constexpr int LDS_KEYS = PLAN_LDS_KEYS;
    uint64_t* keys;
    sage::topk::PickShared& pick;
    float& row_m;
    float& row_Z;
};
template <bool BATCH, bool ONCE>
__global__ __launch_bounds__(THREADS) void tree_attention_plan_kernel(const int* __restrict__ kv_len_arg,
                                                                      const int* __restrict__ n_nodes_arg,
                                                                      const int64_t* __restrict__ kv_start_arg, int nslot_arg,
                                                                      int min_bps_arg, int G_arg, int plan_slabs, int B_arg, int cut_arg, int light_rows_arg,
                                                                      const Params prm, const sage::PlanArgs pl) {
    __shared__ __align__(256) union Both {
        Lds attention;
        PlanLds plan;
        __device__ Both() {}
    } lds;
    if (static_cast<int>(blockIdx.y) < plan_slabs) {        // workgroup-uniform
        // one sequence per launch slot: the slab's first workgroup of sequence blockIdx.z; batches: slab workgroups in turn
        const int b = BATCH ? static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x)
                            : (blockIdx.x == 0 ? static_cast<int>(blockIdx.z) : prm.B);
        if (b >= prm.B) return;
        PlanShared sh{lds.plan.keys, lds.plan.pick, lds.plan.row[0], lds.plan.row[1]};
        sage::plan_sequence<PLAN_OWN, THREADS>(b, pl, sh);
        return;
    }
    attention_workgroup<BATCH, ONCE>(kv_len_arg, n_nodes_arg, nullptr, kv_start_arg, nslot_arg, min_bps_arg, G_arg, B_arg, cut_arg, light_rows_arg, prm, plan_slabs,
                               (LDS_AS Lds*)&lds.attention);   // a verify pass: every node
}

// Merge the splits of one (sequence, node, query head) in split order and write bf16.  One wave per row:
// lane = split for the (max, sum) pairs and their weights, lane = pair of output dims for the accumulation.
// Every partial of the row is requested before the first one is used, so the merge costs one memory round trip.
// ROWS = rows (waves) per workgroup.  MAXS = splits handled per pass (one per lane for the (max, sum) pairs, one
// register each for the accumulation); the host picks the smallest instantiation that covers the launch's slot
// count, which keeps the register count, and with it the number of resident waves, in proportion to the work.
constexpr int MERGE_ROWS_SINGLE = 4;     // one sequence: many small workgroups spread best over the CUs
constexpr int MERGE_ROWS_BATCH = 4;      // (16 rows per workgroup measured 6 % slower on the ragged batch of 8)
constexpr int MERGE_PHASES_BATCH = 32;   // batches: workgroups per (sequence, KV head), each walking the live rows; a
                                         // single sequence gets a wave per possible row (fewer measured no faster)
// A pass asks for as many splits as there are, in steps of MERGE_STEP, where it takes up to MERGE_STEP_UPTO: a batch has 5 to 13 of the 32
// that its instantiation is for, a tree of 64 nodes 16 (whole call: three sequences of 301 to 1999 positions 13.3 -> 12.8 us, seven of
// 300 to 1300 17.1 -> 16.3, seven of 2500 to 8700 with 64 nodes 104 -> 98; 80 layers of 64 nodes 5.94 -> 5.91 ms).  Beyond that the choice
// costs what it saves (41 of 48 splits, ten calls of a drafting pass: 79.4 -> 80.2 us).
constexpr int MERGE_STEP = 8, MERGE_STEP_UPTO = 32;
template <int MAXS, bool BATCH, int ROWS>
__global__ __launch_bounds__(64 * ROWS) void tree_attention_merge_kernel(const int* __restrict__ kv_len_arg,
                                                                         const int* __restrict__ n_nodes_arg,
                                                                         const int* __restrict__ first_node_arg, int nslot_arg,
                                                                         int min_bps_arg, int G_arg, int phases_arg, int B_arg, int cut_arg, int light_rows_arg,
                                                                         const Params prm) {
    static_assert(MAXS <= 64, "one split per lane, one register per split");
    // As in the main kernel, a KV head's blocks are congruent modulo the KV-head count, so with 8 KV heads they run on
    // the XCD whose L2 still holds that head's partials.  Rows of a KV head are numbered as there: node * G + head-in-group.
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // a row's address is wave-uniform: scalar registers
    const int g = blockIdx.x;                                // grid = (KV head, phase, sequence), as in the main kernel
    const float c = prm.scale_log2e;

    // One row: `first_row` = the row in the first of its nsplit partials, the others one slot after the other.
    auto merge_row = [&](int b, int node, int hg, const unsigned char* first_row, int nsplit_v) __attribute__((always_inline)) {
        // wave-uniform by construction; said to the compiler, which cannot see it through the lane exchanges of a batch
        const uintptr_t first_v = reinterpret_cast<uintptr_t>(first_row);
        const uintptr_t first =
            (static_cast<uintptr_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(first_v >> 32)))) << 32) |
            static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(first_v)));   // (the builtin returns int)
        const int nsplit = __builtin_amdgcn_readfirstlane(nsplit_v);
        float2 o = make_float2(0.f, 0.f);
        float m_all = -INFINITY, l_all = 0.f;
        // The splits from s0 on, `cnt` of them, in N registers.
        auto pass = [&](auto n, int s0, int cnt) __attribute__((always_inline)) {
            constexpr int N = decltype(n)::value;
            float ms = -INFINITY, ls = 0.f;
            // The row's partials of this pass as one buffer: uniform base (partial s0), 32-bit offsets, and a size that ends
            // with the row's extent in its last split, so that a load for a split past the last one is answered with zeros
            // by the bounds check instead of by memory.  One add and one load instruction per split.
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
                reinterpret_cast<unsigned char*>(first + static_cast<size_t>(s0) * PART_SLOT_B), 0,
                static_cast<int>(static_cast<unsigned>(cnt - 1) * PART_SLOT_B + PART_ROW_B), 0x00020000);
            {
                const u32x2 pair = __builtin_amdgcn_raw_buffer_load_b64(rows, static_cast<unsigned>(lane) * PART_SLOT_B + D * 2u, 0, 0);
                ms = lane < cnt ? __uint_as_float(pair[0]) : -INFINITY;
                ls = lane < cnt ? __uint_as_float(pair[1]) : 0.f;
            }
            unsigned v[N];                                   // two bf16 output dims of split s
            unsigned off = 4u * lane;                        // the whole offset goes through the per-lane operand: that one is
            asm volatile("" : "+v"(off));                    // bounds-checked, the scalar offset operand is not.  (Opaque, or the
#pragma unroll                                               // offsets are kept in a register each for all the passes below.)
            for (int s = 0; s < N; ++s) {
                v[s] = __builtin_amdgcn_raw_buffer_load_b32(rows, off, 0, 0);
                off += PART_SLOT_B;
            }
            __builtin_amdgcn_sched_barrier(0);               // every load is out before the first wait: one round trip
            const float m_blk = sage::wave_max(ms);
            const float m_new = fmaxf(m_all, m_blk);
            const float keep = (m_all == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((m_all - m_new) * c);
            const float w = (ms == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((ms - m_new) * c);
            l_all = l_all * keep + sage::wave_sum(w * ls);
            o.x *= keep; o.y *= keep;
            m_all = m_new;
#pragma unroll
            for (int s = 0; s < N; ++s) {
                const float ws = sage::lane_value(w, s);        // split s's weight, through a scalar register
                o.x += ws * __uint_as_float(v[s] << 16);
                o.y += ws * __uint_as_float(v[s] & 0xFFFF0000u);
            }
        };
        for (int s0 = 0; s0 < nsplit; s0 += MAXS) {           // MAXS splits at a time
            const int cnt = min(MAXS, nsplit - s0);          // (uniform)
            bool done = false;
            if constexpr (MAXS <= MERGE_STEP_UPTO)
                sage::unrolled<(MAXS - 1) / MERGE_STEP>([&](auto i) __attribute__((always_inline)) {
                    constexpr int N = (decltype(i)::value + 1) * MERGE_STEP;
                    if (!done && cnt <= N) {
                        pass(std::integral_constant<int, N>{}, s0, cnt);
                        done = true;
                    }
                });
            if (!done) pass(std::integral_constant<int, MAXS>{}, s0, cnt);
        }
        const float inv = 1.0f / l_all;
        const uint32_t packed = static_cast<uint32_t>(sage::float_to_bf16_bits(o.x * inv)) |
                                (static_cast<uint32_t>(sage::float_to_bf16_bits(o.y * inv)) << 16);
        reinterpret_cast<uint32_t*>(prm.O + ((static_cast<long>(b) * SAGE_MAX_NODES + node) * prm.Hq + g * prm.G + hg) * D)[lane] = packed;
    };

    // blockIdx = (KV head, phase, sequence); a wave walks the live rows phase * ROWS + wave, + phases * ROWS,
    // ... of its (sequence, KV head), so that rows of nodes past n_nodes cost no workgroup of their own
    const int phases = phases_arg;
    const int phase = blockIdx.y;
    const int b = blockIdx.z;
    auto arguments = [&]() __attribute__((always_inline)) {  // on their way with the sizes
        asm volatile("" : : "s"(prm.part), "s"(prm.O), "s"(prm.Hq), "s"(prm.Hkv), "s"(prm.inv_G), "s"(prm.scale_log2e));
    };
    if (!BATCH) {
        int len_b = __builtin_amdgcn_readfirstlane(kv_len_arg[b]);   // requested together, waited for once
        int n_b = __builtin_amdgcn_readfirstlane(n_nodes_arg[b]);
        int f_b = first_node_arg ? __builtin_amdgcn_readfirstlane(first_node_arg[b]) : 0;
        arguments();
        asm("" : "+s"(len_b), "+s"(n_b), "+s"(f_b));
        const int L = len_b > 0 ? len_b : 0;
        const Split sp = make_split(n_b, f_b, L, G_arg, nslot_arg, static_cast<unsigned>(cut_arg), min_bps_arg);
        const int m = phase * ROWS + wave;                   // a wave per row that a tree can have
        if (sp.col_groups > nslot_arg || m >= sp.rows) return;
        const int cg = static_cast<int>(static_cast<unsigned>(m) / ROWS_PER_WG), node = (m * prm.inv_G) >> 16;
        merge_row(b, sp.first + node, m - node * G_arg,
                  prm.part + slot_at((b * prm.Hkv + g) * nslot_arg + cg * sp.max_split) + static_cast<unsigned>(m) % ROWS_PER_WG * PART_ROW_B,
                  sp.count());
    } else {
        const BatchShape bs = make_batch_shape<false>(kv_len_arg, n_nodes_arg, first_node_arg, nullptr, B_arg, cut_arg, min_bps_arg, G_arg, light_rows_arg, lane,
                                                      arguments);
        const int first_b = __builtin_amdgcn_readlane(bs.first, b);
        const int live = (__builtin_amdgcn_readlane(bs.n, b) - first_b) * G_arg;
        const int seg = __builtin_amdgcn_readlane(bs.seg, b), at = __builtin_amdgcn_readlane(bs.at, b);
        const int last_cost = __builtin_amdgcn_readlane(bs.last_cost, b);
        const int slot_b = g * nslot_arg + __builtin_amdgcn_readlane(bs.groups_before, b);
        for (int m = phase * ROWS + wave; m < live; m += phases * ROWS) {
            const int cg = static_cast<int>(static_cast<unsigned>(m) / ROWS_PER_WG);
            const int cost = m - m % ROWS_PER_WG + ROWS_PER_WG < live ? bs.cost : last_cost;
            const int u0 = at + cg * seg * bs.cost + SEG_COST * cost;   // first block of segment (b, cg)
            const int s_first = div_floor(u0, bs.q), node = (m * prm.inv_G) >> 16;
            merge_row(b, first_b + node, m - node * G_arg, prm.part + slot_at(slot_b + s_first + cg) + static_cast<unsigned>(m) % ROWS_PER_WG * PART_ROW_B,
                      div_floor(u0 + (seg - SEG_COST - 1) * cost, bs.q) - s_first + 1);
        }
    }
}

}  // namespace

namespace sage {

// Launch shape.  A single sequence (and batches of more than 64): slots = workgroups per (sequence, KV head); a slot is
// (KV split, column group); the sequence is cut into about one workgroup per CU (one round, no tail).
// Batches of 2..64 sequences: the tile list of all sequences is cut into `nrange` ranges per KV head, about one
// workgroup per CU in total whatever the lengths turn out to be on the device, and the partial slots of a KV head are one
// per range plus one per (sequence, column group), the most that range and segment boundaries can produce together.
// A range is at least MIN_RANGE_TILES positions, the prologue and epilogue of the pass that it pays anyway: as long as CUs are
// idle, shorter ranges end sooner until they are about that long.  Attention call with the four-wave kernel before this one, us, at
// (SEG_COST blocks, MIN_RANGE_TILES) = (8, 4), (6, 3), (5, 2), (4, 2): three sequences of 301-1999 tokens 14.7, 14.3, 14.0, 13.6; two of
// 212 and 613 13.0, 11.5, 11.7, 12.1; eight of 2205-12133 56.0, 53.4, 54.1, 55.3; six of 500-4000 23.3, 23.5, 22.9, 24.0; twelve of
// 300-5000 with 30 nodes 58.2, 57.7, 59.1, 59.0.  With this one at (6, 3) and (6, 2): the three 14.6 and 13.8, two
// of 4096 and 3500 and other batches the same; but a step with four such calls over the three 77.3 and 77.2, and a cut elsewhere gives
// other bits (0.37 % of the norm).
// The workspace, of which the size stays, counts CAP_SEGMENT_TILES per segment and CAP_RANGE_TILES per range of the longest
// lengths allowed.
constexpr int MAX_BATCH_LANES = 64;      // a lane per sequence in make_batch_shape
constexpr int TILE = 64;                 // tokens: the unit in which the host counts
constexpr int MIN_RANGE_TILES = 3;       // 64-token positions of the line, pass cost included
constexpr int CAP_RANGE_TILES = 8;
constexpr int CAP_SEGMENT_TILES = 4;
struct LaunchShape { int nslot, min_tiles_per_split, nrange; bool batch; };
LaunchShape attention_bf16_shape(int B, int Hkv, int G, int max_kv_len) {
    const int max_groups = (SAGE_MAX_NODES * G + ROWS_PER_WG - 1) / ROWS_PER_WG;
    const int tiles = (max_kv_len + TILE - 1) / TILE + 1;
    LaunchShape sh;
    sh.batch = B >= 2 && B <= MAX_BATCH_LANES;
    sh.nrange = 0;
    if (sh.batch) {
        long want = 256 / Hkv;
        if (want < 1) want = 1;
        const long cap = (static_cast<long>(B) * (tiles + CAP_SEGMENT_TILES) * max_groups + CAP_RANGE_TILES - 1) / CAP_RANGE_TILES;
        if (want > cap) want = cap;
        sh.nrange = static_cast<int>(want);
        sh.min_tiles_per_split = MIN_RANGE_TILES;
        sh.nslot = sh.nrange + B * max_groups;
        return sh;
    }
    if (B <= 1) {
        long want = 256 / Hkv;
        if (want < max_groups) want = max_groups;
        const long cap = static_cast<long>(tiles) * max_groups;
        if (want > cap) want = cap;
        sh.nslot = static_cast<int>(want);
        sh.min_tiles_per_split = 1;
    } else {
        const double est_tiles = 0.6 * B * Hkv * static_cast<double>(tiles);    // ragged batches average below the maximum
        long tps = static_cast<long>(est_tiles / 256.0) + 1;       // about one workgroup per CU in total
        if (tps < 4) tps = 4;
        if (tps > tiles) tps = tiles;
        sh.min_tiles_per_split = static_cast<int>(tps);
        sh.nslot = static_cast<int>((tiles + tps - 1) / tps) * max_groups;
    }
    if (sh.nslot > 256) sh.nslot = 256;               // the merge handles any count; this bounds the workspace
    if (sh.nslot < max_groups) sh.nslot = max_groups;
    return sh;
}

size_t attention_bf16_workspace_bytes(int B, int Hkv, int G, int max_kv_len) {
    const LaunchShape sh = attention_bf16_shape(B, Hkv, G, max_kv_len);
    return (sh.batch ? static_cast<size_t>(1) : static_cast<size_t>(B)) * Hkv * sh.nslot * static_cast<size_t>(PART_SLOT_B);
}

// Whether the attention launch can carry this planning along: a lane holds at most PLAN_OWN slices.
bool attention_bf16_can_carry_plan(const PlanArgs& pl) { return pl.nunits <= 64 * PLAN_OWN; }

// plan == nullptr: the attention alone.  Otherwise the caller has checked attention_bf16_can_carry_plan(*plan).
int tree_attention_bf16(const void* Q, const void* Kc, const void* Vc, const void* Kt, const void* Vt, void* O, int B,
                        int Hq, int Hkv, int d, const int64_t* kv_start, const int* kv_len, int max_kv_len,
                        long kv_token_stride, long kv_head_stride, const uint64_t* anc_mask, const int* n_nodes,
                        const int* first_node, float scale, void* workspace, size_t workspace_bytes, hipStream_t stream,
                        const PlanArgs* plan) {
    const int G = Hq / Hkv;
    if (d != D || G < 1 || G > 16) return SAGE_UNSUPPORTED;   // 64 nodes x 16 heads per KV head = 4 groups of 256 rows
    if ((kv_token_stride % 8) != 0 || (kv_head_stride % 8) != 0) return SAGE_INVALID_ARG;
    if (kv_token_stride > (1L << 24)) return SAGE_UNSUPPORTED;   // the byte offsets inside a 32-token block are 32-bit
    if (!aligned(Q, 16) || !aligned(Kc, 16) || !aligned(Vc, 16) || !aligned(Kt, 16) || !aligned(Vt, 16) || !aligned(workspace, 16))
        return SAGE_INVALID_ARG;
    if (workspace_bytes < attention_bf16_workspace_bytes(B, Hkv, G, max_kv_len)) return SAGE_WORKSPACE_TOO_SMALL;
    if (Hq > 65535 || B > 65535) return SAGE_UNSUPPORTED;

    Params p;
    p.Q = static_cast<const uint16_t*>(Q); p.Kc = static_cast<const uint16_t*>(Kc); p.Vc = static_cast<const uint16_t*>(Vc);
    p.Kt = static_cast<const uint16_t*>(Kt); p.Vt = static_cast<const uint16_t*>(Vt); p.O = static_cast<uint16_t*>(O);
    p.kv_start = kv_start; p.kv_len = kv_len; p.anc_mask = anc_mask; p.n_nodes = n_nodes;
    p.first_node = plan ? nullptr : first_node;
    p.part = static_cast<unsigned char*>(workspace);
    p.kv_token_stride = kv_token_stride; p.kv_head_stride = kv_head_stride;
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.G = G; p.inv_G = (65536 + G - 1) / G;
    const LaunchShape sh = attention_bf16_shape(B, Hkv, G, max_kv_len);
    p.nslot = sh.nslot;
    p.min_blocks_per_split = sh.min_tiles_per_split * (TILE / BLK);
    p.scale_log2e = scale * 1.4426950408889634f;
    p.once_past = static_cast<int>(READ_ONCE_BYTES / (static_cast<long>(B) * Hkv * (2 * ROW_B)));

    p.nrange = sh.nrange;
    // what the kernels need to cut a sequence or a batch (see make_split and make_batch_shape)
    const bool by_product = max_kv_len < (1 << 27) && (p.nslot % 2 == 0 || (SAGE_MAX_NODES * G <= ROWS_PER_WG && p.nslot > 1));
    const int cut = sh.batch ? sh.nrange : by_product ? static_cast<int>(inverse(p.nslot)) : 0;
    // (blocks of different costs only where the line has less than 2^31 positions whatever the lengths are)
    const int light_rows = max_kv_len < (1 << 25) ? LIGHT_ROWS : 1 << 30;
    static_assert(MAX_BATCH_LANES * 4L * ((1L << 25) / BLK + 2 + SEG_COST) * HEAVY_COST + TAIL_BLOCKS * LIGHT_COST < (1L << 31), "64 sequences of four groups");
    const int own_slabs = sh.batch ? p.nrange : p.nslot;
    const dim3 block(THREADS);
    auto launch = [&](auto once) {
        constexpr bool ONCE = decltype(once)::value;
        if (plan) {
            // planning workgroups in slabs of their own ahead of the attention's: one slab whose first workgroup of every
            // sequence plans (one sequence per launch slot), or as many slabs as B workgroups need (batches)
            const int plan_slabs = sh.batch ? (B + Hkv - 1) / Hkv : 1;
            const dim3 grid(Hkv, plan_slabs + own_slabs, sh.batch ? 1 : B);
            if (sh.batch)
                hipLaunchKernelGGL((tree_attention_plan_kernel<true, ONCE>), grid, block, 0, stream, kv_len, n_nodes, kv_start, p.nslot,
                                   p.min_blocks_per_split, G, plan_slabs, B, cut, light_rows, p, *plan);
            else
                hipLaunchKernelGGL((tree_attention_plan_kernel<false, ONCE>), grid, block, 0, stream, kv_len, n_nodes, kv_start, p.nslot,
                                   p.min_blocks_per_split, G, plan_slabs, B, cut, light_rows, p, *plan);
        } else {
            const dim3 grid(Hkv, own_slabs, sh.batch ? 1 : B);
            if (sh.batch)
                hipLaunchKernelGGL((tree_attention_bf16_kernel<true, ONCE>), grid, block, 0, stream, kv_len, n_nodes, first_node, kv_start, p.nslot,
                                   p.min_blocks_per_split, G, B, cut, light_rows, p);
            else
                hipLaunchKernelGGL((tree_attention_bf16_kernel<false, ONCE>), grid, block, 0, stream, kv_len, n_nodes, first_node, kv_start, p.nslot,
                                   p.min_blocks_per_split, G, B, cut, light_rows, p);
        }
    };
    if (max_kv_len > p.once_past) launch(std::true_type{});
    else launch(std::false_type{});
    if (hipGetLastError() != hipSuccess) return SAGE_LAUNCH_FAILED;
    const int mrows = sh.batch ? MERGE_ROWS_BATCH : MERGE_ROWS_SINGLE;
    const int row_blocks = (SAGE_MAX_NODES * G + mrows - 1) / mrows;
    const int want_phases = sh.batch ? MERGE_PHASES_BATCH : row_blocks;
    p.merge_phases = row_blocks < want_phases ? row_blocks : want_phases;
    const dim3 mgrid(Hkv, p.merge_phases, B), mblock(64 * mrows);
    const int max_tiles = (max_kv_len + TILE - 1) / TILE + 1;
    int most = sh.batch ? p.nrange : p.nslot;         // upper bound of the splits of a row: no more than slots, or tiles
    if (most > max_tiles) most = max_tiles;
    // Batches: more than 32 splits (seldom: a sequence with nearly the whole batch's tokens) take several passes of 32, which
    // keeps more waves resident.  A single sequence has few waves to keep, and a second pass is a second round trip to
    // memory: up to 64 splits in one (41 splits of 7 to 21 rows x 4 KV heads: 4.6 -> 4.1 us).
    if (sh.batch) {
        if (most <= 8) hipLaunchKernelGGL((tree_attention_merge_kernel<8, true, MERGE_ROWS_BATCH>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
        else if (most <= 16) hipLaunchKernelGGL((tree_attention_merge_kernel<16, true, MERGE_ROWS_BATCH>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
        else hipLaunchKernelGGL((tree_attention_merge_kernel<32, true, MERGE_ROWS_BATCH>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
    } else {
        if (most <= 8) hipLaunchKernelGGL((tree_attention_merge_kernel<8, false, MERGE_ROWS_SINGLE>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
        else if (most <= 16) hipLaunchKernelGGL((tree_attention_merge_kernel<16, false, MERGE_ROWS_SINGLE>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
        else if (most <= 32) hipLaunchKernelGGL((tree_attention_merge_kernel<32, false, MERGE_ROWS_SINGLE>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
        else if (most <= 48) hipLaunchKernelGGL((tree_attention_merge_kernel<48, false, MERGE_ROWS_SINGLE>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
        else hipLaunchKernelGGL((tree_attention_merge_kernel<64, false, MERGE_ROWS_SINGLE>), mgrid, mblock, 0, stream, kv_len, n_nodes, p.first_node, p.nslot,
                               p.min_blocks_per_split, G, p.merge_phases, B, cut, light_rows, p);
    }
    return launch_status();
}

}  // namespace sage
