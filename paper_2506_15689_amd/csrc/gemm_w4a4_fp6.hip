// Prefill INT4 x INT4 -> INT32 GEMM on the f8f6f4 matrix-core path (paper Sec. 5.2; Fig. 6; Eq. 14).
//
// Both operands arrive in the fp6 operand form of fp6_pack.hip: code q stored as the e2m3 number q/8.
// v_mfma_f32_16x16x128_f8f6f4 with two fp6 operands runs at twice the int8 rate and its fp32 accumulator
// holds S = sum_k (qa/8)(qb/8) exactly (multiples of 1/64, S < 2^17 for K <= 32768).  The integer
// accumulator of the INT4 product is ACC = 64*S; the epilogue de-quantises exactly as the int8 kernels do.
// (16 x 16 x 128 and not 32 x 32 x 64: the chip's power sets the clock under such a loop, and a register-resident one on
// code-valued operands runs at 8.7 POP/s in this shape, 7.6 in the other (in longer launches, basq_diag_mfma_f6, 7.9 .. 8.5).  Products with the weights in the caches, this kernel
// against its predecessor on 32 x 32 x 64, us: 4096 x 8192 x 28672 408 -> 377, 2048 x 4096 x 12288 54.7 -> 50.6, 2048 x 14336 x 4096
// 59.5 -> 54.2, 256 x 4096 x 8192 on 128 x 64 tiles 11.0 -> 9.4.)
//
// Structure: direct-to-LDS buffer loads into a ring of stages, fragments read ahead, XCD-aware tile order.  A stage holds
// 128 codes per row.  The operands are stored as 3 KB blocks of 32 rows x 128 codes (see fp6_pack.hip): a stage is filled by
// 1 KB copies of whole cache lines.  No unpacking: LDS -> registers -> MFMA.
//
// What a K-step's code looks like matters as much as what it moves.  Eight waves of a compute unit, 32 MFMAs and 12 fragments (24
// reads) a wave and step, operands in LDS: 1040 cycles with the MFMAs alone, 1066 with six direct loads a wave, 1120 with the
// reads, 1295 with a vector instruction for the address of each read.  So reads and loads stand evenly between the MFMAs, and a
// step's addresses are constants: it knows its ring stage at compile time.
#include "gemm_fp6_store.h"
#include <type_traits>

namespace basq {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int NUM_XCD = 8;
constexpr int CHUNK = 96;              // bytes of one row per stage: 128 codes
constexpr int BLOCK = 32 * CHUNK;      // one 32-row block of a stage: 2 KB of 16-byte pieces, 1 KB of 8-byte tails

#define LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// Wait until at most N of this wave's direct-to-LDS loads are outstanding and its own LDS reads have
// returned, then join the workgroup barrier (one asm block: the compiler's own barrier would wait for
// every outstanding load and serialise the ring).
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The same where the last n of this wave's stages may still be in flight, n known at run time (the last steps of a tile,
// when no further stage is requested) and uniform over the wave; PER: this wave's loads per stage.
template <int PER, int MAXN>
__device__ __forceinline__ void wait_stages_and_barrier(int n) {
    if constexpr (MAXN > 0) {
        if (n >= MAXN) { wait_loads_and_barrier<PER * MAXN>(); return; }
        wait_stages_and_barrier<PER, MAXN - 1>(n);
    } else {
        wait_loads_and_barrier<0>();
    }
}

#ifndef G6_GROUP_M
#define G6_GROUP_M 4
#endif

template <int BM, int BN, int WAVES_M, int WAVES_N, int KGROUPS, int STAGES, int MINOCC, bool SHORT>
__global__ __launch_bounds__(WAVES_M * WAVES_N * KGROUPS * 64, MINOCC) void gemm_w4a4_fp6_kernel(GemmArgs a, int tiles_m, int tiles_n) {
#if defined(__HIP_DEVICE_COMPILE__)   // the body uses device-only buffer-resource types; the host pass only needs the stub
    constexpr int WAVES = WAVES_M * WAVES_N;                  // of one K group
    constexpr int THREADS = WAVES * KGROUPS * 64;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 16, TN = WN / 16;                 // blocks of 16 rows and of 16 columns
    constexpr int OWN = (TM + KGROUPS - 1) / KGROUPS;         // row blocks of its wave tile that a wave finishes
    // The operand with more blocks is the outer one: its fragments are read half a step ahead, those of the inner one
    // as soon as their last MFMA of a step has gone (see k_step)
    constexpr bool ROWS_OUTER = TM >= TN;
    constexpr int TO = ROWS_OUTER ? TM : TN, TI = ROWS_OUTER ? TN : TM;
    // Outer blocks of a step's first part: half of them, one fewer where there are more outer than inner blocks (six at least),
    // which leaves the barrier, at a part's end, farther from the reads of the next step's operands: 256 x 256, 256 x 192, 160 x 96 and
    // 96 x 96 tiles.  us, half and one fewer: 256 x 256 4096 x 8192 x 28672 381.4 and 376.7, 256 x 192 2048 x 8192 x 12288 88.2
    // and 86.9; 96 x 96 even (320 x 4096 x 4096 9.1).
    constexpr int PART0 = TO >= 6 && TO > TI ? TO / 2 - 1 : TO / 2;
    constexpr int ROWS = BM + BN;
    constexpr int STAGE_BYTES = ROWS * CHUNK;
    constexpr int PIECES = STAGE_BYTES / 1024;                // 1 KB pieces of a stage, one wave-load each
    constexpr int A_PIECES = BM * CHUNK / 1024;               // pieces 0 .. A_PIECES-1 of a stage are activations
    // Direct loads per wave per stage, the same number for all waves: whole pieces, and of the last PIECES % WAVES pieces an equal
    // share, SHARES times 256 bytes (4 a lane); where they do not divide so, or a round holds pieces of both operands as well,
    // the waves without a piece in the last round load nothing there (see issue_one).
    constexpr int WHOLE = PIECES / WAVES, LEFT = PIECES % WAVES;
    constexpr bool BY_BLOCK = LEFT == 0 && WHOLE % 3 == 0;    // whole 32-row blocks a wave
    static_assert(!BY_BLOCK || WHOLE == 3 || A_PIECES % (3 * WAVES) == 0, "blocks of both operands in the first round at most");
    constexpr bool SHARED = LEFT != 0 && LEFT * 4 % WAVES == 0 && A_PIECES % WAVES == 0;
    constexpr bool PADDED = LEFT != 0 && !SHARED;
    constexpr int SHARES = SHARED ? LEFT * 4 / WAVES : 0;
    constexpr int LOADS = WHOLE + (PADDED ? 1 : SHARES);
    static_assert(LEFT == 0 || WHOLE * WAVES >= A_PIECES, "the last pieces are weights");
    static_assert(STAGE_BYTES % 1024 == 0, "a stage is a whole number of 1 KB pieces");
    static_assert(BM % 32 == 0 && BN % 32 == 0, "tiles are made of 32-row blocks");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile");
    static_assert(STAGES >= 3 && LOADS * (STAGES - 2) < 64, "the wait counter counts to 63");
    static_assert(ROWS * 16 <= STAGE_BYTES, "the epilogue constants live in the last stage");
    // With 128 sums a lane (256 x 256) no registers are left to carry the next tile's constants across the K loop: they go to LDS of their
    // own, two tiles' worth beside the ring.  (Carried, they were spilled, and fetched again behind a tile's last MFMA with a full
    // wait.  Whole layers, us: 4096 x 8192 x 28672 447 -> 440, 4096 x 4096 x 28672 252.7 -> 246.7, 8000 x 512 x 14240 94.3 -> 86.7.)
    constexpr bool APART = TM * TN * 4 >= 128;
    static_assert(!APART || (KGROUPS == 1 && !PADDED), "nothing else stands behind the ring");
    static_assert(KGROUPS == 1 || (BM * BN * 4 + ROWS * 16 <= STAGES * STAGE_BYTES && TM % KGROUPS == 0), "K groups exchange their sums through their rings, and each finishes row blocks");

    __shared__ __attribute__((aligned(1024))) uint8_t lds_all[KGROUPS * STAGES * STAGE_BYTES + (PADDED ? 1024 : APART ? 2 * ROWS * 16 : 0)];

    const int tid = threadIdx.x;
    const int lane = tid & 63, swave = __builtin_amdgcn_readfirstlane((tid >> 6) % WAVES);
    const int wm = swave / WAVES_N, wn = swave % WAVES_N;
    // K groups: group g of the workgroup's waves takes a contiguous part of the chunks through a ring of its own.  All take
    // the same number of steps, since they meet at the barriers; the chunks left over by the division go to the last
    // groups, and a group that has one fewer (`idle_last`) leaves the last step's MFMAs out (what it has loaded there is
    // its successor's first chunk).
    const int kgroup = KGROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane((tid >> 6) / WAVES);
    const int chunks = a.K / 128;
    const int ksteps = KGROUPS == 1 ? chunks : (chunks + KGROUPS - 1) / KGROUPS;
    const int short_groups = KGROUPS == 1 ? 0 : ksteps * KGROUPS - chunks;             // groups 0 .. short_groups - 1
    const bool idle_last = KGROUPS > 1 && kgroup < short_groups;
    const int chunk0 = KGROUPS == 1 ? 0 : kgroup * ksteps - (kgroup < short_groups ? kgroup : short_groups);
    uint8_t* const lds = lds_all + kgroup * (STAGES * STAGE_BYTES);                    // this group's ring
    int store_form = (int)a.store_form;                       // fetched here: at the end it would be a memory latency
    asm volatile("" : "+s"(store_form));
    const int rb_a = (int)((a.M + 31) >> 5), rb_w = (a.N + 31) >> 5;   // 32-row blocks per chunk of K
    const unsigned a_step = (unsigned)rb_a * BLOCK, w_step = (unsigned)rb_w * BLOCK;   // bytes from one chunk of K to the next
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.Aq6), 0, (int)(a_step * (unsigned)chunks), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.Wq6), 0, (int)(w_step * (unsigned)chunks), 0x00020000);

    // ---- tile order (XCD-aware: workgroups congruent mod 8 run on one XCD; the tiles a workgroup takes,
    // blockIdx.x + i * gridDim.x, stay congruent when the grid is a multiple of 8 and walk a compact band)
    const int total = tiles_m * tiles_n;
    auto tile_of = [&](int pid, int& tile_m, int& tile_n) {
        int t = pid;
        const int per_xcd = total / NUM_XCD;
        if (pid < per_xcd * NUM_XCD) t = (pid % NUM_XCD) * per_xcd + pid / NUM_XCD;
        constexpr int GROUP_M = G6_GROUP_M;
        const int band = t / (GROUP_M * tiles_n);
        const int first_m = band * GROUP_M;
        const int rows = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
        const int in_band = t - band * GROUP_M * tiles_n;
        // (divisions are vector instructions: without this, in some tilings everything derived from the tile stays in vector
        // registers, and every load, whose block offset must be scalar, is wrapped in a loop over the lanes' values)
        tile_m = __builtin_amdgcn_readfirstlane(first_m + in_band % rows);
        tile_n = __builtin_amdgcn_readfirstlane(in_band / rows);
    };

    // ---- direct loads: load i of wave w copies the 1 KB piece number i*WAVES + w of the stage; three
    // pieces make one 32-row block.  Which block a piece comes from is uniform over the wave, so it goes
    // into the scalar offset of the load; the per-lane part is 16 * lane, except for the 1 KB of 8-byte tails: there the 128
    // bytes of rows 0 .. 15 and of rows 16 .. 31 trade places for the groups 2 and 3, see the fragment addressing.
    // BY_BLOCK: wave w copies whole blocks, number w, WAVES + w, .. of the stage, hence an address per block (256 x 4096 x 8192 on 128 x 128
    // tiles 12.0 -> 11.6 us, 700 x 384 x 3000 5.7 -> 5.4).  All activations of a stage are requested before its weights: loads complete
    // in order, and weights that come from memory hold up activations that the caches have (half of the waves with activations
    // and the others with weights, whole layers with cold weights: 333 x 11008 x 8192 45.6 us, as built 43.3; 117 x 8192 x 23456
    // 44.5 and 42.5; 237 x 14336 x 9408 59.3 and 56.8; 1021 x 11008 x 4096 with cached ones even).
    // Blocks past the matrix are clamped to its last block.
    int soff[LOADS];                                           // scalar: block and part of each of this wave's pieces
    auto set_tile = [&](int tile_m, int tile_n) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int share = swave * SHARES + i - WHOLE;      // number of the 256 bytes among the last pieces
            const int piece = BY_BLOCK ? 3 * (i / 3 * WAVES + swave) + i % 3 : SHARED && i >= WHOLE ? WHOLE * WAVES + share / 4 : i * WAVES + swave;
            int blk = piece / 3;
            const int part = piece % 3;
            if (piece < A_PIECES) {
                blk += tile_m * (BM / 32);
                blk = blk < rb_a ? blk : rb_a - 1;
            } else {
                blk += tile_n * (BN / 32) - BM / 32;
                blk = blk < rb_w ? blk : rb_w - 1;
            }
            soff[i] = blk * BLOCK + part * 1024 + (SHARED && i >= WHOLE ? share % 4 * 256 : 0);
        }
    };
    // issue_one: load number i of a K-step: into the stage at byte stage_off of the ring, from chunk offsets koff_a / koff_w (unsigned
    // 32-bit byte offsets).  No branches, which cost tens of cycles a step: where a round holds pieces of both operands,
    // descriptor and offset are selected; waves without a piece in a padded last round load from past the end of the operand,
    // so that nothing is read, to a place in LDS that nobody reads (96 x 64, 333 x 4096 x 4096: 10.3 -> 9.4 us).  Loads of nothing take the
    // time of loads all the same, though, which shows with weights from memory: shares instead where the pieces divide (us with
    // weights from memory; in the caches.  256 x 192, six of eight waves without a piece: 2048 x 4096 x 12288 padded 61.5; 57.9, by
    // shares 60.1; 57.9, with a branch 59.8; 58.0; 1021 x 8192 x 11008 54.7; 47.3, 52.6; 47.1, 52.3; 47.8.  256 x 128, four of eight:
    // 777 x 14336 x 5008 52.9; 46.4, 50.0; 46.7, 51.1; 47.1; 2048 x 14336 x 4096 69.9; 60.6, 69.3; 61.2, 68.8; 62.7.  96 x 64:
    // 333 x 4096 x 4096 padded 11.2; 8.4, by shares 11.1; 8.9).
    // per-lane source offsets of load i (parts of blocks repeat every three loads) and of the shares
    int src_off[3], share_off[SHARES > 0 ? SHARES : 1];
#pragma unroll
    for (int i = 0; i < 3; ++i) src_off[i] = 16 * ((BY_BLOCK ? i : (i * WAVES + swave) % 3) == 2 ? lane ^ (lane >> 5) * 8 : lane);
#pragma unroll
    for (int i = 0; i < SHARES; ++i) {
        const int share = swave * SHARES + i;
        share_off[i] = 4 * ((WHOLE * WAVES + share / 4) % 3 == 2 && share % 4 >= 2 ? lane ^ 32 : lane);
    }
    const int last_off = PADDED && WHOLE * WAVES + swave >= PIECES ? (int)0xFFFFFF00u : src_off[WHOLE % 3];
    int wave_at = kgroup * (STAGES * STAGE_BYTES) + swave * (BY_BLOCK ? BLOCK : 1024);
    const bool loads_a = 3 * swave < A_PIECES;                 // (BY_BLOCK, first round)
    const __amdgpu_buffer_rsrc_t rsrc_own = loads_a ? rsrc_a : rsrc_w;
    auto issue_one = [&](int stage_off, unsigned koff_a, unsigned koff_w, int i) {
        if (SHARED && i >= WHOLE) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, LDS_PTR(lds + stage_off + WHOLE * WAVES * 1024 + (swave * SHARES + i - WHOLE) * 256), 4, share_off[i - WHOLE],
                                                     (int)(koff_w + (unsigned)soff[i]), 0, 0);
            return;
        }
        if constexpr (BY_BLOCK) {
            // the parts of a block by the load's own offset, which counts in memory and in LDS
            const bool mixed = i < 3 && 3 * WAVES > A_PIECES, is_a = mixed ? loads_a : i * WAVES < A_PIECES;
            const __amdgpu_buffer_rsrc_t rsrc = mixed ? rsrc_own : is_a ? rsrc_a : rsrc_w;
            const unsigned at = (is_a ? koff_a : koff_w) + (unsigned)soff[i / 3 * 3];
            uint8_t* dst = lds_all + wave_at + stage_off + i / 3 * (WAVES * BLOCK);
            if (i % 3 == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(dst), 16, src_off[0], (int)at, 0, 0);
            else if (i % 3 == 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(dst), 16, src_off[1], (int)at, 1024, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, LDS_PTR(dst), 16, src_off[2], (int)at, 2048, 0);
            return;
        }
        const bool last = i >= WHOLE;
        const bool mixed = i * WAVES < A_PIECES && (i + 1) * WAVES > A_PIECES;
        const bool is_a = mixed ? i * WAVES + swave < A_PIECES : i * WAVES < A_PIECES;
        uint8_t* dst = lds_all + wave_at + stage_off + i * WAVES * 1024;
        if (last) dst = i * WAVES + swave < PIECES ? dst : lds_all + KGROUPS * STAGES * STAGE_BYTES;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(is_a ? rsrc_a : rsrc_w, LDS_PTR(dst), 16, last ? last_off : src_off[i % 3],
                                                 (int)((is_a ? koff_a : koff_w) + (unsigned)soff[i]), 0, 0);
    };
    constexpr int LATER = KGROUPS == 1 && BM == 256 && BN < 256 ? 1 : 0;       // by how many half spaces a part's loads stand behind its start (see k_step)
    constexpr int SPLIT = (LOADS + 1) / 2;                     // the first half of a stage's loads (see k_step)
    // Wait until the oldest stage in flight has landed, `ahead` stages having been requested behind it at most
    auto wait_stages = [&](int ahead) { wait_stages_and_barrier<LOADS, STAGES - 2>(ahead); };
    // A tile's first step takes stage `start` of the ring, so that its last STAGES steps take stages 0 .. STAGES - 1: behind `lead`
    // steps that reckon their stage, the others have it at compile time.  Tiles of fewer steps than stages (SHORT) have a
    // kernel of their own: as a second path it cost the others registers (spilled, 256 x 256).
    constexpr int LEAD = STAGES - 2;                           // of a later tile, whose stages have landed already
    constexpr bool ROUNDS = !SHORT;                            // at least STAGES steps
    const int lead = !ROUNDS ? 0 : ksteps >= LEAD + STAGES ? LEAD + (ksteps - LEAD) % STAGES : ksteps % STAGES;
    const int start = (STAGES * 2 - lead) % STAGES;
    const unsigned kbase_a = (unsigned)chunk0 * a_step, kbase_w = (unsigned)chunk0 * w_step;
    auto issue_prologue = [&]() {
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s)
            if (s < ksteps) {
#pragma unroll
                for (int i = 0; i < LOADS; ++i) issue_one((start + s >= STAGES ? start + s - STAGES : start + s) * STAGE_BYTES, kbase_a + s * a_step, kbase_w + s * w_step, i);
            }
    };

    // ---- fragment addressing: lane (frow, fgroup) feeds k = 32*fgroup .. +31 of row frow of a 16-row half of a block:
    // 16 bytes among the pieces, 8 bytes among the tails.  LDS serves 16-byte reads of lanes {0-3, 12-15, 20-27}, {4-11, 16-19,
    // 28-31} and the same of the upper half together, 8-byte reads of 32 lanes at once.  With the groups 0, 3, 1, 2 on lanes
    // 0-15, 16-31, .. (any order will do, if both operands have the same) the first are free of bank conflicts; the second
    // are because the halves of the groups 2 and 3 have traded places.  (In the order 0, 1, 2, 3 half of the LDS cycles were conflicts.)
    const int frow = lane & 15, fgroup = (0x9C >> (2 * (lane >> 4))) & 3;      // 0, 3, 1, 2
    const int moff = 64 * frow + 16 * (fgroup ^ (frow >> 2));
    const int toff = 2048 + 256 * fgroup + 8 * frow, tflip = fgroup >> 1;
    // A wave's WN / 32 column blocks of 32: pairs of adjacent ones (64 columns, a 128-byte line of outputs), and the odd one left over
    // from behind all pairs of the tile.
    constexpr int PAIRED = WN / 64 * 2;
    auto col_block = [&](int j) { return j < PAIRED ? wn * PAIRED + j : WAVES_N * PAIRED + wn; };
    // LDS addresses of the 16-byte reads and of the 8-byte reads of either half of a block, for activations, weights and the odd
    // column block, in every second stage: everything else about a read, also the stage behind, fits its 16-bit offset.
    constexpr int BASES = (STAGES + 1) / 2;
    constexpr bool ODD = WN / 32 != PAIRED;
    struct Base { int main, tail[2]; };
    Base base_a[BASES], base_b[BASES], base_c[ODD ? BASES : 1];
    auto set_base = [&](Base& x, int b, int block) {
        const int at = kgroup * (STAGES * STAGE_BYTES) + 2 * b * STAGE_BYTES + block * BLOCK;
        x.main = at + moff;
        x.tail[0] = at + toff + 128 * tflip;
        x.tail[1] = at + toff + 128 * (1 - tflip);
        asm volatile("" : "+v"(x.main), "+v"(x.tail[0]), "+v"(x.tail[1]));
    };
#pragma unroll
    for (int b = 0; b < BASES; ++b) {
        set_base(base_a[b], b, wm * (WM / 32));
        set_base(base_b[b], b, BM / 32 + wn * PAIRED);
        if (ODD) set_base(base_c[b], b, BM / 32 + WAVES_N * PAIRED + wn);
    }
    static_assert(STAGE_BYTES + (WM / 32) * BLOCK <= 65536 && STAGE_BYTES + (WN / 32) * BLOCK <= 65536, "reach of an offset");

    // Epilogue constants, one 16-byte record per row and column of the tile: in the last stage of the ring, which the next
    // tile's first loads do not touch, or in this tile's half of the LDS behind it (APART).  Kept and read as integers: the compiler
    // puts a wait for every direct-to-LDS load in flight in front of a float-typed LDS read.
    // (with K groups, which take one tile, behind the sums that go through the first group's ring)
    int par_at = APART ? STAGES * STAGE_BYTES : KGROUPS == 1 ? (start + STAGES - 1) % STAGES * STAGE_BYTES : STAGES * STAGE_BYTES - ROWS * 16;
    // The raw values of one record per thread (rows first), requested a tile ahead of their use and converted only where they are put
    // down: a conversion behind the loads would wait for them.
    auto load_par = [&](int tile_m, int tile_n) -> v4i {
        int tid = threadIdx.x;                                // (opaque: nothing derived from it is kept across the main loop)
        asm volatile("" : "+v"(tid));
        v4i raw = {0, 0, 0, 0};
        if (tid < BM) {
            int64_t m = (int64_t)tile_m * BM + tid;
            m = m < a.M ? m : a.M - 1;
            raw = *reinterpret_cast<const v4i*>(a.meta + m);
        } else if (tid < ROWS) {
            int n = tile_n * BN + tid - BM;
            n = n < a.N ? n : a.N - 1;
            raw[0] = a.w_scale[n];
            raw[1] = a.w_zero[n];
            raw[2] = __float_as_int(a.w_sum[n]);
            if (a.out_bias) raw[3] = __float_as_int(a.out_bias[n]);
        }
        return raw;
    };
    static_assert(ROWS <= THREADS, "one record per thread");
    auto put_par = [&](v4i raw, int at) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        if (tid < BM) raw[2] = __float_as_int((float)raw[2]);
        else { raw[0] <<= 16; raw[1] <<= 16; }                    // bf16 -> fp32
        if (ROWS == THREADS || tid < ROWS) reinterpret_cast<v4i*>(lds_all + at)[tid] = raw;
    };

    // ---- persistent loop over this workgroup's tiles
    int pid = blockIdx.x;
    int tile_m, tile_n;
    tile_of(pid, tile_m, tile_n);
    set_tile(tile_m, tile_n);
    v4i par = load_par(tile_m, tile_n);
    issue_prologue();
    if (APART) put_par(par, par_at);
    bool first = true;
    while (true) {
        const int64_t m0 = (int64_t)tile_m * BM;
        const int n0 = tile_n * BN;
        v4f acc[TM][TN];
        // Operand registers: six consecutive VGPRs per fragment (the builtin takes eight, of which the instruction reads the
        // first six in this form).  The two LDS reads of a fragment land in them directly.
        v6i pa[TM], pb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) pa[i] = v6i{0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < TN; ++j) pb[j] = v6i{0, 0, 0, 0, 0, 0};
        auto read_one = [&](v6i& dst, const uint8_t* main_ptr, const uint8_t* tail_ptr) {
            const v4i m = *reinterpret_cast<const v4i*>(main_ptr);
            const v2i t = *reinterpret_cast<const v2i*>(tail_ptr);
            dst[0] = m[0]; dst[1] = m[1]; dst[2] = m[2]; dst[3] = m[3]; dst[4] = t[0]; dst[5] = t[1];
        };
        // half-block number n of an operand, in a stage given by its number (known at compile time) or by its byte offset in the ring
        auto read_half = [&](v6i& dst, const Base* base, auto stage, int n) {
            const int at = n / 2 * BLOCK;
            if constexpr (std::is_same_v<decltype(stage), int>) {
                read_one(dst, lds_all + stage + base[0].main + (at + 1024 * (n & 1)), lds_all + stage + base[0].tail[n & 1] + at);
            } else {
                const Base& x = base[stage / 2];
                read_one(dst, lds_all + x.main + (stage % 2 * STAGE_BYTES + at + 1024 * (n & 1)), lds_all + x.tail[n & 1] + (stage % 2 * STAGE_BYTES + at));
            }
            __builtin_amdgcn_sched_barrier(0);                // one at a time: neighbours would become one read with registers to be moved
        };
        auto read_a = [&](auto stage, int i) { read_half(pa[i], base_a, stage, i); };
        auto read_b = [&](auto stage, int j) {
            if (ODD && j >= 2 * PAIRED) read_half(pb[j], base_c, stage, j - 2 * PAIRED);
            else read_half(pb[j], base_b, stage, j);
        };
        auto read_outer = [&](auto st, int o) { if (ROWS_OUTER) read_a(st, o); else read_b(st, o); };
        auto read_inner = [&](auto st, int i) { if (ROWS_OUTER) read_b(st, i); else read_a(st, i); };
        auto operand = [](v6i x) { return __builtin_shufflevector(x, x, 0, 1, 2, 3, 4, 5, -1, -1); };
        auto mfma = [&](int o, int n) {
            const int i = ROWS_OUTER ? o : n, j = ROWS_OUTER ? n : o;
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(operand(pb[j]), operand(pa[i]), acc[i][j], 2, 2, 0, 0, 0, 0);
        };

#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

        // Stage 0 must have landed: on the first tile the loads of stage 1 may stay in flight; on later
        // tiles both stages were waited for before the previous epilogue's stores went out.  The barrier
        // also ends every wave's use of the epilogue constants before step 0 refills the last stage.
        if (first) {
            wait_stages(ksteps - 1);
        } else {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        // stages this tile starts with that have landed already (beyond stage 0)
        const int landed = first ? 0 : STAGES - 2;
        first = false;
        auto stage_at = [&](int i) { return (i >= STAGES ? i - STAGES : i) * STAGE_BYTES; };
        int prev = stage_at(start + STAGES - 1), cur = stage_at(start), next = stage_at(start + 1);      // stages of steps ks - 1, ks, ks + 1
        asm volatile("" : "+s"(prev), "+s"(cur), "+s"(next));    // opaque: no addresses of their own for a tile's first steps
        // the fragments the first step begins with, in the order in which its MFMAs need them
        read_inner(cur, 0);
#pragma unroll
        for (int t = 0; t < PART0; ++t) read_outer(cur, t);
#pragma unroll
        for (int t = 1; t < TI; ++t) read_inner(cur, t);

        // Part of a K-step: the MFMAs of the outer blocks from .. from + COUNT - 1.
        auto part = [&](auto from_c, auto count_c, auto&& before, auto do_loads, int fill, unsigned koff_a, unsigned koff_w, int first_load, int loads) {
            constexpr int FROM = decltype(from_c)::value, COUNT = decltype(count_c)::value, MFMAS = COUNT * TI;
#pragma unroll
            for (int t = 0; t < MFMAS; ++t) {
                before(t);
                const int n = t / COUNT, o = FROM + (n & 1 ? COUNT - 1 - t % COUNT : t % COUNT);   // back and forth: each shares an operand with the one before
                mfma(o, n);
                __builtin_amdgcn_sched_barrier(0);
                if (decltype(do_loads)::value) {
#pragma unroll
                    for (int u = 0; u < loads; ++u)
                        if ((2 * u + LATER) * MFMAS / (2 * loads) == t) issue_one(fill, koff_a, koff_w, first_load + u);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        // One K-step.  A stage is refilled from the moment every wave has passed the barrier behind its last reads: the
        // first half of the loads of stage ks + STAGES goes out with the second part of step ks, the other
        // half with the first part of step ks + 1.  The last steps, which request nothing, and the very last, which
        // reads no next stage, are copies of their own: with these tests inside a loop, two paths meet in front of MFMAs, and the
        // compiler then waits for every outstanding LDS read there -- including the ones just issued -- instead of only for the
        // operands the MFMAs use (a bubble of an LDS latency per step).
        // Reads and loads evenly between the MFMAs: all waves pass the barrier together, and with a read in front of each of the
        // first MFMAs and a load behind it LDS and loads were what they all waited for (4096 x 8192 x 28672 402 and 390 us).  A part's first
        // load directly behind its first MFMA: half a space later costs where weights come from memory (us, later and so: whole layers on
        // 160 x 96 tiles, 312 x 14336 x 12128 60.3 and 59.3, 135 x 14336 x 13488 57.7 and 56.6; product on 256 x 256, 453 x 11008 x 28576 79.3
        // and 77.8; in the caches even).  Not on 256 x 192 and 256 x 128 tiles, whose products with cached weights are up to 1 % shorter with that
        // half space (2048 x 14336 x 4096 54.8 us and 55.4, 3332 x 8192 x 6704 89.6 and 90.4), with cold ones as long (a layer that is not:
        // 410 x 11008 x 13584 62.3 and 60.6).
        unsigned koff_a = kbase_a + (STAGES - 1) * a_step, koff_w = kbase_w + (STAGES - 1) * w_step;   // the group's chunk ks + STAGES - 1
        auto k_step = [&](auto here, auto behind, auto fill0, auto fill1, auto loads0, auto loads1, auto has_next, auto&& wait) {
            constexpr int REST = TO - PART0;
            asm volatile("" : "+s"(wave_at));               // no LDS address of its own for every load of every stage
            // first part: reads the outer blocks of the second
            part(std::integral_constant<int, 0>{}, std::integral_constant<int, PART0>{},
                 [&](int t) {
#pragma unroll
                     for (int u = 0; u < REST; ++u)
                         if (u * (3 * PART0 * TI) / (4 * REST) == t) read_outer(here, PART0 + u);
                 }, loads0, fill0, koff_a, koff_w, SPLIT, LOADS - SPLIT);
            koff_a += a_step;
            koff_w += w_step;
            // every read of this stage has been issued; pass the barrier (next stage complete and visible: all but
            // the newest STAGES-2 stages have landed)
            wait();
            // second part: reads the next stage's outer blocks of its first part, and every inner block when its last MFMA has gone
            part(std::integral_constant<int, PART0>{}, std::integral_constant<int, REST>{},
                 [&](int t) {
                     if (!decltype(has_next)::value) return;
#pragma unroll
                     for (int u = 0; u < PART0; ++u)
                         if (u * (3 * REST * TI) / (4 * PART0) == t) read_outer(behind, u);
                     if (t > 0 && t % REST == 0) read_inner(behind, t / REST - 1);
                 }, loads1, fill1, koff_a, koff_w, 0, SPLIT);
            if (decltype(has_next)::value) read_inner(behind, TI - 1);
        };
        auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
        // a step on stages reckoned at run time
        auto any_step = [&](auto loads0, auto loads1, auto has_next, auto&& wait) {
            k_step(cur, next, prev, cur, loads0, loads1, has_next, wait);
            prev = cur;
            cur = next;
            next = next == (STAGES - 1) * STAGE_BYTES ? 0 : next + STAGE_BYTES;
        };
        // ... and on stage S
        auto step_on = [&](auto S, auto loads0, auto loads1, auto has_next, auto&& wait) {
            constexpr int here = decltype(S)::value, behind = (here + 1) % STAGES, before = (here + STAGES - 1) % STAGES;
            k_step(S, std::integral_constant<int, behind>{}, before * STAGE_BYTES, here * STAGE_BYTES, loads0, loads1, has_next, wait);
        };
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        if constexpr (ROUNDS) {
#pragma unroll
            for (int i = 0; i < SPLIT; ++i) issue_one(prev, koff_a, koff_w, i);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ROUNDS) {
            // the stages that were waited for before the previous tile's stores went out: no wait here, which would be one for
            // those stores as well
            int ks = 0;
            for (; ks < lead; ++ks)
                any_step(yes, yes, yes, [&]() { if (ks < landed) lds_barrier(); else wait_loads_and_barrier<LOADS * (STAGES - 2)>(); });
            auto round = [&](auto self, auto S) {
                step_on(S, yes, yes, yes, [&]() { wait_loads_and_barrier<LOADS * (STAGES - 2)>(); });
                if constexpr (decltype(S)::value + 1 < STAGES) self(self, std::integral_constant<int, decltype(S)::value + 1>{});
            };
            for (; ks + STAGES < ksteps; ks += STAGES) {
                // The step's code on a 16-byte boundary: where it begins in the middle of an 8-byte pair, which code anywhere in front
                // of it decides, a step of one workgroup per compute unit is 1 % longer (2048 x 4096, K = 14336: 61.2 and 62.3 us).
                asm volatile(".p2align 4");
                round(round, std::integral_constant<int, 0>{});
            }
            // the last STAGES steps, whose requests run out
            auto last = [&](auto self, auto S) {
                constexpr int s = decltype(S)::value;
                if constexpr (s + 1 < STAGES) {
                    auto wait = [&]() { wait_loads_and_barrier<LOADS * (STAGES - 2 - s)>(); };
                    if constexpr (s == 0) step_on(S, yes, no, yes, wait);
                    else step_on(S, no, no, yes, wait);
                    self(self, std::integral_constant<int, s + 1>{});
                } else if (!idle_last) {
                    step_on(S, no, no, no, [&]() { wait_loads_and_barrier<0>(); });
                } else {
                    wait_loads_and_barrier<0>();
                }
            };
            last(last, std::integral_constant<int, 0>{});
        } else {
            int ks = 0;
            auto wait = [&]() { wait_stages(ksteps - 2 - ks); };
            for (; ks + 1 < ksteps; ++ks) any_step(no, no, yes, wait);
            if (!idle_last) any_step(no, no, no, wait);
            else wait_stages(0);
        }
        // every wave has passed the last step's barrier, after which nothing reads the ring: put this tile's constants there
        // (APART: they stand behind it since the tile in front) and request the next tile's first stages, so that their latency
        // hides behind this tile's epilogue
        if (!APART) put_par(par, par_at);
        // K groups: a wave finishes the row blocks of its share, OWN of them, and hands its sums of the others to the waves
        // of the same position in the other groups, through its own ring.  (All sums are exact: any order gives the same bits.)
        const int own0 = kgroup * OWN;
        auto xch_at = [&](int i, int j) { return (((swave * TM + i) * TN + j) * 64 + lane) * 16; };
        if constexpr (KGROUPS > 1) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                if (i / OWN != kgroup) {
#pragma unroll
                    for (int j = 0; j < TN; ++j) *reinterpret_cast<v4i*>(lds + xch_at(i, j)) = __builtin_bit_cast(v4i, acc[i][j]);
                }
        }
        const int next_pid = pid + gridDim.x;
        const bool more = KGROUPS == 1 && next_pid < total;
        int next_m = 0, next_n = 0;
        v4i next_par = {0, 0, 0, 0};
        if (more) {
            tile_of(next_pid, next_m, next_n);
            set_tile(next_m, next_n);
            (APART ? next_par : par) = load_par(next_m, next_n);
            issue_prologue();
        }

        // ---- epilogue (which output an accumulator register holds: gemm_fp6_store.h)
        if (!APART) lds_barrier();                                // LDS only: the next tile's loads stay in flight
        if constexpr (KGROUPS > 1) {
            // the first OWN blocks of `acc` become the sums of this wave's share
#pragma unroll
            for (int i = OWN; i < TM; ++i)
                if (i / OWN == kgroup)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i % OWN][j] = acc[i][j];
#pragma unroll
            for (int o = 1; o < KGROUPS; ++o) {
                const uint8_t* ring = lds_all + (kgroup + o < KGROUPS ? kgroup + o : kgroup + o - KGROUPS) * (STAGES * STAGE_BYTES);
#pragma unroll
                for (int i = 0; i < OWN; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const v4i v = *reinterpret_cast<const v4i*>(ring + xch_at(own0 + i, j));
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i][j][e] += __int_as_float(v[e]);
                    }
            }
        }
        const int row0 = wm * WM + own0 * 16;                     // of the rows this wave finishes
        // (re)derived per tile from an opaque copy of the lane index: everything computed from it below
        // would otherwise be hoisted out of the tile loop and held in registers across the main loop
        int elane = tid;
        asm volatile("" : "+v"(elane));
        elane &= 63;
        const int tok = elane & 15, quad = elane >> 4;
        const v4i* const lrow_par = reinterpret_cast<const v4i*>(lds_all + par_at);
        const v4i* const lcol_par = lrow_par + BM;
        v4i rp[OWN];                                              // scale, lower bound, row sum of this lane's tokens
#pragma unroll
        for (int i = 0; i < OWN; ++i) rp[i] = lrow_par[row0 + i * 16 + tok];
        auto dequant = [&](float s64, v4i row, v4i col) {
            // 64 * S is the integer accumulator, exactly
            const float t = fmaf(64.0f, s64, -(__int_as_float(col[1]) * __int_as_float(row[2])));
            return fmaf(__int_as_float(row[0]) * __int_as_float(col[0]), t,
                        fmaf(__int_as_float(row[1]), __int_as_float(col[2]), __int_as_float(col[3])));
        };
        auto& sums = reinterpret_cast<v4f(&)[OWN][TN]>(acc);
        if (a.acc_out) store_accumulators16<OWN, TN, BM>(a, m0, n0, row0, elane, sums, col_block);
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        // Outputs into registers, where they take the accumulators' place, then the stores.  With one workgroup per compute unit in
        // two halves of the row blocks: the first half's stores go out while the other is worked on (together with the order of
        // the MFMAs: 2048 x 4096 x 12288 60.2 -> 58.8 us, with cached weights 59.5 -> 57.0).  In front of the first stores a wait for
        // the next tile's first stages (requested before this epilogue, so mostly landed): behind them it would be one for the
        // stores too, the counter being one and the same.  (4000 x 2048 x 12288 79.1 -> 75.2; x 6144 on 256 x 128 tiles 45.0 -> 42.6;
        // even from K = 8192 on.)  256 x 256 tiles in one go: their stages are longer on the way, and with long rows and weights from memory the
        // earlier wait costs more than the earlier stores gain (in one go and in halves; with cached weights: 4096 x 8192 x 28672 420.2 and
        // 424.3; 405.2 and 402.4; 2048 x 8192 x 28672 230.5 and 236.9; 221.3 and 219.8; 4096 x 11008 x 16384 308.8 and 312.5; 298.5 and
        // 296.5).  With shorter rows they would gain too (4096 x 4096 x 28672 232.1 and 226.2, 8192 x 512 x 16384 92.0 and 87.4), which would
        // take a second copy of the epilogue.  Nor with two workgroups per compute unit, whose ends overlap as it is (128 x 128
        // tiles 14.7 and 14.9).
        constexpr int FIRST = KGROUPS == 1 && MINOCC * 4 == WAVES && BN < 256 ? (OWN + 1) / 2 : OWN;
        auto finish = [&](auto first_c, auto count_c) {
            constexpr int i0 = decltype(first_c)::value, count = decltype(count_c)::value;
            unsigned outv[count][TN][2];                      // [..][p]: channels 4*quad + 2p, +1
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                v4i cp[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) cp[e] = lcol_par[col_block(j / 2) * 32 + 16 * (j & 1) + 4 * quad + e];
#pragma unroll
                for (int i = 0; i < count; ++i) {
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const float y0 = dequant(acc[i0 + i][j][2 * p], rp[i0 + i], cp[2 * p]);
                        const float y1 = dequant(acc[i0 + i][j][2 * p + 1], rp[i0 + i], cp[2 * p + 1]);
                        outv[i][j][p] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){y0, y1}, b2));   // hardware round-to-nearest-even
                        asm volatile("" : "+v"(outv[i][j][p]));   // computed here: one set of column constants at a time
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (i0 == 0 && (more || APART)) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (i0 == 0 && APART) {                           // behind the last tile too: from a branch the compiler takes waits along in front of the stores
                par_at = 2 * STAGES * STAGE_BYTES + ROWS * 16 - par_at;      // the other half of the LDS behind the ring
                put_par(next_par, par_at);
            }
            store_outputs16<count, TN, BM>(a, (StoreForm)store_form, m0, n0, row0 + 16 * i0, elane, outv, col_block);
        };
        finish(std::integral_constant<int, 0>{}, std::integral_constant<int, FIRST>{});
        if constexpr (FIRST < OWN) finish(std::integral_constant<int, FIRST>{}, std::integral_constant<int, OWN - FIRST>{});
        if (!more) break;
        pid = next_pid; tile_m = next_m; tile_n = next_n;
    }
#endif  // __HIP_DEVICE_COMPILE__
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int KGROUPS, int STAGES, int MINOCC>
int launch_fp6(const GemmArgs& a, hipStream_t s) {
    const int64_t tm = (a.M + BM - 1) / BM;
    const int64_t tn = ((int64_t)a.N + BN - 1) / BN;
    if (tm * tn > 0x7FFFFFFFll) return fail(BASQ_EINVAL, "w4a4_gemm: problem too large for one launch");
    // persistent workgroups: as many as the chip's 256 compute units hold at once (MINOCC waves per
    // SIMD), each walking the tiles blockIdx.x, blockIdx.x + gridDim.x, ...
    // (with K groups each takes one tile)
    constexpr int WAVES = WAVES_M * WAVES_N * KGROUPS;
    const int64_t resident = 256 * (MINOCC * 4 / WAVES);
    static_assert(KGROUPS > 1 || (MINOCC * 4 % WAVES == 0 && MINOCC * 4 >= WAVES), "whole workgroups per compute unit");
    const int64_t grid = KGROUPS > 1 || tm * tn < resident ? tm * tn : resident;
    // Rows that share lines (output_form(); every product into outputs that no cache holds any more, us with the hint and without).
    // Half lines pay for it only where the stores bound the kernel: largest tiles, several rounds of them, few K-steps (8000 x
    // 14240, K = 256 70 and 63; x 28640, K = 1024 even; elsewhere it gains up to 30 %: 998 x 16160, K = 1024).
    // Odder rows do without unless what else there is to do is long against the stores: one round of 128-channel tiles (494 x 10544,
    // K = 11008 42 and 50; 300 x 10768, K = 512 6.6 and 6.7; seven rounds, 1884 x 26416, K = 1024, 66 and 63), one or two of the
    // wider ones with K >= 8192 (1776 x 12496 92 and 98; below, 1884 x 14224, K = 4096 67 and 64).  64-channel tiles: up to 4 %
    // faster without.
    const bool half_lines = (a.ldy & 31) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 63) == 0;
    const bool hides_stores = half_lines  ? !(BM == 256 && BN == 256 && tm * tn > resident && a.K < 1024)
                              : BN == 128 ? tm * tn <= resident
                                          : BN > 128 && a.K >= 8192 && tm * tn <= 2 * resident;
    GemmArgs b = a;
    b.store_form = output_form(a, hides_stores);
    // (split tilings are taken from K = 2048 on, eight steps a group: their kernels of few steps run only where a caller names the tiling)
    if ((a.K / 128 + KGROUPS - 1) / KGROUPS < STAGES)
        hipLaunchKernelGGL((gemm_w4a4_fp6_kernel<BM, BN, WAVES_M, WAVES_N, KGROUPS, STAGES, MINOCC, true>), dim3((unsigned)grid),
                           dim3(WAVES * 64), 0, s, b, (int)tm, (int)tn);
    else
        hipLaunchKernelGGL((gemm_w4a4_fp6_kernel<BM, BN, WAVES_M, WAVES_N, KGROUPS, STAGES, MINOCC, false>), dim3((unsigned)grid),
                           dim3(WAVES * 64), 0, s, b, (int)tm, (int)tn);
    return check_hip(hipGetLastError(), "w4a4_gemm (fp6) launch");
}

// What a tiling costs, in microseconds: `base` once; for every round in which all 256 compute units hold `per_cu` tiles
// round[0] + round[1] * (K / 128); for the tiles left over, the same with the pair of their number per compute unit (a
// compute unit that holds fewer tiles than it can runs each of them faster) and `fill` * (K / 128) more in proportion to
// the share of the chip they fill (the more matrix cores work, the lower the clock).  Least squares over 370 shapes (129 ..
// 4096 tokens, N 1024 .. 28672, K 1024 .. 14336); the standard deviation of the fit is 5-7 % per tiling.
struct Tiling {
    int bm, bn, per_cu;
    double base, round[2], rest[3][2], fill;
};

double tiling_cost(const Tiling& t, int64_t M, int64_t N, int K) {
    const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), slots = 256 * t.per_cu, over = tiles % slots;
    const int64_t left = (over + 255) / 256;                      // tiles per compute unit in the last round, 0 if it is full
    const double ksteps = K / 128;
    double us = t.base + (double)(tiles / slots) * (t.round[0] + t.round[1] * ksteps);
    if (left > 0) us += t.rest[left - 1][0] + (t.rest[left - 1][1] + t.fill * (double)over / (double)slots) * ksteps;
    return us;
}

// Six tilings, fitted to this kernel's predecessor on 32 x 32 x 64 MFMAs: there the cheapest by the table was within 0.3 % of the fastest
// in the mean over those shapes (13 % at worst), whose weights were in the caches.  The present kernel over 250 other shapes (65 .. 4096
// tokens, same N and K): 0.8 % off with weights in the caches (23 % at worst: 295 x 4016, K = 8192 on 64 x 64, 18.8 us against 15.3
// on 128 x 64), 1.6 % with cold ones, 2.0 % up to 333 tokens, where a pass over the weights is what counts and 64 x 64 tiles make too many of
// them (142 x 7120, K = 11008 33.3 us against 24.3).  Where it is far off a split tiling is mostly taken instead: by both tables (below)
// 0.3 % in the caches (9 % at worst) and 1.2 % cold (779 x 2272, K = 1024 9.0 us against 6.1 on 128 x 64; the next 20 %), so the fit stands.
// Choosing among the first, second and fourth by how evenly their tiles fill the chip, as before, was 13 % off in the
// mean and up to 2.6 times: it gave 129 .. 500 tokens tiles too large to occupy the chip (333 x 4096 x 4096: 96 tiles
// of 128 x 128 take 14.1 us, 384 of 64 x 64 11.9 us), and where a round of 256 x 128 tiles fits exactly it takes
// 58.9 us against 62.2 us for 256 x 192 and 66.4 us for 128 x 128 (2048 x 4096, K = 14336; without `fill` the table took
// 256 x 192 there).  128 x 64 is between its neighbours for a few hundred tokens, and for 65 .. 128, one row of tiles where
// 64 x 64 makes two.  At 128 x 12288, K = 4096 the table has the two even and takes 64 x 64: 11.9 us against 11.8 with the weights in
// the caches, 16.8 against 14.1 with cold ones.
constexpr int NUM_TILINGS = BASQ_FP6_TILINGS;
const Tiling tilings[NUM_TILINGS] = {
    {256, 256, 1, 2.9, {10.7, 0.774}, {{6.1, 0.477}}, 0.31},
    {256, 192, 1, 3.0, {9.0, 0.639}, {{4.6, 0.379}}, 0.242},
    {256, 128, 1, 2.3, {5.1, 0.512}, {{4.1, 0.302}}, 0.181},
    {128, 128, 2, 4.1, {3.4, 0.58}, {{0.9, 0.235}, {0.9, 0.487}}, 0.144},
    {128, 64, 2, 2.5, {2.2, 0.406}, {{2.0, 0.209}, {2.4, 0.316}}, 0.068},
    {64, 64, 3, 2.9, {1.3, 0.40}, {{0.7, 0.148}, {1.3, 0.221}, {1.7, 0.339}}, 0.043},
};
// The split tilings: two groups of waves share a tile's channels (KGROUPS = 2), each on a ring of its own; one workgroup a
// compute unit.  Where every compute unit has one tile at most, its time is the chain of its K-steps -- latency of the loads,
// the barrier, the fragment reads -- and two chains of half the length run side by side (same tile, one group against two, K =
// 4096, weights in the caches: 64 x 64 0.86 of the time on up to 64 compute units, 0.91 on up to 256; 128 x 64 0.81 and 0.89; 128 x
// 128 0.88 and 1.03, with cold weights 0.90 and 1.0; K >= 8192 0.78 .. 0.99; K = 1024 even; 333 x 4096 x 4096 11.3 -> 9.5 us).  With a
// second round of tiles they are slower, 1.05 .. 1.6: two one-group workgroups on a compute unit are two chains as well, and
// overlap their ends.  Hence tiles <= 256 and K >= 2048.  Cost: base + (step + fill * share of the chip) * K / 128, least
// squares over 330 shapes (33 .. 4096 tokens) with most weight where a tiling is near the fastest, 4-10 %, on the predecessor.  The
// present kernel, over 250 other shapes: 3.9 % faster with weights in the caches than without these, 5.4 % with cold ones; of the 117
// that take one, four and four are slower by more than 2 %, the worst by 5 %.
struct SplitTiling {
    int bm, bn;
    double base, step, fill;
};
constexpr int NUM_SPLIT_TILINGS = BASQ_FP6_SPLIT_TILINGS;
const SplitTiling split_tilings[NUM_SPLIT_TILINGS] = {
    {64, 64, 3.65, 0.103, 0.029},  {96, 64, 4.06, 0.123, 0.043}, {128, 64, 3.96, 0.146, 0.049},
    {128, 128, 5.07, 0.155, 0.161}, {96, 96, 4.88, 0.136, 0.080}, {160, 96, 5.70, 0.151, 0.156},
};
int cheapest_tiling(int64_t M, int64_t N, int K) {
    // Few K-steps and many rounds are bound by the outputs, which the largest tiles write fastest and the table, fitted on at
    // most seven rounds and from K = 1024 on, prices by their first rounds (23522 x 22162, K = 512: 128 x 128 519 us, 256 x
    // 256 360; 33204 x 14216, K = 256 385 and 284; 4442 x 26256, K = 1536 140 and 120; below four rounds the table is the
    // better guide; K = 2048 and beyond are even).
    if (K < 2048 && ((M + 255) / 256) * ((N + 255) / 256) >= 4 * 256) return 0;
    int best = 0;
    for (int i = 1; i < NUM_TILINGS; ++i)
        if (tiling_cost(tilings[i], M, N, K) < tiling_cost(tilings[best], M, N, K)) best = i;
    return best;
}
// The split tiling to take instead of the cheapest of the others, -1 if there is none.
int cheapest_split_tiling(int64_t M, int64_t N, int K) {
    if (K < 2048) return -1;
    const Tiling& plain = tilings[cheapest_tiling(M, N, K)];
    int best = -1;
    double us = tiling_cost(plain, M, N, K);
    // Between the two forms of one tile the tables are even on a full chip; with long rows the split form is the faster one there
    // too (1021 x 11008 x 4096: 33.7 -> 31.7 us with the weights in the caches, 128 x 128 on 190 .. 256 compute units, K > 8192,
    // 0.91 .. 1.03 with them, 0.86 .. 0.92 cold; 128 x 64 on 192 .. 256 0.94 .. 0.97 with them, 1.03 .. 1.04 cold, 128 x 11008 x 12288
    // 22.2 -> 21.5 and 30.7 -> 31.8 us).
    if (K > 8192 && plain.bm <= 128 && ((M + plain.bm - 1) / plain.bm) * ((N + plain.bn - 1) / plain.bn) <= 256) us = 1e30;
    for (int i = 0; i < NUM_SPLIT_TILINGS; ++i) {
        const SplitTiling& t = split_tilings[i];
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        if (tiles > 256) continue;
        const double c = t.base + (t.step + t.fill * (double)tiles / 256) * (K / 128);
        if (c < us) { us = c; best = i; }
    }
    return best;
}

}  // namespace

// Against the weight-streaming kernel (gemv_w4a4.hip), weights of both forms cold in memory, 17 .. 128 tokens, N 1024 ..
// 28672, K 1024 .. 14336.  Above 64 tokens this kernel is the faster one (128 tokens x 28672, K = 8192: 35 against 59 us; x
// 1024, K = 4096: 7.2 against 11.2 us): the streaming kernel reads every token's codes again per 16 to 64 channels.  Not quite so
// up to 80 tokens with long rows of 4096 .. 8192 channels (65 x 4096, K = 14336: 23.1 against 20.8 us); the line is drawn without
// them.  Up to 32 it never is: its weights are half as large again.
// Between, the line was fitted (5 %) to a streaming kernel that took four waves a workgroup beyond 8192 channels, against this
// kernel's predecessor without the split tilings.  Both have become faster since, this one the more.  Where the line stands: 60
// shapes of 33, 40, 48, 56 and 64 tokens, N 8208 .. 28672, K 1024 .. 14336, products, this kernel's fastest tiling in its place where it
// streams: the kernel taken is 9 % off the faster one in the mean with cold weights and 16 % with weights in the caches.  Cold, calls
// that take this one lose up to 23 % at 40 tokens (x 9712, K = 14336: 28.4 against 23.0 us), 19 % at 48 and 12 % at 56; calls
// that stream lose the more the longer their rows (64 x 21168, K = 11008 51.0 against 32.8; 48 x 20384 43.0 and 32.3; 40 x 19696
// 39.8 and 31.8).  In the caches this one is the faster one wherever it is taken, and up to twice as fast where it is not (64 x 16560, K =
// 14336 58.4 against 28.0).
bool gemm_fp6_beats_streaming(int64_t M, int32_t N, int32_t K) {
    if (M > 64) return true;
    if (M <= 32 || N <= 8192) return false;
    const double k = K / 1024.0, n = N / 4096.0, m = M / 64.0;
    const double streaming = 3.3 + 1.13 * k + (0.374 * k + 0.417) * n * m;
    const double memory = 3.0 + 0.75 * (double)N * (double)K / 5.4e6;             // one pass over the weights
    const double tiles = tiling_cost(tilings[cheapest_tiling(M, N, K)], M, N, K);
    return 1.2 * (tiles > memory ? tiles : memory) < streaming;
}

bool gemm_fp6_applicable(const GemmArgs& a) {
    // buffer addressing: both operands must be smaller than 4 GiB.  K <= 32768: the fp32 accumulator holds the sum of
    // K products of (q_a/8)(q_w/8) -- multiples of 1/64 up to 225 K / 64 -- exactly only while 225 K < 2^24; longer
    // rows take the int8 path, whose INT32 accumulator has no such limit.
    return a.Aq6 && a.Wq6 && a.K % 128 == 0 && a.K <= 32768 && a.M >= 1 &&
           (int64_t)basq_fp6_bytes(a.M, a.K) < 0xFFFFFFFFll && (int64_t)basq_fp6_bytes(a.N, a.K) < 0xFFFFFFFFll;
}

int gemm_fp6_tiling(int64_t M, int32_t N, int32_t K) { return cheapest_tiling(M, N, K); }

int launch_gemm_fp6_tiling(int tiling, const GemmArgs& a, hipStream_t s) {
    switch (tiling) {
        case 0: return launch_fp6<256, 256, 2, 4, 1, 3, 2>(a, s);
        case 1: return launch_fp6<256, 192, 4, 2, 1, 3, 2>(a, s);
        case 2: return launch_fp6<256, 128, 4, 2, 1, 4, 2>(a, s);
        case 3: return launch_fp6<128, 128, 2, 2, 1, 3, 2>(a, s);
        case 4: return launch_fp6<128, 64, 4, 1, 1, 4, 2>(a, s);
        default: return launch_fp6<64, 64, 2, 2, 1, 4, 3>(a, s);
    }
}

int gemm_fp6_split_tiling(int64_t M, int32_t N, int32_t K) { return cheapest_split_tiling(M, N, K); }

int launch_gemm_fp6_split_tiling(int tiling, const GemmArgs& a, hipStream_t s) {
    switch (tiling) {
        case 0: return launch_fp6<64, 64, 2, 2, 2, 4, 2>(a, s);
        case 1: return launch_fp6<96, 64, 3, 2, 2, 4, 3>(a, s);
        case 2: return launch_fp6<128, 64, 2, 2, 2, 4, 2>(a, s);
        case 3: return launch_fp6<128, 128, 2, 2, 2, 3, 2>(a, s);
        case 4: return launch_fp6<96, 96, 3, 1, 2, 4, 2>(a, s);
        default: return launch_fp6<160, 96, 5, 1, 2, 3, 3>(a, s);
    }
}

int launch_gemm_fp6(const GemmArgs& a, hipStream_t s) {
    const int split = cheapest_split_tiling(a.M, a.N, a.K);
    if (split >= 0) return launch_gemm_fp6_split_tiling(split, a, s);
    return launch_gemm_fp6_tiling(cheapest_tiling(a.M, a.N, a.K), a, s);
}

}  // namespace basq
