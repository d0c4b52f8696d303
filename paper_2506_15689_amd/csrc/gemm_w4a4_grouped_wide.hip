// The group-wise INT4 x INT4 GEMM of gemm_w4a4_grouped_fp6.hip (same operands, same sums in the same order, same bits) on
// 256 x 192 tiles, for products large enough to fill the chip with them.
//
// What bounds it: 2200 cycles a group, of which the vector units work 1460 -- the closings' 96 multiply-adds a lane and the rest, 122
// instructions of 4.4 cycles for each of two waves, and the rank-1 updates: an fp32 MFMA runs beside no fp32 vector
// instruction (64 of them 280 cycles, two of the updates 130, both 423), where the fp6 ones do -- and the matrix units 770 more
// beside them.  No single part is the rest: without the loads, the fragment reads, the multiply-adds or the rank-1 updates a
// product is 11 .. 17 % shorter each.  Against 128 x 128 tiles, two workgroups per compute unit, the tile needs 58 % of the direct
// loads and 83 % of the fragment reads per output, which is what it gains: 2048 x 4096 x 12288 98 -> 80 us, 4096 x 4096 x 28672
// 465 -> 386, 1024 x 4096 x 12288 50 -> 42.  (Twelve waves of 64 x 64 outputs on the same tile, three a SIMD: 92 us; their reads
// of LDS stand in the way.  Column blocks in LDS in the order of the operand, four more running addresses: 82.)
//
// Eight waves of 64 x 96 outputs, one workgroup per compute unit that walks its tiles; a ring of three stages, one group each,
// filled by direct loads three groups ahead, across the ends of tiles: a tile's last three groups request the next tile's first
// ones, so its first fragments are in registers when the outputs go out (many tiles: 4096 x 4096 x 28672 417 us with a workgroup
// per tile, 397 as built; one tile a workgroup 41.5 and 42.3).  One copy of the group's code for all of this: with copies for the
// first and the last groups the registers did not suffice.
#include "gemm_fp6_store.h"
#include <type_traits>

namespace basq {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v32f __attribute__((ext_vector_type(32)));

#define GW_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int GW_BM = 256, GW_BN = 192;
constexpr int GW_WAVES_M = 4, GW_WAVES_N = 2, GW_WAVES = GW_WAVES_M * GW_WAVES_N, GW_THREADS = GW_WAVES * 64;
constexpr int GW_TM = 2, GW_TN = 3;                            // 32 x 32 blocks of a wave: 64 x 96 outputs
constexpr int GW_CHUNK = 96;                                   // bytes of one row per stage: 128 codes
constexpr int GW_BLOCK = 32 * GW_CHUNK;                        // a 32-row block of a stage
constexpr int GW_STAGES = 3;
constexpr int GW_A_PIECES = GW_BM * GW_CHUNK / 1024, GW_B_PIECES = GW_BN * GW_CHUNK / 1024;      // 24 and 18 of 1 KB
constexpr int GW_REC_PIECE = GW_A_PIECES + GW_B_PIECES;        // 256 token records of 16 bytes: 4 pieces
constexpr int GW_SUM_PIECE = GW_REC_PIECE + GW_BM * 16 / 1024; // 192 column sums, and 64 words that nobody reads
constexpr int GW_STAGE = (GW_SUM_PIECE + 1) * 1024;
constexpr int GW_LOADS = 6;                                    // direct loads of a wave per stage
constexpr int GW_NUM_XCD = 8;
static_assert(GW_SUM_PIECE + 2 == GW_LOADS * GW_WAVES, "every wave loads as many pieces, the last one twice");
static_assert(GW_A_PIECES == 3 * GW_WAVES && GW_B_PIECES >= 2 * GW_WAVES, "loads 0 .. 2: activations; 3, 4: weights; 5: the rest");
constexpr int GW_COL_AT = GW_STAGES * GW_STAGE;                // column constants of this tile and the next, 16 bytes each
constexpr int GW_LDS_BYTES = GW_COL_AT + 2 * GW_BN * 16;
static_assert(GW_LDS_BYTES <= 160 * 1024, "one workgroup per compute unit");

// Wait until at most N of this wave's direct-to-LDS loads are outstanding and its own LDS reads have returned,
// then join the workgroup barrier (one asm block: the compiler's own barrier would wait for every load).
template <int N>
__device__ __forceinline__ void gw_wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// ---- what a wave requests, as byte offsets; on the host too, where gemm_grouped_wide_strays() holds all of it against the tables.
// Load i < 5 of wave w brings piece 8 i + w of a stage, three of activations and two of weights (three pieces make one 32-row
// block; which block is uniform over the wave and goes into the scalar offset; blocks past the matrix are clamped to its
// last block).  The sixth brings the last two pieces of weights (waves 0 and 1), the group's token records (2 .. 5, 64 rows
// each) or its column sums (6 and 7, both the same), rows and columns clamped likewise.
#define GW_BOTH __host__ __device__ __forceinline__
GW_BOTH int gw_last_piece(int wave) { return (GW_LOADS - 1) * GW_WAVES + (wave < GW_WAVES - 2 ? wave : GW_WAVES - 2); }
GW_BOTH unsigned gw_a_off(int piece, int tile_m, int rb_a) {
    int blk = piece / 3 + tile_m * (GW_BM / 32);
    blk = blk < rb_a ? blk : rb_a - 1;
    return (unsigned)(blk * GW_BLOCK + piece % 3 * 1024);
}
// (the column blocks stand in LDS as the waves own them, one wave's three behind each other: see col_block)
GW_BOTH int gw_slot_block(int slot) {
    const int own = slot % GW_TN, w = slot / GW_TN;
    return own < 2 ? 2 * w + own : 2 * GW_WAVES_N + w;
}
GW_BOTH unsigned gw_b_off(int piece, int tile_n, int rb_w) {
    int blk = gw_slot_block((piece - GW_A_PIECES) / 3) + tile_n * (GW_BN / 32);
    blk = blk < rb_w ? blk : rb_w - 1;
    return (unsigned)(blk * GW_BLOCK + piece % 3 * 1024);
}
GW_BOTH int gw_record_off(int piece, int lane, int tile_m, int64_t M, int ngroups) {
    int64_t m = (int64_t)tile_m * GW_BM + 64 * (piece - GW_REC_PIECE) + lane;
    m = m < M ? m : M - 1;
    return (int)(m * ngroups * 16);
}
GW_BOTH int gw_sum_off(int lane, int tile_n, int N) {                      // (lanes 48 .. 63: what nobody reads)
    int n = tile_n * GW_BN + 32 * gw_slot_block(lane >> 3) + 4 * (lane & 7);
    n = n < N - 4 ? n : N - 4;
    return n * 4;
}
// Behind the last tile: nothing, from lane offsets past the end of any table.  A lane is left out where its offset reaches the table's
// size less the scalar offset, and that difference must not wrap: the scalar offsets go back to the first groups, of which every
// table has the GW_STAGES that are requested here.
GW_BOTH void gw_request_nothing(int& lane_off, int& last_voff, unsigned& koff_a, unsigned& koff_w, unsigned& koff_l) {
    lane_off = last_voff = (int)0xFFFFFF00u;
    koff_a = koff_w = koff_l = 0;
}

__global__ __launch_bounds__(GW_THREADS, 2) void gemm_w4a4_grouped_wide_kernel(GemmArgs a, const int32_t* w_gsum, int tiles_m, int tiles_n) {
#if defined(__HIP_DEVICE_COMPILE__)   // the body uses device-only buffer-resource types; the host pass only needs the stub
    __shared__ __attribute__((aligned(1024))) uint8_t lds[GW_LDS_BYTES];

    // ---- tile order (workgroups congruent mod 8 run on one XCD; the tiles a workgroup takes, blockIdx.x + i * gridDim.x, stay
    // congruent, the grid being a multiple of 8 wherever there is a second one, and walk a compact band)
    const int total = tiles_m * tiles_n;
    auto tile_of = [&](int pid, int& tile_m, int& tile_n) {
        int t = pid;
        const int per_xcd = total / GW_NUM_XCD;
        if (pid < per_xcd * GW_NUM_XCD) t = (pid % GW_NUM_XCD) * per_xcd + pid / GW_NUM_XCD;
        constexpr int GROUP_M = 4;
        const int band = t / (GROUP_M * tiles_n);
        const int first_m = band * GROUP_M;
        const int rows = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
        const int in_band = t - band * GROUP_M * tiles_n;
        // (divisions are vector instructions: keep what follows from them scalar)
        tile_m = __builtin_amdgcn_readfirstlane(first_m + in_band % rows);
        tile_n = __builtin_amdgcn_readfirstlane(in_band / rows);
    };

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int swave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = swave / GW_WAVES_N, wn = swave % GW_WAVES_N;
    const int ngroups = a.K / 128;
    int store_form = (int)a.store_form;                       // fetched here: at the end it would be a memory latency
    asm volatile("" : "+s"(store_form));
    const int rb_a = (int)((a.M + 31) >> 5), rb_w = (a.N + 31) >> 5;   // 32-row blocks per chunk of K
    const unsigned a_step = (unsigned)rb_a * GW_BLOCK, w_step = (unsigned)rb_w * GW_BLOCK;   // bytes from one chunk to the next
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.Aq6), 0, (int)(a_step * (unsigned)ngroups), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.Wq6), 0, (int)(w_step * (unsigned)ngroups), 0x00020000);

    // ---- direct loads: six of 1 KB per wave and stage (which ones: gw_last_piece and below)
    int lane_off = lane * 16;
    const int last_piece = gw_last_piece(swave);
    const bool last_w = last_piece < GW_REC_PIECE, last_rec = !last_w && last_piece < GW_SUM_PIECE;
    const unsigned last_step = last_w ? w_step : last_rec ? 16u : (unsigned)a.N * 4u;
    const __amdgpu_buffer_rsrc_t rsrc_l = __builtin_amdgcn_make_buffer_rsrc(
        last_w ? (void*)const_cast<uint8_t*>(a.Wq6) : last_rec ? (void*)const_cast<basq_tokmeta*>(a.meta) : (void*)const_cast<int32_t*>(w_gsum), 0,
        last_w ? (int)(w_step * (unsigned)ngroups) : last_rec ? (int)(a.M * ngroups * 16) : (int)((int64_t)ngroups * a.N * 4), 0x00020000);
    unsigned soff[GW_LOADS - 1], koff_a, koff_w, koff_l;                   // koff: of the next group to request
    int last_voff;
    auto request_from = [&](int tile_m, int tile_n) {                      // the next group to request is the first of this tile
#pragma unroll
        for (int i = 0; i < GW_LOADS - 1; ++i)
            soff[i] = i * GW_WAVES < GW_A_PIECES ? gw_a_off(i * GW_WAVES + swave, tile_m, rb_a) : gw_b_off(i * GW_WAVES + swave, tile_n, rb_w);
        const int rec = gw_record_off(last_piece, lane, tile_m, a.M, ngroups), sum = gw_sum_off(lane, tile_n, a.N);
        last_voff = last_w ? lane_off : last_rec ? rec : sum;
        koff_a = koff_w = 0;
        koff_l = last_w ? gw_b_off(last_piece, tile_n, rb_w) : 0;
    };
    auto issue_one = [&](int stage_off, int i) {
        const int at = stage_off + (i * GW_WAVES + swave) * 1024;
        if (i * GW_WAVES < GW_A_PIECES)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, GW_LDS_PTR(lds + at), 16, lane_off, (int)(koff_a + soff[i]), 0, 0);
        else if (i < GW_LOADS - 1)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, GW_LDS_PTR(lds + at), 16, lane_off, (int)(koff_w + soff[i]), 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_l, GW_LDS_PTR(lds + stage_off + last_piece * 1024), 16, last_voff, (int)koff_l, 0, 0);
    };
    auto next_request = [&]() { koff_a += a_step; koff_w += w_step; koff_l += last_step; };

    // ---- fragment addressing: lane (frow, fhalf) feeds k = 64*kb + 32*fhalf .. +31 of its row, i.e. group
    // f = 2*kb + fhalf of the row's block: 16 bytes among the pieces, 8 bytes among the tails
    const int frow = lane & 31, fhalf = lane >> 5;
    const int toff = 2048 + 256 * fhalf + 8 * frow;                        // k-block 1: 512 bytes further
    const int a_row = wm * GW_TM * GW_BLOCK;
    // a wave's column blocks: a pair of adjacent ones (64 columns, a 128-byte line of outputs), and one from behind all pairs
    auto col_block = [&](int j) { return j < 2 ? wn * 2 + j : GW_WAVES_N * 2 + wn; };
    const int b_row = GW_A_PIECES * 1024 + wn * GW_TN * GW_BLOCK;
    // running byte addresses of the reads: of the stage that is read next
    int ma[2], mb[2], ta = a_row + toff, tb = b_row + toff;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int moff = 64 * frow + 16 * ((2 * kb + fhalf) ^ ((frow >> 2) & 3));
        ma[kb] = a_row + moff;
        mb[kb] = b_row + moff;
        asm volatile("" : "+v"(ma[kb]), "+v"(mb[kb]));
    }
    int rec_at = GW_REC_PIECE * 1024 + (wm * GW_TM * 32 + frow) * 16, sum_at = GW_SUM_PIECE * 1024 + (wn * GW_TN * 32 + frow) * 4;
    asm volatile("" : "+v"(ta), "+v"(tb), "+v"(rec_at), "+v"(sum_at));

    // Column constants (sw, sw * zp, c) of a tile.  Requested as raw bits on every path, so that no conversion, with a wait for
    // everything in flight in front of it, stands behind the request.
    const int my_col = tid < GW_BN ? tid : GW_BN - 1;
    struct Column { uint16_t scale, zero; float bias; };
    auto load_column = [&](int tile_n) -> Column {
        int col = tile_n * GW_BN + my_col;
        col = col < a.N ? col : a.N - 1;
        return {a.w_scale[col], a.w_zero[col], a.out_bias ? a.out_bias[col] : 0.0f};
    };
    v4i* lcol = reinterpret_cast<v4i*>(lds + GW_COL_AT);
    auto put_column = [&](int buffer, Column c) {
        // Used here first, and by every wave: a conversion that moves up would wait for its load there, and where only some waves
        // use theirs the others wait for them later, between the stores.
        asm volatile("" : "+v"(c.scale), "+v"(c.zero), "+v"(c.bias));
        const float sw = bf16_to_f32(c.scale), zp = bf16_to_f32(c.zero);
        if (tid < GW_BN) lcol[buffer * GW_BN + tid] = v4i{__float_as_int(sw), __float_as_int(sw * zp), __float_as_int(c.bias), 0};
    };

    // F / 64: facc[j] holds the row blocks i = 0, 1 of column block j, 16 registers each
    v32f facc[GW_TN];
#pragma unroll
    for (int j = 0; j < GW_TN; ++j)
#pragma unroll
        for (int r = 0; r < 32; ++r) facc[j][r] = 0.0f;
    float rsum[GW_TM] = {0.0f, 0.0f};                                      // R_m of this lane's tokens (lane % 32)
    // operand registers: six consecutive VGPRs per fragment; the builtin takes eight, the fp6 form reads six
    // The third column block's fragments take the first one's place.
    v8i pa[2][GW_TM], pb[2][2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int j = 0; j < 2; ++j) pb[kb][j] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < 2; ++i) pa[kb][i] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
    }
    v4i rec[GW_TM];                                                        // a group's records of this lane's tokens ..
    int csum[GW_TN];                                                       // .. and sums of its channels
    auto read_one = [&](v8i& dst, const uint8_t* main_ptr, const uint8_t* tail_ptr) {
        const v4i mv = *reinterpret_cast<const v4i*>(main_ptr);
        const v2i tv = *reinterpret_cast<const v2i*>(tail_ptr);
        dst[0] = mv[0]; dst[1] = mv[1]; dst[2] = mv[2]; dst[3] = mv[3]; dst[4] = tv[0]; dst[5] = tv[1];
        // (tail reads of one base that stand side by side are merged into paired ones, whose result cannot land in two operand tuples)
        asm volatile("" ::: "memory");
    };
    auto read_a = [&](int kb, int i) { read_one(pa[kb][i], lds + ma[kb] + i * GW_BLOCK, lds + ta + i * GW_BLOCK + 512 * kb); };
    auto read_b = [&](int kb, int j) { read_one(pb[kb][j & 1], lds + mb[kb] + j * GW_BLOCK, lds + tb + j * GW_BLOCK + 512 * kb); };
    // As integers: the compiler puts a wait for every outstanding direct-to-LDS load in front of a float-typed LDS read.
    auto read_records = [&](int t) { rec[t] = *reinterpret_cast<const v4i*>(lds + rec_at + t * 32 * 16); };
    auto read_sums = [&]() {
#pragma unroll
        for (int j = 0; j < GW_TN; ++j) csum[j] = *reinterpret_cast<const int*>(lds + sum_at + j * 32 * 4);
    };
    int stage = 0;                                                         // byte offset of the stage being read
    auto next_stage = [&]() {
        const bool wrap = stage == (GW_STAGES - 1) * GW_STAGE;
        const int d = wrap ? -(GW_STAGES - 1) * GW_STAGE : GW_STAGE;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) { ma[kb] += d; mb[kb] += d; }
        ta += d; tb += d; rec_at += d; sum_at += d;
        stage += d;
    };
    const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // S_g of the blocks (i, j).  The weights are the first MFMA operand: accumulator register r of lane l belongs to token
    // l % 32 of the row block and to output channel 8*(r/4) + 4*(l/32) + r%4 of the column block.
    v16f acc[GW_TM][GW_TN] = {{zero, zero, zero}, {zero, zero, zero}};
    auto close_half = [&](int i, int j, int half, float scale) {           // F' += s_mg * S_g, eight registers
#pragma unroll
        for (int r = 8 * half; r < 8 * half + 8; ++r) facc[j][16 * i + r] = fmaf(scale, acc[i][j][r], facc[j][16 * i + r]);
        asm volatile("" : "+v"(facc[j]));                                  // here, not where the sums are next used
    };

    // ---- the first tile's first three groups
    int pid = blockIdx.x, tile_m, tile_n;
    tile_of(pid, tile_m, tile_n);
    const Column first_column = load_column(tile_n);
    request_from(tile_m, tile_n);
#pragma unroll
    for (int g = 0; g < GW_STAGES; ++g) {
#pragma unroll
        for (int i = 0; i < GW_LOADS; ++i) issue_one(g * GW_STAGE, i);
        next_request();
    }
    put_column(0, first_column);
    gw_wait_loads_and_barrier<2 * GW_LOADS>();
    read_b(0, 0); read_b(1, 0);
    read_records(0); read_records(1); read_sums();
    read_b(0, 1); read_b(1, 1);
    read_a(0, 0); read_a(1, 0); read_a(0, 1); read_a(1, 1);
    __builtin_amdgcn_sched_barrier(0);

    float prev_s[2] = {0.0f, 0.0f};                                        // scales of the group before
    // One group per pass: blocks (i, j) = (0,0), (1,0), (1,1), (0,1), (0,2), (1,2), two MFMAs each.  The barrier, in front of block
    // (0,1), ends every wave's reads of this stage, which the group three further on refills from here on, and begins those
    // of the next one: each fragment as soon as its registers have had their last use.  Behind every MFMA go eight multiply-adds
    // of a closing, one block late.
    auto group = [&]() {
        const int here = stage;
        float s[2] = {0.0f, 0.0f}, zlane = 0.0f, c1 = 0.0f, c2 = 0.0f;
#pragma unroll
        for (int t = 0; t < 4 * GW_TN; ++t) {
            const int j = t >> 2, i = ((t >> 1) ^ j) & 1, kb = t & 1;
            if (t == 6) gw_wait_loads_and_barrier<GW_LOADS>();
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(pb[kb][j & 1], pa[kb][i], kb == 0 ? zero : acc[i][j], 2, 2, 0, 0, 0, 0);
            if (t == 2) {
                // the constants, not before: they were the last to be read
                s[0] = __int_as_float(rec[0][0]); s[1] = __int_as_float(rec[1][0]);
                const float z0 = __int_as_float(rec[0][1]), z1 = __int_as_float(rec[1][1]);
                zlane = fhalf ? z1 : z0;                                   // block l / 32 of the rank-1 update
                const float c0 = 0.015625f * (float)csum[0];
                c1 = 0.015625f * (float)csum[1];
                c2 = 0.015625f * (float)csum[2];
                rsum[0] += fmaf(s[0], (float)rec[0][2], 128.0f * z0);
                rsum[1] += fmaf(s[1], (float)rec[1][2], 128.0f * z1);
                asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(rsum[0]), "+v"(rsum[1]), "+v"(c1), "+v"(c2));
                facc[0] = __builtin_amdgcn_mfma_f32_32x32x1f32(c0, zlane, facc[0], 0, 0, 0);
            }
            if (t == 4) facc[1] = __builtin_amdgcn_mfma_f32_32x32x1f32(c1, zlane, facc[1], 0, 0, 0);
            if (t == 8) facc[2] = __builtin_amdgcn_mfma_f32_32x32x1f32(c2, zlane, facc[2], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (t == 2) read_b(0, 2);
            if (t == 3) { read_b(1, 2); next_stage(); }
            if (t == 6) { read_records(0); read_records(1); }
            if (t == 7) { read_sums(); read_b(0, 1); }
            if (t == 8) { read_a(0, 0); read_b(1, 1); }
            if (t == 9) read_a(1, 0);
            if (t == 10) { read_b(0, 0); read_a(0, 1); }
            if (t == 11) { read_b(1, 0); read_a(1, 1); }
            if (t >= 6) issue_one(here, t - 6);
            if (t == 11) next_request();
            __builtin_amdgcn_sched_barrier(0);
            // behind MFMAs 2b + 1 and 2b + 2: the halves of block b - 1, of this group or of the one before
            constexpr int BLOCKS = GW_TM * GW_TN;
            const int c = (t - 1 + 2 * BLOCKS) / 2 % BLOCKS == 0 ? BLOCKS - 1 : (t - 1 + 2 * BLOCKS) / 2 % BLOCKS - 1;
            const int ci = (c ^ (c >> 1)) & 1;
            close_half(ci, c >> 1, (t & 1) ^ 1, t >= 3 ? s[ci] : prev_s[ci]);
            __builtin_amdgcn_sched_barrier(0);
        }
        prev_s[0] = s[0];
        prev_s[1] = s[1];
    };
    int buffer = 0;                                                        // of this tile's column constants
    while (true) {
        // Every group requests the one three further on: the last three those of the next tile, whose first fragments are read
        // with the last group, or nothing, from past the end of the operands.  The second and third group of a later tile
        // have landed before the stores of the tile in front go out (the wait in `finish`).  Its first two groups need no wait for
        // loads, then, but the one copy of their code has it, and there it is a wait for those stores: for all but six of them in the
        // first group, for the rest in the second.
        const int next_pid = pid + gridDim.x;
        const bool more = next_pid < total;
        int next_m = 0, next_n = 0;
        int g = 0;
#pragma unroll 1
        for (int end = ngroups - GW_STAGES; end <= ngroups; end += GW_STAGES) {
#pragma unroll 1
            for (; g < end; ++g) {
                asm volatile(".p2align 4");
                group();
            }
            if (end == ngroups) break;
            if (more) {
                tile_of(next_pid, next_m, next_n);
                request_from(next_m, next_n);
            } else {
                gw_request_nothing(lane_off, last_voff, koff_a, koff_w, koff_l);
            }
        }
        const Column next_column = load_column(more ? next_n : tile_n);
        close_half(0, GW_TN - 1, 1, prev_s[0]);
        close_half(1, GW_TN - 1, 0, prev_s[1]);
        close_half(1, GW_TN - 1, 1, prev_s[1]);

        // ---- epilogue: the pair of column blocks first, whose stores go out while the odd one is worked on
        auto result = [&](int i, int j, int r, v4i col) {
            return fmaf(__int_as_float(col[0]), 64.0f * facc[j][16 * i + r], fmaf(-__int_as_float(col[1]), rsum[i], __int_as_float(col[2])));
        };
        typedef float f2 __attribute__((ext_vector_type(2)));
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        // (from an opaque copy of the lane index: what follows from it would otherwise be held in registers across the groups)
        int elane = lane;
        asm volatile("" : "+v"(elane));
        const v4i* cols = lcol + buffer * GW_BN + 4 * (elane >> 5);
        auto finish = [&](auto first_c, auto count_c) {
            constexpr int j0 = decltype(first_c)::value, count = decltype(count_c)::value;
            unsigned outv[GW_TM][count][4][2];
#pragma unroll
            for (int j = 0; j < count; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v4i cp[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) cp[e] = cols[col_block(j0 + j) * 32 + 8 * q + e];
#pragma unroll
                    for (int i = 0; i < GW_TM; ++i)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const float y0 = result(i, j0 + j, 4 * q + 2 * p, cp[2 * p]), y1 = result(i, j0 + j, 4 * q + 2 * p + 1, cp[2 * p + 1]);
                            outv[i][j][q][p] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){y0, y1}, b2));   // hardware round-to-nearest-even
                            asm volatile("" : "+v"(outv[i][j][q][p]));         // computed here: one set of column constants at a time
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (j0 == 0) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the next tile's second and third group
                put_column(buffer ^ 1, next_column);
            }
            store_outputs<GW_TM, count, GW_BM>(a, (StoreForm)store_form, (int64_t)tile_m * GW_BM, tile_n * GW_BN, wm * GW_TM * 32, elane, outv,
                                               [&](int j) { return col_block(j0 + j); });
        };
        finish(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
        finish(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
        if (!more) break;
#pragma unroll
        for (int j = 0; j < GW_TN; ++j)
#pragma unroll
            for (int r = 0; r < 32; ++r) facc[j][r] = 0.0f;
        rsum[0] = rsum[1] = prev_s[0] = prev_s[1] = 0.0f;
        buffer ^= 1;
        pid = next_pid; tile_m = next_m; tile_n = next_n;
    }
#endif  // __HIP_DEVICE_COMPILE__
}

}  // namespace

// The requests of an M x K x N product that leave their table, in any byte of a lane's 16, or are not dropped behind a last tile:
// counted on the host, with the kernel's own offsets.
int64_t gemm_grouped_wide_strays(int64_t M, int32_t N, int32_t K) {
    const int ngroups = K / 128, tiles_m = (int)((M + GW_BM - 1) / GW_BM), tiles_n = (N + GW_BN - 1) / GW_BN;
    const int rb_a = (int)((M + 31) >> 5), rb_w = (N + 31) >> 5;
    const unsigned a_step = (unsigned)rb_a * GW_BLOCK, w_step = (unsigned)rb_w * GW_BLOCK;
    const uint64_t a_size = (uint64_t)a_step * ngroups, w_size = (uint64_t)w_step * ngroups;
    const uint64_t rec_size = (uint64_t)M * ngroups * 16, sum_size = (uint64_t)ngroups * N * 4;
    int64_t strays = 0;
    auto check = [&](uint64_t size, unsigned scalar, int lane_offset, bool wanted) {
        const unsigned vector = (unsigned)lane_offset;
        strays += scalar > size || (wanted ? scalar + (uint64_t)vector + 16 > size : vector < size - scalar);
    };
    for (int tile = 0; tile < tiles_m * tiles_n; ++tile)
        for (int wave = 0; wave < GW_WAVES; ++wave)
            for (int lane = 0; lane < 64; ++lane) {
                const int tile_m = tile % tiles_m, tile_n = tile / tiles_m, last_piece = gw_last_piece(wave);
                const bool last_w = last_piece < GW_REC_PIECE, last_rec = !last_w && last_piece < GW_SUM_PIECE;
                int lane_off = lane * 16;
                int last_voff = last_w ? lane_off : last_rec ? gw_record_off(last_piece, lane, tile_m, M, ngroups) : gw_sum_off(lane, tile_n, N);
                unsigned koff_a = 0, koff_w = 0, koff_l = last_w ? gw_b_off(last_piece, tile_n, rb_w) : 0;
                for (int g = 0; g < ngroups + GW_STAGES; ++g) {
                    if (g == ngroups) gw_request_nothing(lane_off, last_voff, koff_a, koff_w, koff_l);
                    for (int i = 0; i < GW_LOADS - 1; ++i) {
                        const bool of_a = i * GW_WAVES < GW_A_PIECES;
                        const int piece = i * GW_WAVES + wave;
                        check(of_a ? a_size : w_size, of_a ? koff_a + gw_a_off(piece, tile_m, rb_a) : koff_w + gw_b_off(piece, tile_n, rb_w), lane_off, g < ngroups);
                    }
                    check(last_w ? w_size : last_rec ? rec_size : sum_size, koff_l, last_voff, g < ngroups);
                    koff_a += a_step;
                    koff_w += w_step;
                    koff_l += last_w ? w_step : last_rec ? 16u : (unsigned)N * 4u;
                }
            }
    return strays;
}

bool gemm_grouped_wide_applicable(const GemmArgs& a, const int32_t* w_gsum) {
    // four column sums a lane and load: their rows start on 16-byte boundaries
    return a.K >= 128 * GW_STAGES && a.N % 4 == 0 && (reinterpret_cast<uintptr_t>(w_gsum) & 15) == 0 && gemm_grouped_fp6_applicable(a);
}

// Microseconds of both tilings, least squares over 120 shapes (100 .. 4096 tokens, N 1024 .. 28672, K 1024 .. 14336, 90 and more
// of the large tiles), 6-7 %: rounds in which every compute unit is full, and a last one by the number of tiles a compute unit
// holds there and the share of the chip that they fill.  Rows of odd lines cost the large tiles more with outputs that no cache
// holds (their stores wait on nobody else's work), so there they have to be 4 % cheaper: without that 2552 x 10224, K = 8192 205 us
// against 201, 377 x 24208, K = 1024 19.0 against 18.2, 334 x 23824 5 % off.  Over 304 shapes (100 .. 4096 tokens, N 1024 .. 28672, K 384 ..
// 14336, 100 and more of the large tiles) the large tiles are then nowhere more than 2 % behind the small ones where they are
// taken; the small ones are taken where the large are up to 22 % faster (4091 x 24512, K = 1536 173 and 141; K < 1024 and
// several rounds of tiles), with cold weights the choice is 0.8 % off the faster tiling in the mean.
// Where they are even: one round of large tiles, three quarters full (K = 4096: 2272 x 3584, 171 tiles, 36.0 us narrow and 40.9;
// 3816 x 2480, 195 tiles, 47.9 and 41.9); a second one just begun loses (1775 x 8176, 301 tiles, 60.8 and 78.1).
bool gemm_grouped_wide_is_faster(int64_t M, int32_t N, int32_t K) {
    if (K < 128 * GW_STAGES) return false;
    const double g = K / 128;
    const int64_t small = ((M + 127) / 128) * (((int64_t)N + 127) / 128), small_over = small % 512, small_left = (small_over + 255) / 256;
    const int64_t large = ((M + GW_BM - 1) / GW_BM) * (((int64_t)N + GW_BN - 1) / GW_BN), large_over = large % 256;
    double narrow = 2.9 + (double)(small / 512) * (3.0 + 0.882 * g), wide = 4.5 + (double)(large / 256) * (7.5 + 1.068 * g);
    if (small_left > 0) narrow += (small_left == 1 ? 2.3 + 0.386 * g : 3.0 + 0.639 * g) + 0.266 * g * (double)small_over / 512;
    if (large_over > 0) wide += 4.5 + 0.653 * g + 0.469 * g * (double)large_over / 256;
    return wide < (N % 32 != 0 ? 0.96 : 1.0) * narrow;
}

int launch_gemm_grouped_wide(const GemmArgs& a, const int32_t* w_gsum, hipStream_t s) {
    const int64_t tm = (a.M + GW_BM - 1) / GW_BM, tn = ((int64_t)a.N + GW_BN - 1) / GW_BN;
    if (tm * tn > 0x7FFFFFFFll) return fail(BASQ_EINVAL, "w4a4_gemm_grouped: problem too large for one launch");
    GemmArgs b = a;
    // Rows of half lines with the hint, odder ones without, whatever K and the number of tiles: one workgroup per compute unit does not
    // hide what the hint costs there (outputs that no cache holds any more, us with and without; 128 x 128 tiles.  Half lines: 2567 x
    // 4000, K = 384 11.9 and 14.0; 12.1; 1585 x 27872, K = 2048 90.8 and 104.9; 103.5; 917 x 12256, K = 4096 44.3 and 46.3; 55.0.  Odder:
    // 3132 x 3536, K = 512 18.0 and 13.3; 14.4; 2591 x 4176, K = 1024 20.5 and 16.8; 18.7; 2739 x 14224, K = 4096 160.8 and 152.1;
    // 156.8; 4020 x 8784, K = 8192 226.9 and 224.6; 267.3; but 385 x 19792, K = 384 13.5 and 14.2; 14.1).
    b.store_form = output_form(a, (a.ldy & 31) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 63) == 0);
    const int64_t grid = tm * tn < 256 ? tm * tn : 256;           // persistent workgroups, one per compute unit
    hipLaunchKernelGGL(gemm_w4a4_grouped_wide_kernel, dim3((unsigned)grid), dim3(GW_THREADS), 0, s, b, w_gsum, (int)tm, (int)tn);
    return check_hip(hipGetLastError(), "w4a4_gemm_grouped (wide) launch");
}

}  // namespace basq
