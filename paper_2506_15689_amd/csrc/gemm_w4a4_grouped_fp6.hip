// The group-wise INT4 x INT4 GEMM of gemm_w4a4_grouped.hip on the f8f6f4 matrix-core path (Eq. 4 applied per group
// of 128 channels; the product itself as in Sec. 5.2):
//
//     Y[m,n] = sw_n * ( sum_g ( s_mg ACC_g[m,n] + z_mg colsum_g[n] ) - zp_n * R_m ) + c_n
//
// Operands in the fp6 operand form (fp6_pack.hip: code q stored as the e2m3 number q/8), so a group's accumulator is
// S_g = ACC_g / 64 in fp32, exactly, and needs no conversion before it is scaled.  One LDS stage of the ring is one
// chunk of 128 codes = one group, and its constants (128 token records, 128 column sums).  Every group is closed into the
// fp32 sum F' = F / 64 as F' = fma(s_mg, S_g, fma(z_mg, colsum_g / 64, F')) (every term is the exact 1/64 of the int8
// kernel's, so F' * 64 has that kernel's bits).
//
// What bounds it: per wave and group 8 MFMAs (256 cycles) and the closing of 64 x 64 outputs.  The inner multiply-add is
// an outer product of tokens and channels, so it is a rank-1 update on the matrix cores: v_mfma_f32_32x32x1_2b_f32 does
// two 32 x 32 blocks in 64 cycles with the single rounding of fma (checked bit for bit over normal and subnormal values),
// against 128 for 32 vector instructions, and it takes one column sum and one lower bound per lane instead of 32 sums
// from LDS (it runs beside no fp32 vector instruction: 64 of them 280 cycles, two updates 130, both 423).  The outer one is 64
// vector instructions (256 cycles), which run beside the fp6 MFMAs of the same wave if nothing makes them wait: eight behind every MFMA (32 cycles each), one block late.  With sixteen behind every second MFMA a
// group took a wave alone on its SIMD 1230 cycles, as built 1020 (64 x 4096 x 4096 20.4 -> 17.6 us, 700 x 5008, K = 8192 38.9 ->
// 33.7); two waves a SIMD share the loads into LDS and its reads, and gain less (2048 x 4096 x 12288 98 - 102 us, now 92 - 98; without
// the loads 70, the multiply-adds 80, the fragment reads 82, the rank-1 updates 87).  The reads take running addresses, two
// instructions a read less than a stage's address each time; a branch in the loop costs tens of cycles (unpeeled, with the
// tests for the last groups inside, 24.3 us for 64 x 4096 x 4096).  256 x 128 tiles, a quarter less to load: 98.6.
// Products that fill the chip with 256 x 192 tiles take those (gemm_w4a4_grouped_wide.hip).  Here
// 128 x 128 tiles, four waves of 64 x 64, two workgroups per compute unit, a ring of three stages filled by
// direct-to-LDS loads two to three groups ahead.
#include "gemm_fp6_store.h"
#include <type_traits>

namespace basq {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v32f __attribute__((ext_vector_type(32)));

#define G6G_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int G6G_BM = 128, G6G_BN = 128;
constexpr int G6G_WAVES_N = 2, G6G_WAVES = 4, G6G_THREADS = 256;
constexpr int G6G_WM = 64, G6G_TM = 2, G6G_TN = 2;
constexpr int G6G_CHUNK = 96;                                  // bytes of one row per stage: 128 codes
constexpr int G6G_BLOCK = 32 * G6G_CHUNK;                      // a 32-row block of a stage
constexpr int G6G_STAGES = 3;
// LDS: the activations of all stages, then their weights, records and column sums.  A read of any stage is then one address per
// lane plus an offset that the instruction carries (64 KB at most), not an addition per read and step.
constexpr int G6G_A_STAGE = G6G_BM * G6G_CHUNK, G6G_B_STAGE = G6G_BN * G6G_CHUNK;      // 12 KB each
constexpr int G6G_REC_STAGE = G6G_BM * 16, G6G_SUM_STAGE = G6G_BN * 4;
constexpr int G6G_B_AT = G6G_STAGES * G6G_A_STAGE, G6G_REC_AT = G6G_B_AT + G6G_STAGES * G6G_B_STAGE;
constexpr int G6G_SUM_AT = G6G_REC_AT + G6G_STAGES * G6G_REC_STAGE;
constexpr int G6G_LDS_BYTES = G6G_SUM_AT + G6G_STAGES * G6G_SUM_STAGE;
constexpr int G6G_PIECES = (G6G_A_STAGE + G6G_B_STAGE) / 1024; // 1 KB pieces of a stage's operands, one wave-load each
constexpr int G6G_LOADS = G6G_PIECES / G6G_WAVES;              // operand loads per wave per stage
constexpr int G6G_A_LOADS = (G6G_BM * G6G_CHUNK / 1024) / G6G_WAVES;   // ... of which the first ones are activations
constexpr int G6G_ALL_LOADS = G6G_LOADS + 1;                   // ... and one more brings constants
constexpr int G6G_NUM_XCD = 8;
static_assert(G6G_PIECES % G6G_WAVES == 0 && (G6G_BM * G6G_CHUNK / 1024) % G6G_WAVES == 0, "whole rounds of loads");
static_assert(2 * G6G_LDS_BYTES <= 160 * 1024, "two workgroups per compute unit");

// Wait until at most N of this wave's direct-to-LDS loads are outstanding and its own LDS reads have returned,
// then join the workgroup barrier (one asm block: the compiler's own barrier would wait for every load).
template <int N>
__device__ __forceinline__ void g6g_wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

__global__ __launch_bounds__(G6G_THREADS, 2) void gemm_w4a4_grouped_fp6_kernel(GemmArgs a, const int32_t* w_gsum, int tiles_m, int tiles_n) {
#if defined(__HIP_DEVICE_COMPILE__)   // the body uses device-only buffer-resource types; the host pass only needs the stub
    __shared__ __attribute__((aligned(1024))) uint8_t lds[G6G_LDS_BYTES];

    // ---- tile assignment (ids congruent mod 8 run on one XCD and walk a compact band)
    int tile_m, tile_n;
    {
        const int total = tiles_m * tiles_n;
        const int pid = blockIdx.x;
        int t = pid;
        const int per_xcd = total / G6G_NUM_XCD;
        if (pid < per_xcd * G6G_NUM_XCD) t = (pid % G6G_NUM_XCD) * per_xcd + pid / G6G_NUM_XCD;
        constexpr int GROUP_M = 4;
        const int band = t / (GROUP_M * tiles_n);
        const int first_m = band * GROUP_M;
        const int rows = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
        const int in_band = t - band * GROUP_M * tiles_n;
        // (divisions are vector instructions: keep what follows from them scalar)
        tile_m = __builtin_amdgcn_readfirstlane(first_m + in_band % rows);
        tile_n = __builtin_amdgcn_readfirstlane(in_band / rows);
    }

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / G6G_WAVES_N, wn = wave % G6G_WAVES_N;
    const int swave = __builtin_amdgcn_readfirstlane(wave);
    const int64_t m0 = (int64_t)tile_m * G6G_BM;
    const int n0 = tile_n * G6G_BN;
    const int ngroups = a.K / 128;
    int store_form = (int)a.store_form;                       // fetched here: at the end it would be a memory latency
    asm volatile("" : "+s"(store_form));
    const int rb_a = (int)((a.M + 31) >> 5), rb_w = (a.N + 31) >> 5;   // 32-row blocks per chunk of K
    const unsigned a_step = (unsigned)rb_a * G6G_BLOCK, w_step = (unsigned)rb_w * G6G_BLOCK;   // bytes from one chunk to the next
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.Aq6), 0, (int)(a_step * (unsigned)ngroups), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.Wq6), 0, (int)(w_step * (unsigned)ngroups), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_m = __builtin_amdgcn_make_buffer_rsrc(const_cast<basq_tokmeta*>(a.meta), 0, (int)(a.M * ngroups * 16), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_c = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(w_gsum), 0, (int)((int64_t)ngroups * a.N * 4), 0x00020000);

    // ---- direct loads.  Operand load i of wave w copies the 1 KB piece i*4 + w of the stage (three pieces make one
    // 32-row block; which block is uniform over the wave and goes into the scalar offset; blocks past the matrix are
    // clamped to its last block).  One more load per wave brings a group's constants: waves 0, 1 the token records
    // of rows 64w + lane, waves 2, 3 the column sums of columns 64(w-2) + lane (clamped likewise).
    const int lane_off = lane * 16;
    int soff[G6G_LOADS];
#pragma unroll
    for (int i = 0; i < G6G_LOADS; ++i) {
        const int piece = i * G6G_WAVES + swave;
        int blk = piece / 3;
        const int part = piece % 3;
        if (i < G6G_A_LOADS) {
            blk += tile_m * (G6G_BM / 32);
            blk = blk < rb_a ? blk : rb_a - 1;
        } else {
            blk += tile_n * (G6G_BN / 32) - G6G_BM / 32;
            blk = blk < rb_w ? blk : rb_w - 1;
        }
        soff[i] = blk * G6G_BLOCK + part * 1024;
    }
    int pvoff;
    if (swave < 2) {
        int64_t m = m0 + 64 * swave + lane;
        m = m < a.M ? m : a.M - 1;
        pvoff = (int)(m * ngroups * 16);
    } else {
        int n = n0 + 64 * (swave - 2) + lane;
        n = n < a.N ? n : a.N - 1;
        pvoff = n * 4;
    }
    // load number i of group g, into stage `stage` of the ring; the last one is the constants'
    auto issue_one = [&](int stage, int g, int i) {
        if (i < G6G_A_LOADS)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, G6G_LDS_PTR(lds + stage * G6G_A_STAGE + (i * G6G_WAVES + swave) * 1024), 16, lane_off, (int)((unsigned)g * a_step + (unsigned)soff[i]), 0, 0);
        else if (i < G6G_LOADS)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_w, G6G_LDS_PTR(lds + G6G_B_AT + stage * G6G_B_STAGE + ((i - G6G_A_LOADS) * G6G_WAVES + swave) * 1024), 16, lane_off, (int)((unsigned)g * w_step + (unsigned)soff[i]), 0, 0);
        else if (swave < 2)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_m, G6G_LDS_PTR(lds + G6G_REC_AT + stage * G6G_REC_STAGE + swave * 1024), 16, pvoff, g * 16, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_c, G6G_LDS_PTR(lds + G6G_SUM_AT + stage * G6G_SUM_STAGE + (swave - 2) * 256), 4, pvoff, g * a.N * 4, 0, 0);
    };

    // ---- fragment addressing: lane (frow, fhalf) feeds k = 64*kb + 32*fhalf .. +31 of its row, i.e. group
    // f = 2*kb + fhalf of the row's block: 16 bytes among the pieces, 8 bytes among the tails
    const int frow = lane & 31, fhalf = lane >> 5;
    const int toff = 2048 + 256 * fhalf + 8 * frow;                        // k-block 1: 512 bytes further
    const int a_row = wm * G6G_TM * G6G_BLOCK;
    const int b_row = G6G_B_AT + wn * G6G_TN * G6G_BLOCK;
    // Byte addresses of the reads in stage 0.  The 8-byte tail reads have one opaque register each: reads whose addresses
    // share a visible base get merged into paired reads, whose result could not land in two operand tuples without register
    // copies.
    int ma[2], mb[2], ta[2][G6G_TM], tb[2][G6G_TN];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int moff = 64 * frow + 16 * ((2 * kb + fhalf) ^ ((frow >> 2) & 3));
        ma[kb] = a_row + moff;
        mb[kb] = b_row + moff;
        asm volatile("" : "+v"(ma[kb]), "+v"(mb[kb]));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            ta[kb][i] = a_row + i * G6G_BLOCK + toff + 512 * kb;
            tb[kb][i] = b_row + i * G6G_BLOCK + toff + 512 * kb;
            asm volatile("" : "+v"(ta[kb][i]), "+v"(tb[kb][i]));
        }
    }
    int rec_at = G6G_REC_AT + (wm * G6G_WM + frow) * 16, sum_at = G6G_SUM_AT + (wn * G6G_TN * 32 + frow) * 4;
    asm volatile("" : "+v"(rec_at), "+v"(sum_at));

    // F / 64: facc[j] holds the row blocks i = 0, 1 of column block j, 16 registers each
    v32f facc[G6G_TN];
#pragma unroll
    for (int j = 0; j < G6G_TN; ++j)
#pragma unroll
        for (int r = 0; r < 32; ++r) facc[j][r] = 0.0f;
    float rsum[G6G_TM] = {0.0f, 0.0f};                                     // R_m of this lane's tokens (lane % 32)
    // operand registers: six consecutive VGPRs per fragment; the builtin takes eight, the fp6 form reads six
    v8i pa[2][G6G_TM], pb[2][G6G_TN];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 2; ++i) pa[kb][i] = pb[kb][i] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
    // constants of a group: the records of this lane's tokens, the sums of its channels
    v4i rec[G6G_TM];
    int csum[G6G_TN];
    auto read_one = [&](v8i& dst, const uint8_t* main_ptr, const uint8_t* tail_ptr) {
        const v4i m = *reinterpret_cast<const v4i*>(main_ptr);
        const v2i t = *reinterpret_cast<const v2i*>(tail_ptr);
        dst[0] = m[0]; dst[1] = m[1]; dst[2] = m[2]; dst[3] = m[3]; dst[4] = t[0]; dst[5] = t[1];
    };
    auto read_a = [&](int kb, int i) { read_one(pa[kb][i], lds + ma[kb] + i * G6G_BLOCK, lds + ta[kb][i]); };
    auto read_b = [&](int kb, int j) { read_one(pb[kb][j], lds + mb[kb] + j * G6G_BLOCK, lds + tb[kb][j]); };
    // As integers: the compiler puts a wait for every outstanding direct-to-LDS load in front of a float-typed LDS read.
    auto read_constants = [&](int t) {
        rec[t] = *reinterpret_cast<const v4i*>(lds + rec_at + t * 32 * 16);
        csum[t] = *reinterpret_cast<const int*>(lds + sum_at + t * 32 * 4);
    };
    int stage = 0;
    auto next_stage = [&]() {
        const bool wrap = stage == G6G_STAGES - 1;
        const int d = wrap ? -(G6G_STAGES - 1) : 1;
        static_assert(G6G_A_STAGE == G6G_B_STAGE, "one step for both operands");
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            ma[kb] += d * G6G_A_STAGE; mb[kb] += d * G6G_A_STAGE;
#pragma unroll
            for (int i = 0; i < 2; ++i) { ta[kb][i] += d * G6G_A_STAGE; tb[kb][i] += d * G6G_A_STAGE; }
        }
        rec_at += d * G6G_REC_STAGE;
        sum_at += d * G6G_SUM_STAGE;
        stage = wrap ? 0 : stage + 1;
    };
    const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // S_g of the four blocks (i, j).  The weights are the first MFMA operand: accumulator register r of lane l belongs to token
    // l % 32 of the row block and to output channel 8*(r/4) + 4*(l/32) + r%4 of the column block.
    v16f acc[G6G_TM][G6G_TN] = {{zero, zero}, {zero, zero}};
    auto close_half = [&](int i, int j, int half, float scale) {           // F' += s_mg * S_g, eight registers
#pragma unroll
        for (int r = 8 * half; r < 8 * half + 8; ++r) facc[j][16 * i + r] = fmaf(scale, acc[i][j][r], facc[j][16 * i + r]);
        asm volatile("" : "+v"(facc[j]));                                  // here, not where the sums are next used
    };

    // ---- prologue: the first three groups.  A wave's loads complete in the order it issued them, so "at most n
    // outstanding" below always names the newest n.
#pragma unroll
    for (int g = 0; g < G6G_STAGES; ++g)
        if (g < ngroups) {
#pragma unroll
            for (int i = 0; i < G6G_ALL_LOADS; ++i) issue_one(g, g, i);
        }
    if (ngroups > 2) g6g_wait_loads_and_barrier<2 * G6G_ALL_LOADS>();
    else if (ngroups > 1) g6g_wait_loads_and_barrier<G6G_ALL_LOADS>();
    else g6g_wait_loads_and_barrier<0>();
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        read_b(kb, 0);
        read_a(kb, 0);
        read_constants(kb);
    }
    __builtin_amdgcn_sched_barrier(0);

    // One group per pass: blocks (i, j) = (0,0), (1,0), (0,1), (1,1), two MFMAs each.  Fragments B0 and A0 and the constants were
    // read during the group before; A1 and B1 are read with the first block.  The barrier, in front of the first MFMA of block
    // (0,1), ends every wave's reads of stage g, which group g + 3 refills from here on, and begins those of stage g + 1: B0
    // and A0, whose last uses are blocks (1,0) and (0,1), with a block and a half to arrive, and the constants.
    // Behind every MFMA go eight multiply-adds of a closing, one block late: the two pipes take 32 cycles each, side by side
    // (sixteen behind every second MFMA left each pipe idle in turns).
    float prev_s[2] = {0.0f, 0.0f};                                        // scales of the group before, for its blocks (., 1)
    auto group = [&](int g, auto loads_c, auto newest_c) {
        constexpr bool loads = decltype(loads_c)::value;
        constexpr int newest = decltype(newest_c)::value;                  // loads that may be in flight at the barrier
        const int here = stage;
        float s[2] = {0.0f, 0.0f}, zlane = 0.0f, c1 = 0.0f;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int i = (t >> 1) & 1, j = t >> 2, kb = t & 1;
            if (t == 4) g6g_wait_loads_and_barrier<newest>();
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(pb[kb][j], pa[kb][i], kb == 0 ? zero : acc[i][j], 2, 2, 0, 0, 0, 0);
            if (t == 2) {
                // the constants, not before: they were the last to be read; out of their registers before t = 6 reads the next
                s[0] = __int_as_float(rec[0][0]); s[1] = __int_as_float(rec[1][0]);
                const float z0 = __int_as_float(rec[0][1]), z1 = __int_as_float(rec[1][1]);
                zlane = fhalf ? z1 : z0;                                   // block l / 32 of the rank-1 update
                const float c0 = 0.015625f * (float)csum[0];
                c1 = 0.015625f * (float)csum[1];
                rsum[0] += fmaf(s[0], (float)rec[0][2], 128.0f * z0);
                rsum[1] += fmaf(s[1], (float)rec[1][2], 128.0f * z1);
                asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(rsum[0]), "+v"(rsum[1]), "+v"(c1));
                facc[0] = __builtin_amdgcn_mfma_f32_32x32x1f32(c0, zlane, facc[0], 0, 0, 0);
            }
            if (t == 4) facc[1] = __builtin_amdgcn_mfma_f32_32x32x1f32(c1, zlane, facc[1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (t < 2) { read_a(t, 1); read_b(t, 1); }
            if (t == 2) next_stage();
            if (t == 4) { read_b(0, 0); read_a(0, 0); }
            if (t == 5) { read_b(1, 0); read_a(1, 0); }
            if (t == 6) { read_constants(0); read_constants(1); }
            if (loads && t >= 4) {
                issue_one(here, g + G6G_STAGES, 2 * (t - 4));
                if (2 * (t - 4) + 1 < G6G_ALL_LOADS) issue_one(here, g + G6G_STAGES, 2 * (t - 4) + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            // behind MFMAs 2b + 1 and 2b + 2: the halves of block b - 1, of this group or of the one before
            const int c = (t + 5) / 2 % 4;
            close_half(c & 1, c >> 1, (t & 1) ^ 1, t >= 3 ? s[c & 1] : prev_s[c & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        prev_s[0] = s[0];
        prev_s[1] = s[1];
    };
    constexpr std::integral_constant<int, G6G_ALL_LOADS> one_stage{};
    constexpr std::integral_constant<int, 0> none{};
    int g = 0;
    for (; g + G6G_STAGES < ngroups; ++g) {
        asm volatile(".p2align 4");
        group(g, std::true_type{}, one_stage);
    }
    for (; g + 2 < ngroups; ++g) group(g, std::false_type{}, one_stage);
    for (; g < ngroups; ++g) group(g, std::false_type{}, none);
    close_half(0, 1, 1, prev_s[0]);
    close_half(1, 1, 0, prev_s[1]);
    close_half(1, 1, 1, prev_s[1]);
    __syncthreads();

    // ---- epilogue: column constants through LDS (sw, sw * zp, c), rows already in registers
    v4i* lcol = reinterpret_cast<v4i*>(lds);
    if (tid < G6G_BN) {
        int n = n0 + tid;
        n = n < a.N ? n : a.N - 1;
        const float sw = bf16_to_f32(a.w_scale[n]), zp = bf16_to_f32(a.w_zero[n]);
        const float c = a.out_bias ? a.out_bias[n] : 0.0f;
        lcol[tid] = v4i{__float_as_int(sw), __float_as_int(sw * zp), __float_as_int(c), 0};
    }
    __syncthreads();
    auto result = [&](int i, int j, int r, v4i col) {
        return fmaf(__int_as_float(col[0]), 64.0f * facc[j][16 * i + r], fmaf(-__int_as_float(col[1]), rsum[i], __int_as_float(col[2])));
    };
    auto col_block = [&](int j) { return wn * G6G_TN + j; };
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    unsigned outv[G6G_TM][G6G_TN][4][2];
#pragma unroll
    for (int j = 0; j < G6G_TN; ++j) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v4i cp[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) cp[e] = lcol[col_block(j) * 32 + 8 * q + 4 * fhalf + e];
#pragma unroll
            for (int i = 0; i < G6G_TM; ++i)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const float y0 = result(i, j, 4 * q + 2 * p, cp[2 * p]), y1 = result(i, j, 4 * q + 2 * p + 1, cp[2 * p + 1]);
                    outv[i][j][q][p] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2){y0, y1}, b2));   // hardware round-to-nearest-even
                    asm volatile("" : "+v"(outv[i][j][q][p]));         // computed here: one set of column constants at a time
                }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    store_outputs<G6G_TM, G6G_TN, G6G_BM>(a, (StoreForm)store_form, m0, n0, wm * G6G_WM, lane, outv, col_block);
#endif  // __HIP_DEVICE_COMPILE__
}

}  // namespace

bool gemm_grouped_fp6_applicable(const GemmArgs& a) {
    const int64_t ngroups = a.K / 128;
    // buffer addressing: every table must be smaller than 4 GiB
    return a.Aq6 && a.Wq6 && a.K % 128 == 0 && a.M >= 1 && (int64_t)basq_fp6_bytes(a.M, a.K) < 0xFFFFFFFFll &&
           (int64_t)basq_fp6_bytes(a.N, a.K) < 0xFFFFFFFFll && a.M * ngroups * 16 < 0xFFFFFFFFll &&
           ngroups * a.N * 4 < 0x7FFFFFFFll;
}

int launch_gemm_grouped_fp6(const GemmArgs& a, const int32_t* w_gsum, hipStream_t s) {
    if (a.M == 0) return BASQ_OK;
    if (gemm_grouped_wide_applicable(a, w_gsum) && gemm_grouped_wide_is_faster(a.M, a.N, a.K)) return launch_gemm_grouped_wide(a, w_gsum, s);
    return launch_gemm_grouped_fp6_narrow(a, w_gsum, s);
}

int launch_gemm_grouped_fp6_narrow(const GemmArgs& a, const int32_t* w_gsum, hipStream_t s) {
    const int64_t tm = (a.M + G6G_BM - 1) / G6G_BM;
    const int64_t tn = ((int64_t)a.N + G6G_BN - 1) / G6G_BN;
    if (tm * tn > 0x7FFFFFFFll) return fail(BASQ_EINVAL, "w4a4_gemm_grouped: problem too large for one launch");
    GemmArgs b = a;
    // shared lines: with the hint from K = 1024 on (3000 x 20016, K = 4096 225 us with and 229 without; 1000 x 26416, K = 1024 42 and
    // 46), with half lines (2048 x 12320, K = 512 25 and 29) and where all workgroups are in flight at once (1000 x 5008, K = 512
    // 8.9 and 9.7); otherwise the stores bound it (3000 x 20016, K = 512 58 and 52)
    b.store_form = output_form(a, a.K >= 1024 || (a.ldy & 31) == 0 || tm * tn <= 512);
    hipLaunchKernelGGL(gemm_w4a4_grouped_fp6_kernel, dim3((unsigned)(tm * tn)), dim3(G6G_THREADS), 0, s, b, w_gsum, (int)tm, (int)tn);
    return check_hip(hipGetLastError(), "w4a4_gemm_grouped (fp6) launch");
}

}  // namespace basq
