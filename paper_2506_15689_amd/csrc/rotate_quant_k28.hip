// Fast rotate + bias + quantise kernel for rot_size == K == 14336 = 28 * 512: the rotation is
// H_28 (x) H_512 (Paley type-I H_28; paper Sec. 5.2 splits a large non-power-of-two rotation in one
// Cooley-Tukey step).  Channel k = i*512 + j, i the H_28 index.
//
// Two wavefronts share a token (four up to 256 tokens, see the split kernel); wave half h owns output rows i' in [16h, 16h+16) (rows >= 28 idle).
//   1. H_28 along i on the matrix core, exact: lane (g = l/16, m = l%16) loads rows i = 8g+t, t = 0..7,
//      columns j = 128*jb + 8m .. +8 (16 B each), transposes the 8x8 bf16 block in registers
//      (v_perm), and feeds it as A (row = column group m, k = i) to one bf16 MFMA per column
//      offset jj against the +-1 matrix H_28 (k = i, n = i').  After it a lane holds, for its
//      i' = 16h + l%16, the columns j = 128*jb + 32*(l/16) + 8*r + jj.
//   2. H_512 along j in fp32: seven butterfly stages over register bits (jj, r, jb) and two over
//      lane bits 4 and 5, done by swapping register halves with v_permlane16_swap / v_permlane32_swap
//      so that both operands of a butterfly sit in one lane.
//   3. Every lane now owns 128 consecutive channels: normalise, bias (from LDS), min/max, the two
//      waves of the token combine their ranges through LDS, quantise, pack, store.
#include "basq_internal.h"

#include <type_traits>

namespace basq {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v4i __attribute__((ext_vector_type(4)));

#define K28_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int K28 = 14336;
constexpr int K28_CUS = 256;
constexpr int K28_VEC_BYTES = K28 * 4;              // b^c or s^a in LDS
constexpr int K28_BLOCK_BYTES = 8 * 1024;           // a column block of a token in LDS: 32 rows x 128 columns in bf16

struct H28Cols {
    uint32_t col[28];   // bit i of col[j] set  <=>  H28[i][j] == -1
};

template <int CTRL>
__device__ __forceinline__ float dppf(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ int dppi(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}

#define BFLY28(x, y) do { const float _a = (x), _b = (y); (x) = _a + _b; (y) = _a - _b; } while (0)

// butterfly across lane bit 5 (SWAP32) or lane bit 4 for the register pair (x, y): afterwards x holds
// the sums and y the differences; the lane bit now tells which of the two former registers it was
template <bool SWAP32>
__device__ __forceinline__ void cross_lane_bfly(float& x, float& y) {
    unsigned a = __float_as_uint(x), b = __float_as_uint(y);
    if (SWAP32) {
        auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0]; b = r[1];
    } else {
        auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0]; b = r[1];
    }
    const float fa = __uint_as_float(a), fb = __uint_as_float(b);
    x = fa + fb;
    y = fa - fb;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() would also wait for the global
// loads of the next token and for the code stores, which nothing on the other side of the barrier reads.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Wait until at most N of this wave's memory operations are outstanding (they complete in the order they were issued).
template <int N>
__device__ __forceinline__ void wait_memory() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// A 4-byte LDS write that the compiler does not see as one: it would wait for every direct load into LDS in flight.
__device__ __forceinline__ void lds_write(const void* p, int v) {
    asm volatile("ds_write_b32 %0, %1" ::"v"((int)(uintptr_t)K28_LDS_PTR(p)), "v"(v) : "memory");
}

#if defined(__HIP_DEVICE_COMPILE__)   // device-only buffer-resource types
// 16-byte loads of column block jb of a token: rows 8g .. 8g+7.  Buffer loads on a descriptor that ends with
// the token: rows >= 28 lie past its end and read as zero without a branch -- with a branch per row the paths
// that meet afterwards carry different numbers of loads in flight and every wait becomes a wait for all of them,
// the prefetched block of the next token included.  `x` is uniform over the wave.  (`bytes` = 0: a token that does not
// exist, nothing is read.)
__device__ __forceinline__ void k28_load_block(v4u (&R)[8], const uint16_t* x, int jb, int bytes, int lane) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x), 0, bytes, 0x00020000);
    const int voff = 8192 * (lane >> 4) + 16 * (lane & 15) + 256 * jb;   // bytes; row i = 8g + t starts at 1024 i
#pragma unroll
    for (int t = 0; t < 8; ++t)
        R[t] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 1024 * t, 0, 2 /* non-temporal */));
}

// b^c and s^a into LDS by direct loads: 16 bytes q of the 512-byte run of channels 512 i' + 128 g + 4 q .. + 3 stand at place
// q ^ (i' % 16), so that 16 lanes of a read (i' = 0 .. 15) spread over the banks, and a direct load reads whole lines.
template <int WAVES, bool HAS_BIAS, bool HAS_SCALE>
__device__ __forceinline__ void k28_stage_vectors(const RotateQuantArgs& a, uint8_t* lds, int wave, int lane) {
    static_assert(K28_VEC_BYTES % (1024 * WAVES) == 0, "whole rounds of direct loads");
#pragma unroll
    for (int i = 0; i < K28_VEC_BYTES / 1024 / WAVES; ++i) {
        const int piece = i * WAVES + wave;
        const int voff = (lane >> 5) * 512 + 16 * ((lane & 31) ^ ((piece >> 1) & 15));
        if (HAS_BIAS)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.bias), 0, K28_VEC_BYTES, 0x00020000),
                                                     K28_LDS_PTR(lds + piece * 1024), 16, voff, piece * 1024, 0, 0);
        if (HAS_SCALE)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.act_scale), 0, K28_VEC_BYTES, 0x00020000),
                                                     K28_LDS_PTR(lds + (HAS_BIAS ? K28_VEC_BYTES : 0) + piece * 1024), 16, voff, piece * 1024, 0, 0);
    }
}

// B operand: H_28[k = 8g + t][n = ip], zero outside 28 x 28; `signs`: column ip of the matrix
__device__ __forceinline__ v8bf k28_bop(uint32_t signs, bool row_valid, int g) {
    typedef short v8s __attribute__((ext_vector_type(8)));
    v8s tmp;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int i = 8 * g + t;
        short v = 0;
        if (row_valid && i < 28) v = (short)(((signs >> i) & 1u) ? 0xBF80 : 0x3F80);
        tmp[t] = v;
    }
    return __builtin_bit_cast(v8bf, tmp);
}

// H_28 of one column block: d[jj][r]
__device__ __forceinline__ void k28_h28_block(const v4u (&R)[8], v8bf bop, float (&d)[8][4]) {
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
        v4u A;
        const int w = jj >> 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // bytes of (hi, lo) = (R[2u+1][w], R[2u][w]); even jj takes the low halves, odd jj the high halves
            A[u] = (jj & 1) ? __builtin_amdgcn_perm(R[2 * u + 1][w], R[2 * u][w], 0x07060302u)
                            : __builtin_amdgcn_perm(R[2 * u + 1][w], R[2 * u][w], 0x05040100u);
        }
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, A), bop, acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) d[jj][r] = acc[r];
    }
}

// the stages over jj (j0..2) and r (j3..4) of one column block
__device__ __forceinline__ void k28_block_stages(float (&d)[8][4]) {
#pragma unroll
    for (int s = 1; s < 8; s <<= 1)
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            if ((jj & s) == 0)
#pragma unroll
                for (int r = 0; r < 4; ++r) BFLY28(d[jj][r], d[jj + s][r]);
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
        BFLY28(d[jj][0], d[jj][1]);
        BFLY28(d[jj][2], d[jj][3]);
        BFLY28(d[jj][0], d[jj][2]);
        BFLY28(d[jj][1], d[jj][3]);
    }
}

// Range of a wave's values, the same in every lane
__device__ __forceinline__ void k28_wave_range(float& mn, float& mx) {
    mn = fminf(mn, dppf<0xB1>(mn)); mx = fmaxf(mx, dppf<0xB1>(mx));
    mn = fminf(mn, dppf<0x4E>(mn)); mx = fmaxf(mx, dppf<0x4E>(mx));
    mn = fminf(mn, dppf<0x141>(mn)); mx = fmaxf(mx, dppf<0x141>(mx));
    mn = fminf(mn, dppf<0x140>(mn)); mx = fmaxf(mx, dppf<0x140>(mx));
    float lo4[4], hi4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        lo4[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mn), 16 * q));
        hi4[q] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mx), 16 * q));
    }
    mn = fminf(fminf(lo4[0], lo4[1]), fminf(lo4[2], lo4[3]));
    mx = fmaxf(fmaxf(hi4[0], hi4[1]), fmaxf(hi4[2], hi4[3]));
}

__device__ __forceinline__ int k28_wave_sum(int sum) {
    sum += dppi<0xB1>(sum);
    sum += dppi<0x4E>(sum);
    sum += dppi<0x141>(sum);
    sum += dppi<0x140>(sum);
    return __builtin_amdgcn_readlane(sum, 0) + __builtin_amdgcn_readlane(sum, 16) +
           __builtin_amdgcn_readlane(sum, 32) + __builtin_amdgcn_readlane(sum, 48);
}

// Codes of the 32 channels d[jj][r] of group jb of a lane (chunk 4*i' + g of the fp6 layout): 16 bytes in the 4-bit form, their sum, and
// with `store6` the fp6 form, stored.
__device__ __forceinline__ void k28_quantise_group(const RotateQuantArgs& a, const float (&d)[8][4], float inv, float nlo, bool row_valid,
                                                   bool store6, int64_t m, int64_t rb6, int chunk, int jb, uint32_t (&words)[4], int& sum) {
    v16f qe, qo;                                           // the clamped values before rounding: low / high nibbles
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        uint32_t ev = 0, od = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float t0 = __builtin_amdgcn_fmed3f(fmaf(d[2 * p][r], inv, nlo), 0.0f, 15.0f);
            const float t1 = __builtin_amdgcn_fmed3f(fmaf(d[2 * p + 1][r], inv, nlo), 0.0f, 15.0f);
            ev = __builtin_amdgcn_cvt_pk_u8_f32(t0, p, ev);
            od = __builtin_amdgcn_cvt_pk_u8_f32(t1, p, od);
            qe[4 * r + p] = t0;
            qo[4 * r + p] = t1;
        }
        if (row_valid) {
            sum = __builtin_amdgcn_udot4(ev, 0x01010101u, sum, false);
            sum = __builtin_amdgcn_udot4(od, 0x01010101u, sum, false);
        }
        words[r] = ev | (od << 4);
    }
    if (store6) {
        // The 32 codes once more, as e2m3 numbers q/8, straight from the clamped values: the
        // packed conversion divides by its scale operand, rounds to nearest-even (on the e2m3 grid below 2
        // that is t/8 -> rint(t)/8, ties as in the integer conversion) and interleaves its two sources.
        const v6i f6 = __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(qe, qo, 8.0f);
        const int rr = (int)(m & 31);
        uint8_t* blk = a.Aq6 + ((int64_t)chunk * rb6 + (m >> 5)) * 3072;
        *reinterpret_cast<uint4*>(blk + 64 * rr + 16 * (jb ^ ((rr >> 2) & 3))) =
            make_uint4((uint32_t)f6[0], (uint32_t)f6[1], (uint32_t)f6[2], (uint32_t)f6[3]);
        *reinterpret_cast<uint2*>(blk + 2048 + 256 * jb + 8 * rr) = make_uint2((uint32_t)f6[4], (uint32_t)f6[5]);
    }
}
#endif  // __HIP_DEVICE_COMPILE__

// What bounds it: 2450 vector instructions per wave and token, 17 us for 2048 tokens, if the memory is busy beside them.
//
// The vectors b^c and s^a go to LDS by direct loads requested behind the first token's and not waited for before they are
// used.  (A loop of loads and LDS writes in front of everything was 16 memory latencies in a row: one token 10.5 us, without
// 8.2; 1024 tokens 20.4 and 17.5; 64 with both vectors 16.7 and 10.8.)
//
// STAGED = 0: a wave has one token, and a compute unit takes the next workgroup when it has done with one.
// STAGED > 0: workgroups stay and walk over the tokens.  The column blocks 1 .. STAGED of the next token are requested straight
// into LDS as soon as both waves of the token have read them, and are there when it begins, as is block 0, in registers.  (With
// block 0 alone requested ahead every round began with a memory latency and 20 KB a token.)  Four tokens and one vector take
// 152 KB of LDS, so four tokens (eight waves) share a workgroup; with both vectors there is room for one block of a token.
// Which one is taken where: launch_k28_flags().
template <int TOKENS, bool HAS_BIAS, bool HAS_SCALE, bool ROT_OUT, int STAGED>
__global__ __launch_bounds__(TOKENS * 128, TOKENS == 2 && !(HAS_BIAS && HAS_SCALE) ? 2 : 1) void rotate_quant_k28_kernel(RotateQuantArgs a, float norm, H28Cols hc) {
#if defined(__HIP_DEVICE_COMPILE__)   // the body uses device-only buffer-resource types; the host pass only needs the stub
    constexpr int WAVES = 2 * TOKENS;
    constexpr int VECTORS = (HAS_BIAS ? 1 : 0) + (HAS_SCALE ? 1 : 0);
    constexpr int SCALE_AT = HAS_BIAS ? K28_VEC_BYTES : 0;
    constexpr int STAGE_AT = VECTORS * K28_VEC_BYTES;
    constexpr int RED_AT = STAGE_AT + TOKENS * STAGED * K28_BLOCK_BYTES;
    constexpr int VEC_PIECES = K28_VEC_BYTES / 1024 / WAVES;           // 1 KB pieces of a vector that a wave brings
    __shared__ __attribute__((aligned(1024))) uint8_t lds[RED_AT + 2 * TOKENS * 32];
    int* red = reinterpret_cast<int*>(lds + RED_AT);   // [parity][token in block][half][mn, mx, sum, -]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave & 1, tok_in_blk = wave >> 1;
    const int g = lane >> 4, m16 = lane & 15;
    const int ip = 16 * half + m16;                // output row i'
    const bool row_valid = ip < 28;
    const uint32_t signs = hc.col[row_valid ? ip : 27];  // requested first: a wait for it waits for nothing else

    // Workgroups g, g+8, ... share an XCD; renumbered so that 32 consecutive tokens (one block of the fp6 output) go to one,
    // meet in its L2 and their pieces merge there: runs of 32 / TOKENS workgroups, as far as all XCDs have one.
    constexpr int RUN = 32 / TOKENS;
    int vblock = blockIdx.x;
    if (vblock < (int)gridDim.x / (8 * RUN) * (8 * RUN)) {
        const int xcd = vblock & 7, i = vblock >> 3;
        vblock = ((i / RUN) * 8 + xcd) * RUN + i % RUN;
    }
    const int64_t rb6 = (a.M + 31) >> 5;                    // 32-row blocks per chunk of the fp6 output
    const int64_t tokens_per_round = (int64_t)gridDim.x * TOKENS;
    const int64_t m_first = (int64_t)vblock * TOKENS;
    // Blocks 1 .. STAGED of a token straight into LDS, in the lanes' order: wave half h brings rows 8g + 4h .. 8g + 4h + 3.
    uint8_t* const staged = lds + STAGE_AT + tok_in_blk * STAGED * K28_BLOCK_BYTES;
    auto stage_blocks = [&](int64_t tok, int bytes) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.X + tok * a.ldx), 0, bytes, 0x00020000);
        const int voff = 8192 * g + 16 * m16 + 4096 * half;
#pragma unroll
        for (int jb = 1; jb <= STAGED; ++jb)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, K28_LDS_PTR(staged + (jb - 1) * K28_BLOCK_BYTES + (4 * half + t) * 1024), 16,
                                                         voff + 256 * jb + 1024 * t, 0, 0, 2 /* non-temporal */);
    };
    auto load_block = [&](v4u (&R)[8], int64_t tok, int jb, int bytes) { k28_load_block(R, a.X + tok * a.ldx, jb, bytes, lane); };
    v4u R[4][8];
    {
        const int64_t m = m_first + tok_in_blk;
        const int64_t mm = m < a.M ? m : a.M - 1;
        if (STAGED > 0 && half == 1 && g == 3) {
            // rows 28 .. 31 lie past the token's end: zeros, also if such a load should write nothing
#pragma unroll
            for (int jb = 0; jb < STAGED; ++jb)
#pragma unroll
                for (int t = 4; t < 8; ++t) *reinterpret_cast<v4i*>(staged + jb * K28_BLOCK_BYTES + t * 1024 + lane * 16) = v4i{0, 0, 0, 0};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        load_block(R[0], mm, 0, K28 * 2);
        if (STAGED > 0) stage_blocks(mm, K28 * 2);
        else
#pragma unroll
            for (int jb = 1; jb < 4; ++jb) load_block(R[jb], mm, jb, K28 * 2);
    }
    k28_stage_vectors<WAVES, HAS_BIAS, HAS_SCALE>(a, lds, wave, lane);
    __builtin_amdgcn_sched_barrier(0);
    const int vec_row = row_valid ? ip : 27;           // (rows past the matrix: any values, they go nowhere)
    int vec_at = vec_row * 2048 + g * 512 + 16 * (vec_row & 15);
    // As integers: the compiler puts a wait for every outstanding direct load in front of a float-typed LDS read.
    auto vec4 = [&](int base, int q) { return *reinterpret_cast<const v4i*>(lds + base + ((vec_at ^ (16 * (q & 15))) + 256 * (q >> 4))); };

    const v8bf bop = k28_bop(signs, row_valid, g);
    if (STAGED > 0) {
        wait_memory<VECTORS * VEC_PIECES>();
        lds_barrier();
    }
    // The row sums of the two halves meet one token late, at the next token's barrier, so that a token
    // costs one barrier: red is double buffered by token parity.
    int parity = 0;
    int64_t prev_m = -1;
    float prev_s = 0.f, prev_lo = 0.f;
    for (int64_t m0 = m_first;; m0 += tokens_per_round, parity ^= 1) {
        const int64_t m = m0 + tok_in_blk;
        const bool tok_valid = m < a.M;
        const int64_t mm = tok_valid ? m : a.M - 1;      // keep every wave on the same barrier schedule

        // ---- H_28 on the matrix core.  Blocks that were not requested a token ago are requested together now, while the
        // accumulators that will replace them are not live yet.
        float d[4][8][4];                                  // [jb][jj][r]
        if (STAGED > 0) {
#pragma unroll
            for (int jb = STAGED + 1; jb < 4; ++jb) load_block(R[jb], mm, jb, K28 * 2);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (jb >= 1 && jb <= STAGED)
                    R[jb][t] = __builtin_bit_cast(v4u, *reinterpret_cast<const v4i*>(staged + (jb - 1) * K28_BLOCK_BYTES + t * 1024 + lane * 16));
            k28_h28_block(R[jb], bop, d[jb]);
        }
        // first block of this wave's next token: its latency hides behind the butterflies below
        const bool more = STAGED > 0 && m0 + tokens_per_round < a.M;
        const int64_t next = m + tokens_per_round < a.M ? m + tokens_per_round : a.M - 1;
        if (STAGED > 0) load_block(R[0], next, 0, more ? K28 * 2 : 0);
        __builtin_amdgcn_sched_barrier(0);

        // ---- H_512: register stages jj (j0..2), r (j3..4), jb (j7..8) ------------------------------------
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) k28_block_stages(d[jb]);
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                BFLY28(d[0][jj][r], d[1][jj][r]);
                BFLY28(d[2][jj][r], d[3][jj][r]);
                BFLY28(d[0][jj][r], d[2][jj][r]);
                BFLY28(d[1][jj][r], d[3][jj][r]);
            }
        // ---- lane stages: j5 (lane bit 4) pairs jb bit 0, j6 (lane bit 5) pairs jb bit 1.  Afterwards
        // register index jb means (j5, j6) and lane bits (4, 5) mean (j7, j8).
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                cross_lane_bfly<false>(d[0][jj][r], d[1][jj][r]);
                cross_lane_bfly<false>(d[2][jj][r], d[3][jj][r]);
                cross_lane_bfly<true>(d[0][jj][r], d[2][jj][r]);
                cross_lane_bfly<true>(d[1][jj][r], d[3][jj][r]);
            }

        // ---- this lane owns channels ip*512 + 128*g + c, c = 32*jb + 8*r + jj ---------------------------
        const int ch0 = ip * 512 + 128 * g;
        if (VECTORS > 0 && m0 == m_first) {                // the vectors have arrived, every wave's part of them
            wait_memory<(STAGED > 0 ? 8 : 0)>();             // (behind them only the next token's block 0)
            lds_barrier();
        }
        float mn = INFINITY, mx = -INFINITY;
        asm volatile("" : "+v"(vec_at));                   // (32 addresses kept over the tokens would be spilled)
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int q2 = 0; q2 < 2; ++q2) {
                    const int c = 32 * jb + 8 * r + 4 * q2;
                    v4i bb = {0, 0, 0, 0}, ss = {0, 0, 0, 0};
                    if (HAS_BIAS) bb = vec4(0, c >> 2);
                    if (HAS_SCALE) ss = vec4(SCALE_AT, c >> 2);
                    float rr[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float rv = d[jb][4 * q2 + e][r] * norm;
                        rr[e] = rv;
                        const float bv = __int_as_float(bb[e]);
                        const float v = HAS_SCALE ? fmaf(rv, __int_as_float(ss[e]), -bv) : rv - bv;
                        d[jb][4 * q2 + e][r] = v;
                        mn = fminf(mn, v);
                        mx = fmaxf(mx, v);
                    }
                    if (ROT_OUT && row_valid && tok_valid)
                        *reinterpret_cast<float4*>(a.rot_out + m * (int64_t)K28 + ch0 + c) = make_float4(rr[0], rr[1], rr[2], rr[3]);
                }
        if (!row_valid) { mn = INFINITY; mx = -INFINITY; }
        k28_wave_range(mn, mx);                            // then the two halves of the token through LDS
        const int* myred = red + (parity * TOKENS + tok_in_blk) * 8;
        const int* otherred = red + ((parity ^ 1) * TOKENS + tok_in_blk) * 8;
        if (lane == 0) {
            lds_write(myred + half * 4, __float_as_int(mn));
            lds_write(myred + half * 4 + 1, __float_as_int(mx));
        }
        lds_barrier();
        mn = fminf(__int_as_float(myred[0]), __int_as_float(myred[4]));
        mx = fmaxf(__int_as_float(myred[1]), __int_as_float(myred[5]));
        if (half == 0 && lane == 0 && prev_m >= 0) {       // finish the previous token
            basq_tokmeta mt;
            mt.scale = prev_s; mt.lo = prev_lo;
            mt.rowsum = otherred[2] + otherred[6];
            mt.reserved = 0;
            a.meta[prev_m] = mt;
        }
        // Behind the barrier every wave has read its token's blocks: the next one's may come.  (Also where there is none: the
        // compiler counts the requests behind block 0, and with a branch here it would wait for the code stores as well.)
        if (STAGED > 0) stage_blocks(next, more ? K28 * 2 : 0);
        __builtin_amdgcn_sched_barrier(0);

        const float lo = a.clip_lo * mn;
        const float hi = a.clip_hi * mx;
        float s = __fdiv_rn(hi - lo, 15.0f);
        if (!(s > 0.0f && s < INFINITY)) s = 1.0f;
        const float inv = __fdiv_rn(1.0f, s);
        const float nlo = -(lo * inv);

        int sum = 0;
        uint32_t words[4][4];                              // [jb][r]: 16 bytes of codes per jb
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
            k28_quantise_group(a, d[jb], inv, nlo, row_valid, a.Aq6 && row_valid && tok_valid, m, rb6, 4 * ip + g, jb, words[jb], sum);
        // A lane holds 64 consecutive output bytes as four 16-byte pieces.  Transposing the pieces over
        // (jb, g) lets every store instruction write whole 64-byte segments (piece jb of lane g goes to
        // register g of lane jb), instead of four partial writes per segment.
        // (The 4-bit form is optional when the fp6 form is written.)
        if (a.Aq) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                auto s0 = __builtin_amdgcn_permlane16_swap(words[0][r], words[1][r], false, false);
                auto s1 = __builtin_amdgcn_permlane16_swap(words[2][r], words[3][r], false, false);
                auto t0 = __builtin_amdgcn_permlane32_swap(s0[0], s1[0], false, false);
                auto t1 = __builtin_amdgcn_permlane32_swap(s0[1], s1[1], false, false);
                words[0][r] = t0[0]; words[2][r] = t0[1];
                words[1][r] = t1[0]; words[3][r] = t1[1];
            }
            if (row_valid && tok_valid) {
                uint8_t* orow = a.Aq + m * (int64_t)(K28 / 2) + ip * 256 + 16 * g;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    nt_store16(orow + 64 * j, make_uint4(words[j][0], words[j][1], words[j][2], words[j][3]));
            }
        }
        sum = k28_wave_sum(sum);
        if (lane == 0) lds_write(myred + half * 4 + 2, sum);
        prev_m = tok_valid ? m : -1;
        prev_s = s; prev_lo = lo;
        if (!more) break;
        // The next token's blocks are in LDS.  Behind their requests this wave stored at least four pieces of codes (its token
        // exists, or there would be no more), which may still be on their way.
        wait_memory<4>();
        lds_barrier();
    }
    if (STAGED > 0) wait_memory<0>();                      // nothing may be on its way into LDS when the workgroup ends
    lds_barrier();
    if (half == 0 && lane == 0 && prev_m >= 0) {
        const int* lastred = red + (parity * TOKENS + tok_in_blk) * 8;
        basq_tokmeta mt;
        mt.scale = prev_s; mt.lo = prev_lo;
        mt.rowsum = lastred[2] + lastred[6];
        mt.reserved = 0;
        a.meta[prev_m] = mt;
    }
#endif  // __HIP_DEVICE_COMPILE__
}

// Few tokens: one to a workgroup, four waves.  A call this small is all latency -- a wave alone on its SIMD takes five to six cycles
// an instruction, 5.6 us for the 2450 of half a token -- and the split divides the chain: wave (half, part) takes output rows
// [16 half, 16 half + 16) of column blocks 2 part and 2 part + 1.  Parts exchange by way of LDS in front of the stage over the
// upper block bit, after which a wave has columns jj = 4 part .. + 3 of all four blocks, and behind the range, after which it
// has its two blocks' 32-channel groups whole again.  Every sum is that of the two-wave kernel, in its order.
// With two waves a token one took 8.2 us, 64 9.5 and 256 10.9; as built 6.1, 6.9 and 8.4 (64 with both vectors 10.8 and 8.0).  LDS holds
// one workgroup per compute unit, so more than 256 tokens would take two rounds (257 .. 512 on two waves 10.9 - 12.6).
template <bool HAS_BIAS, bool HAS_SCALE>
__global__ __launch_bounds__(256, 1) void rotate_quant_k28_split_kernel(RotateQuantArgs a, float norm, H28Cols hc) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int VECTORS = (HAS_BIAS ? 1 : 0) + (HAS_SCALE ? 1 : 0);
    constexpr int SCALE_AT = HAS_BIAS ? K28_VEC_BYTES : 0;
    constexpr int XCH_AT = VECTORS * K28_VEC_BYTES, RED_AT = XCH_AT + 4 * 8 * 1024;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[RED_AT + 4 * 16];
    int* red = reinterpret_cast<int*>(lds + RED_AT);       // [wave][mn, mx, sum, -]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave & 1, part = wave >> 1;
    const int g = lane >> 4, m16 = lane & 15;
    const int ip = 16 * half + m16;
    const bool row_valid = ip < 28;
    const uint32_t signs = hc.col[row_valid ? ip : 27];    // requested first: a wait for it waits for nothing else
    int64_t m = blockIdx.x;                                // 32 consecutive tokens on one XCD, as in the two-wave kernel
    if ((gridDim.x & 127) == 0) m = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    v4u R[2][8];
#pragma unroll
    for (int b = 0; b < 2; ++b) k28_load_block(R[b], a.X + m * a.ldx, 2 * part + b, K28 * 2, lane);
    k28_stage_vectors<4, HAS_BIAS, HAS_SCALE>(a, lds, wave, lane);
    __builtin_amdgcn_sched_barrier(0);
    const v8bf bop = k28_bop(signs, row_valid, g);

    float d[2][8][4];                                      // [jb - 2 part][jj][r]
#pragma unroll
    for (int b = 0; b < 2; ++b) k28_h28_block(R[b], bop, d[b]);
#pragma unroll
    for (int b = 0; b < 2; ++b) k28_block_stages(d[b]);
#pragma unroll
    for (int jj = 0; jj < 8; ++jj)
#pragma unroll
        for (int r = 0; r < 4; ++r) BFLY28(d[0][jj][r], d[1][jj][r]);

    v4i* const mine = reinterpret_cast<v4i*>(lds + XCH_AT) + wave * 512 + lane;
    const v4i* const theirs = reinterpret_cast<const v4i*>(lds + XCH_AT) + (wave ^ 2) * 512 + lane;
    auto put = [&](int slot, const float (&v)[4]) {
        mine[64 * slot] = v4i{__float_as_int(v[0]), __float_as_int(v[1]), __float_as_int(v[2]), __float_as_int(v[3])};
    };
    float e[4][4][4];                                      // [jb][jj - 4 part][r]
    auto exchange_columns = [&](auto part_c) {
        constexpr int P = decltype(part_c)::value;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) put(4 * b + k, d[b][4 * (1 - P) + k]);
        lds_barrier();
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const v4i o = theirs[64 * (4 * b + k)];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float own = d[b][4 * P + k][r], other = __int_as_float(o[r]);
                    e[b][k][r] = P ? other : own;
                    e[2 + b][k][r] = P ? own : other;
                    BFLY28(e[b][k][r], e[2 + b][k][r]);
                }
            }
    };
    if (part) exchange_columns(std::integral_constant<int, 1>{});
    else exchange_columns(std::integral_constant<int, 0>{});
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            cross_lane_bfly<false>(e[0][k][r], e[1][k][r]);
            cross_lane_bfly<false>(e[2][k][r], e[3][k][r]);
            cross_lane_bfly<true>(e[0][k][r], e[2][k][r]);
            cross_lane_bfly<true>(e[1][k][r], e[3][k][r]);
        }

    // the vectors have arrived, every wave's part of them, and every wave has read its partner's columns
    wait_memory<0>();
    lds_barrier();
    const int vec_row = row_valid ? ip : 27;               // (rows past the matrix: any values, they go nowhere)
    const int vec_at = vec_row * 2048 + g * 512 + 16 * ((vec_row & 15) ^ part);
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int q = 8 * jb + 2 * r;                  // + part
            const uint8_t* const at = lds + ((vec_at ^ (16 * (q & 15))) + 256 * (q >> 4));
            v4i bb = {0, 0, 0, 0}, ss = {0, 0, 0, 0};
            if (HAS_BIAS) bb = *reinterpret_cast<const v4i*>(at);
            if (HAS_SCALE) ss = *reinterpret_cast<const v4i*>(at + SCALE_AT);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float rv = e[jb][k][r] * norm, bv = __int_as_float(bb[k]);
                const float v = HAS_SCALE ? fmaf(rv, __int_as_float(ss[k]), -bv) : rv - bv;
                e[jb][k][r] = v;
                mn = fminf(mn, v);
                mx = fmaxf(mx, v);
            }
        }
    if (!row_valid) { mn = INFINITY; mx = -INFINITY; }
    k28_wave_range(mn, mx);
    if (lane == 0) {
        red[4 * wave] = __float_as_int(mn);
        red[4 * wave + 1] = __float_as_int(mx);
    }
    auto exchange_blocks = [&](auto part_c) {
        constexpr int P = decltype(part_c)::value;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) put(4 * b + k, e[2 * (1 - P) + b][k]);
        lds_barrier();
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const v4i o = theirs[64 * (4 * b + k)];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    d[b][4 * P + k][r] = e[2 * P + b][k][r];
                    d[b][4 * (1 - P) + k][r] = __int_as_float(o[r]);
                }
            }
    };
    if (part) exchange_blocks(std::integral_constant<int, 1>{});
    else exchange_blocks(std::integral_constant<int, 0>{});
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        mn = fminf(mn, __int_as_float(red[4 * w]));
        mx = fmaxf(mx, __int_as_float(red[4 * w + 1]));
    }

    const float lo = a.clip_lo * mn;
    const float hi = a.clip_hi * mx;
    float s = __fdiv_rn(hi - lo, 15.0f);
    if (!(s > 0.0f && s < INFINITY)) s = 1.0f;
    const float inv = __fdiv_rn(1.0f, s);
    const float nlo = -(lo * inv);
    int sum = 0;
    const int64_t rb6 = (a.M + 31) >> 5;
    uint32_t words[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
        k28_quantise_group(a, d[b], inv, nlo, row_valid, a.Aq6 && row_valid, m, rb6, 4 * ip + g, 2 * part + b, words[b], sum);
    if (a.Aq && row_valid) {
        uint8_t* dst = a.Aq + m * (int64_t)(K28 / 2) + ip * 256 + 64 * g + 32 * part;
#pragma unroll
        for (int b = 0; b < 2; ++b) *reinterpret_cast<uint4*>(dst + 16 * b) = make_uint4(words[b][0], words[b][1], words[b][2], words[b][3]);
    }
    sum = k28_wave_sum(sum);
    if (lane == 0) red[4 * wave + 2] = sum;
    lds_barrier();
    if (threadIdx.x == 0) {
        basq_tokmeta mt;
        mt.scale = s; mt.lo = lo;
        mt.rowsum = red[2] + red[6] + red[10] + red[14];
        mt.reserved = 0;
        a.meta[m] = mt;
    }
#endif  // __HIP_DEVICE_COMPILE__
}

template <int TOKENS, bool HB, bool HS, bool ROT_OUT, int STAGED>
int launch_k28_form(const RotateQuantArgs& a, hipStream_t s, float norm, const H28Cols& hc) {
    int64_t blocks = (a.M + TOKENS - 1) / TOKENS;
    if (STAGED > 0 && blocks > K28_CUS) blocks = K28_CUS;
    if (blocks > 0x7FFFFFFFll) return fail(BASQ_EINVAL, "rotate_quant (28x512): too many tokens for one launch");
    hipLaunchKernelGGL((rotate_quant_k28_kernel<TOKENS, HB, HS, ROT_OUT, STAGED>), dim3((unsigned)blocks), dim3(TOKENS * 128), 0, s, a, norm, hc);
    return check_hip(hipGetLastError(), "rotate_quant (28x512) launch");
}

// Up to a token a compute unit: four waves a token.  Otherwise two tokens to a workgroup of one round (two of them fit a compute
// unit, one with both vectors in LDS), but workgroups of four tokens that stay where they are faster:
//  - with both vectors, from 513 tokens on;
//  - with at most one for codes in the 4-bit form alone, if the last round of 1024 tokens leaves at most a tenth of all rounds empty
//    (b^c given, staying workgroups and two-token ones: 1400 tokens 25.2 and 21.7 us, 1800 26.2 and 26.0, 2048 26.9 and 27.7,
//    2049 34.1 and 29.6, 2600 36.4 and 35.7, 2800 36.5 and 37.1, 4100 55.4 and 51.5, 5000 57.8 and 60.5, 8192 86.4 and 96.4).
//    Calls that write the fp6 form are faster on two-token workgroups (1025 26.4 and 20.1, 2048 31.8 and 31.6, 3000 45.0 and 43.9,
//    8192 109.7 and 105.2, 16384 218 and 205), as are those that write the rotation out, where the staying ones spill (2048 98.9
//    and 66.9; 8192 417 and 270).
template <bool HB, bool HS>
int launch_k28_flags(const RotateQuantArgs& a, hipStream_t s, float norm, const H28Cols& hc) {
    if (a.rot_out) return launch_k28_form<2, HB, HS, true, 0>(a, s, norm, hc);
    if (a.M <= K28_CUS) {
        hipLaunchKernelGGL((rotate_quant_k28_split_kernel<HB, HS>), dim3((unsigned)a.M), dim3(256), 0, s, a, norm, hc);
        return check_hip(hipGetLastError(), "rotate_quant (28x512, split) launch");
    }
    constexpr bool BOTH = HB && HS;
    constexpr int64_t ROUND = 4 * K28_CUS;
    const int64_t room = (a.M + ROUND - 1) / ROUND * ROUND;
    const bool stay = BOTH ? a.M > 2 * K28_CUS : !a.Aq6 && a.M > ROUND && room - a.M <= room / 10;
    if (stay) return launch_k28_form<4, HB, HS, false, BOTH ? 1 : 3>(a, s, norm, hc);
    return launch_k28_form<2, HB, HS, false, 0>(a, s, norm, hc);
}

}  // namespace

bool rotate_quant_k28_applicable(const RotateQuantArgs& a) {
    return a.group == a.K && a.has28 && a.rot_size == K28 && a.K == K28 && (a.Aq != nullptr || a.Aq6 != nullptr) &&
           a.meta != nullptr;
}

int launch_rotate_quant_k28(const RotateQuantArgs& a, hipStream_t s) {
    H28Cols hc{};
    const int8_t* h = hadamard28_host();
    for (int j = 0; j < 28; ++j) {
        uint32_t mk = 0;
        for (int i = 0; i < 28; ++i) if (h[i * 28 + j] < 0) mk |= 1u << i;
        hc.col[j] = mk;
    }
    const float norm = (float)(1.0 / sqrt((double)K28));
    const bool hb = a.bias != nullptr, hs = a.act_scale != nullptr;
    if (hb && hs) return launch_k28_flags<true, true>(a, s, norm, hc);
    if (hb) return launch_k28_flags<true, false>(a, s, norm, hc);
    if (hs) return launch_k28_flags<false, true>(a, s, norm, hc);
    return launch_k28_flags<false, false>(a, s, norm, hc);
}

}  // namespace basq
