// The whole layer in ONE launch for few small tokens: rot_size == K in {512, 1024, 2048}, weights in the streaming layout.  At this
// size the two-kernel path is two dependent launches of 3 - 4 us for a fraction of a microsecond of memory traffic, so every
// workgroup rotates and quantises four tokens itself, one a wave -- the routine of rotate_quant_small_kernel, hence the same bits --
// while its weights are on their way, and multiplies them with 64 output channels, 16 a wave.  A token is rotated by all
// ceil(N / 64) workgroups that need it, which is what bounds the rule (linear_small_applicable).
// (Eq. 14 / Eq. 15 rotation, bias and scale, Eq. 4 quantiser, Sec. 5.2 INT4 product.)
//
//   phase 0   a wave requests its token, its values of b^c and s^a, its weights (K / 128 pieces of 16 bytes a lane) and its constants,
//             in the order in which they are used: loads complete in the order of issue
//   phase 1   rotation, range, codes: codes and token record go to LDS
//   phase 2   16 x 16 x 64 int8 MFMA on weights (registers) and codes (LDS; rows of tokens that do not exist are zero), a wave
//             holds the whole sum of its channels; de-quantisation and store
#include "rotate_block_piece.h"

namespace basq {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int LS_WAVES = 4, LS_TOKENS = 4, LS_ROWS = 16 * LS_WAVES;

template <int NP, bool HAS_BIAS, bool HAS_SCALE>
__global__ __launch_bounds__(LS_WAVES * 64, NP == 4 ? 2 : 4) void linear_small_kernel(RotateQuantArgs q, GemmArgs g, float norm) {
    constexpr bool FOLD_NORM = NP == 2;                 // as in rotate_quant_small_kernel
    constexpr int K = 512 * NP, KB = K / 2, CHUNKS = KB / 64;
    constexpr int XQ_STRIDE = KB + 16;                  // the tokens of a quarter wave read pieces that fall on different banks
    __shared__ __attribute__((aligned(16))) uint8_t xq[LS_TOKENS * XQ_STRIDE];
    __shared__ __attribute__((aligned(16))) basq_tokmeta lmeta[LS_TOKENS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = (int)g.M;
    const int m0 = blockIdx.y * LS_TOKENS, m = m0 + wave;
    const int n0 = blockIdx.x * LS_ROWS + 16 * wave;    // this wave's channels
    const bool some = n0 < g.N;

    const P2Lane pl = p2_lane(lane);
    const int eout = rb_eout(lane);
    uint4 raw[NP];
    float2 bb[NP][4], ss[NP][4];
    const int mm = m < M ? m : M - 1;                   // (a wave without a token rotates the last one and keeps it to itself)
#pragma unroll
    for (int c = 0; c < NP; ++c) raw[c] = *reinterpret_cast<const uint4*>(q.X + (int64_t)mm * q.ldx + 512 * c + 8 * pl.chunk);
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (HAS_BIAS) bb[c][r] = *reinterpret_cast<const float2*>(q.bias + 512 * c + eout + 8 * r);
            if (HAS_SCALE) ss[c][r] = *reinterpret_cast<const float2*>(q.act_scale + 512 * c + eout + 8 * r);
        }
    __builtin_amdgcn_sched_barrier(0);
    const uint8_t* wblk = g.Wq + (int64_t)(some ? n0 : 0) * KB + lane * 16;      // piece `lane` of each of the block's KBs
    v4i w[CHUNKS];
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) w[i] = *reinterpret_cast<const v4i*>(wblk + i * 1024);
    // Constants of channel lane % 16: scale and sum in lanes whose bit 4 is clear, zero point and bias in the others.  Addresses are selected
    // and not the loads: behind a branch the compiler waits for the weights before it reuses a register (raw: a conversion would wait too).
    const int row = lane & 15, sub = lane >> 4;
    const int on = n0 + row < g.N ? n0 + row : g.N - 1;
    const int cst2 = (sub & 1 ? g.w_zero : g.w_scale)[on];
    const float cst4 = ((sub & 1) && g.out_bias ? g.out_bias : g.w_sum)[on];
    __builtin_amdgcn_sched_barrier(0);

    v8bf bop[2];
    rb_make_bop<9, FOLD_NORM ? 5 : 0>(lane, bop);
    float v[NP][2][4];
#pragma unroll
    for (int c = 0; c < NP; ++c) rb_rotate_piece(raw[c], bop, v[c]);
    rb_pair_pieces<NP>(v);
    const RbRange x = rb_token_range<NP, FOLD_NORM, HAS_BIAS, HAS_SCALE, false>(v, bb, ss, norm, q.clip_lo, q.clip_hi, nullptr);
    int sum = 0;
    const int q4 = lane & 3, seg = rb_segment(lane);
#pragma unroll
    for (int c = 0; c < NP; ++c)
        *reinterpret_cast<uint32_t*>(xq + wave * XQ_STRIDE + 256 * c + 16 * seg + 4 * q4) = rb_codes(v[c], x.inv, x.nlo, lane, true, sum);
    sum = wave_sum_i(sum);
    if (lane == 0) {
        basq_tokmeta mt;
        mt.scale = x.s; mt.lo = x.lo; mt.rowsum = sum; mt.reserved = 0;
        lmeta[wave] = mt;
    }
    p2_lds_barrier();                                   // (not __syncthreads(): the weights may still be on their way)

    const bool t_ok = row < LS_TOKENS && m0 + row < M;
    const uint8_t* xrow = xq + (t_ok ? row : 0) * XQ_STRIDE + sub * 16;
    v4i acc = {0, 0, 0, 0}, acc2 = {0, 0, 0, 0};      // two chains: low and high nibbles
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        v4i xv = {0, 0, 0, 0};
        if (t_ok) xv = *reinterpret_cast<const v4i*>(xrow + i * 64);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[i] & 0x0F0F0F0F, xv & 0x0F0F0F0F, acc, 0, 0, 0);
        acc2 = __builtin_amdgcn_mfma_i32_16x16x64_i8((w[i] >> 4) & 0x0F0F0F0F, (xv >> 4) & 0x0F0F0F0F, acc2, 0, 0, 0);
    }
    acc += acc2;
    // accumulator register r of lane l: channel 4*(l/16) + r, token l%16
    const basq_tokmeta mt = lmeta[t_ok ? row : 0];
    uint16_t y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int from = 4 * (4 * sub + r);
        const float sw = __int_as_float(__builtin_amdgcn_ds_bpermute(from, cst2) << 16);
        const float zp = __int_as_float(__builtin_amdgcn_ds_bpermute(from + 64, cst2) << 16);
        const float ws = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(cst4)));
        const float cb = g.out_bias ? __int_as_float(__builtin_amdgcn_ds_bpermute(from + 64, __float_as_int(cst4))) : 0.0f;
        const float t = (float)acc[r] - zp * (float)mt.rowsum;
        y[r] = f32_to_bf16(fmaf(mt.scale * sw, t, fmaf(mt.lo, ws, cb)));
    }
    if (!t_ok) return;
    const int n = n0 + 4 * sub;
    uint16_t* out = g.Y + (int64_t)(m0 + row) * g.ldy + n;
    if (n + 4 <= g.N && (reinterpret_cast<uintptr_t>(out) & 7) == 0) {
        *reinterpret_cast<uint2*>(out) = make_uint2(y[0] | (uint32_t)y[1] << 16, y[2] | (uint32_t)y[3] << 16);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (n + r < g.N) out[r] = y[r];
    }
}

template <int NP>
int launch_ls(const RotateQuantArgs& q, const GemmArgs& g, hipStream_t s) {
    const bool hb = q.bias != nullptr, hs = q.act_scale != nullptr;
    const float norm = (float)(1.0 / sqrt((double)q.K));
    const dim3 grid((unsigned)((g.N + LS_ROWS - 1) / LS_ROWS), (unsigned)((g.M + LS_TOKENS - 1) / LS_TOKENS)), block(LS_WAVES * 64);
#define LS_LAUNCH(HB, HS) hipLaunchKernelGGL((linear_small_kernel<NP, HB, HS>), grid, block, 0, s, q, g, norm)
    if (hb && hs) LS_LAUNCH(true, true);
    else if (hb) LS_LAUNCH(true, false);
    else if (hs) LS_LAUNCH(false, true);
    else LS_LAUNCH(false, false);
#undef LS_LAUNCH
    return check_hip(hipGetLastError(), "linear_small launch");
}

}  // namespace

// As many workgroups as rotate no longer than the launch and the wait between two kernels take: 512 with one or two pieces a token,
// 256 with four (a workgroup's rotation is twice as long, and half as many are in flight).  Whole layers from a graph, cold weights,
// us, two launches and one: K = 1024, 64 x 1024 (256 workgroups) 7.2 and 4.3, 1 x 28672 (448) 9.2 and 6.3, 16 x 8192 (512) 6.8 and 6.0,
// 32 x 4096 with both vectors (512) 7.0 and 6.1, 64 x 4096 (1024) 7.7 and 8.2, 64 x 8192 8.3 and 13.1; K = 512, 128 x 1024 (512) 7.5 and
// 4.4, 64 x 8192 (2048) 7.3 and 9.0; K = 2048, 1 x 2048 with both vectors (32) 6.4 and 6.4, 16 x 2048 (128) 7.1 and 6.0, 64 x 1024
// (256) 9.1 and 6.0.  The lines were drawn when the constants' loads still waited for the weights; a little beyond them one
// launch would be the faster one now (8 x 1024 x 28672, 896, 9.8 and 8.8; 128 x 512 x 2048, 1024, 7.7 and 5.9; 64 x 2048 x 2048,
// 512, 9.5 and 8.5, with both vectors 9.8 and 9.2).
bool linear_small_applicable(const RotateQuantArgs& q, const GemmArgs& g) {
    if (q.has28 || q.rot_size != q.K || q.group != q.K || !(q.K == 512 || q.K == 1024 || q.K == 2048) || q.rot_out != nullptr ||
        g.acc_out != nullptr || g.w_layout != BASQ_W_DECODE16 || g.M < 1 || g.M > 128)
        return false;
    const int64_t groups = (g.M + LS_TOKENS - 1) / LS_TOKENS * (((int64_t)g.N + LS_ROWS - 1) / LS_ROWS);
    return groups <= (q.K == 2048 ? 256 : 512);
}

int launch_linear_small(const RotateQuantArgs& q, const GemmArgs& g, hipStream_t s) {
    if (q.K == 512) return launch_ls<1>(q, g, s);
    if (q.K == 1024) return launch_ls<2>(q, g, s);
    return launch_ls<4>(q, g, s);
}

}  // namespace basq
