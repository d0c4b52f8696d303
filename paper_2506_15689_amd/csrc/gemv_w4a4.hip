// Weight-streaming W4A4 product for few tokens (M <= 128: decode, batched decode, speculative decoding): one
// pass over the packed 4-bit weights, bound by HBM bandwidth up to about 64 tokens.  Same arithmetic as the
// prefill GEMM (ACC in INT32, fused de-quantisation).
//
// A workgroup owns one to four tiles of 16 output channels; its waves split K.  Each lane issues a batch of 16-byte weight
// loads before it consumes any, so the whole weight matrix is in flight at once.  The 16 x 16 x 64 int8 MFMA
// takes 16 weight rows as one operand and 16 (zero padded) tokens as the other; more tokens are more token
// tiles against the same weight registers.  Nibbles are split into low/high words exactly as in the prefill
// kernel.
//
// Weight layouts.  The MFMA operand puts 16 different rows on the 16 lanes of a quarter wave, so on
// canonical [N, K/2] weights every load instruction touches 16 rows x 64 bytes and each 128-byte line
// is fetched in eight 16-byte pieces.  The streaming layout (BASQ_W_DECODE16) stores the 1 KB a wave
// load needs contiguously, in lane order: 4 KB contiguous per workgroup step.
#include "basq_internal.h"

#include <type_traits>

namespace basq {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int GV_ROWS = 16;                         // output channels per tile

typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));

// The end of the kernel, a workgroup's sums to outputs, in two forms.  request() fetches the epilogue's constants and token
// records in front of the weight stream, so that their latency overlaps it: without a branch (clamped indices) and as raw bits
// -- a conversion there would wait for them before the first weight load is issued, and a record fetched in the epilogue is a
// memory latency at the very end.  finish() takes the waves' accumulators: register r of lane l is weight row 4*(l/16) + r,
// token l%16 of its tile.
//
// Up to 16 tokens, one or two tiles: the sums meet by LDS atomics (integer adds: any order gives the same bits) and a thread
// finishes one output of each tile.  (As below, one wave would finish them all: 4 x 8192 x 28672 24.9 -> 25.9 us.)
template <int WAVES, int TILES>
struct GvFewTiles {
    static constexpr int NT = TILES, LDS_INTS = NT * 256;
    int orow, otok, M;
    uint16_t sw_bits[TILES], zp_bits[TILES];
    float ws[TILES], cb[TILES];
    basq_tokmeta mt;
    __device__ __forceinline__ void request(const GemmArgs& a, int n0, int tid, int* part) {
        static_assert(WAVES * 64 == 256, "a thread per output of a tile");
#pragma unroll
        for (int i = 0; i < NT; ++i) part[i * 256 + tid] = 0;
        orow = tid & 15; otok = tid >> 4; M = (int)a.M;
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int on = n0 + GV_ROWS * t + orow;
            const int on_c = on < a.N ? on : a.N - 1;
            sw_bits[t] = a.w_scale[on_c];
            zp_bits[t] = a.w_zero[on_c];
            ws[t] = a.w_sum[on_c];
            cb[t] = 0.0f;
            if (a.out_bias) cb[t] = a.out_bias[on_c];
        }
        mt = a.meta[otok < M ? otok : M - 1];
    }
    __device__ __forceinline__ void finish(const GemmArgs& a, int n0, int lane, const v4i (&acc)[NT], int* part) const {
        __syncthreads();                                // every wave has zeroed its share of `part`
#pragma unroll
        for (int at = 0; at < NT; ++at)
#pragma unroll
            for (int r = 0; r < 4; ++r) atomicAdd(&part[at * 256 + (4 * (lane >> 4) + r) * 16 + (lane & 15)], acc[at][r]);
        __syncthreads();
        if (otok >= M) return;
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int on = n0 + GV_ROWS * t + orow;
            if (on >= a.N) continue;
            const int av = part[t * 256 + orow * 16 + otok];
            const float sw = bf16_to_f32(sw_bits[t]), zp = bf16_to_f32(zp_bits[t]);
            const float tv = (float)av - zp * (float)mt.rowsum;
            const float y = fmaf(mt.scale * sw, tv, fmaf(mt.lo, ws[t], cb[t]));
            a.Y[(int64_t)otok * a.ldy + on] = f32_to_bf16(y);
            if (a.acc_out) a.acc_out[(int64_t)otok * a.N + on] = av;
        }
    }
};

// More tokens: every wave puts its sums down and finishes whole tiles, a lane four adjacent channels of one token: 8-byte stores
// and vector loads of the constants.  (A thread per output, with atomics, 2-byte stores and a rounding in software, spent 1300
// cycles here on four tiles and 2700 on eight, 540 and 1300 as built: 17 x 4096 x 4096 5.2 -> 4.8 us, 64 x 8192 x 8192 15.2 -> 14.3,
// 128 x 8192 x 28672 63.3 -> 59.3.)  A wave keeps to the token tiles wave % TT (and, TT > WAVES, every WAVES-th from there), over all weight
// tiles or a share of them, so that it requests a record per token tile and the constants per weight tile.  With both per output
// tile, up to 40 loads a lane in front of the weights, calls that fill few of their token tiles were slower than with a thread
// per output (65 x 1024 x 28672 19.0 us, per output 18.0, as built 17.3); with the constants channel by channel in a workgroup that
// has channels past the last, that workgroup alone took 2 us longer (65 x 1024 x 8208 8.9, 7.1, as built 6.9).
template <int WAVES, int TILES, int TT>
struct GvManyTiles {
    static constexpr int NT = TILES * TT, LDS_INTS = WAVES * NT * 256;
    static constexpr int OWN_TT = TT > WAVES ? TT / WAVES : 1;             // token tiles of a wave, WAVES apart
    static constexpr int T_STEP = TT < WAVES ? WAVES / TT : 1;             // its weight tiles are T_STEP apart
    static constexpr int OWN_T = (TILES + T_STEP - 1) / T_STEP;
    static_assert(TT > WAVES ? TT % WAVES == 0 : WAVES % TT == 0, "every wave has as many token tiles");
    int wave, tt0, t0, M;
    bool whole;                                         // every channel of the workgroup exists
    uint2 sw_bits[OWN_T], zp_bits[OWN_T];
    float4 ws[OWN_T], cb[OWN_T];
    basq_tokmeta mts[OWN_TT];
    __device__ __forceinline__ void request(const GemmArgs& a, int n0, int tid, int*) {
        const int lane = tid & 63, row = lane & 15, sub = lane >> 4;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6); M = (int)a.M;
        tt0 = wave % TT; t0 = wave / TT;
        whole = n0 + GV_ROWS * TILES <= a.N;
#pragma unroll
        for (int k = 0; k < OWN_T; ++k) {
            const int t = t0 + k * T_STEP < TILES ? t0 + k * T_STEP : TILES - 1;   // (a wave without a k-th tile: in bounds)
            const int on = n0 + GV_ROWS * t + 4 * sub;
            cb[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (a.N >= 4) {
                const int at4 = on < a.N - 4 ? on : a.N - 4;       // past the last four channels: those, put in their places by finish()
                __builtin_memcpy(&sw_bits[k], a.w_scale + at4, 8);
                __builtin_memcpy(&zp_bits[k], a.w_zero + at4, 8);
                __builtin_memcpy(&ws[k], a.w_sum + at4, 16);
                if (a.out_bias) __builtin_memcpy(&cb[k], a.out_bias + at4, 16);
            } else {
                int c[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) c[r] = on + r < a.N ? on + r : a.N - 1;
                sw_bits[k] = make_uint2(a.w_scale[c[0]] | (uint32_t)a.w_scale[c[1]] << 16, a.w_scale[c[2]] | (uint32_t)a.w_scale[c[3]] << 16);
                zp_bits[k] = make_uint2(a.w_zero[c[0]] | (uint32_t)a.w_zero[c[1]] << 16, a.w_zero[c[2]] | (uint32_t)a.w_zero[c[3]] << 16);
                ws[k] = make_float4(a.w_sum[c[0]], a.w_sum[c[1]], a.w_sum[c[2]], a.w_sum[c[3]]);
                if (a.out_bias) cb[k] = make_float4(a.out_bias[c[0]], a.out_bias[c[1]], a.out_bias[c[2]], a.out_bias[c[3]]);
            }
        }
#pragma unroll
        for (int s = 0; s < OWN_TT; ++s) {
            const int tok = 16 * (tt0 + s * WAVES) + row;
            mts[s] = a.meta[tok < M ? tok : M - 1];
        }
    }
    __device__ __forceinline__ void finish(const GemmArgs& a, int n0, int lane, const v4i (&acc)[NT], int* lds) const {
        v4i* part = reinterpret_cast<v4i*>(lds);            // [wave][tile][lane]
        const int row = lane & 15, sub = lane >> 4;
#pragma unroll
        for (int at = 0; at < NT; ++at) part[(wave * NT + at) * 64 + lane] = acc[at];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < OWN_T; ++k) {
            const int t = t0 + k * T_STEP, on = n0 + GV_ROWS * t + 4 * sub;
            if (t >= TILES) break;
            uint2 sw2 = sw_bits[k], zp2 = zp_bits[k];
            float4 ws4 = ws[k], cb4 = cb[k];
            const int shift = on - (a.N - 4);                      // 1 .. 3: that many of the lane's channels lie past the last
            if (!whole && a.N >= 4 && shift > 0) {
                auto down16 = [&](uint2 v) {
                    const uint64_t w = ((uint64_t)v.y << 32 | v.x) >> (16 * (shift & 3));
                    return make_uint2((uint32_t)w, (uint32_t)(w >> 32));
                };
                auto down32 = [&](float4 v) {
                    return make_float4(shift == 1 ? v.y : shift == 2 ? v.z : v.w, shift == 1 ? v.z : v.w, v.w, v.w);
                };
                sw2 = down16(sw2); zp2 = down16(zp2);
                ws4 = down32(ws4); cb4 = down32(cb4);
            }
#pragma unroll
            for (int s = 0; s < OWN_TT; ++s) {
                const int tt = tt0 + s * WAVES, at = t * TT + tt, tok = 16 * tt + row;
                if (16 * tt >= M) continue;                        // no token there
                v4i av = part[at * 64 + lane];
#pragma unroll
                for (int w = 1; w < WAVES; ++w) av += part[(w * NT + at) * 64 + lane];
                if (tok >= M) continue;
                const basq_tokmeta mt = mts[s];
                const float rowsum = (float)mt.rowsum;
                auto dequant = [&](int acc, float sw, float zp, float wsum, float c) {
                    return fmaf(mt.scale * sw, (float)acc - zp * rowsum, fmaf(mt.lo, wsum, c));
                };
                auto lo16 = [](uint32_t v) { return __uint_as_float(v << 16); };
                auto hi16 = [](uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); };
                const f2 y01 = {dequant(av[0], lo16(sw2.x), lo16(zp2.x), ws4.x, cb4.x), dequant(av[1], hi16(sw2.x), hi16(zp2.x), ws4.y, cb4.y)};
                const f2 y23 = {dequant(av[2], lo16(sw2.y), lo16(zp2.y), ws4.z, cb4.z), dequant(av[3], hi16(sw2.y), hi16(zp2.y), ws4.w, cb4.w)};
                const uint2 out = make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(y01, b2)),       // round-to-nearest-even
                                             __builtin_bit_cast(uint32_t, __builtin_convertvector(y23, b2)));
                uint16_t* dst = a.Y + (int64_t)tok * a.ldy + on;
                if (whole || on + 4 <= a.N) {
                    __builtin_memcpy(dst, &out, 8);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (on + r < a.N) dst[r] = (uint16_t)((r < 2 ? out.x : out.y) >> (16 * (r & 1)));
                }
                if (a.acc_out) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (on + r < a.N) a.acc_out[(int64_t)tok * a.N + on + r] = av[r];
                }
            }
        }
    }
};

// STEPS: 64-byte k-chunks per lane held in registers at once (all of their loads are in flight together).
// TILES: 16-row weight tiles per workgroup; they share the activation operand, which at 16 tokens is as many
//        L2 bytes per workgroup as one tile's weights.
// TT:    16-token tiles (M <= 16 * TT); they share the weight registers.
// WAVES: wavefronts per workgroup, which split K.
template <bool STREAM_LAYOUT, int WAVES, int STEPS, int TILES, int TT>
__global__ __launch_bounds__(WAVES * 64) void gemv_w4a4_kernel(GemmArgs a) {
    constexpr int NT = TILES * TT;                  // accumulator tiles per wave
    constexpr bool TWO_CHAINS = NT <= 2;            // few tiles: low and high nibbles on separate MFMA chains
    typedef std::conditional_t<TT == 1, GvFewTiles<WAVES, TILES>, GvManyTiles<WAVES, TILES, TT>> End;
    __shared__ __attribute__((aligned(16))) int part[End::LDS_INTS];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * (GV_ROWS * TILES);
    const int KB = a.K / 2;
    const int nchunks = KB / 64;               // 64-byte chunks per row (K % 128 == 0 checked by the caller)
    const int row = lane & 15, sub = lane >> 4;
    const int M = (int)a.M;

    // chunk c of this lane: canonical = 16 bytes of row n at 64c + 16sub; streaming = piece `lane` of the
    // 16-row block's c-th KB (rows past N are stored as zeros there; a whole block past N does not exist)
    const uint8_t* wrow[TILES];
    bool w_ok[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int nt0 = n0 + GV_ROWS * t, n = nt0 + row;
        w_ok[t] = STREAM_LAYOUT ? nt0 < a.N : n < a.N;
        wrow[t] = STREAM_LAYOUT ? a.Wq + (int64_t)(w_ok[t] ? nt0 : 0) * KB + lane * 16
                                : a.Wq + (int64_t)(w_ok[t] ? n : 0) * KB + sub * 16;
    }
    constexpr int WSTEP = STREAM_LAYOUT ? 1024 : 64;
    // the same lane index selects the token of tile tt on the other operand
    const uint8_t* arow[TT];
    bool t_ok[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        t_ok[tt] = 16 * tt + row < M;
        arow[tt] = a.Aq + (int64_t)(t_ok[tt] ? 16 * tt + row : 0) * KB + sub * 16;
    }

    End end;
    end.request(a, n0, tid, part);

    v4i acc[NT], acc2[TWO_CHAINS ? NT : 1];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < (TWO_CHAINS ? NT : 1); ++i) acc2[i] = v4i{0, 0, 0, 0};
    for (int c0 = wave; c0 < nchunks; c0 += WAVES * STEPS) {
        v4i w[TILES][STEPS], x[TT][STEPS];
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            const int c = c0 + i * WAVES;
            const bool ok = c < nchunks;
            // the weights are read once per call: streaming (non-temporal) loads
#pragma unroll
            for (int t = 0; t < TILES; ++t)
                w[t][i] = (ok && w_ok[t]) ? __builtin_nontemporal_load(reinterpret_cast<const v4i*>(wrow[t] + c * WSTEP))
                                          : v4i{0, 0, 0, 0};
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                x[tt][i] = (ok && t_ok[tt]) ? *reinterpret_cast<const v4i*>(arow[tt] + c * 64) : v4i{0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
            v4i wlo[TILES], whi[TILES];
#pragma unroll
            for (int t = 0; t < TILES; ++t) { wlo[t] = w[t][i] & 0x0F0F0F0F; whi[t] = (w[t][i] >> 4) & 0x0F0F0F0F; }
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const v4i xlo = x[tt][i] & 0x0F0F0F0F, xhi = (x[tt][i] >> 4) & 0x0F0F0F0F;
#pragma unroll
                for (int t = 0; t < TILES; ++t) {
                    const int at = t * TT + tt;
                    acc[at] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wlo[t], xlo, acc[at], 0, 0, 0);
                    if (TWO_CHAINS) acc2[at] = __builtin_amdgcn_mfma_i32_16x16x64_i8(whi[t], xhi, acc2[at], 0, 0, 0);
                    else acc[at] = __builtin_amdgcn_mfma_i32_16x16x64_i8(whi[t], xhi, acc[at], 0, 0, 0);
                }
            }
        }
    }
    if (TWO_CHAINS) {
#pragma unroll
        for (int at = 0; at < NT; ++at) acc[at] += acc2[at];
    }
    end.finish(a, n0, lane, acc, part);
}

// canonical [N, K/2] -> streaming layout: one thread per 16-byte piece of the output
__global__ __launch_bounds__(256) void pack_decode16_kernel(const uint8_t* __restrict__ Wq, int N, int KB,
                                                            uint8_t* __restrict__ out, int64_t pieces) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= pieces) return;
    const int nchunks = KB / 64;
    const int ln = (int)(p & 63);
    const int64_t kb = p >> 6;                       // (block, chunk)
    const int c = (int)(kb % nchunks);
    const int64_t n = (kb / nchunks) * 16 + (ln & 15);
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < N) v = *reinterpret_cast<const uint4*>(Wq + n * KB + 64 * c + 16 * (ln >> 4));
    *reinterpret_cast<uint4*>(out + p * 16) = v;
}

}  // namespace

int launch_pack_decode16(const uint8_t* Wq, int32_t N, int32_t K, uint8_t* out, hipStream_t s) {
    const int KB = K / 2;
    const int64_t pieces = (int64_t)((N + 15) / 16) * (KB / 64) * 64;
    const int64_t blocks = (pieces + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return fail(BASQ_EINVAL, "pack_decode: matrix too large");
    hipLaunchKernelGGL(pack_decode16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, Wq, N, KB, out, pieces);
    return check_hip(hipGetLastError(), "pack_decode launch");
}

template <bool SL, int WAVES, int STEPS, int TILES, int TT>
static void launch_gemv_cfg(const GemmArgs& a, hipStream_t s, int blocks16) {
    hipLaunchKernelGGL((gemv_w4a4_kernel<SL, WAVES, STEPS, TILES, TT>), dim3((unsigned)((blocks16 + TILES - 1) / TILES)),
                       dim3(WAVES * 64), 0, s, a);
}

template <bool SL, int STEPS, int TT>
static void launch_gemv_tiles(const GemmArgs& a, hipStream_t s, int blocks16) {
    // More weight tiles per workgroup = fewer passes over the activations, which is what bounds the kernel from
    // 32 tokens on -- as long as the workgroups still fill the chip (measured on N = 4096, 12288, 28672).  Up to 512 tiles
    // there is one workgroup per compute unit or less, and its time is the chain of a wave's batches of loads: eight
    // waves, and a tile each as long as every compute unit gets one at most (17 tokens, K = 14336, N = 4096: 18.9 us with four
    // waves on two tiles, 16.8 with four on one, 10.6 with eight on one; N = 8192, K = 4096: 7.7 -> 6.7; eight on one for
    // N = 6144: 12.5 against 10.8 at 64 tokens; eight on two for N = 12288: 9.0 against 8.3).  Rows that four waves hold in
    // one batch have no chain to shorten (17 tokens, K = 1024, N = 8192: 4.4 us with eight waves, 4.0 with four; N = 1024 3.5
    // with either; 65 tokens, K = 512, N = 8192: 6.1 against 5.6).
    const bool one_batch = a.K / 128 <= 4 * STEPS;
    // 33 .. 64 tokens over 512 .. 1024 tiles: eight waves on the three or four tiles that give every compute unit one workgroup,
    // which has twice the loads in flight of four waves on two (cold weights: 64 x 4096 x 12288 14.1 -> 10.7 us, x 16384 14.5 -> 11.7,
    // 64 x 8192 x 12288 24.3 -> 17.8; 64 x 4096 x 20000, beyond, 19.2 and 18.3; up to 32 tokens even; rows of one batch 5.7 and 6.4).
    if constexpr (TT == 4) {
        if (blocks16 > 512 && blocks16 <= 768 && !one_batch) { launch_gemv_cfg<SL, 8, 4, 3, TT>(a, s, blocks16); return; }
        if (blocks16 > 768 && blocks16 <= 1024 && !one_batch) { launch_gemv_cfg<SL, 8, 2, 4, TT>(a, s, blocks16); return; }
    }
    if (blocks16 >= 1536) launch_gemv_cfg<SL, 4, STEPS, 4, TT>(a, s, blocks16);
    else if (blocks16 > 512 || (one_batch && blocks16 > 256)) launch_gemv_cfg<SL, 4, STEPS, 2, TT>(a, s, blocks16);
    else if (one_batch) launch_gemv_cfg<SL, 4, STEPS, 1, TT>(a, s, blocks16);
    else if (blocks16 > 256) launch_gemv_cfg<SL, 8, STEPS, 2, TT>(a, s, blocks16);
    else launch_gemv_cfg<SL, 8, STEPS, 1, TT>(a, s, blocks16);
}

template <bool SL>
static void launch_gemv_layout(const GemmArgs& a, hipStream_t s) {
    const int blocks16 = (a.N + GV_ROWS - 1) / GV_ROWS;
    if (a.M <= 16) {
        // long rows: twice the loads in flight per lane (measured: K = 8192 gains 6 %, K = 4096 loses 5 %)
        const bool deep = a.K / 128 > 32;
        // two tiles per workgroup once the activations weigh in (more than 8 tokens) and the chip stays filled
        if (a.M > 8 && blocks16 >= 4 * 256) launch_gemv_cfg<SL, 4, 8, 2, 1>(a, s, blocks16);
        // 65 .. 112 chunks per row (K = 14336): all of a lane's loads in one batch instead of one and a ragged one
        // (measured 8.0 us against 8.8 us on N = 4096)
        else if (a.K / 128 > 64 && a.K / 128 <= 112) launch_gemv_cfg<SL, 4, 28, 1, 1>(a, s, blocks16);
        else if (deep) launch_gemv_cfg<SL, 4, 16, 1, 1>(a, s, blocks16);
        else launch_gemv_cfg<SL, 4, 8, 1, 1>(a, s, blocks16);
    } else if (a.M <= 32) {
        launch_gemv_tiles<SL, 2, 2>(a, s, blocks16);
    } else if (a.M <= 64) {
        launch_gemv_tiles<SL, 2, 4>(a, s, blocks16);
    } else {
        launch_gemv_tiles<SL, 1, 8>(a, s, blocks16);
    }
}

int launch_gemv_decode(const GemmArgs& a, hipStream_t s) {
    if (a.M == 0) return BASQ_OK;
    if (a.M > GEMV_MAX_TOKENS) return fail(BASQ_EINVAL, "weight-streaming kernel: more than %d tokens", GEMV_MAX_TOKENS);
    if (a.w_layout == BASQ_W_DECODE16) launch_gemv_layout<true>(a, s);
    else launch_gemv_layout<false>(a, s);
    return check_hip(hipGetLastError(), "w4a4_gemv launch");
}

}  // namespace basq
