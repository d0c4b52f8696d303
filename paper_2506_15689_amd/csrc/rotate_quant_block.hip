// Fast rotate + bias + quantise kernels for BLOCKWISE rotations: rot_size n in {128, 256, 512} applied to every
// block of n channels of a longer token (K a multiple of n and of 256, K <= 16384), per-token ranges.  This is the
// shape of a layer whose width has no Hadamard matrix of its own size in this library -- e.g. the 11008 = 43 * 256
// wide MLP of the 7B LLaMA-2 that the paper's Sec. 5.2 times -- rotated in blocks instead (paper Sec. 3.1 rotation,
// Eq. 14 bias, Eq. 15 scale, Eq. 4 quantiser with the per-token range of Sec. 5).
//
// One workgroup of four wavefronts per token; a wave takes the 512-channel pieces w, w+4, ... of the token and
// keeps them in registers (8 values per lane per piece) across the two passes that a per-token range needs.
// No LDS except for the workgroup's range and row sum.
//
// Inside a piece, channel e (9 bits):
//   load      lane l reads 8 consecutive bf16 (16 B) at chunk(l): e = 8*chunk + t, chunk bits (e3..e8) <- lane bits
//             (2,3,0,1,4,5), as in the K = 4096/8192 kernel (P2Lane).
//   MFMA      the stages over (e0,e1,e2,e7,e8) -- only (e0,e1,e2,e7) for n = 256, (e0,e1,e2) for n = 128 -- as one
//             16x16x32 bf16 MFMA pair against a +-1 (n = 256: +-2^-4, the exact normalisation) block-diagonal
//             operand: exact.  Afterwards e0 = h, (e5,e6) = r, lane bits (0..5) = (e1,e2,e7,e8,e3,e4).
//   stages    e5, e6 on the accumulator registers; e3, e4 across lane bits 4 and 5 by swapping register halves
//             (v_permlane16_swap / v_permlane32_swap) so that both operands of a butterfly sit in one lane.
//             Afterwards: e0 = h, (e3,e4) = r, lane bits (0..5) = (e1,e2,e7,e8,e5,e6).
//   codes     a lane's four bytes (two codes each) are 4 bytes apart and the four lanes of a quad fill the gaps:
//             a 4 x 4 byte transpose inside the quad (DPP + v_perm) gives every lane one aligned dword of the
//             16-byte segment, and a store instruction writes 256 contiguous bytes of the row.
//   fp6 form  made from those dwords inside the quad, about 30 vector instructions a piece on top of 100.  A repacking
//             launch behind the kernel cost 4-6 us up to 2048 tokens and a pass over the codes beyond (the layer with 64
//             output channels, K = 11008 in blocks of 256: 1021 tokens 87 -> 33 us with the product's share, 16384 tokens
//             249 -> 187 us).  Calls that want both forms of many tokens still repack (rotate_quant.hip).
//
// Whole tokens of 512, 1024 or 2048 channels (rotate_quant_small_kernel) are one to four such pieces of ONE wave.  They
// took the generic kernel of one workgroup per token in LDS: K = 1024, 64 tokens 5.3 -> 3.1 us, 4096 tokens 23.0 -> 5.3 us,
// 65536 tokens 311 -> 42.8 us (3.9 TB/s; the rest is vector instructions, 16 values a lane).
#include "rotate_block_piece.h"

namespace basq {

namespace {

constexpr int RB_WAVES = 4;
constexpr int RB_THREADS = RB_WAVES * 64;
constexpr int RB_PMAX = 8;                          // pieces per wave: K <= 4 * 8 * 512

// The channel from which a lane requests its values of b^c and s^a for piece p of its wave, two at +8*r, r = 0..3.  Past the
// token (the missing half of a last piece, pieces that do not exist) the values are not used: channels of the first 256, which
// the smallest token has too.
__host__ __device__ __forceinline__ int rb_vector_at(int K, int wave, int p, int eout) {
    const int e0 = 512 * (wave + RB_WAVES * p) + eout;
    return e0 < K ? e0 : eout & 255;
}
// The same codes in the fp6 operand form (fp6_pack.hip): the four lanes of a quad hold a group of 32 codes, whose
// 24-byte string of 6-bit fields is 48 bits from each lane.  Lane q4 of the quad stores dword q4 of the first 16 bytes,
// lanes 0 and 1 one dword of the last 8 each.  `group16` and `group8`: where the group's two parts go.
__device__ __forceinline__ void rb_store_fp6(uint32_t word, int q4, uint8_t* group16, uint8_t* group8) {
    uint32_t f[4];                                                       // two 6-bit fields each
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = ((word >> (8 * i)) & 15u) | (((word >> (8 * i + 4)) & 15u) << 6);
    const uint32_t lo = f[0] | (f[1] << 12) | (f[2] << 24);             // bits 0..31 of the lane's 48
    const uint32_t hi = (f[2] >> 8) | (f[3] << 4);                      // bits 32..47
    // dwords 0..3: L0.lo; L0.hi, L1.lo (low half); L1.lo (high half), L1.hi; L2.lo
    const uint32_t plo = rb_dpp_u<0x90>(lo), phi = rb_dpp_u<0x90>(hi);   // from lanes 0, 0, 1, 2 of the quad
    const uint32_t sel = q4 == 1 ? 0x05040100u : q4 == 2 ? 0x05040302u : 0x03020100u;
    *reinterpret_cast<uint32_t*>(group16 + 4 * q4) = __builtin_amdgcn_perm(q4 == 1 ? lo : phi, q4 == 1 ? phi : plo, sel);
    // dwords 4, 5: L2.hi, L3.lo (low half); L3.lo (high half), L3.hi
    const uint32_t lo3 = rb_dpp_u<0xFF>(lo), hi3 = rb_dpp_u<0xFF>(hi), hi2 = rb_dpp_u<0xAA>(hi);
    const uint32_t tail = q4 == 0 ? __builtin_amdgcn_perm(lo3, hi2, 0x05040100u) : __builtin_amdgcn_perm(hi3, lo3, 0x05040302u);
    if (q4 < 2) *reinterpret_cast<uint32_t*>(group8 + 4 * q4) = tail;
}

// Workgroup number of this block, renumbered so that runs of RUN consecutive workgroups of `total` go to one XCD (blocks
// congruent mod 8 do): the 8-byte tails that 32 neighbouring tokens write next to each other then meet in one L2.
template <int RUN>
__device__ __forceinline__ unsigned rb_renumber(unsigned bid, unsigned total) {
    const unsigned full = total / (8 * RUN) * (8 * RUN);
    const unsigned base = bid < full ? 0 : full, run = bid < full ? RUN : (total - full) / 8;
    const unsigned b = bid - base, xcd = b % 8, i = b / 8;
    if (bid >= full && i >= run) return bid;                            // the last total % 8
    return base + (i / (run ? run : 1) * 8 + xcd) * run + i % (run ? run : 1);
}

// Where the groups of one token that this lane's quad holds go in the fp6 form.
struct RbFp6 {
    uint8_t *group16, *group8;      // of piece 0
    int64_t piece_bytes;            // four chunks of 128 codes
    __device__ __forceinline__ RbFp6(const RotateQuantArgs& a, int64_t m, int seg) {
        const int64_t rb6 = (a.M + 31) >> 5;
        const int r = (int)(m & 31), f = seg & 3;
        uint8_t* block = a.Aq6 + ((int64_t)(seg >> 2) * rb6 + (m >> 5)) * 3072;
        group16 = block + 64 * r + 16 * (f ^ ((r >> 2) & 3));
        group8 = block + 2048 + 256 * f + 8 * r;
        piece_bytes = 4 * rb6 * 3072;
    }
    __device__ __forceinline__ void store(uint32_t word, int q4, int piece) const {
        rb_store_fp6(word, q4, group16 + piece * piece_bytes, group8 + piece * piece_bytes);
    }
};

// PMAX: pieces that a wave has at most.
// (Two waves a SIMD: allowed more than 256 registers, the compiler gives the MFMAs' results to accumulation registers, and a move each
// brings them back.  With that, DPP moves without an old value, and a quad's bytes transposed in two steps: K = 11008, 1021 tokens
// 13.54 -> 13.13 us, 64 5.43 -> 5.13; rotate_quant_small_kernel, K = 1024, 4096 tokens 5.11 -> 4.82.  Not where the rotation is
// written out: the registers saved let one more wave in, and the memory is slower with that many rows of fp32 under way: without b^c
// and s^a, K = 11008, 1777 tokens 38.5 us with two and 31.9 as built, K = 8192 in blocks of 128, 9000 tokens 110.5 and 99.4.)
template <int LOG2N, bool FP6, int PMAX, bool HAS_BIAS, bool HAS_SCALE, bool ROT_OUT>
__global__ __launch_bounds__(RB_THREADS, ROT_OUT ? 1 : 2) void rotate_quant_block_kernel(RotateQuantArgs a, float norm) {
    constexpr bool FOLD_NORM = LOG2N == 8;           // 1/sqrt(256) = 2^-4 sits in the MFMA operand
    __shared__ float red_mn[RB_WAVES], red_mx[RB_WAVES];
    __shared__ int red_sum[RB_WAVES];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t m = FP6 ? rb_renumber<32>(blockIdx.x, gridDim.x) : blockIdx.x;   // (its divisions are 0.3 us in front of the first load)
    const int K = a.K;
    const int np = (K + 511) >> 9;                    // pieces of the token (the last one may be half: K % 512 = 256)
    const P2Lane pl = p2_lane(lane);
    v8bf bop[2];
    rb_make_bop<LOG2N, FOLD_NORM ? 4 : 0>(lane, bop);

    const int eout = rb_eout(lane);

    // ---- all of this wave's pieces are requested at once ------------------------------------------------------
    const uint16_t* x = a.X + m * a.ldx;
    uint4 raw[PMAX];
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        const int ein = 512 * (wave + RB_WAVES * p) + 8 * pl.chunk;
        raw[p] = ein < K ? nt_load16(x + ein) : make_uint4(0, 0, 0, 0);
    }

    // ---- pass 1: rotate, bias, range ---------------------------------------------------------------------------
    // b^c and s^a of a piece are requested a piece ahead, without a branch (past the token: see rb_vector_at):
    // requested where they are used they were a cache latency in front of every piece (K = 11008: 1 token 5.9 -> 4.3 us, 256 8.4 -> 6.7,
    // 2048 25.8 -> 24.2, 4096 49.2 -> 45.6).  The token's loads without their branches, on a descriptor that ends with it: 4.4, 6.9,
    // 24.6, 46.9.
    float2 bb[2][4], ss[2][4];
    auto request_vectors = [&](int p) {
        const int at = rb_vector_at(K, wave, p, eout);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (HAS_BIAS) bb[p & 1][r] = *reinterpret_cast<const float2*>(a.bias + at + 8 * r);
            if (HAS_SCALE) ss[p & 1][r] = *reinterpret_cast<const float2*>(a.act_scale + at + 8 * r);
        }
    };
    if (PMAX > 1 || wave < np) request_vectors(0);
    float v[PMAX][2][4];
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        const int c = wave + RB_WAVES * p;
        if (c < np) {                                  // uniform over the wave
            if (p + 1 < PMAX) request_vectors(p + 1);
            __builtin_amdgcn_sched_barrier(0);
            float d[2][4];
            rb_rotate_piece(raw[p], bop, d);
            const int e0 = 512 * c + eout;
            const bool ok = e0 < K;                    // a half piece: the lanes of its missing 256 channels
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = e0 + 8 * r;              // channels e (h = 0) and e + 1 (h = 1)
                const float2 b2 = HAS_BIAS ? bb[p & 1][r] : make_float2(0.f, 0.f), s2 = HAS_SCALE ? ss[p & 1][r] : make_float2(1.f, 1.f);
                float r0 = d[0][r], r1 = d[1][r];
                if (!FOLD_NORM) { r0 = r0 * norm; r1 = r1 * norm; }
                if (ROT_OUT && ok) *reinterpret_cast<float2*>(a.rot_out + m * (int64_t)K + e) = make_float2(r0, r1);
                const float v0 = HAS_SCALE ? fmaf(r0, s2.x, -b2.x) : r0 - b2.x;
                const float v1 = HAS_SCALE ? fmaf(r1, s2.y, -b2.y) : r1 - b2.y;
                v[p][0][r] = v0;
                v[p][1][r] = v1;
                if (ok) {
                    mn = fminf(mn, fminf(v0, v1));
                    mx = fmaxf(mx, fmaxf(v0, v1));
                }
            }
        }
    }
    mn = wave_min_f(mn);
    mx = wave_max_f(mx);
    if (lane == 0) { red_mn[wave] = mn; red_mx[wave] = mx; }
    __syncthreads();
    mn = fminf(fminf(red_mn[0], red_mn[1]), fminf(red_mn[2], red_mn[3]));
    mx = fmaxf(fmaxf(red_mx[0], red_mx[1]), fmaxf(red_mx[2], red_mx[3]));

    const float lo = a.clip_lo * mn;
    const float hi = a.clip_hi * mx;
    float s = __fdiv_rn(hi - lo, 15.0f);
    if (!(s > 0.0f && s < INFINITY)) s = 1.0f;
    const float inv = __fdiv_rn(1.0f, s);
    const float nlo = -(lo * inv);

    // ---- pass 2: quantise, pack, store -------------------------------------------------------------------------
    int sum = 0;
    const int q4 = lane & 3, seg = rb_segment(lane);
    const bool codes = !FP6 || a.Aq != nullptr;          // the 4-bit form is optional beside the fp6 form
    uint8_t* orow = codes ? a.Aq + m * (int64_t)(K / 2) + 16 * seg + 4 * q4 : nullptr;
    const RbFp6 f6(a, m, seg);
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        const int c = wave + RB_WAVES * p;
        if (c < np) {
            const bool ok = 512 * c + eout < K;
            const uint32_t word = rb_codes(v[p], inv, nlo, lane, ok, sum);
            if (ok) {
                if (codes) *reinterpret_cast<uint32_t*>(orow + 256 * c) = word;
                if (FP6) f6.store(word, q4, c);
            }
        }
    }
    sum = wave_sum_i(sum);
    if (lane == 0) red_sum[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        basq_tokmeta mt;
        mt.scale = s; mt.lo = lo; mt.rowsum = red_sum[0] + red_sum[1] + red_sum[2] + red_sum[3]; mt.reserved = 0;
        a.meta[m] = mt;
    }
}

// rot_size == K = 512 * NP, NP in {1, 2, 4}: the token is one rotation block of up to four pieces, which one wavefront
// holds (8 values per lane per piece).  The stages over e9 (, e10) pair its pieces register by register; nothing crosses
// waves, so there is no LDS and no barrier, and the four waves of a workgroup take four tokens.  b^c and s^a stay in
// registers over a wave's tokens, the next token is requested before the current one is worked on.
// Registers as in the blockwise kernel, but two waves a SIMD do not pay for K = 2048 with both vectors either (4000 tokens 11.5 us, as
// built 9.3; three waves fit both ways), and with one of them and the rotation written out a fourth wave is kept away, as above
// (20000 tokens, fp6 form too, 80.9 and 76.7 us).
template <int NP, bool HAS_BIAS, bool HAS_SCALE, bool ROT_OUT>
__global__ __launch_bounds__(RB_THREADS, ROT_OUT || (NP == 4 && HAS_BIAS && HAS_SCALE) ? 1 : 2) void rotate_quant_small_kernel(RotateQuantArgs a, float norm) {
    constexpr bool FOLD_NORM = NP == 2;                // 1/sqrt(1024) = 2^-5 sits in the MFMA operand
    if (NP == 4 && ROT_OUT && HAS_BIAS != HAS_SCALE) asm volatile("" ::: "v128");
    constexpr int K = 512 * NP;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const P2Lane pl = p2_lane(lane);
    v8bf bop[2];
    rb_make_bop<9, FOLD_NORM ? 5 : 0>(lane, bop);
    const int eout = rb_eout(lane), q4 = lane & 3, seg = rb_segment(lane);
    const int64_t step = (int64_t)gridDim.x * RB_WAVES;
    int64_t m = (int64_t)(a.Aq6 ? rb_renumber<8>(blockIdx.x, gridDim.x) : blockIdx.x) * RB_WAVES + wave;
    if (m >= a.M) return;
    uint4 raw[NP];
#pragma unroll
    for (int c = 0; c < NP; ++c) raw[c] = nt_load16(a.X + m * a.ldx + 512 * c + 8 * pl.chunk);
    float2 bb[NP][4], ss[NP][4];
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (HAS_BIAS) bb[c][r] = *reinterpret_cast<const float2*>(a.bias + 512 * c + eout + 8 * r);
            if (HAS_SCALE) ss[c][r] = *reinterpret_cast<const float2*>(a.act_scale + 512 * c + eout + 8 * r);
        }
    while (true) {
        float v[NP][2][4];
#pragma unroll
        for (int c = 0; c < NP; ++c) rb_rotate_piece(raw[c], bop, v[c]);
        const int64_t next = m + step;
        if (next < a.M) {
#pragma unroll
            for (int c = 0; c < NP; ++c) raw[c] = nt_load16(a.X + next * a.ldx + 512 * c + 8 * pl.chunk);
        }
        rb_pair_pieces<NP>(v);                         // e9, e10
        const RbRange x = rb_token_range<NP, FOLD_NORM, HAS_BIAS, HAS_SCALE, ROT_OUT>(v, bb, ss, norm, a.clip_lo, a.clip_hi,
                                                                                       ROT_OUT ? a.rot_out + m * (int64_t)K + eout : nullptr);
        int sum = 0;
        uint8_t* orow = a.Aq ? a.Aq + m * (int64_t)(K / 2) + 16 * seg + 4 * q4 : nullptr;
        const RbFp6 f6(a, m, seg);
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            const uint32_t word = rb_codes(v[c], x.inv, x.nlo, lane, true, sum);
            if (a.Aq) *reinterpret_cast<uint32_t*>(orow + 256 * c) = word;
            if (a.Aq6) f6.store(word, q4, c);
        }
        sum = wave_sum_i(sum);
        if (lane == 0) {
            basq_tokmeta mt;
            mt.scale = x.s; mt.lo = x.lo; mt.rowsum = sum; mt.reserved = 0;
            a.meta[m] = mt;
        }
        if (next >= a.M) return;
        m = next;
    }
}

template <int LOG2N, bool FP6, int PMAX>
int launch_rb_pieces(const RotateQuantArgs& a, hipStream_t s, float norm) {
    const bool hb = a.bias != nullptr, hs = a.act_scale != nullptr, ro = a.rot_out != nullptr;
    const dim3 grid((unsigned)a.M), block(RB_THREADS);
#define RB_LAUNCH(HB, HS, RO) hipLaunchKernelGGL((rotate_quant_block_kernel<LOG2N, FP6, PMAX, HB, HS, RO>), grid, block, 0, s, a, norm)
    if (hb && hs) { if (ro) RB_LAUNCH(true, true, true); else RB_LAUNCH(true, true, false); }
    else if (hb) { if (ro) RB_LAUNCH(true, false, true); else RB_LAUNCH(true, false, false); }
    else if (hs) { if (ro) RB_LAUNCH(false, true, true); else RB_LAUNCH(false, true, false); }
    else { if (ro) RB_LAUNCH(false, false, true); else RB_LAUNCH(false, false, false); }
#undef RB_LAUNCH
    return check_hip(hipGetLastError(), "rotate_quant (blockwise) launch");
}

// A kernel for each number of pieces a wave has, up to three (K <= 6144): the vectors requested for a piece that does not exist, and
// the registers of eight pieces, cost short tokens 3 - 11 % where the chip is full (both vectors, requested in place, a piece ahead in the
// kernel for eight pieces, as built: K = 512 in blocks of 128, 2048 tokens 5.8, 6.2, 3.8 us, 16384 34.0, 35.7, 18.2; K = 2048, 1021
// tokens 4.8, 5.2, 4.6; K = 4096 6.9, 7.2, 6.6; K = 5632 8.2, 8.8, 8.2).  With four pieces one of its own is the faster one with b^c (K = 8192,
// 4096 tokens 26.0 -> 24.2) and the slower one for both forms of the codes without (26.6 -> 27.6); beyond, one less in eight counts
// little.
template <int LOG2N, bool FP6>
int launch_rb_form(const RotateQuantArgs& a, hipStream_t s, float norm) {
    const int pieces = (a.K + 512 * RB_WAVES - 1) / (512 * RB_WAVES);
    if (pieces == 1) return launch_rb_pieces<LOG2N, FP6, 1>(a, s, norm);
    if (pieces == 2) return launch_rb_pieces<LOG2N, FP6, 2>(a, s, norm);
    if (pieces == 3) return launch_rb_pieces<LOG2N, FP6, 3>(a, s, norm);
    return launch_rb_pieces<LOG2N, FP6, RB_PMAX>(a, s, norm);
}

// A kernel of its own for codes alone: with the fp6 form behind a test of its pointer they took 3-9 % longer (K = 512 in blocks
// of 128: 1 token 2.78 -> 3.00 us, 40000 tokens 77 -> 84; K = 4096 in blocks of 128: 40000 tokens 143 -> 147).
template <int LOG2N>
int launch_rb(const RotateQuantArgs& a, hipStream_t s, float norm) {
    return a.Aq6 ? launch_rb_form<LOG2N, true>(a, s, norm) : launch_rb_form<LOG2N, false>(a, s, norm);
}

template <int NP>
int launch_rs(const RotateQuantArgs& a, hipStream_t s, float norm) {
    const bool hb = a.bias != nullptr, hs = a.act_scale != nullptr, ro = a.rot_out != nullptr;
    // one token per wave up to 8192 tokens, then every wave walks on (eight waves per SIMD at most)
    const int64_t want = (a.M + RB_WAVES - 1) / RB_WAVES;
    const dim3 grid((unsigned)(want < 2048 ? want : 2048)), block(RB_THREADS);
#define RS_LAUNCH(HB, HS, RO) hipLaunchKernelGGL((rotate_quant_small_kernel<NP, HB, HS, RO>), grid, block, 0, s, a, norm)
    if (hb && hs) { if (ro) RS_LAUNCH(true, true, true); else RS_LAUNCH(true, true, false); }
    else if (hb) { if (ro) RS_LAUNCH(true, false, true); else RS_LAUNCH(true, false, false); }
    else if (hs) { if (ro) RS_LAUNCH(false, true, true); else RS_LAUNCH(false, true, false); }
    else { if (ro) RS_LAUNCH(false, false, true); else RS_LAUNCH(false, false, false); }
#undef RS_LAUNCH
    return check_hip(hipGetLastError(), "rotate_quant (small token) launch");
}

}  // namespace

bool rotate_quant_block_applicable(const RotateQuantArgs& a) {
    // per-token ranges; n = 512 needs whole 512-channel pieces, 128 and 256 also take a last piece of 256 channels
    return a.group == a.K && !a.has28 && (a.rot_size == 128 || a.rot_size == 256 || a.rot_size == 512) &&
           a.K % 256 == 0 && a.K % a.rot_size == 0 && a.K <= RB_WAVES * RB_PMAX * 512 &&
           (a.Aq != nullptr || a.Aq6 != nullptr) && a.meta != nullptr && a.M <= 0x7FFFFFFFll;
}

int rotate_quant_block_vector_channels(int32_t K) {
    int end = 0;
    const int np = (K + 511) / 512;
    for (int wave = 0; wave < RB_WAVES; ++wave)
        for (int p = 0; p < RB_PMAX && (p == 0 || wave + RB_WAVES * (p - 1) < np); ++p)    // piece p is requested with piece p - 1
            for (int lane = 0; lane < 64; ++lane) {
                const int last = rb_vector_at(K, wave, p, rb_eout(lane)) + 8 * 3 + 1;
                if (last >= end) end = last + 1;
            }
    return end;
}

bool rotate_quant_small_applicable(const RotateQuantArgs& a) {
    return a.group == a.K && !a.has28 && a.rot_size == a.K && (a.K == 512 || a.K == 1024 || a.K == 2048) &&
           (a.Aq != nullptr || a.Aq6 != nullptr) && a.meta != nullptr;
}

int launch_rotate_quant_small(const RotateQuantArgs& a, hipStream_t s) {
    const float norm = (float)(1.0 / sqrt((double)a.rot_size));
    if (a.K == 512) return launch_rs<1>(a, s, norm);
    if (a.K == 1024) return launch_rs<2>(a, s, norm);
    return launch_rs<4>(a, s, norm);
}

int launch_rotate_quant_block(const RotateQuantArgs& a, hipStream_t s) {
    const float norm = (float)(1.0 / sqrt((double)a.rot_size));
    if (a.rot_size == 128) return launch_rb<7>(a, s, norm);
    if (a.rot_size == 256) return launch_rb<8>(a, s, norm);
    return launch_rb<9>(a, s, norm);
}

}  // namespace basq
