// A 512-channel piece of a token through rotation and quantiser, in the registers of one wave; shared by the blockwise and
// small-token kernels (rotate_quant_block.hip, where the layout is described) and the one-launch layer of small tokens
// (linear_small.hip), hence the same bits.
#ifndef BASQ_ROTATE_BLOCK_PIECE_H
#define BASQ_ROTATE_BLOCK_PIECE_H

#include "rotate_pow2_token.h"

namespace basq {
namespace {

// butterfly across lane bit 5 (SWAP32) or lane bit 4 for the register pair (x, y): afterwards x holds the sums and y
// the differences, and the lane bit tells which of the two former registers a lane's pair came from
template <bool SWAP32>
__device__ __forceinline__ void rb_cross_lane_bfly(float& x, float& y) {
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

// B operand of the MFMA: k = 8*(lane/16) + t carries input bits (e0,e1,e2,e7,e8), column lane%16 of half h carries
// output bits (h; e1,e2,e7,e8).  H over the low LOG2N-4 of those five bits, identity over the rest.
// Entries +-2^-SHIFT.
template <int LOG2N, int SHIFT>
__device__ __forceinline__ void rb_make_bop(int lane, v8bf (&bop)[2]) {
    constexpr int MASK = (1 << (LOG2N - 4)) - 1;       // 7 -> 0b00111, 8 -> 0b01111, 9 -> 0b11111
    const int jp = lane & 15, g = lane >> 4;
    const uint16_t mag = (uint16_t)((127 - SHIFT) << 7);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        v8s tmp;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int kin = t | (g << 3), jout = h | (jp << 1);
            const bool same_block = ((kin ^ jout) & ~MASK & 31) == 0;
            const short v = (short)(mag | ((__builtin_popcount(kin & jout & MASK) & 1) ? 0x8000 : 0));
            tmp[t] = same_block ? v : (short)0;
        }
        bop[h] = __builtin_bit_cast(v8bf, tmp);
    }
}

template <int CTRL>
__device__ __forceinline__ uint32_t rb_dpp_u(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// The stages of one piece: MFMA, then e5, e6 in registers, then e3, e4 across lane bits 4 and 5.
__device__ __forceinline__ void rb_rotate_piece(const uint4& raw, const v8bf (&bop)[2], float (&d)[2][4]) {
    const v8bf aop = __builtin_bit_cast(v8bf, raw);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bop[h], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) d[h][r] = acc[r];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        BFLY(d[h][0], d[h][1]);                // e5
        BFLY(d[h][2], d[h][3]);
        BFLY(d[h][0], d[h][2]);                // e6
        BFLY(d[h][1], d[h][3]);
        rb_cross_lane_bfly<false>(d[h][0], d[h][1]);   // e3 <-> lane bit 4; register bit r0 now means e3
        rb_cross_lane_bfly<false>(d[h][2], d[h][3]);
        rb_cross_lane_bfly<true>(d[h][0], d[h][2]);    // e4 <-> lane bit 5; register bit r1 now means e4
        rb_cross_lane_bfly<true>(d[h][1], d[h][3]);
    }
}

// where a lane's values of a piece end up: e = rb_eout + h + 8*r0 + 16*r1
__host__ __device__ __forceinline__ int rb_eout(int lane) {
    return 2 * (lane & 1) + 4 * ((lane >> 1) & 1) + 128 * ((lane >> 2) & 1) + 256 * ((lane >> 3) & 1) +
           32 * ((lane >> 4) & 1) + 64 * ((lane >> 5) & 1);
}
// the 32-channel segment of the piece whose codes the lane's quad holds
__device__ __forceinline__ int rb_segment(int lane) {
    return ((lane >> 4) & 1) + 2 * ((lane >> 5) & 1) + 4 * ((lane >> 2) & 1) + 8 * ((lane >> 3) & 1);
}

// Codes of a lane's eight values; returns the aligned dword of eight consecutive channels' codes, channels
// 32*segment + 8*(lane%4) .. +7 of the piece, and adds the lane's own codes to `sum` if `count`.
__device__ __forceinline__ uint32_t rb_codes(const float (&v)[2][4], float inv, float nlo, int lane, bool count, int& sum) {
    uint32_t ev = 0, od = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float t0 = __builtin_amdgcn_fmed3f(fmaf(v[0][r], inv, nlo), 0.0f, 15.0f);
        const float t1 = __builtin_amdgcn_fmed3f(fmaf(v[1][r], inv, nlo), 0.0f, 15.0f);
        ev = __builtin_amdgcn_cvt_pk_u8_f32(t0, r, ev);          // round-half-to-even, NaN -> 0
        od = __builtin_amdgcn_cvt_pk_u8_f32(t1, r, od);
    }
    if (count) {
        sum = __builtin_amdgcn_udot4(ev, 0x01010101u, sum, false);
        sum = __builtin_amdgcn_udot4(od, 0x01010101u, sum, false);
    }
    // byte r of `w`: the row's byte at 256*c + 16*seg + q4 + 4*r.  Quad transpose: lane q4 ends with the bytes
    // q4 of its quad's four words, i.e. the aligned dword at ... + 4*q4.
    const uint32_t w = ev | (od << 4);
    // with the neighbour: bytes 0, 2 (even lanes) or 1, 3 of both; with the lane after that: one 16-bit half of both
    const uint32_t sel1 = lane & 1 ? 0x03070105u : 0x06020400u, sel2 = lane & 2 ? 0x03020706u : 0x05040100u;
    const uint32_t x = __builtin_amdgcn_perm(rb_dpp_u<0xB1>(w), w, sel1);
    return __builtin_amdgcn_perm(rb_dpp_u<0x4E>(x), x, sel2);
}

// A whole token of NP pieces in one wave: the stages over e9 (, e10) pair its pieces register by register.
template <int NP>
__device__ __forceinline__ void rb_pair_pieces(float (&v)[NP][2][4]) {
#pragma unroll
    for (int st = 1; st < NP; st <<= 1)
#pragma unroll
        for (int c = 0; c < NP; ++c)
            if ((c & st) == 0)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) BFLY(v[c][h][r], v[c + st][h][r]);
}

// ... its range, behind normalisation, s^a and b^c (bb, ss: this lane's values, two at +8*r of each piece); rot_row: where the
// fp32 rotation goes (ROT_OUT), from this lane's first channel on.
struct RbRange { float s, lo, inv, nlo; };
template <int NP, bool FOLD_NORM, bool HAS_BIAS, bool HAS_SCALE, bool ROT_OUT>
__device__ __forceinline__ RbRange rb_token_range(float (&v)[NP][2][4], const float2 (&bb)[NP][4], const float2 (&ss)[NP][4], float norm,
                                                  float clip_lo, float clip_hi, float* rot_row) {
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float r0 = v[c][0][r], r1 = v[c][1][r];
            if (!FOLD_NORM) { r0 = r0 * norm; r1 = r1 * norm; }
            if (ROT_OUT) *reinterpret_cast<float2*>(rot_row + 512 * c + 8 * r) = make_float2(r0, r1);
            const float b0 = HAS_BIAS ? bb[c][r].x : 0.0f, b1 = HAS_BIAS ? bb[c][r].y : 0.0f;
            const float v0 = HAS_SCALE ? fmaf(r0, ss[c][r].x, -b0) : r0 - b0;
            const float v1 = HAS_SCALE ? fmaf(r1, ss[c][r].y, -b1) : r1 - b1;
            v[c][0][r] = v0;
            v[c][1][r] = v1;
            mn = fminf(mn, fminf(v0, v1));
            mx = fmaxf(mx, fmaxf(v0, v1));
        }
    mn = wave_min_f(mn);
    mx = wave_max_f(mx);
    RbRange x;
    x.lo = clip_lo * mn;
    const float hi = clip_hi * mx;
    x.s = __fdiv_rn(hi - x.lo, 15.0f);
    if (!(x.s > 0.0f && x.s < INFINITY)) x.s = 1.0f;
    x.inv = __fdiv_rn(1.0f, x.s);
    x.nlo = -(x.lo * x.inv);
    return x;
}

}  // namespace
}  // namespace basq

#endif
