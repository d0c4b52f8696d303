// Output stores shared by the fp6 GEMM kernels.
#pragma once

#include "basq_internal.h"

namespace basq {

namespace {

// A wave's outputs to memory.  With the weights as the first operand of the 32 x 32 MFMA, accumulator register r of lane l
// belongs to token l % 32 of a row block and to output channel 8*(r/4) + 4*(l/32) + r%4 of a column block, so four adjacent
// channels are two dwords of packed bf16: outv[i][j][q][p] = channels 8q + 4*(l/32) + 2p, +1 of row block i, column block j.
//
// Lane bit 5 (which four of eight channels) trades places with the low bit of q, lane bit 4 (token) with its high bit, and
// in a pair of column blocks lane bit 3 (token) with the block: a lane then owns 16 bytes of one token's row, and a store
// covers whole 128-byte lines of eight rows.  Against dword stores of 64-byte runs a wave issues 16 stores instead of 64
// for 128 x 64 outputs (a compute unit takes 16 cycles per store instruction of either width); 16-byte stores of 64-byte
// runs were slower than the dword stores (449 against 433 us on 4096 x 8192 x 28672; as built 424), and without the
// non-temporal hint these were too (439).
//
//   row0            first row of the wave inside the tile; m0, n0: the tile's first row and column
//   col_block(j)    column block of the tile (32 columns each) of the wave's block j; blocks 2k and 2k + 1 are adjacent
// Any ldy >= N, N and Y a bf16 tensor can have; FORM says what they allow (see store_outputs).
template <StoreForm FORM, int TM, int TN, int BM, class ColBlock>
__device__ __forceinline__ void store_outputs_as(const GemmArgs& a, int64_t m0, int n0, int row0, int lane, const unsigned (&outv)[TM][TN][4][2], ColBlock&& col_block) {
    const int piece = 2 * ((lane >> 4) & 1) + (lane >> 5);
    const int row_end = (int)(a.M - m0 < BM ? a.M - m0 : BM), col_end = a.N - n0;       // of the matrix, from the tile's start
    auto store16 = [&](int row, int col, unsigned o0, unsigned o1, unsigned o2, unsigned o3) {      // within the tile
        if (row >= row_end || col >= col_end) return;
        uint16_t* dst = a.Y + (m0 + row) * a.ldy + n0 + col;
        const basq_v4u v = {o0, o1, o2, o3};
        if (FORM == StoreForm::whole_nt) {
            nt_store16(dst, make_uint4(o0, o1, o2, o3));
        } else if (FORM == StoreForm::whole) {
            *reinterpret_cast<basq_v4u*>(dst) = v;
        } else if (col + 8 <= col_end) {
            __builtin_memcpy(dst, &v, 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (col + 2 * e + 1 < col_end) { const unsigned d = v[e]; __builtin_memcpy(dst + 2 * e, &d, 4); }
                else if (col + 2 * e < col_end) dst[2 * e] = (uint16_t)v[e];
            }
        }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        unsigned z[TN][2][4];                                 // [block][token / 16][dword] of 16 bytes: piece `piece` of token l % 16
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const auto u = __builtin_amdgcn_permlane32_swap(outv[i][j][0][p], outv[i][j][1][p], false, false);
                const auto v = __builtin_amdgcn_permlane32_swap(outv[i][j][2][p], outv[i][j][3][p], false, false);
                z[j][0][p] = u[0]; z[j][0][2 + p] = u[1];
                z[j][1][p] = v[0]; z[j][1][2 + p] = v[1];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const auto u = __builtin_amdgcn_permlane16_swap(z[j][0][e], z[j][1][e], false, false);
                z[j][0][e] = u[0]; z[j][1][e] = u[1];
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < TN; j += 2) {
                if (j + 1 < TN) {
                    unsigned lo[4], hi[4];                    // tokens 0..7 and 8..15 of the sixteen (row rotation by 8 lanes)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        lo[e] = (unsigned)__builtin_amdgcn_update_dpp((int)z[j][h][e], (int)z[j + 1][h][e], 0x128, 0xF, 0xC, false);
                        hi[e] = (unsigned)__builtin_amdgcn_update_dpp((int)z[j + 1][h][e], (int)z[j][h][e], 0x128, 0xF, 0x3, false);
                    }
                    const int row = row0 + i * 32 + 16 * h + (lane & 7), col = (col_block(j) + ((lane >> 3) & 1)) * 32 + 8 * piece;
                    store16(row, col, lo[0], lo[1], lo[2], lo[3]);
                    store16(row + 8, col, hi[0], hi[1], hi[2], hi[3]);
                } else {
                    store16(row0 + i * 32 + 16 * h + (lane & 15), col_block(j) * 32 + 8 * piece, z[j][h][0], z[j][h][1], z[j][h][2], z[j][h][3]);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Rows that start on 16-byte boundaries and hold whole pieces of 8 channels leave as aligned 16-byte stores, with the
// non-temporal hint where output_form() says so.  Everything else takes 16-byte stores at the
// alignment there is; only the last piece of a row of N % 8 != 0 channels goes by pairs of channels.  (1021 tokens, K = 4096:
// N = 32000 70 us, 32001 91 us in rows of 32001 and 78 us in rows of 32008; with 2-byte stores for odd N or ldy, which from
// this register layout go to 32 rows an instruction, 211 and 225 us, and dword stores for even N were 7-14 % slower: 2048 x
// 12290 75.6 us, as built 65.2.)
template <int TM, int TN, int BM, class ColBlock>
__device__ __forceinline__ void store_outputs(const GemmArgs& a, StoreForm form, int64_t m0, int n0, int row0, int lane, const unsigned (&outv)[TM][TN][4][2], ColBlock&& col_block) {
    if (form == StoreForm::whole_nt)
        store_outputs_as<StoreForm::whole_nt, TM, TN, BM>(a, m0, n0, row0, lane, outv, col_block);
    else if (form == StoreForm::whole)
        store_outputs_as<StoreForm::whole, TM, TN, BM>(a, m0, n0, row0, lane, outv, col_block);
    else
        store_outputs_as<StoreForm::any, TM, TN, BM>(a, m0, n0, row0, lane, outv, col_block);
}

// The same out of 16 x 16 blocks: accumulator register r of lane l belongs to token l % 16 and channel 4*(l/16) + r of a block,
// outv[i][j][p] = channels 4*(l/16) + 2p, +1 of row block i, column block j of 16 (j / 2 of 32: col_block).  Lane bit 4 (channel)
// trades places with the low bit of j, and in a pair of 32-column blocks lane bit 3 (token) with the block: as above a lane owns 16 bytes of
// one token's row and a store covers whole lines of eight rows, at half the swaps between lanes.
template <StoreForm FORM, int TM, int TN, int BM, class ColBlock>
__device__ __forceinline__ void store_outputs16_as(const GemmArgs& a, int64_t m0, int n0, int row0, int lane, const unsigned (&outv)[TM][TN][2], ColBlock&& col_block) {
    const int piece = 2 * ((lane >> 4) & 1) + (lane >> 5);
    const int row_end = (int)(a.M - m0 < BM ? a.M - m0 : BM), col_end = a.N - n0;       // of the matrix, from the tile's start
    auto store16 = [&](int row, int col, unsigned o0, unsigned o1, unsigned o2, unsigned o3) {      // within the tile
        if (row >= row_end || col >= col_end) return;
        uint16_t* dst = a.Y + (m0 + row) * a.ldy + n0 + col;
        const basq_v4u v = {o0, o1, o2, o3};
        if (FORM == StoreForm::whole_nt) {
            nt_store16(dst, make_uint4(o0, o1, o2, o3));
        } else if (FORM == StoreForm::whole) {
            *reinterpret_cast<basq_v4u*>(dst) = v;
        } else if (col + 8 <= col_end) {
            __builtin_memcpy(dst, &v, 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (col + 2 * e + 1 < col_end) { const unsigned d = v[e]; __builtin_memcpy(dst + 2 * e, &d, 4); }
                else if (col + 2 * e < col_end) dst[2 * e] = (uint16_t)v[e];
            }
        }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        unsigned z[TN / 2][4];                                // 16 bytes: piece `piece` of token l % 16
#pragma unroll
        for (int j = 0; j < TN / 2; ++j)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const auto u = __builtin_amdgcn_permlane16_swap(outv[i][2 * j][p], outv[i][2 * j + 1][p], false, false);
                z[j][p] = u[0]; z[j][2 + p] = u[1];
            }
#pragma unroll
        for (int j = 0; j < TN / 2; j += 2) {
            if (j + 1 < TN / 2) {
                unsigned lo[4], hi[4];                        // tokens 0..7 and 8..15 of the sixteen (row rotation by 8 lanes)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    lo[e] = (unsigned)__builtin_amdgcn_update_dpp((int)z[j][e], (int)z[j + 1][e], 0x128, 0xF, 0xC, false);
                    hi[e] = (unsigned)__builtin_amdgcn_update_dpp((int)z[j + 1][e], (int)z[j][e], 0x128, 0xF, 0x3, false);
                }
                const int row = row0 + i * 16 + (lane & 7), col = (col_block(j) + ((lane >> 3) & 1)) * 32 + 8 * piece;
                store16(row, col, lo[0], lo[1], lo[2], lo[3]);
                store16(row + 8, col, hi[0], hi[1], hi[2], hi[3]);
            } else {
                store16(row0 + i * 16 + (lane & 15), col_block(j) * 32 + 8 * piece, z[j][0], z[j][1], z[j][2], z[j][3]);
            }
        }
        if (i & 1) __builtin_amdgcn_sched_barrier(0);
    }
}

template <int TM, int TN, int BM, class ColBlock>
__device__ __forceinline__ void store_outputs16(const GemmArgs& a, StoreForm form, int64_t m0, int n0, int row0, int lane, const unsigned (&outv)[TM][TN][2], ColBlock&& col_block) {
    if (form == StoreForm::whole_nt)
        store_outputs16_as<StoreForm::whole_nt, TM, TN, BM>(a, m0, n0, row0, lane, outv, col_block);
    else if (form == StoreForm::whole)
        store_outputs16_as<StoreForm::whole, TM, TN, BM>(a, m0, n0, row0, lane, outv, col_block);
    else
        store_outputs16_as<StoreForm::any, TM, TN, BM>(a, m0, n0, row0, lane, outv, col_block);
}

typedef float fp6_acc_t __attribute__((ext_vector_type(4)));

// The optional dump of the integer accumulators (64 * acc) into a.acc_out, rows of N int32.  One channel a dword: lane bit 3 (token)
// trades places with the column block, so that a store covers 32 channels of eight rows (2048 x 4096, K = 4096, the predecessor
// on 32 x 32 blocks: 29 us with the dump, 23.7 without; dword stores into 32 rows an instruction: 128 us).
template <int TM, int TN, int BM, class ColBlock>
__device__ __forceinline__ void store_accumulators16(const GemmArgs& a, int64_t m0, int n0, int row0, int lane, const fp6_acc_t (&acc)[TM][TN], ColBlock&& col_block) {
    const int row_end = (int)(a.M - m0 < BM ? a.M - m0 : BM), col_end = a.N - n0;
    auto store16 = [&](int row, int col, const int (&v)[4]) {
        if (row >= row_end) return;
        int32_t* dst = a.acc_out + (m0 + row) * a.N + n0 + col;
        if (col + 4 <= col_end) {
            __builtin_memcpy(dst, v, 16);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (col + e < col_end) dst[e] = v[e];
        }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
            int lo[4], hi[4];                                 // tokens 0..7 and 8..15 of the sixteen (row rotation by 8 lanes)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v0 = __float2int_rn(64.0f * acc[i][j][e]), v1 = __float2int_rn(64.0f * acc[i][j + 1][e]);
                lo[e] = __builtin_amdgcn_update_dpp(v0, v1, 0x128, 0xF, 0xC, false);
                hi[e] = __builtin_amdgcn_update_dpp(v1, v0, 0x128, 0xF, 0x3, false);
            }
            const int row = row0 + i * 16 + (lane & 7), col = col_block(j / 2) * 32 + 16 * ((lane >> 3) & 1) + 4 * (lane >> 4);
            store16(row, col, lo);
            store16(row + 8, col, hi);
            __builtin_amdgcn_sched_barrier(0);
        }
}

// How the outputs leave.  With the non-temporal hint they don't displace the operands from the caches (4096 x
// 28672, K = 8192: 406 us with, 420 without; 2048 x 12288, K = 4096 56 and 58; 333 x 4096 even) -- where rows are whole
// 128-byte lines.  A line that two rows share is otherwise written in two parts (every product into outputs that no cache holds
// any more: 33204 x 14216, K = 256 467 us with, 262 without; 5293 x 5840, K = 256 29 and 23; 4096 x 9008, K = 2048 65 and 54),
// which pays only where something else takes longer: where operands that are read many times do not stay in the 256 MB beside
// the outputs (4096 x 28656, K = 8192 409 and 419; 4096 x 16432, K = 11008 348 and 370; but 16384 x 9008, K = 4096 308 and 294,
// 3000 x 20016, K = 8192 even), and where the launch says so.  With a reader of Y right behind (a copy of
// it timed with the product) the hint costs 0 to 3 % up to 50 MB of outputs (333 x 4096 14.0 and 13.8 us, 2048 x 12288 78.0 and 75.7)
// and still gains 3 % at 4096 x 28672, K = 8192.
// `hides_stores`: the launch's other work hides what shared lines cost with the hint (each launch has its rule and figures).
StoreForm output_form(const GemmArgs& a, bool hides_stores) {
    const uintptr_t y = reinterpret_cast<uintptr_t>(a.Y);
    if ((a.ldy & 7) != 0 || (a.N & 7) != 0 || (y & 15) != 0) return StoreForm::any;
    if (((a.ldy & 63) == 0 && (y & 127) == 0) || hides_stores) return StoreForm::whole_nt;
    const double operands = 0.75 * a.K * ((double)a.M + a.N);
    const bool spill = operands > (double)(128 << 20) && operands + 2.0 * (double)a.M * a.N > (double)(256 << 20);
    return spill ? StoreForm::whole_nt : StoreForm::whole;
}

}  // namespace

}  // namespace basq
