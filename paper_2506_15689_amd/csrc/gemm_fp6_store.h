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
// Needs even ldy and N and 4-byte aligned Y; where ldy, N and Y allow 16-byte pieces they are stored whole.
template <int TM, int TN, int BM, class ColBlock>
__device__ __forceinline__ void store_outputs(const GemmArgs& a, int64_t m0, int n0, int row0, int lane, const unsigned (&outv)[TM][TN][4][2], ColBlock&& col_block) {
    const bool wide = (a.ldy & 7) == 0 && (a.N & 7) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 15) == 0;
    const int piece = 2 * ((lane >> 4) & 1) + (lane >> 5);
    const int row_end = (int)(a.M - m0 < BM ? a.M - m0 : BM), col_end = a.N - n0;       // of the matrix, from the tile's start
    auto store16 = [&](int row, int col, unsigned o0, unsigned o1, unsigned o2, unsigned o3) {      // within the tile
        if (row >= row_end) return;
        uint16_t* dst = a.Y + (m0 + row) * a.ldy + n0 + col;
        if (wide) {
            if (col < col_end) nt_store16(dst, make_uint4(o0, o1, o2, o3));
        } else {
            const unsigned o[4] = {o0, o1, o2, o3};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + 2 * e < col_end) *reinterpret_cast<uint32_t*>(dst + 2 * e) = o[e];
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

}  // namespace

}  // namespace basq
