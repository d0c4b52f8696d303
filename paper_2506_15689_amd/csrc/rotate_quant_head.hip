// Per-head rotate + bias + quantise: rot_size == group == 128 (the online Hadamard on q and k, R_qk, and
// the per-head asymmetric INT4 of the KV cache: paper Sec. 4 "online rotations", Sec. 5 "Deployment
// Details" and Sec. 5.2).  Every 128-channel head is rotated by H_128 / sqrt(128) and gets its own range
// and token record, so a 512-channel piece of a token (four heads) is an independent work item: one
// wavefront per item, nothing but registers in between.
//
// Channel bits of an item: e0..e6 inside the head, e7,e8 the head.
//   load   lane l reads 8 consecutive bf16 (e0..e2); its 16-byte unit is (e3,e4) <- lane bits (4,5),
//          (e5,e6) <- lane bits (0,1), (e7,e8) <- lane bits (2,3): a wave load is 1 KB, fully coalesced.
//   MFMA   A = 16 rows (lane%16 = e5..e8) x 32 (k = 8*(lane/16) + t = e0..e4), B = H_32 with its columns
//          permuted so that output bit e0 is the half index h and (e1..e4) the output lane%16.  Exact: bf16
//          inputs, +-1 entries.  Afterwards lane (col = e1..e4, lane/16 = e7,e8) holds d[h][r], r = (e5,e6).
//   stages e5, e6 on the four r registers.  The head of a value is lane/16: its 16 lanes are one DPP row.
//   bias (LDS copy), range over 8 registers and the row, quantise; the four bytes of a lane (one per r)
//   are transposed inside each quad so that a lane stores one dword and a wave 256 contiguous bytes.
#include "basq_internal.h"
#include <type_traits>

namespace basq {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef short v8s __attribute__((ext_vector_type(8)));

constexpr int RH_WAVES = 4;
constexpr int RH_THREADS = RH_WAVES * 64;

// (every CTRL used takes each lane's value from a lane of the row: no old value to keep)
template <int CTRL>
__device__ __forceinline__ float rh_dppf(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ int rh_dppi(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
#define RH_BFLY(x, y) do { const float _a = (x), _b = (y); (x) = _a + _b; (y) = _a - _b; } while (0)

struct RhMin { __device__ __forceinline__ float operator()(float a, float b) const { return fminf(a, b); } };
struct RhMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct RhAdd { __device__ __forceinline__ int operator()(int a, int b) const { return a + b; } };
__device__ __forceinline__ float rh_quad(float v, std::integral_constant<int, 1>) { return rh_dppf<0xB1>(v); }
__device__ __forceinline__ int rh_quad(int v, std::integral_constant<int, 1>) { return rh_dppi<0xB1>(v); }
__device__ __forceinline__ float rh_quad(float v, std::integral_constant<int, 2>) { return rh_dppf<0x4E>(v); }
__device__ __forceinline__ int rh_quad(int v, std::integral_constant<int, 2>) { return rh_dppi<0x4E>(v); }
__device__ __forceinline__ float rh_ror4(float v) { return rh_dppf<0x124>(v); }
__device__ __forceinline__ int rh_ror4(int v) { return rh_dppi<0x124>(v); }
__device__ __forceinline__ float rh_ror8(float v) { return rh_dppf<0x128>(v); }
__device__ __forceinline__ int rh_ror8(int v) { return rh_dppi<0x128>(v); }

// Reduction of NI items at once over the 16 lanes of a DPP row; lane l ends with the result of item l % NI.  With four
// items 11 instructions instead of 16: a lane hands over what its neighbour collects.
template <int NI, class T, class Op>
__device__ __forceinline__ T rh_reduce(const T (&v)[NI], int lane, Op op) {
    constexpr std::integral_constant<int, 1> x1{};
    constexpr std::integral_constant<int, 2> x2{};
    const bool b0 = lane & 1, b1 = lane & 2;
    T r;
    if constexpr (NI == 4) {
        const T p = op(b0 ? v[1] : v[0], rh_quad(b0 ? v[0] : v[1], x1));
        const T q = op(b0 ? v[3] : v[2], rh_quad(b0 ? v[2] : v[3], x1));
        r = op(b1 ? q : p, rh_quad(b1 ? p : q, x2));
    } else if constexpr (NI == 2) {
        r = op(b0 ? v[1] : v[0], rh_quad(b0 ? v[0] : v[1], x1));
        r = op(r, rh_quad(r, x2));
    } else {
        r = op(v[0], rh_quad(v[0], x1));
        r = op(r, rh_quad(r, x2));
    }
    r = op(r, rh_ror4(r));
    return op(r, rh_ror8(r));
}
// the value that lane t of the quad (t < NI: the lane that holds item t) has
template <int NI>
__device__ __forceinline__ float rh_item(float v, int t) {
    if (NI == 1) return v;
    return t == 0 ? rh_dppf<0x00>(v) : t == 1 ? rh_dppf<0x55>(v) : t == 2 ? rh_dppf<0xAA>(v) : rh_dppf<0xFF>(v);
}

// NI consecutive items of a token per step of a wave (NI divides the items per token): their loads are in flight together,
// the next step's are requested before this step's are worked on, and what is per head -- two divisions and the rest of the
// range arithmetic, 30 instructions that one item repeats on the 16 lanes of a head -- is done for the NI items on
// different lanes at once.  What bounds it is vector-instruction issue, 100 per item: 120 while the compiler, allowed more than 256
// registers a lane, kept the MFMAs' results in accumulation registers, and every DPP move had a zero put into its result first;
// 8192 tokens of K = 4096 20.5 -> 19.2 us.  Where the rotation is written out they may stay there: a wave a SIMD more is slower then
// (1777 tokens with s^a 11.5 us, as built 11.2).
// K = 4096, one item a step and nothing requested ahead -> with both: 1024 tokens 8.0 -> 6.5 us, 4096 tokens 15.7 -> 13.7,
// 8192 tokens 25.4 -> 21.2, 65536 tokens 156 -> 127; K = 8192, 16384 tokens 102 -> 69 (before the staging below took its present
// form, and on another machine than its figures).  NI = 2 throughout: 24.1 us at 8192 tokens; eight workgroups per compute unit: 16.5 us at 4096.
template <int NI, bool HAS_BIAS, bool HAS_SCALE, bool ROT_OUT>
__global__ __launch_bounds__(RH_THREADS, ROT_OUT ? 1 : 2) void rotate_quant_head_kernel(RotateQuantArgs a, float norm) {
    // bias and s^a laid out so that lane l of piece (c, r) reads the float2 at ((c*4 + r)*64 + l)
    extern __shared__ __attribute__((aligned(16))) float rh_lds[];
    const int K = a.K;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, g = lane >> 4;
    float2* lbias = reinterpret_cast<float2*>(rh_lds);
    float2* lscale = reinterpret_cast<float2*>(rh_lds + (HAS_BIAS ? K : 0));
    const int unit = g | ((lane & 3) << 2) | (((lane >> 2) & 3) << 4);       // 16-byte unit of the lane inside an item

    const int spt = K / (512 * NI);                            // steps per token
    const int hpt = K / 128;                                   // heads (token records) per token
    // Step = (token m, item group c), uniform over the wave: kept in scalar registers and advanced without a
    // division (stride = sq tokens + sr groups).
    const int swave = __builtin_amdgcn_readfirstlane(wave);
    const int64_t first = (int64_t)blockIdx.x * RH_WAVES + swave;
    const int64_t stride = (int64_t)gridDim.x * RH_WAVES;
    const int64_t sq = stride / spt;
    const int sr = (int)(stride - sq * spt);
    int64_t m = first / spt;
    int c = (int)(first - m * spt);
    uint4 raw[NI];
    auto request = [&](int64_t tok, int grp) {
#pragma unroll
        for (int t = 0; t < NI; ++t) raw[t] = nt_load16(a.X + tok * a.ldx + 512 * (NI * grp + t) + 8 * unit);
    };
    if (m < a.M) request(m, c);                                // before the staging below, whose barrier would wait for more

    if (HAS_BIAS || HAS_SCALE) {
        // Up to eight pieces requested before the first is written (a piece at a time is a memory latency each, eight in a row in
        // front of everything at K = 4096: 1 token 3.2 -> 2.6 us, 1024 6.5 -> 5.7, 8192 23.0 -> 21.3; K = 8192, 333 tokens 6.9 -> 5.8).
        static_assert(RH_THREADS == 256, "a piece is an item: float2 number f of the staged copy is lane f%64, r = (f/64)%4, c = f/256");
        const int at = threadIdx.x, items = K / 512;
        const int e = 128 * ((at & 63) >> 4) + 32 * (at >> 6) + 2 * (at & 15);
        auto stage = [&](int c0, auto count_c) {
            constexpr int COUNT = decltype(count_c)::value;
            float2 bv[COUNT], sv[COUNT];
#pragma unroll
            for (int i = 0; i < COUNT; ++i) {
                if (HAS_BIAS) bv[i] = *reinterpret_cast<const float2*>(a.bias + 512 * (c0 + i) + e);
                if (HAS_SCALE) sv[i] = *reinterpret_cast<const float2*>(a.act_scale + 512 * (c0 + i) + e);
            }
#pragma unroll
            for (int i = 0; i < COUNT; ++i) {
                if (HAS_BIAS) lbias[256 * (c0 + i) + at] = bv[i];
                if (HAS_SCALE) lscale[256 * (c0 + i) + at] = sv[i];
            }
        };
        int c0 = 0;
        for (; c0 + 8 <= items; c0 += 8) stage(c0, std::integral_constant<int, 8>{});
        if (items & 4) { stage(c0, std::integral_constant<int, 4>{}); c0 += 4; }
        if (items & 2) { stage(c0, std::integral_constant<int, 2>{}); c0 += 2; }
        if (items & 1) stage(c0, std::integral_constant<int, 1>{});
        __syncthreads();
    }

    // B operand: column j' = lane%16 of half h, k = 8*(lane/16) + t; input bits (t0,t1,t2,g0,g1) = e0..e4,
    // output bits (h, j'0..j'3) = e0..e4: sign = parity(popcount(kin & jout))
    v8bf bop[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        v8s tmp;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int kin = t | (g << 3), jout = h | (col << 1);
            tmp[t] = (short)(0x3F80 | ((__builtin_popcount(kin & jout) & 1) ? 0x8000 : 0));
        }
        bop[h] = __builtin_bit_cast(v8bf, tmp);
    }
    // byte transpose inside a quad, lane i collects byte i of the four lanes: with the neighbour bytes 0, 2 (even lanes) or 1, 3
    // of both, then with the lane after that one 16-bit half of both
    const int qi = lane & 3;
    const unsigned sel1 = lane & 1 ? 0x03070105u : 0x06020400u, sel2 = lane & 2 ? 0x03020706u : 0x05040100u;

    while (m < a.M) {
        float d[NI][2][4];
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const v8bf aop = __builtin_bit_cast(v8bf, raw[t]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4f acc = {0.f, 0.f, 0.f, 0.f};
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aop, bop[h], acc, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) d[t][h][r] = acc[r];
            }
        }
        int64_t next_m = m + sq;
        int next_c = c + sr;
        if (next_c >= spt) { next_c -= spt; ++next_m; }
        if (next_m < a.M) request(next_m, next_c);

        float mn[NI], mx[NI];
#pragma unroll
        for (int t = 0; t < NI; ++t) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                RH_BFLY(d[t][h][0], d[t][h][1]);
                RH_BFLY(d[t][h][2], d[t][h][3]);
                RH_BFLY(d[t][h][0], d[t][h][2]);
                RH_BFLY(d[t][h][1], d[t][h][3]);
            }
            // this lane's values: channels 512*item + 128g + 32r + 2col + h
            const int item = NI * c + t;
            mn[t] = INFINITY; mx[t] = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float2 bb = make_float2(0.f, 0.f), ss = make_float2(1.f, 1.f);
                if (HAS_BIAS) bb = lbias[(item * 4 + r) * 64 + lane];
                if (HAS_SCALE) ss = lscale[(item * 4 + r) * 64 + lane];
                const float r0 = d[t][0][r] * norm, r1 = d[t][1][r] * norm;
                if (ROT_OUT)
                    *reinterpret_cast<float2*>(a.rot_out + m * (int64_t)K + 512 * item + 128 * g + 32 * r + 2 * col) = make_float2(r0, r1);
                const float v0 = HAS_SCALE ? fmaf(r0, ss.x, -bb.x) : r0 - bb.x;
                const float v1 = HAS_SCALE ? fmaf(r1, ss.y, -bb.y) : r1 - bb.y;
                d[t][0][r] = v0; d[t][1][r] = v1;
                mn[t] = fminf(mn[t], fminf(v0, v1));
                mx[t] = fmaxf(mx[t], fmaxf(v0, v1));
            }
        }
        // the record of item lane % NI, head g
        const float lo = a.clip_lo * rh_reduce(mn, lane, RhMin{});
        const float hi = a.clip_hi * rh_reduce(mx, lane, RhMax{});
        float s = __fdiv_rn(hi - lo, 15.0f);
        if (!(s > 0.0f && s < INFINITY)) s = 1.0f;
        const float inv = __fdiv_rn(1.0f, s);
        const float nlo = -(lo * inv);

        int sums[NI];
#pragma unroll
        for (int t = 0; t < NI; ++t) {
            const float inv_t = rh_item<NI>(inv, t), nlo_t = rh_item<NI>(nlo, t);
            uint32_t ev = 0, od = 0;                            // byte r: the code of channel 2col (+1) of 32-block r
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float t0 = __builtin_amdgcn_fmed3f(fmaf(d[t][0][r], inv_t, nlo_t), 0.0f, 15.0f);
                const float t1 = __builtin_amdgcn_fmed3f(fmaf(d[t][1][r], inv_t, nlo_t), 0.0f, 15.0f);
                ev = __builtin_amdgcn_cvt_pk_u8_f32(t0, r, ev);     // round-half-to-even, NaN -> 0
                od = __builtin_amdgcn_cvt_pk_u8_f32(t1, r, od);
            }
            const int sum = __builtin_amdgcn_udot4(ev, 0x01010101u, 0, false);
            sums[t] = __builtin_amdgcn_udot4(od, 0x01010101u, sum, false);
            const uint32_t mine = ev | (od << 4);                   // byte r = the packed byte at 256*item + 64g + 16r + col
            const uint32_t x = __builtin_amdgcn_perm((unsigned)rh_dppi<0xB1>((int)mine), mine, sel1);
            const uint32_t word = __builtin_amdgcn_perm((unsigned)rh_dppi<0x4E>((int)x), x, sel2);
            // lane (quad q = col/4, i = col%4) now holds bytes 256*item + 64g + 16i + 4q .. +3
            *reinterpret_cast<uint32_t*>(a.Aq + m * (int64_t)(K / 2) + 256 * (NI * c + t) + 64 * g + 16 * qi + 4 * (col >> 2)) = word;
        }
        const int sum = rh_reduce(sums, lane, RhAdd{});
        if (col < NI) {                                         // lane col of a head: item col
            basq_tokmeta mt;
            mt.scale = s; mt.lo = lo; mt.rowsum = sum; mt.reserved = 0;
            a.meta[m * hpt + 4 * (NI * c + col) + g] = mt;
        }
        m = next_m;
        c = next_c;
    }
}

template <int NI, bool HB, bool HS>
int launch_head_flags(const RotateQuantArgs& a, hipStream_t s) {
    const int64_t steps = a.M * (int64_t)(a.K / (512 * NI));
    const int64_t want = (steps + RH_WAVES - 1) / RH_WAVES;
    // workgroups per compute unit at most; with several items a step four, so that a wave has steps to prefetch
    const int64_t cap = 256 * (NI == 1 ? 8 : 4);
    const unsigned blocks = (unsigned)(want < cap ? want : cap);
    const size_t lds = (size_t)a.K * sizeof(float) * ((HB ? 1 : 0) + (HS ? 1 : 0));
    const float norm = (float)(1.0 / sqrt(128.0));
    if (a.rot_out)
        hipLaunchKernelGGL((rotate_quant_head_kernel<NI, HB, HS, true>), dim3(blocks), dim3(RH_THREADS), lds, s, a, norm);
    else
        hipLaunchKernelGGL((rotate_quant_head_kernel<NI, HB, HS, false>), dim3(blocks), dim3(RH_THREADS), lds, s, a, norm);
    return check_hip(hipGetLastError(), "rotate_quant (per head) launch");
}

template <int NI>
int launch_head(const RotateQuantArgs& a, hipStream_t s) {
    if (a.bias && a.act_scale) return launch_head_flags<NI, true, true>(a, s);
    if (a.bias) return launch_head_flags<NI, true, false>(a, s);
    if (a.act_scale) return launch_head_flags<NI, false, true>(a, s);
    return launch_head_flags<NI, false, false>(a, s);
}

}  // namespace

bool rotate_quant_head_applicable(const RotateQuantArgs& a) {
    // the staged bias and s^a must fit the default 64 KB of dynamic LDS
    const size_t lds = (size_t)a.K * sizeof(float) * ((a.bias ? 1 : 0) + (a.act_scale ? 1 : 0));
    return !a.has28 && a.rot_size == 128 && a.group == 128 && a.K % 512 == 0 && a.Aq != nullptr && a.meta != nullptr &&
           a.Aq6 == nullptr && lds <= 64 * 1024;
}

int launch_rotate_quant_head(const RotateQuantArgs& a, hipStream_t s) {
    // several items a step where a token has them and a step per wave still leaves no SIMD with fewer than two waves
    const int64_t items = a.M * (int64_t)(a.K / 512);
    if (a.K % 2048 == 0 && items >= 4 * 2048) return launch_head<4>(a, s);
    if (a.K % 1024 == 0 && items >= 2 * 2048) return launch_head<2>(a, s);
    return launch_head<1>(a, s);
}

}  // namespace basq
