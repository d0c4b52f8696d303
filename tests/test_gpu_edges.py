"""GPU parity on the edges of the fast rotate+quant kernels, through the C ABI against the CPU oracle.

Degenerate tokens (Eq. 4 has no answer for a token whose range is empty or not finite; the reading taken is
s = 1, NaN -> code 0, min/max ignore NaN) on every specialised kernel and on both sides of each of their
token-count switches, always as: the GPU's fp32 rotation of the checked rows (`rot_out`) -> oracle.quantize_tokens
-> codes and the BITS of scale, lower bound and row sum must equal what the kernel under test wrote for those rows.
The kernel under test runs WITHOUT `rot_out` (that is what selects the fast variants), with and without the fp6 copy.
Then: the many-token path, the one-launch decode kernel, and the group-wise layer at full benchmark size."""
import sys

import numpy as np
import pytest
import torch

import oracle
import layout_ref
from paper_2506_15689_amd import binding as B
from paper_2506_15689_amd import synth_inputs as si

import parity_util as pu

pytestmark = pytest.mark.gpu

DEV = "cuda"
N_SPECIAL = 10


def announce(msg):
    print(f"[edge] {msg}", flush=True)
    sys.stdout.flush()


def plant_degenerate_rows(X: torch.Tensor, first: int) -> None:
    """Overwrites rows first .. first + N_SPECIAL - 1 of X (bf16 [M, K]) with the degenerate tokens."""
    K = X.shape[1]
    X[first:first + N_SPECIAL] = 0.0                      # +0: all-zero token (constant when there is no bias)
    X[first + 1, 0] = 1.0                                 # rotates to the constant 1/sqrt(n) in its first block
    X[first + 2, K // 3] = float("nan")                   # NaN in every channel of that block after the rotation
    X[first + 3, 5] = float("inf")                        # +-inf everywhere in the block
    X[first + 4, K - 1] = float("-inf")
    X[first + 5, 3] = float("inf")                        # two infinities of one block: inf - inf = NaN in half of
    X[first + 5, 64] = float("inf")                       # the outputs, +-inf in the rest
    X[first + 6, :] = 3.0e38                              # finite inputs whose sums overflow
    X[first + 7, 0] = 2.0 ** -126                         # rotates into the subnormal range
    X[first + 8, :] = -1.5                                # one non-zero output per rotation block, the rest exact zeros
    X[first + 9, :] = float("nan")                        # nothing finite at all


def gpu_inputs(M, K, seed, *, with_bias, with_scale):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    X = (torch.randn((M, K), generator=gen, device=DEV) * 1.5).to(torch.bfloat16)
    X[:, 7] *= 20.0                                       # an outlier channel (Sec. 3.1)
    bias = (torch.randn(K, generator=gen, device=DEV) * 0.3) if with_bias else None
    sa = (torch.rand(K, generator=gen, device=DEV) * 0.45 + 0.8) if with_scale else None
    return X, bias, sa


def rows_to_check(M, specials, rng, n_random=64):
    rows = set()
    for f in specials:
        rows |= set(range(f, f + N_SPECIAL))
    rows |= {0, M - 1}
    rows |= set(int(v) for v in rng.choice(M, size=min(n_random, M), replace=False))
    return np.array(sorted(rows))


def check_fp6_copy(Aq, A6, K, row_blocks):
    """The fp6 copy against the repacking kernel everywhere (whole 32-row blocks; the bytes of rows past M in the
    last block are undefined) and against the layout reference on the given 32-row blocks."""
    M = Aq.shape[0]
    A6b = torch.zeros_like(A6)
    B.basq_pack_fp6(Aq, A6b)
    torch.cuda.synchronize()
    RB = (M + 31) // 32
    full = M // 32
    v, vb = A6.view(K // 128, RB, 3072), A6b.view(K // 128, RB, 3072)
    assert torch.equal(v[:, :full], vb[:, :full]), "fp6 copy written by the quantiser differs from the repacked codes"
    for rb in row_blocks:
        if rb < 0 or rb >= full:
            continue
        codes = oracle.unpack_codes(Aq[32 * rb:32 * rb + 32].cpu().numpy())
        ref6 = layout_ref.pack_fp6(codes).reshape(K // 128, 3072)
        np.testing.assert_array_equal(v[:, rb].cpu().numpy(), ref6, err_msg=f"fp6 copy, row block {rb}")


# K = 4096: several waves per token up to 512 tokens, one wave per token in four-wave workgroups up to 2047,
# eight-wave workgroups up to 32767, and from 32768 tokens on with the fp6 copy the staged tails.
# K = 8192: split up to 256, four waves to 2047, eight waves to 4096, four waves beyond, staged tails from 32768;
# with s^a (staged in LDS beside b^c) eight waves from 1025 tokens on.
# K = 14336: four waves per token up to 256 tokens, then two: workgroups of two tokens, and of four that stay for several rounds
# with both b^c and s^a from 513 tokens on, otherwise for codes alone where the last round of 1024 tokens is filled well enough
# (1844 and not 1843).
SWITCH_CASES = [
    (4096, 12), (4096, 512), (4096, 513), (4096, 2047), (4096, 2048), (4096, 2061), (4096, 32768 + 13),
    (8192, 11), (8192, 256), (8192, 257), (8192, 1024), (8192, 1025), (8192, 2047), (8192, 2048), (8192, 4096), (8192, 4097), (8192, 12301), (8192, 32768 + 13),
    (14336, 11), (14336, 131), (14336, 256), (14336, 257), (14336, 512), (14336, 513), (14336, 1024), (14336, 1025), (14336, 1030), (14336, 1843), (14336, 1844), (14336, 2048 + 5), (14336, 3071),
]


@pytest.mark.parametrize("K,M", SWITCH_CASES)
@pytest.mark.parametrize("with_bias,with_scale", [(False, False), (True, False), (True, True)])
def test_degenerate_tokens_on_the_fast_kernels(K, M, with_bias, with_scale):
    if M > 20000 and with_scale:
        pytest.skip("the many-token variants do not depend on s^a; covered with and without the bias")
    announce(f"degenerate tokens K={K} M={M} bias={with_bias} scale={with_scale}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=with_bias, with_scale=with_scale)
    specials = sorted({0, M - N_SPECIAL} | ({M // 2 - 3} if M >= 4 * N_SPECIAL else set()))
    for f in reversed(specials):                          # the set at row 0 is planted last and stays whole
        plant_degenerate_rows(X, f)
    rng = np.random.default_rng(K + M)
    rows = rows_to_check(M, specials, rng)
    clip_lo, clip_hi = 0.9, 0.95
    # without the fp6 copy
    Aq, meta = B.alloc_activation_buffers(M, K, DEV)
    Aq.fill_(0xEE); meta.fill_(-7)
    B.basq_rotate_quant(X, K, bias, sa, clip_lo, clip_hi, Aq, meta)
    ref = pu.check_rows_against_oracle(X, rows, K, bias, sa, clip_lo, clip_hi, Aq, meta, what="no fp6 copy")
    # what the reading of a degenerate token promises, on the oracle's own output (rows of the first planted set)
    pos = {int(r): i for i, r in enumerate(rows)}
    f0 = specials[0]
    if not with_bias and not with_scale:
        i = pos[f0]                                       # the all-zero token is constant: s := 1, every code 0
        assert ref.scale[i, 0] == 1.0 and ref.lo[i, 0] == 0.0 and not ref.codes[i].any()
        i = pos[f0 + 1]                                   # a constant c > 0 with unequal clips: range [0.9 c, 0.95 c]
        assert ref.scale[i, 0] > 0 and set(np.unique(ref.codes[i])) == {15}
    i = pos[f0 + 9]
    assert ref.scale[i, 0] == 1.0 and not ref.codes[i].any(), "an all-NaN token has no finite range: s = 1, codes 0"
    i = pos[f0 + 2]
    assert not ref.codes[i].any(), "NaN -> code 0"
    # with the fp6 copy: same codes and records, and the copy holds the same codes
    Aq2, meta2 = B.alloc_activation_buffers(M, K, DEV)
    A6 = B.alloc_fp6_buffer(M, K, DEV).zero_()
    B.basq_rotate_quant(X, K, bias, sa, clip_lo, clip_hi, Aq2, meta2, Aq6=A6)
    torch.cuda.synchronize()
    pu.check_rows_against_oracle(X, rows, K, bias, sa, clip_lo, clip_hi, Aq2, meta2, what="with the fp6 copy")
    assert torch.equal(Aq2, Aq) and torch.equal(meta2[:, :3], meta[:, :3]), "codes or records change with the fp6 copy"
    check_fp6_copy(Aq2, A6, K, sorted({f // 32 for f in specials} | {(M - 1) // 32 - 1}))
    # the fp6 form alone (what the one-call layer asks for on the fp6 matrix path): same records, same fp6 bytes
    meta3 = torch.full_like(meta2, -7)
    A6c = B.alloc_fp6_buffer(M, K, DEV).zero_()
    B.basq_rotate_quant(X, K, bias, sa, clip_lo, clip_hi, None, meta3, Aq6=A6c)
    torch.cuda.synchronize()
    full = M // 32
    assert torch.equal(meta3[:, :3], meta2[:, :3]), "records change when the 4-bit codes are left out"
    assert torch.equal(A6c.view(K // 128, -1, 3072)[:, :full], A6.view(K // 128, -1, 3072)[:, :full]), \
        "fp6 form changes when the 4-bit codes are left out"
    # properties on all rows
    rs = meta[:, 2].to(torch.int64)
    assert torch.equal(rs, (Aq & 0x0F).to(torch.int64).sum(dim=1) + (Aq >> 4).to(torch.int64).sum(dim=1))


@pytest.mark.parametrize("K,M,rot,group", [(4096, 70, 128, 128), (2048, 600, 128, 128), (8192, 37, 128, 128),
                                           (4096, 12, 4096, 128), (8192, 70, 8192, 128), (1024, 33, 64, 64)])
@pytest.mark.parametrize("with_bias", [False, True])
def test_degenerate_tokens_with_groupwise_ranges(K, M, rot, group, with_bias):
    """Per-head kernel (rot = group = 128), the one-wave-per-token kernel with a range per four lanes
    (rot = K, group = 128) and the generic kernel: a degenerate GROUP next to ordinary ones in the same token."""
    announce(f"degenerate groups K={K} M={M} rot={rot} group={group} bias={with_bias}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M + group, with_bias=with_bias, with_scale=False)
    specials = [0, M - N_SPECIAL]
    for f in reversed(specials):
        plant_degenerate_rows(X, f)
    # ordinary tokens with one dead head: all-zero, NaN and inf confined to one rotation block (rot = 128 only)
    if rot == 128 and M > 30:
        X[12, 256:384] = 0.0
        X[13, 128 + 5] = float("nan")
        X[14, 384 + 9] = float("inf")
    rows = np.arange(M) if M <= 80 else np.union1d(rows_to_check(M, specials, np.random.default_rng(M), n_random=48), [12, 13, 14])
    ng = K // group
    Aq = torch.full((M, K // 2), 0xEE, dtype=torch.uint8, device=DEV)
    meta = torch.full((M * ng, 4), -7, dtype=torch.int32, device=DEV)
    B.basq_rotate_quant(X, rot, bias, sa, 0.9, 0.95, Aq, meta, group_size=group)
    torch.cuda.synchronize()
    pu.check_rows_against_oracle(X, rows, rot, bias, sa, 0.9, 0.95, Aq, meta, group=group, what="group-wise")


@pytest.mark.parametrize("K,M,rot", [(11008, 300, 256), (1280, 70, 128), (2048, 41, 512), (768, 33, 256), (16384, 25, 512)])
@pytest.mark.parametrize("with_bias,with_scale", [(False, False), (True, False), (True, True)])
def test_degenerate_tokens_on_the_blockwise_kernel(K, M, rot, with_bias, with_scale):
    """Blockwise rotations of 128, 256 and 512 channels with per-token ranges (the register-resident blockwise
    kernel; K = 11008 and 768 end in a half piece of 256 channels): the degenerate tokens at both ends of the batch,
    and ordinary tokens with one dead rotation block (zero, NaN, inf confined to it)."""
    announce(f"degenerate tokens, blockwise K={K} M={M} rot={rot} bias={with_bias} scale={with_scale}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M + rot, with_bias=with_bias, with_scale=with_scale)
    specials = [0, M - N_SPECIAL]
    for f in reversed(specials):
        plant_degenerate_rows(X, f)
    X[12, rot:2 * rot] = 0.0
    X[13, rot + 5] = float("nan")
    X[14, K - rot + 9] = float("inf")
    rows = np.arange(M) if M <= 80 else np.union1d(rows_to_check(M, specials, np.random.default_rng(M), n_random=48), [12, 13, 14])
    Aq, meta = B.alloc_activation_buffers(M, K, DEV)
    Aq.fill_(0xEE); meta.fill_(-7)
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, rot, bias, sa, 0.9, 0.95, Aq, meta, Aq6=A6)
    torch.cuda.synchronize()
    pu.check_rows_against_oracle(X, rows, rot, bias, sa, 0.9, 0.95, Aq, meta, what="blockwise")
    check_fp6_copy(Aq, A6, K, row_blocks=[0, (M // 32) - 1])


@pytest.mark.parametrize("K", [4096, 8192])
@pytest.mark.parametrize("M", [1, 2, 4])
@pytest.mark.parametrize("with_bias", [False, True])
def test_degenerate_tokens_through_the_one_launch_decode_kernel(K, M, with_bias):
    """basq_linear_fused with at most four tokens on the streaming layout is one kernel that rotates, quantises and
    multiplies; its codes never reach memory, so the output is what is compared: with oracle.linear on the GPU's
    rotation of the same tokens (a separate call), NaN-aware -- where the reference is finite the usual tolerance,
    elsewhere the same kind of non-finite value -- and bit for bit with the two-call path."""
    N = 264
    lay = si.make_tiny(max(M, 16), K, N, seed=K + M)
    case = pu.make_case(lay, use_bias=with_bias, use_out_bias=with_bias)
    d = pu.to_device(case)
    kinds = {1: [[9], [0], [3], [6]], 2: [[0, 2], [3, 7]], 4: [[0, 1, 2, 3], [5, 6, 8, 9]]}[M]
    Wd = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device=DEV)
    B.basq_pack_decode(d.Wq, Wd)
    for kind in kinds + [None]:
        announce(f"one-launch decode K={K} M={M} bias={with_bias} degenerate kinds={kind}")
        X = d.X[:M].clone()
        if kind is not None:
            scratch = torch.zeros((N_SPECIAL, K), dtype=torch.bfloat16, device=DEV)
            plant_degenerate_rows(scratch, 0)
            for i, k in enumerate(kind):
                X[i] = scratch[k]
        Y1 = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=DEV)
        ws = torch.empty(max(B.basq_workspace_bytes(M, K, N), 256), dtype=torch.uint8, device=DEV)
        B.basq_linear_fused(X, K, d.bias, None, case.clip_lo, case.clip_hi, Wd, d.w_scale, d.w_zero, d.w_sum,
                            d.out_bias, Y1, ws, w_layout=B.BASQ_W_DECODE16, N=N)
        # the two-call path on the same tokens, with the rotation dumped for the oracle
        Aq, meta = B.alloc_activation_buffers(M, K, DEV)
        r = torch.empty((M, K), dtype=torch.float32, device=DEV)
        Y2 = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=DEV)
        B.basq_rotate_quant(X, K, d.bias, None, case.clip_lo, case.clip_hi, Aq, meta, r)
        B.basq_w4a4_gemm(Aq, meta, Wd, d.w_scale, d.w_zero, d.w_sum, d.out_bias, Y2, w_layout=B.BASQ_W_DECODE16, N=N)
        torch.cuda.synchronize()
        y1, y2 = si.bf16_bits(Y1.cpu()), si.bf16_bits(Y2.cpu())
        np.testing.assert_array_equal(y1, y2, err_msg="one launch vs two calls")
        x = oracle.bf16_to_f32(si.bf16_bits(X.cpu()))
        with np.errstate(all="ignore"):
            ref = oracle.linear(x, K, case.bias, None, case.clip_lo, case.clip_hi, case.wq, case.c, r=r.cpu().numpy())
        np.testing.assert_array_equal(oracle.unpack_codes(Aq.cpu().numpy()), ref.tq.codes)
        y = oracle.bf16_to_f32(y1).astype(np.float64)
        # bf16's largest finite value: beyond it the reference itself rounds to infinity
        fin = np.isfinite(ref.y) & (np.abs(ref.y) < 3.0e38)
        assert np.isfinite(y[fin]).all(), "a finite reference output came out non-finite"
        for m in range(M):                                # row by row: a degenerate token's outputs can be huge
            if fin[m].any():
                top = float(np.abs(ref.y[m][fin[m]]).max())
                assert np.abs(y[m][fin[m]] - ref.y[m][fin[m]]).max() <= pu.Y_TOL * max(top, 1e-30), f"token {m}"
        nan_ref = np.isnan(ref.y)
        assert np.isnan(y[nan_ref]).all(), "NaN in the reference, a number on the GPU"
        inf_ref = np.isinf(ref.y)
        assert (y[inf_ref] == ref.y[inf_ref]).all(), "infinite reference output: the GPU's differs"


@pytest.mark.parametrize("K", [8192, 4096])
def test_grouped_layer_at_benchmark_size(K):
    """The group-wise layer (activation ranges per 128 channels) at the size and in the launch configuration the
    benchmark times with --group-size 128 -- C5 (K = 8192: 64 groups) and C2 (K = 4096) -- checked on sampled token
    rows x output channels that include the first and last tiles: codes and group records bit-exact on the GPU's
    rotation, outputs within one bf16 step of oracle.linear_grouped on the same codes, within 2e-2 of max|ref| from
    X; the fp6 path (benchmarked) and the int8 path bit-identical on ALL elements."""
    name = "C5" if K == 8192 else "C2"
    cfg = si.CONFIGS[name]
    G = 128
    lay = si.make_layer(cfg)
    M, N = cfg.M, cfg.N
    ng = K // G
    announce(f"grouped layer at full size: {name} M={M} K={K} N={N}")
    rng = np.random.default_rng(cfg.index + 100)
    edge = 34
    rows = np.array(sorted(set(range(edge)) | set(range(M - edge, M)) | set(int(v) for v in rng.choice(M, 40, replace=False))))
    cols = np.array(sorted(set(range(edge)) | set(range(N - edge, N)) | set(int(v) for v in rng.choice(N, 400, replace=False))))
    xc = oracle.bf16_to_f32(si.bf16_bits(lay.X_calib))
    bc = oracle.channel_bias(xc, cfg.rot_size)
    w_s = oracle.bf16_to_f32(si.bf16_bits(lay.W_rot[torch.from_numpy(cols)]))
    wq_s = oracle.quantize_weights(w_s)
    c_s = oracle.fused_bias(wq_s, bc, None)

    W = lay.W_rot.to(DEV)
    Wq, w_scale, w_zero, w_sum = B.alloc_weight_buffers(N, K, DEV)
    B.basq_quantize_weights(W, Wq, w_scale, w_zero, w_sum)
    del W
    bias = torch.from_numpy(bc).to(DEV)
    out_bias = torch.empty(N, dtype=torch.float32, device=DEV)
    B.basq_fused_bias(Wq, w_scale, w_zero, bias, None, out_bias)
    gsum = torch.empty((ng, N), dtype=torch.int32, device=DEV)
    B.basq_group_colsums(Wq, G, gsum)
    W6 = B.alloc_fp6_buffer(N, K, DEV)
    B.basq_pack_fp6(Wq, W6)
    X = lay.X.to(DEV)
    Aq = torch.empty((M, K // 2), dtype=torch.uint8, device=DEV)
    meta = torch.empty((M * ng, 4), dtype=torch.int32, device=DEV)
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, cfg.rot_size, bias, None, cfg.clip, cfg.clip, Aq, meta, group_size=G, Aq6=A6)
    Y6 = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.basq_w4a4_gemm_grouped(Aq, meta, G, Wq, w_scale, w_zero, gsum, out_bias, Y6, Aq6=A6, Wq6=W6)
    Y8 = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.basq_w4a4_gemm_grouped(Aq, meta, G, Wq, w_scale, w_zero, gsum, out_bias, Y8)
    torch.cuda.synchronize()
    assert torch.equal(Y6.view(torch.int16), Y8.view(torch.int16)), "fp6 and int8 group-wise GEMMs differ"
    assert not torch.isnan(Y6).any()

    t_rows, t_cols = torch.from_numpy(rows).to(DEV), torch.from_numpy(cols).to(DEV)
    np.testing.assert_array_equal(oracle.unpack_codes(Wq[t_cols].cpu().numpy()), wq_s.codes)
    np.testing.assert_array_equal(gsum[:, t_cols].cpu().numpy(), oracle.group_colsums(wq_s, G), err_msg="group column sums")
    ref_q = pu.check_rows_against_oracle(X, rows, cfg.rot_size, bias, None, cfg.clip, cfg.clip, Aq, meta, group=G,
                                      what="group-wise ranges at full size")
    x_s = oracle.bf16_to_f32(si.bf16_bits(lay.X[torch.from_numpy(rows)]))
    # the oracle's layer on the codes just verified: its quantiser is deterministic, so feed it the same rotation
    Xs = X[t_rows].contiguous()
    r = torch.empty((len(rows), K), dtype=torch.float32, device=DEV)
    B.basq_rotate_quant(Xs, cfg.rot_size, bias, None, cfg.clip, cfg.clip,
                        torch.empty((len(rows), K // 2), dtype=torch.uint8, device=DEV),
                        torch.empty((len(rows) * ng, 4), dtype=torch.int32, device=DEV), r, group_size=G)
    torch.cuda.synchronize()
    ref_i = oracle.linear_grouped(x_s, cfg.rot_size, bc, None, cfg.clip, cfg.clip, G, wq_s, c_s, r=r.cpu().numpy())
    np.testing.assert_array_equal(ref_i.tq.codes, ref_q.codes)
    y = oracle.bf16_to_f32(si.bf16_bits(Y6[t_rows][:, t_cols].cpu())).astype(np.float64)
    top = float(np.abs(ref_i.y).max())
    worst = float((np.abs(y - ref_i.y) - 2.0 ** -8 * np.abs(ref_i.y)).max() / top)
    assert worst <= 1e-5, f"worst excess over one bf16 step: {worst} of max|ref| on identical codes"
    ref = oracle.linear_grouped(x_s, cfg.rot_size, bc, None, cfg.clip, cfg.clip, G, wq_s, c_s)
    err = float(np.abs(y - ref.y).max() / np.abs(ref.y).max())
    assert err <= pu.Y_TOL, f"output error {err}"
    d = ref_q.codes.astype(np.int32) - ref.tq.codes.astype(np.int32)
    assert (d != 0).mean() <= pu.FLIP_TOL and (np.abs(d[d != 0]) == 1).all()
    announce(f"ok rows={len(rows)} cols={len(cols)} y_err={err:.2e} flips={(d != 0).mean():.2e}")


def test_worst_case_accumulator_on_both_matrix_paths():
    """The fp6 path is exact because S = sum (q_a/8)(q_w/8) fits the fp32 accumulator: at the longest row it takes,
    K = 32768, with every code 15 on both sides the INT32 accumulator of Sec. 5.2's INT4 GEMM must be 225 K on the
    fp6 path and on the int8 path; a few columns of smaller codes check that nothing saturates on the way."""
    K, M, N = 32768, 200, 72
    codes_a = torch.full((M, K // 2), 0xFF, dtype=torch.uint8, device=DEV)
    codes_w = torch.full((N, K // 2), 0xFF, dtype=torch.uint8, device=DEV)
    codes_w[5] = 0x11                                      # every code 1: ACC = 15 K
    codes_w[6] = 0xF0                                      # alternating 0, 15: ACC = 225 K / 2
    meta = torch.zeros((M, 4), dtype=torch.int32, device=DEV)
    meta[:, 0] = torch.tensor(1.0).view(torch.int32)       # scale 1, lower bound 0
    meta[:, 2] = 15 * K
    w_scale = torch.ones(N, dtype=torch.bfloat16, device=DEV)
    w_zero = torch.zeros(N, dtype=torch.bfloat16, device=DEV)
    w_sum = torch.zeros(N, dtype=torch.float32, device=DEV)
    A6, W6 = B.alloc_fp6_buffer(M, K, DEV), B.alloc_fp6_buffer(N, K, DEV)
    B.basq_pack_fp6(codes_a, A6)
    B.basq_pack_fp6(codes_w, W6)
    want = np.full((M, N), 225 * K, dtype=np.int64)
    want[:, 5] = 15 * K
    want[:, 6] = 225 * K // 2
    for name, kw in (("int8", {}), ("fp6", dict(Aq6=A6, Wq6=W6))):
        announce(f"worst-case accumulator, {name} path")
        acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
        Y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        B.basq_w4a4_gemm(codes_a, meta, codes_w, w_scale, w_zero, w_sum, None, Y, acc, **kw)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(acc.cpu().numpy().astype(np.int64), want, err_msg=f"{name} path")
    # and the oracle's triple loop agrees on a few rows
    ref = oracle.int_gemm(oracle.unpack_codes(codes_a[:2].cpu().numpy()), oracle.unpack_codes(codes_w.cpu().numpy()))
    np.testing.assert_array_equal(ref, want[:2])


@pytest.mark.parametrize("N,K,with_bias,with_layer_bias", [(72, 512, True, True), (100, 1792, True, False),
                                                           (40, 4096, False, True), (33, 256, False, False)])
def test_prepare_weights_against_the_oracle(N, K, with_bias, with_layer_bias):
    """basq_prepare_weights: w_sum bit-exact against the oracle's weight quantiser, the fused bias of Eq. 14 against
    oracle.fused_bias (both accumulate in fp64; summation order differs), the prepacked weights equal to the layout
    reference; and the same numbers as the single-purpose helpers."""
    lay = si.make_tiny(8, K, N, seed=N + K)
    w = oracle.bf16_to_f32(si.bf16_bits(lay.W_rot))
    wq = oracle.quantize_weights(w)
    rng = np.random.default_rng(N)
    bc = rng.standard_normal(K).astype(np.float32) if with_bias else None
    lb = rng.standard_normal(N).astype(np.float32) if with_layer_bias else None
    Wq = torch.from_numpy(oracle.pack_codes(wq.codes)).to(DEV)
    w_scale, w_zero = si.bits_to_bf16(wq.scale_bits).to(DEV), si.bits_to_bf16(wq.zero_bits).to(DEV)
    tb = None if bc is None else torch.from_numpy(bc).to(DEV)
    tl = None if lb is None else torch.from_numpy(lb).to(DEV)
    w_sum = torch.full((N,), float("nan"), dtype=torch.float32, device=DEV)
    out_bias = torch.full((N,), float("nan"), dtype=torch.float32, device=DEV)
    W6 = B.alloc_fp6_buffer(N, K, DEV).zero_() if K % 128 == 0 else None
    B.basq_prepare_weights(Wq, w_scale, w_zero, tb, tl, w_sum, out_bias, W6)
    ob2 = torch.empty_like(out_bias)
    B.basq_fused_bias(Wq, w_scale, w_zero, tb, tl, ob2)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(w_sum.cpu().numpy().view(np.uint32), wq.wsum.view(np.uint32), err_msg="w_sum bits")
    ref = oracle.fused_bias(wq, bc, lb)
    np.testing.assert_allclose(out_bias.cpu().numpy(), ref, rtol=1e-6, atol=1e-6)
    assert torch.equal(out_bias, ob2), "basq_prepare_weights and basq_fused_bias disagree"
    if W6 is not None:
        full = (N // 32) * 32                              # bytes of rows past N in the last block are undefined
        got = W6.cpu().numpy().reshape(K // 128, -1, 3072)
        want = layout_ref.pack_fp6(wq.codes).reshape(K // 128, -1, 3072)
        np.testing.assert_array_equal(got[:, :full // 32], want[:, :full // 32], err_msg="prepacked weights")


@pytest.mark.parametrize("M", [524288 + 45, 1048576 + 19])
def test_packed_operands_of_two_to_four_gib_and_beyond(M):
    """The matrix-path kernels address their packed operands with 32-bit unsigned byte offsets, so an operand may be
    up to 4 GiB.  524288 + 45 tokens of K = 8192 (four times the largest batch of Sec. 5.2's prefill table, 131072
    tokens) make the 4-bit activations 2.0 GiB and their fp6 form 3.0 GiB: the rows behind byte 2^31 of either form
    must come out as the oracle computes them -- codes and records bit-exact, accumulators bit-exact on both matrix
    paths, outputs within one bf16 step on identical codes -- and the two paths must agree on every element.
    1048576 + 19 tokens put both forms beyond 4 GiB: the quantiser and the repacking kernel index with 64 bits, and
    the product falls back to the kernel that does too (with or without the fp6 operands); same checks, around byte
    2^32 as well."""
    K, N = 8192, 192
    announce(f"packed operands of {M * (K // 2) / 2 ** 30:.2f} GiB (4-bit) and {M * K * 0.75 / 2 ** 30:.2f} GiB (fp6): M={M} K={K} N={N}")
    gen = torch.Generator(device=DEV).manual_seed(2031)
    X = torch.empty((M, K), dtype=torch.bfloat16, device=DEV)
    for i in range(0, M, 65536):
        n = min(65536, M - i)
        X[i:i + n] = (torch.randn((n, K), generator=gen, device=DEV) * 1.5).to(torch.bfloat16)
    X[:, 7] *= 20.0
    bias = torch.randn(K, generator=gen, device=DEV) * 0.3
    W = (torch.randn((N, K), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    Wq, w_scale, w_zero, w_sum = B.alloc_weight_buffers(N, K, DEV)
    B.basq_quantize_weights(W, Wq, w_scale, w_zero, w_sum)
    out_bias = torch.empty(N, dtype=torch.float32, device=DEV)
    B.basq_fused_bias(Wq, w_scale, w_zero, bias, None, out_bias)
    W6 = B.alloc_fp6_buffer(N, K, DEV)
    B.basq_pack_fp6(Wq, W6)

    Aq, meta = B.alloc_activation_buffers(M, K, DEV)
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    assert Aq.numel() > 2 ** 31 and A6.numel() > 2 ** 31 and (Aq.numel() < 2 ** 32) == (M < 1048576)
    clip = 0.9
    B.basq_rotate_quant(X, K, bias, None, clip, clip, Aq, meta, Aq6=A6)
    torch.cuda.synchronize()
    # rows around byte 2^31 of the 4-bit form (row 524288), the first and last rows, and a random sample; the fp6
    # form is laid out chunk by chunk of 128 channels, so every row has codes on both sides of its byte 2^31
    rng = np.random.default_rng(2031)
    cross4 = 2 ** 31 // (K // 2)
    chunk6 = 2 ** 31 // (3072 * ((M + 31) // 32))                 # the 128-channel chunk of the fp6 form that straddles 2^31
    rows = set(range(8)) | set(range(cross4 - 40, min(M, cross4 + 45))) | set(range(M - 45, M))
    if M > 2 * cross4:
        rows |= set(range(2 * cross4 - 40, min(M, 2 * cross4 + 45)))      # byte 2^32
    rows |= set(int(v) for v in rng.choice(M, 64, replace=False))
    rows = np.array(sorted(rows))
    announce(f"  4-bit form crosses 2^31 at row {cross4}; fp6 form inside chunk {chunk6} of {K // 128} "
             f"(every row has codes behind it); {len(rows)} rows sampled")
    ref_q = pu.check_rows_against_oracle(X, rows, K, bias, None, clip, clip, Aq, meta, what="operands beyond 2 GiB")
    check_fp6_copy(Aq, A6, K, row_blocks=[0, cross4 // 32 - 1, cross4 // 32, M // 32 - 1])
    torch.cuda.empty_cache()

    acc8 = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
    Y8 = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.basq_w4a4_gemm(Aq, meta, Wq, w_scale, w_zero, w_sum, out_bias, Y8, acc8)
    acc6 = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
    Y6 = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.basq_w4a4_gemm(Aq, meta, Wq, w_scale, w_zero, w_sum, out_bias, Y6, acc6, Aq6=A6, Wq6=W6)
    torch.cuda.synchronize()
    assert torch.equal(acc6, acc8), "accumulators of the fp6 and int8 paths differ"
    assert torch.equal(Y6.view(torch.int16), Y8.view(torch.int16)), "outputs of the fp6 and int8 paths differ"
    assert not torch.isnan(Y6).any()

    wq_ref = oracle.quantize_weights(oracle.bf16_to_f32(si.bf16_bits(W.cpu())))
    np.testing.assert_array_equal(oracle.unpack_codes(Wq.cpu().numpy()), wq_ref.codes)
    c_ref = oracle.fused_bias(wq_ref, bias.cpu().numpy(), None)
    t_rows = torch.from_numpy(rows).to(DEV)
    acc_ref = oracle.int_gemm_blas(ref_q.codes, wq_ref.codes)
    np.testing.assert_array_equal(acc6[t_rows].cpu().numpy(), acc_ref, err_msg="accumulators behind 2^31")
    y_ref = oracle.dequant(acc_ref, ref_q, wq_ref, c_ref)
    y = oracle.bf16_to_f32(si.bf16_bits(Y6[t_rows].cpu())).astype(np.float64)
    top = float(np.abs(y_ref).max())
    worst = float((np.abs(y - y_ref) - 2.0 ** -8 * np.abs(y_ref)).max() / top)
    assert worst <= 1e-5, f"worst excess over one bf16 step: {worst} of max|ref| on identical codes"
    announce(f"ok worst excess {worst:.2e}")


@pytest.mark.parametrize("K", [128, 256, 384, 512, 640, 896])
@pytest.mark.parametrize("M,N,pad", [(129, 64, 0), (300, 1000, 0), (257, 514, 2), (131, 333, 1), (700, 20480, 8), (1030, 4100, 4), (2000, 12300, 4),
                                     (61, 24584, 2), (64, 28672, 0), (65, 72, 0), (128, 2050, 2)])
def test_fp6_product_over_few_k_steps(K, M, N, pad):
    """Every length of the K loop around the depth of its ring of LDS stages (no steady step at all, one, several), each
    with ragged tiles and each alignment of the output rows, on the tiling that the shape takes: the bits of
    the int8 path (exact integer products, the same epilogue arithmetic, so no tolerance).  The last four are token
    counts that the weight-streaming kernel also takes (it is what they are compared with)."""
    announce(f"fp6 product M={M} N={N} K={K} pad={pad}")
    assert B.basq_diag_fp6_tiling(M, K, N) >= 0, "not a case of the fp6 product"
    gen = torch.Generator(device=DEV).manual_seed(K + M)
    A = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device=DEV, generator=gen)
    W = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device=DEV, generator=gen)
    A6, W6 = B.alloc_fp6_buffer(M, K), B.alloc_fp6_buffer(N, K)
    B.basq_pack_fp6(A, A6)
    B.basq_pack_fp6(W, W6)
    codes = A.to(torch.int32)
    meta = torch.zeros((M, 4), dtype=torch.int32, device=DEV)
    meta.view(torch.float32)[:, 0] = torch.rand(M, device=DEV, generator=gen) + 0.1
    meta.view(torch.float32)[:, 1] = -torch.rand(M, device=DEV, generator=gen)
    meta[:, 2] = ((codes & 15) + (codes >> 4)).sum(dim=1)
    sw = (torch.rand(N, device=DEV, generator=gen) + 0.1).to(torch.bfloat16)
    zp = torch.randint(0, 16, (N,), device=DEV, generator=gen).to(torch.bfloat16)
    ws, c = torch.randn(N, device=DEV, generator=gen), torch.randn(N, device=DEV, generator=gen)
    out = []
    for a6, w6 in ((A6, W6), (None, None)):
        Y = torch.full((M + 1, N + pad), -7.0, dtype=torch.bfloat16, device=DEV)
        B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, Y[:M, :N], Aq6=a6, Wq6=w6)
        assert bool((Y[M] == -7.0).all()) and bool((Y[:, N:] == -7.0).all()), "wrote outside the output"
        out.append(Y[:M, :N].contiguous())
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))


@pytest.mark.parametrize("K", [512, 1024, 2048])
@pytest.mark.parametrize("M", [21, 63, 257, 300, 8192 + 37])
@pytest.mark.parametrize("with_bias,with_scale", [(False, False), (True, True)])
def test_small_token_rotations(K, M, with_bias, with_scale):
    """rot_size == K in {512, 1024, 2048}, one wave per token: the token counts around a workgroup, a run of workgroups of
    one XCD and the persistent loop, with the degenerate tokens at both ends; and the rotation against the dense one in
    fp64 (fp32 sums of at most 2048 terms of a token's size: 2e-5 of its largest value is 100 roundings)."""
    announce(f"small tokens K={K} M={M} bias={with_bias} scale={with_scale}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=with_bias, with_scale=with_scale)
    specials = [0, M - N_SPECIAL]
    for f in reversed(specials):
        plant_degenerate_rows(X, f)
    rows = rows_to_check(M, specials, np.random.default_rng(M), n_random=48)
    Aq, meta = B.alloc_activation_buffers(M, K, DEV)
    Aq.fill_(0xEE); meta.fill_(-7)
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, K, bias, sa, 0.9, 0.95, Aq, meta, Aq6=A6)
    torch.cuda.synchronize()
    pu.check_rows_against_oracle(X, rows, K, bias, sa, 0.9, 0.95, Aq, meta, what="small token")
    check_fp6_copy(Aq, A6, K, row_blocks=[0, (M // 32) - 1])
    Xf = X[N_SPECIAL:N_SPECIAL + 1].contiguous()
    r = torch.empty((1, K), device=DEV)
    B.basq_rotate_quant(Xf, K, None, None, 1.0, 1.0, torch.empty((1, K // 2), dtype=torch.uint8, device=DEV),
                        torch.empty((1, 4), dtype=torch.int32, device=DEV), r)
    H = torch.ones((1, 1), dtype=torch.float64)
    while H.shape[0] < K:
        H = torch.cat([torch.cat([H, H], 1), torch.cat([H, -H], 1)], 0)
    want = Xf.double().cpu() @ H / K ** 0.5
    assert float((r.double().cpu() - want).abs().max()) <= 2e-5 * float(want.abs().max())


@pytest.mark.parametrize("K,rot,N", [(1024, 1024, 72), (11008, 256, 40), (1536, 512, 136)])
@pytest.mark.parametrize("M", [129, 300, 1021])
def test_layer_on_the_fp6_form_alone(K, rot, N, M):
    """Where the one-call layer lets the quantiser leave the 4-bit codes out (M > 128 with fp6 weights): the bits of the
    two calls that write and read both forms."""
    announce(f"fp6 form alone K={K} rot={rot} M={M}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=True, with_scale=True)
    gen = torch.Generator(device=DEV).manual_seed(M)
    W = (torch.randn((N, K), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    Wq, sw, zp, ws = B.alloc_weight_buffers(N, K)
    B.basq_quantize_weights(W, Wq, sw, zp, ws)
    c, W6 = torch.empty(N, device=DEV), B.alloc_fp6_buffer(N, K)
    B.basq_prepare_weights(Wq, sw, zp, bias, None, ws, c, W6)
    Aq, meta = B.alloc_activation_buffers(M, K, DEV)
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, rot, bias, sa, 0.9, 0.9, Aq, meta, Aq6=A6)
    two, one = (torch.empty((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    B.basq_w4a4_gemm(Aq, meta, Wq, sw, zp, ws, c, two, Aq6=A6, Wq6=W6)
    work = torch.empty(B.basq_workspace_bytes(M, K, N), dtype=torch.uint8, device=DEV)
    B.basq_linear_fused(X, rot, bias, sa, 0.9, 0.9, Wq, sw, zp, ws, c, one, work, Wq6=W6)
    assert torch.equal(one.view(torch.int16), two.view(torch.int16))


@pytest.mark.parametrize("K,M", [(4096, 1023), (4096, 1024), (4096, 3077), (8192, 513), (2048, 4099), (1024, 2049), (3072, 701),
                                 (1536, 1500)])
@pytest.mark.parametrize("with_bias,with_scale", [(True, False), (True, True)])
def test_per_head_steps_of_several_items(K, M, with_bias, with_scale):
    """The per-head kernel with one, two and four 512-channel items a step (by width and token count), on both sides of the
    token count where it changes and with a last step that only some waves have, dead heads next to ordinary ones."""
    announce(f"per-head steps K={K} M={M} scale={with_scale}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=with_bias, with_scale=with_scale)
    specials = [0, M - N_SPECIAL]
    for f in reversed(specials):
        plant_degenerate_rows(X, f)
    X[12, 256:384] = 0.0
    X[13, 128 + 5] = float("nan")
    X[14, 384 + 9] = float("inf")
    rows = np.union1d(rows_to_check(M, specials, np.random.default_rng(M), n_random=48), [12, 13, 14])
    Aq = torch.full((M, K // 2), 0xEE, dtype=torch.uint8, device=DEV)
    meta = torch.full((M * (K // 128), 4), -7, dtype=torch.int32, device=DEV)
    B.basq_rotate_quant(X, 128, bias, sa, 0.9, 0.95, Aq, meta, group_size=128)
    torch.cuda.synchronize()
    pu.check_rows_against_oracle(X, rows, 128, bias, sa, 0.9, 0.95, Aq, meta, group=128, what="per head")
    assert not bool((meta[:, 3] == -7).any()), "a record was not written"


@pytest.mark.parametrize("N", [40, 4096, 4112, 8192, 8208])
@pytest.mark.parametrize("M", [17, 33, 65])
@pytest.mark.parametrize("K", [128, 512, 640, 1024, 1152])
def test_streaming_product_where_its_workgroups_change(K, M, N):
    """The weight-streaming kernel on both sides of the output widths at which it takes more waves or tiles a workgroup
    (256 and 512 tiles of 16 channels) and of the row lengths from which it takes more waves, fewer chunks of K than waves:
    its INT32 accumulators against the exact product of the codes (fp64 matmul of integers below 2^53)."""
    announce(f"streaming product M={M} N={N} K={K}")
    gen = torch.Generator(device=DEV).manual_seed(N + M)
    A = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device=DEV, generator=gen)
    W = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device=DEV, generator=gen)
    Wd = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device=DEV)
    B.basq_pack_decode(W, Wd)
    meta = torch.ones((M, 4), dtype=torch.int32, device=DEV)
    one = torch.ones(N, dtype=torch.bfloat16, device=DEV)
    ws = torch.zeros(N, device=DEV)
    codes = [torch.stack([t & 15, t >> 4], dim=2).view(t.shape[0], K).double().cpu() for t in (A, W)]
    want = (codes[0] @ codes[1].T).to(torch.int32)
    for w, layout in ((Wd, B.BASQ_W_DECODE16), (W, B.BASQ_W_CANONICAL)):
        acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
        Y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        B.basq_w4a4_gemm(A, meta, w, one, one, ws, None, Y, acc, w_layout=layout, N=N)
        assert torch.equal(acc.cpu(), want)


@pytest.mark.parametrize("K,M", [(4096, 33), (4096, 2051), (8192, 70), (8192, 1030), (8192, 2051), (8192, 2344), (8192, 4099),
                                 (4096, 7000)])
@pytest.mark.parametrize("with_bias,with_scale", [(False, False), (True, True)])
def test_fp6_form_of_groupwise_codes(K, M, with_bias, with_scale):
    """Full rotation with groups of 128: the fp6 form that the quantiser writes beside the codes is the repacked codes, and
    codes and records are those of the call without it."""
    announce(f"fp6 form of groups K={K} M={M} bias={with_bias} scale={with_scale}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=with_bias, with_scale=with_scale)
    for f in reversed([0, M - N_SPECIAL]):
        plant_degenerate_rows(X, f)
    Aq, meta, Aq2, meta2 = (torch.full(s, 0x5E, dtype=t, device=DEV) for s, t in 2 * [((M, K // 2), torch.uint8), ((M * (K // 128), 4), torch.int32)])
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, K, bias, sa, 0.9, 0.95, Aq, meta, Aq6=A6, group_size=128)
    B.basq_rotate_quant(X, K, bias, sa, 0.9, 0.95, Aq2, meta2, group_size=128)
    assert torch.equal(Aq, Aq2) and torch.equal(meta, meta2)
    check_fp6_copy(Aq, A6, K, row_blocks=[0, (M // 32) - 1])


def random_product(M, N, K, seed, groups=1):
    """Random codes in every form the products take, records and weight constants of ordinary size."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rand = lambda *shape: torch.rand(*shape, device=DEV, generator=gen)
    A = torch.randint(0, 256, (M, K // 2), dtype=torch.uint8, device=DEV, generator=gen)
    W = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device=DEV, generator=gen)
    A6, W6 = B.alloc_fp6_buffer(M, K), B.alloc_fp6_buffer(N, K)
    B.basq_pack_fp6(A, A6)
    B.basq_pack_fp6(W, W6)
    meta = torch.zeros((M * groups, 4), dtype=torch.int32, device=DEV)
    meta.view(torch.float32)[:, 0] = rand(M * groups) + 0.1
    meta.view(torch.float32)[:, 1] = -rand(M * groups)
    codes = A.to(torch.int32).view(M * groups, K // 2 // groups)
    meta[:, 2] = ((codes & 15) + (codes >> 4)).sum(dim=1)
    sw = (rand(N) + 0.1).to(torch.bfloat16)
    zp = torch.randint(0, 16, (N,), device=DEV, generator=gen).to(torch.bfloat16)
    return A, A6, meta, W, W6, sw, zp, rand(N), rand(N)


def output_view(M, N, ldy, offset):
    """A bf16 [M, N] view with rows of ldy elements that starts `offset` elements into its (poisoned) buffer."""
    buf = torch.full((M * ldy + offset + 8,), -7.0, dtype=torch.bfloat16, device=DEV)
    return buf, torch.as_strided(buf, (M, N), (ldy, 1), offset)


OUTPUT_FORMS = [(300, 333, 333, 0), (300, 334, 336, 0), (129, 1000, 1001, 1), (1021, 4094, 4094, 2), (260, 775, 776, 8),
                (700, 12289, 12289, 3), (515, 773, 776, 0), (1500, 20482, 20488, 0)]


@pytest.mark.parametrize("M,N,ldy,offset", OUTPUT_FORMS)
@pytest.mark.parametrize("grouped", [False, True])
def test_fp6_products_into_rows_of_any_alignment(M, N, ldy, offset, grouped):
    """Output rows that end inside a 16-byte piece and start on any 2-byte boundary: the int8 kernels' bits, nothing beside
    them."""
    K = 384
    announce(f"output rows M={M} N={N} ldy={ldy} offset={offset} grouped={grouped}")
    A, A6, meta, W, W6, sw, zp, ws, c = random_product(M, N, K, seed=M + N, groups=K // 128 if grouped else 1)
    gsum = torch.empty((K // 128, N), dtype=torch.int32, device=DEV)
    B.basq_group_colsums(W, 128, gsum)
    got = []
    for a6, w6 in ((A6, W6), (None, None)):
        buf, Y = output_view(M, N, ldy, offset)
        dump = torch.full((M * N + 8,), -9, dtype=torch.int32, device=DEV)
        if grouped:
            B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, gsum, c, Y, Aq6=a6, Wq6=w6)
        else:
            B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, Y, dump[:M * N].view(M, N), Aq6=a6, Wq6=w6)
            plain_buf, plain = output_view(M, N, ldy, offset)
            B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, plain, Aq6=a6, Wq6=w6)
            assert torch.equal(plain_buf.view(torch.int16), buf.view(torch.int16)), "outputs with and without the accumulators"
        assert bool((dump[M * N:] == -9).all())
        got.append((Y.clone(), dump))
        Y.fill_(-7.0)
        assert bool((buf == -7.0).all()), "wrote outside the output"
    assert torch.equal(got[0][1], got[1][1])
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16))


# tile of each tiling (tokens, channels) and how many workgroups of it are resident at once
FP6_TILES = [(256, 256, 256), (256, 192, 256), (256, 128, 256), (128, 128, 512), (128, 64, 512), (64, 64, 768)]


@pytest.mark.parametrize("K", [128, 256, 384, 512, 640, 896])
@pytest.mark.parametrize("tiling", range(B.FP6_TILINGS))
def test_every_tiling_of_the_fp6_product(tiling, K):
    """Each tiling by name: lengths of the K loop around the depth of its ring of stages, tiles ragged in both directions,
    fewer tokens and channels than a tile, every kind of output row, and more tiles than are resident at once (so that a
    workgroup goes on to another tile): the bits of the kernels without the fp6 operands, nothing beside the output."""
    bm, bn, resident = FP6_TILES[tiling]
    rows = 9                                                # of tiles, of the case that overflows the chip
    shapes = [(1, 1, 1, 0), (33, 72, 72, 0), (bm, bn, bn, 0), (bm + 1, bn - 1, bn, 8), (2 * bm - 31, 3 * bn + 32, 3 * bn + 40, 0),
              (300, 1000, 1000, 0), (131, 333, 333, 1), (257, 514, 516, 2),
              (rows * bm - 45, (resident // rows + 2) * bn + 8, (resident // rows + 2) * bn + 8, 0)]
    for M, N, ldy, offset in shapes:
        announce(f"tiling {tiling} M={M} N={N} K={K} ldy={ldy} offset={offset}")
        A, A6, meta, W, W6, sw, zp, ws, c = random_product(M, N, K, seed=M + N)
        buf, Y = output_view(M, N, ldy, offset)
        with_acc = N < 2000
        acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV) if with_acc else None
        B.basq_diag_w4a4_gemm_fp6(tiling, meta, K, sw, zp, ws, c, Y, acc, A6, W6)
        want = torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV)
        want_acc = torch.full((M, N), -2, dtype=torch.int32, device=DEV) if with_acc else None
        B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, want, want_acc)
        assert torch.equal(Y.contiguous().view(torch.int16), want.view(torch.int16))
        assert not with_acc or torch.equal(acc, want_acc)
        Y.fill_(-7.0)
        assert bool((buf == -7.0).all()), "wrote outside the output"


@pytest.mark.parametrize("M", [17, 33, 49, 64, 65])
@pytest.mark.parametrize("N,K", [(8193, 2304), (8208, 4096), (12281, 2304), (12289, 2304), (16384, 4096), (16390, 1024), (35, 4096), (61, 384)])
def test_streaming_product_where_waves_share_the_outputs(M, N, K):
    """17 and more tokens: a wave finishes whole tiles, four channels a lane, on either side of the rules that choose waves and
    tiles per workgroup, with channels past the last and rows of outputs at any alignment: the bits of the tiled int8 kernel on
    the same tokens among 129 (exact integer sums, the same epilogue)."""
    announce(f"streaming product M={M} N={N} K={K}")
    A, _, meta, W, _, sw, zp, ws, c = random_product(129, N, K, seed=M + N)
    want = torch.empty((129, N), dtype=torch.bfloat16, device=DEV)
    want_acc = torch.empty((129, N), dtype=torch.int32, device=DEV)
    B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, want, want_acc)
    Wd = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device=DEV)
    B.basq_pack_decode(W, Wd)
    for layout, w in ((B.BASQ_W_CANONICAL, W), (B.BASQ_W_DECODE16, Wd)):
        for ldy, offset in ((N, 0), (N + 3, 1)):
            buf, Y = output_view(M, N, ldy, offset)
            acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
            B.basq_w4a4_gemm(A[:M], meta[:M], w, sw, zp, ws, c, Y, acc, w_layout=layout, N=N)
            assert torch.equal(Y.contiguous().view(torch.int16), want[:M].view(torch.int16))
            assert torch.equal(acc, want_acc[:M])
            Y.fill_(-7.0)
            assert bool((buf == -7.0).all()), "wrote outside the output"


@pytest.mark.parametrize("M,N,K", [(M, N, 1152) for M in (17, 32, 65, 113, 128) for N in (24560, 24561, 24577)] +
                         [(128, N, 2304) for N in (8193, 12289, 16390)] +
                         [(M, N, 256) for M in (17, 48, 128) for N in (1, 2, 3, 4, 5, 7, 18, 31)])
def test_streaming_product_on_the_widest_and_narrowest_outputs(M, N, K):
    """The same around 1535 and 1536 tiles of channels, where four of them go to a workgroup, with all token tiles filled,
    and with fewer channels than a lane finishes."""
    test_streaming_product_where_waves_share_the_outputs(M, N, K)


@pytest.mark.parametrize("K", [384, 512, 640, 1152])
def test_wide_tiles_of_the_group_wise_product(K):
    """The 256 x 192 tiling by name: lengths of the loop over the groups from the depth of the ring on, tiles ragged in both
    directions, fewer tokens and channels than a tile, every kind of output row, more tiles than compute units (a workgroup goes on
    to another tile), constants from very small to very large: the int8 kernel's bits, nothing beside the output.  The tables
    that it reads by direct loads may end anywhere, but its column sums start on a 16-byte boundary; where they do not, or N
    is no multiple of 4, the call takes the other tiling."""
    G = K // 128
    shapes = [(1, 4, 4, 0), (33, 72, 72, 0), (256, 192, 192, 0), (257, 188, 192, 8), (481, 612, 620, 0), (300, 1000, 1001, 1),
              (515, 196, 198, 2), (9 * 256 - 45, 30 * 192 + 8, 30 * 192 + 8, 0)]
    for M, N, ldy, offset in shapes:
        announce(f"wide group-wise tiling M={M} N={N} K={K} ldy={ldy} offset={offset}")
        A, A6, meta, W, W6, sw, zp, _, c = random_product(M, N, K, seed=M + N, groups=G)
        rows = torch.arange(M, device=DEV).repeat_interleave(G)
        meta.view(torch.float32)[:, :2] *= torch.pow(2.0, ((rows * 7) % 5 - 2).float() * 24)[:, None]
        gsum = torch.empty((G, N), dtype=torch.int32, device=DEV)
        B.basq_group_colsums(W, 128, gsum)
        want = torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV)
        B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, gsum, c, want)
        for bias in (c, None):
            buf, Y = output_view(M, N, ldy, offset)
            B.basq_diag_w4a4_gemm_grouped_fp6(1, meta, K, sw, zp, gsum, bias, Y, A6, W6)
            if bias is None:
                B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, gsum, None, want)
            assert torch.equal(Y.contiguous().view(torch.int16), want.view(torch.int16))
            Y.fill_(-7.0)
            assert bool((buf == -7.0).all()), "wrote outside the output"
        shifted = torch.empty(G * N + 1, dtype=torch.int32, device=DEV)[1:].view(G, N).copy_(gsum)
        with pytest.raises(B.BasqError):
            B.basq_diag_w4a4_gemm_grouped_fp6(1, meta, K, sw, zp, shifted, None, want, A6, W6)
        got = torch.empty_like(want)
        B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, shifted, None, got, Aq6=A6, Wq6=W6)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("K", [384, 512, 640])
def test_wide_group_wise_tiles_of_three_to_a_workgroup(K):
    """More than two tiles for each compute unit: a workgroup takes back the first buffer of column constants and hands its ring
    over twice, from each position that the number of groups can leave it in."""
    M, N, G = 17 * 256 - 45, 31 * 192, K // 128
    announce(f"three wide group-wise tiles a workgroup K={K}")
    A, A6, meta, W, W6, sw, zp, _, c = random_product(M, N, K, seed=K, groups=G)
    gsum = torch.empty((G, N), dtype=torch.int32, device=DEV)
    B.basq_group_colsums(W, 128, gsum)
    want, got = (torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, gsum, c, want)
    B.basq_diag_w4a4_gemm_grouped_fp6(1, meta, K, sw, zp, gsum, c, got, A6, W6)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("K", [128, 256, 384, 640, 1152])
def test_small_tiles_of_the_group_wise_product(K):
    """The 128 x 128 tiling by name, which large products no longer take by themselves: from one group on, ragged tiles, odd rows,
    more tiles than are in flight at once."""
    G = K // 128
    for M, N, ldy, offset in [(1, 1, 1, 0), (33, 72, 72, 0), (128, 128, 128, 0), (129, 127, 130, 1), (481, 612, 620, 0), (300, 1001, 1001, 3),
                              (9 * 256 - 45, 30 * 192 + 8, 30 * 192 + 8, 0)]:
        announce(f"small group-wise tiling M={M} N={N} K={K} ldy={ldy} offset={offset}")
        A, A6, meta, W, W6, sw, zp, _, c = random_product(M, N, K, seed=M + N, groups=G)
        gsum = torch.empty((G, N), dtype=torch.int32, device=DEV)
        B.basq_group_colsums(W, 128, gsum)
        want = torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV)
        B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, gsum, c, want)
        buf, Y = output_view(M, N, ldy, offset)
        B.basq_diag_w4a4_gemm_grouped_fp6(0, meta, K, sw, zp, gsum, c, Y, A6, W6)
        assert torch.equal(Y.contiguous().view(torch.int16), want.view(torch.int16))
        Y.fill_(-7.0)
        assert bool((buf == -7.0).all()), "wrote outside the output"


def test_group_wise_products_on_either_tiling():
    """Shapes on both sides of the rule that chooses between the tilings, through the public call."""
    chosen = set()
    for M, N, K in [(256, 2048, 1024), (1024, 12288, 1024), (1020, 12292, 4096), (1020, 12290, 4096), (3345, 2720, 2048)]:
        announce(f"group-wise product M={M} N={N} K={K}")
        chosen.add(B.basq_diag_grouped_tiling(M, K, N))
        A, A6, meta, W, W6, sw, zp, _, c = random_product(M, N, K, seed=M + N, groups=K // 128)
        gsum = torch.empty((K // 128, N), dtype=torch.int32, device=DEV)
        B.basq_group_colsums(W, 128, gsum)
        got = []
        for forms in ({"Aq6": A6, "Wq6": W6}, {}):
            Y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
            B.basq_w4a4_gemm_grouped(A, meta, 128, W, sw, zp, gsum, c, Y, **forms)
            got.append(Y.view(torch.int16))
        assert torch.equal(*got)
    assert chosen == {0, 1}


@pytest.mark.parametrize("steps", [8, 9, 10, 11, 12, 13])
@pytest.mark.parametrize("tiling", range(B.FP6_TILINGS))
def test_fp6_tiles_of_every_number_of_steps_around_the_ring(tiling, steps):
    """A tile's first steps reckon their ring stage, the others have it fixed in rounds of as many as there are stages: every remainder
    of the rounds, at least one of them, and more tiles than are resident, so that a workgroup begins anew where the tile in front
    has left the ring.  Exact sums: the bits of the kernels without the fp6 operands."""
    bm, bn, _ = FP6_TILES[tiling]
    K = 128 * steps
    for M, N in [(bm + 3, bn + 8), (9 * bm - 45, (30 if bn > 128 else 100) * bn + 8)]:
        announce(f"tiling {tiling} steps={steps} M={M} N={N}")
        A, A6, meta, W, W6, sw, zp, ws, c = random_product(M, N, K, seed=steps)
        Y, want = (torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
        B.basq_diag_w4a4_gemm_fp6(tiling, meta, K, sw, zp, ws, c, Y, None, A6, W6)
        B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, want)
        assert torch.equal(Y.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("K", [256, 384, 1024])
@pytest.mark.parametrize("with_bias", [True, False])
def test_fp6_three_of_the_largest_tiles_to_a_workgroup(K, with_bias):
    """256 x 256 tiles keep their constants in one of two places in turn, written while the other is read: three tiles to most workgroups
    and two to the others, ragged on either side, and a reader of every constant."""
    M, N = 256 * 25 - 3, 256 * 23 - 40                          # 575 tiles on 256 workgroups
    announce(f"three tiles M={M} N={N} K={K} bias={with_bias}")
    A, A6, meta, W, W6, sw, zp, ws, c = random_product(M, N, K, seed=K)
    c = c if with_bias else None
    Y, want = (torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    B.basq_diag_w4a4_gemm_fp6(0, meta, K, sw, zp, ws, c, Y, None, A6, W6)
    B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, want)
    assert torch.equal(Y.view(torch.int16), want.view(torch.int16))


SPLIT_TILES = [(64, 64), (96, 64), (128, 64), (128, 128), (96, 96), (160, 96)]


@pytest.mark.parametrize("K", [128, 256, 384, 640, 896, 1024, 2176])
@pytest.mark.parametrize("tiling", range(B.FP6_SPLIT_TILINGS))
def test_every_split_tiling_of_the_fp6_product(tiling, K):
    """The tilings in which two groups of waves share a tile's channels, by name: one chunk (the first group has none), odd and
    even numbers of them around the depth of a group's ring, ragged tiles, every kind of output row, more tiles than compute
    units: the bits of the kernels without the fp6 operands (exact sums, the same epilogue), nothing beside the output."""
    bm, bn = SPLIT_TILES[tiling]
    shapes = [(1, 1, 1, 0), (33, 72, 72, 0), (bm, bn, bn, 0), (bm + 1, bn - 1, bn, 8), (2 * bm - 31, 3 * bn + 32, 3 * bn + 40, 0),
              (131, 333, 333, 1), (257, 514, 516, 2), (9 * bm - 45, 32 * bn + 8, 32 * bn + 8, 0)]
    for M, N, ldy, offset in shapes:
        announce(f"split tiling {tiling} M={M} N={N} K={K} ldy={ldy} offset={offset}")
        A, A6, meta, W, W6, sw, zp, ws, c = random_product(M, N, K, seed=M + N)
        buf, Y = output_view(M, N, ldy, offset)
        acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
        B.basq_diag_w4a4_gemm_fp6(tiling, meta, K, sw, zp, ws, c, Y, acc, A6, W6, split=True)
        want = torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV)
        want_acc = torch.full((M, N), -2, dtype=torch.int32, device=DEV)
        B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, want, want_acc)
        assert torch.equal(Y.contiguous().view(torch.int16), want.view(torch.int16))
        assert torch.equal(acc, want_acc)
        Y.fill_(-7.0)
        assert bool((buf == -7.0).all()), "wrote outside the output"


@pytest.mark.parametrize("M,K,rot,N,product", [
    (61, 4096, 4096, 12288, "fp6"), (46, 4096, 4096, 12288, "stream"), (47, 4096, 4096, 12288, "fp6"),    # the rule's edge
    (61, 4096, 4096, 8192, "stream"), (42, 4096, 4096, 8208, "fp6"), (39, 1024, 1024, 12288, "fp6"),
    (60, 1024, 256, 12296, "fp6"), (64, 896, 128, 28672, "layer streams"),
    (65, 4096, 4096, 200, "fp6"), (128, 8192, 8192, 72, "fp6"), (100, 2048, 2048, 333, "fp6"), (96, 1536, 512, 136, "fp6"),
    (65, 640, 128, 200, "layer streams"), (128, 896, 128, 333, "layer streams"), (128, 14336, 14336, 40, "fp6"),
    (129, 640, 128, 200, "fp6"), (129, 4096, 4096, 72, "fp6")])
def test_layer_with_both_weight_forms(M, K, rot, N, product):
    """The one-call layer with streaming-layout and fp6 weights, the way a serving program keeps them, over the token counts
    at which either product may take it and with quantisers that write the fp6 form themselves and one that does not ("layer
    streams": the fp6 product would take the codes, but only from a launch of its own): the bits of the layer without the
    fp6 weights.  The workspace is poisoned, so a product that reads codes which were left out shows."""
    announce(f"both weight forms M={M} K={K} rot={rot} N={N}: {product}")
    assert (B.basq_diag_fp6_tiling(M, K, N) >= 0) == (product != "stream")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=True, with_scale=True)
    gen = torch.Generator(device=DEV).manual_seed(N)
    W = (torch.randn((N, K), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    Wq, sw, zp, ws = B.alloc_weight_buffers(N, K)
    B.basq_quantize_weights(W, Wq, sw, zp, ws)
    c, W6 = torch.empty(N, device=DEV), B.alloc_fp6_buffer(N, K)
    B.basq_prepare_weights(Wq, sw, zp, bias, None, ws, c, W6)
    Wd = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device=DEV)
    B.basq_pack_decode(Wq, Wd)
    work = torch.empty(B.basq_workspace_bytes(M, K, N), dtype=torch.uint8, device=DEV)

    def layer(poison, w6, w=Wd, layout=B.BASQ_W_DECODE16):
        work.fill_(poison)
        Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        B.basq_linear_fused(X, rot, bias, sa, 0.9, 0.9, w, sw, zp, ws, c, Y, work, Wq6=w6, w_layout=layout, N=N)
        return Y.view(torch.int16)

    want = layer(0, None, Wq, B.BASQ_W_CANONICAL)
    assert torch.equal(layer(0x5A, W6), want) and torch.equal(layer(0xFF, W6), want)
    if M <= B.STREAM_MAX_TOKENS:
        assert torch.equal(layer(0xFF, None), want)


@pytest.mark.parametrize("M,N,K,with_acc,at_most", [(1021, 32001, 4096, False, 2.0), (2048, 4096, 4096, True, 2.5),
                                                    (33204, 14216, 256, False, 1.6)])
def test_fp6_product_is_not_slow_on_odd_rows_or_with_the_accumulators(M, N, K, with_acc, at_most):
    """Against the same product into rows of whole 128-byte lines without the dump.  Stores of two bytes into 32 different
    rows made it 3.0 and 5.4 times as long, non-temporal stores of lines that two rows share 1.9 times; as built at most 1.35
    times.  The bound is about halfway and the quickest of several runs is taken."""
    reps = 8
    announce(f"time of odd rows M={M} N={N} K={K} acc={with_acc}")

    def quickest(n, acc):
        A, A6, meta, W, W6, sw, zp, ws, c = random_product(M, n, K, seed=n)
        Y = torch.empty((M, n), dtype=torch.bfloat16, device=DEV)
        dump = torch.empty((M, n), dtype=torch.int32, device=DEV) if acc else None
        best = float("inf")
        for _ in range(5):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, Y, dump, Aq6=A6, Wq6=W6)
            torch.cuda._sleep(400000)                       # the launches below queue up behind it
            begin.record()
            for _ in range(reps):
                B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, c, Y, dump, Aq6=A6, Wq6=W6)
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end) / reps)
        return best

    even = quickest(N // 64 * 64, False)
    odd = quickest(N, with_acc)
    announce(f"  {1000 * odd:.1f} us against {1000 * even:.1f} us")
    assert odd <= at_most * even


@pytest.mark.parametrize("K,rot,M,with_scale", [(512, 128, 8192, False), (512, 128, 8197, False), (2048, 512, 8229, True),
                                                (11008, 256, 6096, True), (11008, 256, 6097, True)])
def test_fp6_form_of_blockwise_codes_where_its_writer_changes(K, rot, M, with_scale):
    """Blockwise rotations with both forms of the codes on both sides of the size from which a second launch repacks them:
    the fp6 form is that of the codes, and codes and records are those of the call without it."""
    announce(f"fp6 form of blockwise codes K={K} rot={rot} M={M} scale={with_scale}")
    X, bias, sa = gpu_inputs(M, K, seed=K + M, with_bias=True, with_scale=with_scale)
    for f in reversed([0, M - N_SPECIAL]):
        plant_degenerate_rows(X, f)
    Aq, meta, Aq2, meta2 = (torch.full(s, 0x5E, dtype=t, device=DEV) for s, t in 2 * [((M, K // 2), torch.uint8), ((M, 4), torch.int32)])
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, rot, bias, sa, 0.9, 0.95, Aq, meta, Aq6=A6)
    B.basq_rotate_quant(X, rot, bias, sa, 0.9, 0.95, Aq2, meta2)
    assert torch.equal(Aq, Aq2) and torch.equal(meta, meta2)
    check_fp6_copy(Aq, A6, K, row_blocks=[0, (M // 32) - 1, M // 32])


@pytest.mark.parametrize("M,with_rot", [(16383, True), (16384, True), (32767, False), (32768, False)])
def test_fp6_form_of_groupwise_codes_where_its_writer_changes(M, with_rot):
    """Full rotation with groups of 128 on both sides of the token counts from which a second launch repacks the codes: the
    fp6 form is that of the codes, and codes, records and rotation are those of the call without it."""
    K = 4096
    announce(f"fp6 form of groups M={M} rotation out={with_rot}")
    X, bias, _ = gpu_inputs(M, K, seed=M, with_bias=True, with_scale=False)
    got = []
    for a6 in (B.alloc_fp6_buffer(M, K, DEV), None):
        Aq = torch.full((M, K // 2), 0x5E, dtype=torch.uint8, device=DEV)
        meta = torch.full((M * (K // 128), 4), 0x5E, dtype=torch.int32, device=DEV)
        r = torch.empty((M, K), device=DEV) if with_rot else None
        B.basq_rotate_quant(X, K, bias, None, 0.9, 0.95, Aq, meta, r, Aq6=a6, group_size=128)
        got.append((Aq, meta, r, a6))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert not with_rot or torch.equal(got[0][2], got[1][2])
    check_fp6_copy(got[0][0], got[0][3], K, row_blocks=[0, (M // 32) - 1])


@pytest.mark.parametrize("kind", ["ordinary", "cancelling", "wide exponents", "tiny", "large"])
@pytest.mark.parametrize("K", [128, 384, 1024])
def test_group_sums_bit_for_bit(K, kind):
    """The group-wise fp6 kernels keep F / 64 and take z * colsum by a matrix instruction; the int8 kernel keeps F by fp32
    multiply-adds.  On either tiling of the fp6 product (the large one from three groups on) all 24 bits of F must agree: with unit weight scales, no zero points and out_bias = -(what was read so far)
    three calls bring F out in pieces of eight bits (each difference is exact: what is subtracted is the rounded sum)."""
    announce(f"group sums K={K} {kind}")
    M, N, G = 6, 1500, K // 128
    A, A6, meta, W, W6, _, _, _, _ = random_product(M, N, K, seed=K + len(kind), groups=G)
    gen = torch.Generator(device=DEV).manual_seed(K)
    rand = lambda: torch.rand(M * G, device=DEV, generator=gen)
    scale, lo = rand() + 0.1, -rand()
    if kind == "cancelling":                                    # products of some 10^4 against bounds of the other sign
        lo = -scale * (7.5 + 0.01 * rand())
    elif kind == "wide exponents":
        scale, lo = torch.exp2(40 * rand() - 20), torch.exp2(40 * rand() - 20) * (rand() - 0.5).sign()
    elif kind != "ordinary":
        f = 1e-30 if kind == "tiny" else 1e30
        scale, lo = scale * f, lo * f
    meta.view(torch.float32)[:, 0], meta.view(torch.float32)[:, 1] = scale, lo
    gsum = torch.empty((G, N), dtype=torch.int32, device=DEV)
    B.basq_group_colsums(W, 128, gsum)
    one, zero = torch.ones(N, dtype=torch.bfloat16, device=DEV), torch.zeros(N, dtype=torch.bfloat16, device=DEV)
    for m in range(M):
        got = []
        a6, mt = B.alloc_fp6_buffer(1, K), meta[m * G:(m + 1) * G]
        B.basq_pack_fp6(A[m:m + 1], a6)
        # the int8 kernel, the call with the fp6 forms, which takes the small tiles for one token, and the large ones by name
        for tiling in (None, 0, 1) if G >= 3 else (None, 0):
            read = torch.zeros(N, device=DEV)
            pieces = []
            for _ in range(3):
                Y = torch.empty((1, N), dtype=torch.bfloat16, device=DEV)
                if tiling == 1:
                    B.basq_diag_w4a4_gemm_grouped_fp6(1, mt, K, one, zero, gsum, -read, Y, a6, W6)
                else:
                    forms = {} if tiling is None else dict(Aq6=a6, Wq6=W6)
                    B.basq_w4a4_gemm_grouped(A[m:m + 1], mt, 128, W, one, zero, gsum, -read, Y, **forms)
                pieces.append(Y[0].view(torch.int16).clone())
                read = read + Y[0].float()
            got.append(torch.stack(pieces))
        for tiling, pieces in enumerate(got[1:]):
            assert torch.equal(got[0], pieces), f"token {m}, tiling {tiling}: {int((got[0] != pieces).sum())} pieces differ"


@pytest.mark.parametrize("K,M", [(8192, 2049), (8192, 2344), (8192, 3999), (8192, 5000), (4096, 8192 + 8), (4096, 9000),
                                 (4096, 33100), (8192, 33100)])
def test_fp6_form_of_codes_in_a_partly_filled_last_round(K, M):
    """The one-wave kernel with a last round of tokens that only some of its workgroups have: every token's codes and records
    are those of the call without the fp6 form, and the fp6 form, its ragged last block included, is that of the codes."""
    announce(f"last round K={K} M={M}")
    X, bias, _ = gpu_inputs(M, K, seed=K + M, with_bias=True, with_scale=False)
    Aq, meta, Aq2, meta2 = (torch.full(s, 0x5E, dtype=t, device=DEV) for s, t in 2 * [((M, K // 2), torch.uint8), ((M, 4), torch.int32)])
    A6 = B.alloc_fp6_buffer(M, K, DEV)
    B.basq_rotate_quant(X, K, bias, None, 0.9, 0.95, Aq, meta, Aq6=A6)
    B.basq_rotate_quant(X, K, bias, None, 0.9, 0.95, Aq2, meta2)
    assert torch.equal(Aq, Aq2) and torch.equal(meta, meta2)
    check_fp6_copy(Aq, A6, K, row_blocks=[0, (M // 32) - 1])
    if M % 32:                                              # the rows of the last, ragged block: through the product with unit weights
        N = 32
        W = torch.full((N, K // 2), 0x11, dtype=torch.uint8, device=DEV)
        W6 = B.alloc_fp6_buffer(N, K, DEV)
        B.basq_pack_fp6(W, W6)
        one, zero = torch.ones(N, dtype=torch.bfloat16, device=DEV), torch.zeros(N, dtype=torch.bfloat16, device=DEV)
        acc = torch.full((M, N), -1, dtype=torch.int32, device=DEV)
        Y = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        B.basq_w4a4_gemm(Aq, meta, W, one, zero, torch.zeros(N, device=DEV), None, Y, acc, Aq6=A6, Wq6=W6)
        assert torch.equal(acc, meta[:, 2:3].expand(M, N)), "row sums of the fp6 form"


@pytest.mark.parametrize("K", [512, 1024, 2048])
def test_small_tokens_in_one_launch(K):
    """The one-launch layer of few small tokens against the two calls (the quantiser, then the product on canonical weights): four tokens
    and 64 channels to a workgroup, so token and channel counts around multiples of these, up to the most that it takes and one
    beyond; with and without b^c, s^a and the layer bias, rows of every alignment, tokens of a wider matrix, dead and NaN tokens."""
    gen = torch.Generator(device=DEV).manual_seed(K)
    rand = lambda *shape: torch.rand(*shape, device=DEV, generator=gen)
    most = (256 if K == 2048 else 512) * 64
    for M, N, ldy, offset, vectors in [(1, 1, 1, 0, 3), (1, 16, 17, 1, 0), (3, 15, 15, 3, 1), (4, 64, 64, 0, 2), (5, 63, 68, 4, 3), (7, 65, 66, 2, 0), (64, 1000, 1000, 0, 3),
                                       (33, 130, 132, 0, 1), (128, 200, 201, 0, 2), (127, 77, 80, 8, 3), (4, most, most, 0, 1), (4, most + 1, most + 1, 0, 3)]:
        announce(f"small tokens in one launch M={M} N={N} K={K} ldy={ldy} offset={offset} vectors={vectors}")
        _, _, _, W, W6, sw, zp, ws, c = random_product(M, N, K, seed=M + N)
        wide = torch.randn((M, K + 24), device=DEV, generator=gen).to(torch.bfloat16)
        if M > 3:
            wide[1] = 0
            wide[M - 1, 5] = float("nan")
            wide[2, 7] = float("inf")
        X = wide[:, :K]
        bias = rand(K) - 0.5 if vectors & 1 else None
        scale = rand(K) + 0.5 if vectors & 2 else None
        out_bias = c if vectors & 1 else None
        Wd = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device=DEV)
        B.basq_pack_decode(W, Wd)
        A, meta = B.alloc_activation_buffers(M, K, DEV)
        want = torch.full((M, N), -7.0, dtype=torch.bfloat16, device=DEV)
        B.basq_rotate_quant(X, K, bias, scale, 0.9, 0.8, A, meta)
        B.basq_w4a4_gemm(A, meta, W, sw, zp, ws, out_bias, want)
        workspace = torch.empty(B.basq_workspace_bytes(M, K, N), dtype=torch.uint8, device=DEV)
        for six in (None, W6):
            buf, Y = output_view(M, N, ldy, offset)
            assert B.basq_diag_one_launch(X, K, bias, scale, Y, B.BASQ_W_DECODE16) == (N <= most)
            B.basq_linear_fused(X, K, bias, scale, 0.9, 0.8, Wd, sw, zp, ws, out_bias, Y, workspace, Wq6=six, w_layout=B.BASQ_W_DECODE16, N=N)
            got = Y.contiguous()
            assert torch.equal(got.isnan(), want.isnan())
            assert torch.equal(got.nan_to_num(0.0).view(torch.int16), want.nan_to_num(0.0).view(torch.int16))
            Y.fill_(-7.0)
            assert bool((buf == -7.0).all()), "wrote outside the output"


@pytest.mark.parametrize("M,K,shift", [(64, 1024, 0), (128, 512, 0), (31, 1024, 8), (16, 2048, 0), (1, 4096, 0), (4, 4096, 0), (3, 4096, 8)])
def test_small_layers_in_place(M, K, shift):
    """Outputs over the layer's own tokens, or over the tokens shifted by some channels: as with outputs elsewhere."""
    gen = torch.Generator(device=DEV).manual_seed(M + K)
    _, _, _, W, _, sw, zp, ws, c = random_product(M, K, K, seed=M + K)
    Wd = torch.empty(B.basq_decode_bytes(K, K), dtype=torch.uint8, device=DEV)
    B.basq_pack_decode(W, Wd)
    X = torch.randn((M, K), device=DEV, generator=gen).to(torch.bfloat16)
    workspace = torch.empty(B.basq_workspace_bytes(M, K, K), dtype=torch.uint8, device=DEV)
    layer = lambda x, y: B.basq_linear_fused(x, K, None, None, 0.9, 0.8, Wd, sw, zp, ws, c, y, workspace, w_layout=B.BASQ_W_DECODE16, N=K)
    want = torch.empty_like(X)
    assert B.basq_diag_one_launch(X, K, None, None, want, B.BASQ_W_DECODE16)
    layer(X, want)
    for _ in range(20):
        buf = torch.zeros(M * K + shift, dtype=torch.bfloat16, device=DEV)
        x, y = buf[shift:].view(M, K), buf[:M * K].view(M, K)
        x.copy_(X)
        assert not B.basq_diag_one_launch(x, K, None, None, y, B.BASQ_W_DECODE16)
        layer(x, y)
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("over", ["bias", "act_scale"])
@pytest.mark.parametrize("K,N", [(512, 1024), (1024, 2048), (2048, 4096), (4096, 4096)])
def test_small_layers_over_a_channel_vector(K, N, over):
    """Outputs over b^c or s^a, which have been read when the first output is written: as with outputs elsewhere."""
    gen = torch.Generator(device=DEV).manual_seed(K)
    _, _, _, W, _, sw, zp, ws, c = random_product(1, N, K, seed=K)
    Wd = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device=DEV)
    B.basq_pack_decode(W, Wd)
    X = torch.randn((1, K), device=DEV, generator=gen).to(torch.bfloat16)
    vectors = {"bias": torch.rand(K, device=DEV, generator=gen) - 0.5, "act_scale": torch.rand(K, device=DEV, generator=gen) + 0.5}
    workspace = torch.empty(B.basq_workspace_bytes(1, K, N), dtype=torch.uint8, device=DEV)
    layer = lambda v, y: B.basq_linear_fused(X, K, v["bias"], v["act_scale"], 0.9, 0.8, Wd, sw, zp, ws, c, y, workspace, w_layout=B.BASQ_W_DECODE16, N=N)
    want = torch.empty((1, N), dtype=torch.bfloat16, device=DEV)
    layer(vectors, want)
    for _ in range(20):
        mine = {k: v.clone() for k, v in vectors.items()}
        y = mine[over].view(torch.bfloat16)[:N].view(1, N)
        assert not B.basq_diag_one_launch(X, K, mine["bias"], mine["act_scale"], y, B.BASQ_W_DECODE16)
        layer(mine, y)
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))


def test_fp6_ceiling_loop_multiplies_codes():
    """The loop that the benchmark's fp6 ceiling is measured with: sixteen 16 x 16 x 128 products a wave and round of operands that hold
    codes q as the e2m3 numbers q/8.  The checksums of a wave add up to the products of the operands' column sums, exactly."""
    seed = np.arange(64 * 8, dtype=np.uint64)[:, None] * 32 + np.arange(32, dtype=np.uint64)
    h = seed * 0x9E3779B1 & 0xFFFFFFFF
    h = (h ^ (h >> 15)) * 0x85EBCA77 & 0xFFFFFFFF
    codes = np.zeros(h.shape, dtype=np.int64)
    for bit in range(12, 27):
        codes += (h >> bit & 1).astype(np.int64)
    codes = codes.reshape(4, 16, 2, 4, 32).sum(axis=(1, 3))          # [lane / 16][a or b][channel]: over rows and operands
    total = int((codes[:, 0] * codes[:, 1]).sum())
    for iters in (1, 3):
        out = torch.zeros(512, dtype=torch.float32, device=DEV)
        B.basq_diag_mfma_f6(out, 2, iters)
        waves = out.cpu().double().view(2, 4, 64).sum(-1) * 64
        assert int(waves[0, 0]) == int(waves[1, 0]) == iters * total
