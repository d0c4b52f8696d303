"""The C-ABI library without a GPU: it loads, exports every symbol the header declares, and turns
bad arguments into error codes before anything would be launched."""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle
from paper_2506_15689_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2506_15689_amd import build
        build.build_lib(verbose=False)
    return B.load()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "basq.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(basq_[a-z0-9_]+)\s*\(", header))
    assert {"basq_rotate_quant", "basq_w4a4_gemm", "basq_linear_fused"} <= declared
    for name in declared:
        assert hasattr(lib, name), f"{name} declared in basq.h but not exported"
    assert declared == set(B.EXPORTS)


def test_version_and_error_text(lib):
    assert B.basq_version() >= 100
    rc = lib.basq_rotate_quant(None, 4, 100, 100, 64, None, None, 0.9, 0.9, 4, 0, None, None, None, None, None)
    assert rc == B.BASQ_EINVAL and "multiple of 32" in B.basq_last_error()


@pytest.mark.parametrize("missing", ["_raw_stream", "_raw_device"])
def test_current_stream_without_torchs_undocumented_functions(monkeypatch, missing):
    """The handle of the current stream comes from two functions that torch does not document; without either it is the
    Stream object's, also once the GPU is in use."""
    class Stream:
        cuda_stream = 0x5678

    monkeypatch.setattr(B, "_raw_stream", lambda device: 0x1234)
    monkeypatch.setattr(B, "_raw_device", lambda: 0)
    monkeypatch.setattr(B.torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(B.torch.cuda, "current_stream", lambda: Stream)
    assert B._stream(None) == 0x1234
    monkeypatch.setattr(B, missing, None)
    assert B._stream(None) == 0x5678
    assert B._stream(Stream) == 0x5678


def test_fp6_tilings_by_name(lib):
    """Which tiling a shape takes is known without a GPU; a product by name is refused where it could not run."""
    T = B.basq_diag_fp6_tiling
    assert T(4096, 8192, 28672) == 0 and T(2048, 4096, 12288) == 1 and T(2048, 14336, 4096) == 2
    assert T(1021, 11008, 4096) == 3 and T(260, 11008, 4096) == 4 and T(333, 4096, 4096) == 5
    # few K-steps and four rounds of the largest tiles, and just below
    assert T(1024, 512, 256 * 256) == 0 and T(1024, 512, 256 * 255) != 0 and T(33204, 256, 14216) == 0
    # shapes whose product runs elsewhere
    assert T(32, 4096, 28672) == T(61, 4096, 8192) == T(200, 4096 + 64, 512) == T(200, 32768 + 128, 512) == T(0, 4096, 4096) == -1
    assert T(61, 4096, 12288) >= 0 and T(65, 128, 1) >= 0
    call = lambda t, K=256, a=FAKE, w=FAKE, y=FAKE: lib.basq_diag_w4a4_gemm_fp6(
        t, FAKE, 64, K, 64, FAKE, FAKE, FAKE, None, y, 64, None, a, w, None)
    assert call(-1) == call(B.FP6_TILINGS) == B.BASQ_EINVAL
    assert call(0, a=None) == call(0, w=None) == call(0, y=None) == call(0, K=192) == B.BASQ_EINVAL
    assert call(0, a=ctypes.c_void_p(0x1008)) == B.BASQ_EINVAL
    assert call(0, K=32768 + 128) == B.BASQ_EUNSUPPORTED


def test_fp6_split_tilings_by_name(lib):
    """Which split tiling a shape takes, and that a product by name is refused where it could not run."""
    T = B.basq_diag_fp6_split_tiling
    assert T(333, 4096, 4096) == 1 and T(1021, 11008, 4096) == 3 and T(61, 4096, 12288) == 0
    # many tiles, few K-steps with many rounds, and shapes whose product runs elsewhere
    assert T(4096, 8192, 28672) == T(2048, 4096, 12288) == T(33204, 256, 14216) == T(32, 4096, 28672) == T(0, 4096, 4096) == -1
    call = lambda t, K=256, a=FAKE: lib.basq_diag_w4a4_gemm_fp6_split(
        t, FAKE, 64, K, 64, FAKE, FAKE, FAKE, None, FAKE, 64, None, a, FAKE, None)
    assert call(-1) == call(B.FP6_SPLIT_TILINGS) == call(0, a=None) == call(0, K=192) == B.BASQ_EINVAL
    assert call(0, K=32768 + 128) == B.BASQ_EUNSUPPORTED


def test_grouped_tilings_by_name(lib):
    """Which tiling a group-wise shape takes, and that a product by name is refused where it could not run."""
    T = B.basq_diag_grouped_tiling
    assert T(2048, 4096, 12288) == T(3345, 8192, 2720) == 1
    # odd output widths, rows shorter than the ring, too few tiles, and a second round of them just begun
    assert T(2048, 4096, 12290) == T(2048, 256, 12288) == T(333, 4096, 4096) == T(1775, 4096, 8176) == 0
    # rows of odd lines, where the large tiles have to be the cheaper ones by a margin; the same in rows of whole and half lines
    assert T(279, 1024, 24272) == T(2552, 8192, 10224) == T(1729, 1536, 27280) == 0
    assert T(279, 1024, 24256) == T(279, 1024, 24288) == T(3684, 1024, 3088) == 1
    assert T(0, 4096, 4096) == T(4, 192, 4096) == -1
    # an operand or a table of 4 GiB, which the fp6 form cannot address: the largest that it takes, and one more of each
    assert T(256, 32768, 174752) >= 0 and T(174752, 32768, 256) >= 0
    assert T(256, 32768, 174752 + 32) == T(174752 + 32, 32768, 256) == -1
    call = lambda t, K=512, N=64, a=FAKE, gs=FAKE: lib.basq_diag_w4a4_gemm_grouped_fp6(
        t, FAKE, 64, K, N, FAKE, FAKE, gs, None, FAKE, 64, a, FAKE, None)
    assert call(-1) == call(2) == call(0, a=None) == call(1, gs=None) == call(0, K=192) == B.BASQ_EINVAL
    assert call(1, K=256) == call(1, N=62) == call(1, gs=ctypes.c_void_p(0x1004)) == B.BASQ_EUNSUPPORTED


def test_wide_group_wise_tiling_requests_nothing_outside_its_tables(lib):
    """Blocks, records and sums past the matrix are clamped to its last ones, and what is requested behind a workgroup's last tile
    is dropped, which takes scalar offsets inside the table: one token, few channels and the shortest rows are the tables that
    such an offset leaves first."""
    for K in (384, 512, 1152):
        for M, N in [(1, 4), (1, 64), (1, 200), (2, 4), (33, 60), (257, 188), (300, 388)]:
            assert B.basq_diag_grouped_wide_strays(M, K, N) == 0, (M, K, N)
    assert [B.basq_diag_grouped_wide_strays(*s) for s in [(0, 384, 4), (1, 256, 4), (1, 384, 6), (1, 400, 4)]] == [-1] * 4


def test_blockwise_rotation_requests_no_channel_past_the_token(lib):
    """b^c and s^a have K values each; what is requested for the missing half of a last piece, and for pieces that do not
    exist, must lie inside them too, down to the smallest token (K = 256, half a piece)."""
    for K in range(256, 16384 + 1, 256):
        assert B.basq_diag_block_vector_channels(K) == K
    assert [lib.basq_diag_block_vector_channels(K) for K in (0, 128, 384, 16640)] == [B.BASQ_EINVAL] * 4


def one_launch(lib, M, K, N, rot=None, x=0x10000000, y=0x40000000, bias=None, scale=None, layout=B.BASQ_W_DECODE16, ldx=None, ldy=None):
    return lib.basq_diag_one_launch(x, M, K, ldx or K, rot or K, bias, scale, N, layout, y, ldy or N)


def test_layers_in_one_launch(lib):
    """The rules by size, each on either side of its line."""
    one = lambda *shape, **kw: one_launch(lib, *shape, **kw)
    for K in (4096, 8192):
        assert [one(1, K, 1), one(4, K, 4096), one(5, K, 4096), one(4, K, 4097), one(0, K, 64)] == [1, 1, 0, 0, 0]
    for K in (512, 1024):
        assert [one(128, K, 1024), one(128, K, 1025), one(129, K, 64), one(4, K, 32768), one(5, K, 32768), one(4, K, 32769)] == [1, 0, 0, 1, 0, 0]
    assert [one(64, 2048, 1024), one(64, 2048, 1025), one(1, 2048, 16384), one(1, 2048, 16385)] == [1, 0, 1, 0]
    assert [one(1, 256, 64), one(1, 14336, 64), one(1, 11008, 64, rot=256), one(1, 1024, 64, rot=512)] == [0] * 4
    assert [one(1, K, 64, layout=B.BASQ_W_CANONICAL) for K in (1024, 4096)] == [0, 0]
    assert one(1, 1024, 64, ldx=1020) == one(1, 1024, 64, ldy=63) == one(1, 1024, 64, y=None) == B.BASQ_EINVAL


@pytest.mark.parametrize("M,K,N", [(1, 4096, 4096), (4, 4096, 1000), (2, 8192, 4096), (1, 512, 512), (64, 1024, 1024), (16, 2048, 2048)])
def test_outputs_over_a_layers_inputs_take_two_launches(lib, M, K, N):
    """Workgroups of a one-launch layer read all of their tokens, b^c and s^a, in no order against the stores of the others: outputs over
    any byte of these, by whole buffers and by the last or first byte that they share."""
    x, ldx, ldy = 0x40000000, K + 16, N + 24
    x_bytes, y_bytes, v_bytes = 2 * ((M - 1) * ldx + K), 2 * ((M - 1) * ldy + N), 4 * K
    one = lambda y, **kw: one_launch(lib, M, K, N, x=x, y=y, ldx=ldx, ldy=ldy, **kw)
    assert [one(x), one(x + x_bytes - 2), one(x - y_bytes + 2), one(x + 2 * K - 2)] == [0] * 4
    assert [one(x + x_bytes), one(x - y_bytes)] == [1, 1]
    # against the bytes themselves: tokens and outputs that share rows of one matrix, and rows of different lengths
    for ldx, ldy, shift in [(K + N + 8, K + N + 8, 2 * d) for d in (0, 1, 8, K - 1, K, K + 1, K + 8, K + 9)] + [(K + N + 8, ldy, 2 * d) for d in (K, K + 8, K + N + 8 + K)]:
        bytes_of = lambda start, ld, n: {start + 2 * (m * ld + i) for m in range(M) for i in range(n)}
        shared = bytes_of(0, ldx, K) & bytes_of(shift, ldy, N)
        assert one_launch(lib, M, K, N, x=x, y=x + shift, ldx=ldx, ldy=ldy) == (not shared), (ldx, ldy, shift)
    for vector in ("bias", "scale"):
        at = {vector: 0x70000000}
        assert [one(0x70000000, **at), one(0x70000000 + v_bytes - 2, **at), one(0x70000000 - y_bytes + 2, **at)] == [0] * 3
        assert [one(0x70000000 + v_bytes, **at), one(0x70000000 - y_bytes, **at), one(0x70000000)] == [1] * 3


FAKE = ctypes.c_void_p(0x1000)      # aligned, never dereferenced: validation fails first


@pytest.mark.parametrize("kw,code", [
    (dict(M=-1), B.BASQ_EINVAL),
    (dict(K=0), B.BASQ_EINVAL),
    (dict(K=48), B.BASQ_EINVAL),
    (dict(ldx=1016), B.BASQ_EINVAL),
    (dict(ldx=1028), B.BASQ_EINVAL),
    (dict(rot=1000), B.BASQ_EUNSUPPORTED),
    (dict(rot=28), B.BASQ_EUNSUPPORTED),
    (dict(rot=768), B.BASQ_EUNSUPPORTED),
    (dict(K=1024, rot=512 * 3), B.BASQ_EUNSUPPORTED),
    (dict(K=1024 + 512, ldx=2048, rot=1024), B.BASQ_EINVAL),
    (dict(bits=8), B.BASQ_EUNSUPPORTED),
    (dict(bits=3), B.BASQ_EUNSUPPORTED),
    (dict(group=100), B.BASQ_EINVAL),                                 # not a multiple of 32
    (dict(group=96), B.BASQ_EINVAL),                                  # does not divide K
    (dict(K=1056, ldx=1056, rot=32, group=96, Aq6=FAKE), B.BASQ_EINVAL),   # fp6 form with groups: still K % 128 == 0
    (dict(clip_lo=0.0), B.BASQ_EINVAL),
    (dict(clip_hi=1.5), B.BASQ_EINVAL),
    (dict(clip_lo=float("nan")), B.BASQ_EINVAL),
    (dict(X=None), B.BASQ_EINVAL),
    (dict(X=ctypes.c_void_p(0x1008)), B.BASQ_EINVAL),
    (dict(Aq=None), B.BASQ_EINVAL),
    (dict(Aq=None, Aq6=FAKE), B.BASQ_EUNSUPPORTED),                   # the fp6 form alone: only where the quantiser writes it itself
    (dict(Aq=None, Aq6=FAKE, K=4096, ldx=4096, rot=4096, group=128), B.BASQ_EUNSUPPORTED),
    (dict(meta=None), B.BASQ_EINVAL),
    (dict(K=65536, ldx=65536, rot=65536), B.BASQ_EUNSUPPORTED),
    (dict(K=1056, ldx=1056, rot=32, Aq6=FAKE), B.BASQ_EINVAL),        # fp6 form needs K % 128 == 0
    (dict(Aq6=ctypes.c_void_p(0x1008)), B.BASQ_EINVAL),
    (dict(bias=ctypes.c_void_p(0x1004)), B.BASQ_EINVAL),              # b^c and s^a are read four channels at a time
    (dict(sa=ctypes.c_void_p(0x1008)), B.BASQ_EINVAL),
])
def test_rotate_quant_rejects_bad_arguments(lib, kw, code):
    a = dict(X=FAKE, M=4, K=1024, ldx=1024, rot=1024, bias=None, sa=None, clip_lo=0.9, clip_hi=0.9, bits=4,
             group=0, Aq=FAKE, meta=FAKE, rot_out=None, Aq6=None)
    a.update(kw)
    rc = lib.basq_rotate_quant(a["X"], a["M"], a["K"], a["ldx"], a["rot"], a["bias"], a["sa"], a["clip_lo"],
                               a["clip_hi"], a["bits"], a["group"], a["Aq"], a["meta"], a["rot_out"], a["Aq6"], None)
    assert rc == code, B.basq_last_error()
    assert B.basq_last_error() != ""


@pytest.mark.parametrize("kw,code", [
    (dict(M=-2), B.BASQ_EINVAL),
    (dict(K=100), B.BASQ_EINVAL),
    (dict(N=0), B.BASQ_EINVAL),
    (dict(layout=7), B.BASQ_EUNSUPPORTED),
    (dict(ldy=100), B.BASQ_EINVAL),
    (dict(Wq=None), B.BASQ_EINVAL),
    (dict(w_scale=None), B.BASQ_EINVAL),
    (dict(w_zero=None), B.BASQ_EINVAL),
    (dict(w_sum=None), B.BASQ_EINVAL),
    (dict(Aq=None), B.BASQ_EINVAL),
    (dict(Y=None), B.BASQ_EINVAL),
    (dict(Aq=ctypes.c_void_p(0x1004)), B.BASQ_EINVAL),
    (dict(Y=ctypes.c_void_p(0x1001)), B.BASQ_EINVAL),
    (dict(Aq6=FAKE), B.BASQ_EINVAL),                                  # fp6 operands: both or neither
    (dict(Wq6=FAKE), B.BASQ_EINVAL),
    (dict(K=1056, Aq6=FAKE, Wq6=FAKE), B.BASQ_EINVAL),
    (dict(Aq6=FAKE, Wq6=ctypes.c_void_p(0x1004)), B.BASQ_EINVAL),
])
def test_gemm_rejects_bad_arguments(lib, kw, code):
    a = dict(Aq=FAKE, meta=FAKE, M=8, K=1024, Wq=FAKE, N=256, layout=0, w_scale=FAKE, w_zero=FAKE, w_sum=FAKE,
             out_bias=None, Y=FAKE, ldy=256, acc=None, Aq6=None, Wq6=None)
    a.update(kw)
    rc = lib.basq_w4a4_gemm(a["Aq"], a["meta"], a["M"], a["K"], a["Wq"], a["N"], a["layout"], a["w_scale"],
                            a["w_zero"], a["w_sum"], a["out_bias"], a["Y"], a["ldy"], a["acc"], a["Aq6"], a["Wq6"],
                            None)
    assert rc == code, B.basq_last_error()


def test_fused_call_checks_workspace(lib):
    need = B.basq_workspace_bytes(64, 1024, 256)
    assert need >= 64 * 512 + 64 * 16 and need % 256 == 0
    assert need >= 64 * 512 + 64 * 16 + B.basq_fp6_bytes(64, 1024)
    args = [FAKE, 64, 1024, 1024, 1024, None, None, 0.9, 0.9, 4, 0, FAKE, 256, 0, FAKE, FAKE, FAKE, None, FAKE, 256,
            None]
    assert lib.basq_linear_fused(*args, ctypes.c_void_p(0x2000), need - 1, None) == B.BASQ_EWORKSPACE
    assert "workspace too small" in B.basq_last_error()
    assert lib.basq_linear_fused(*args, None, need, None) == B.BASQ_EINVAL
    assert lib.basq_linear_fused(*args, ctypes.c_void_p(0x2010), need, None) == B.BASQ_EINVAL
    odd = list(args)
    odd[2] = odd[3] = 1056; odd[4] = 32                                     # fp6 weights need K % 128 == 0
    odd[-1] = FAKE
    assert lib.basq_linear_fused(*odd, ctypes.c_void_p(0x2000), 1 << 20, None) == B.BASQ_EINVAL


def test_static_workspace_call_rejects_what_does_not_fit(lib):
    """basq_linear_fused_static: shapes whose codes and records exceed the library's own workspace fail on the
    host, before the workspace is even looked up (so this runs without a GPU)."""
    args = lambda M, K: [FAKE, M, K, K, K, None, None, 0.9, 0.9, 4, 0, FAKE, 256, 0, FAKE, FAKE, FAKE, None, FAKE, 256,
                         None, None]
    assert B.basq_workspace_bytes(4096, 8192, 256) > B.STATIC_WORKSPACE_BYTES
    assert lib.basq_linear_fused_static(*args(4096, 8192)) == B.BASQ_EWORKSPACE
    assert "workspace" in B.basq_last_error()
    assert lib.basq_linear_fused_static(*args(-1, 1024)) == B.BASQ_EINVAL
    assert lib.basq_linear_fused_static(*args(8, 1000)) == B.BASQ_EINVAL
    header = open(os.path.join(ROOT, "include", "basq.h")).read()
    m = re.search(r"#define\s+BASQ_STATIC_WORKSPACE_BYTES\s+\((\d+)u\s*<<\s*(\d+)\)", header)
    assert m and int(m.group(1)) << int(m.group(2)) == B.STATIC_WORKSPACE_BYTES


def test_fp6_form_sizes_and_argument_checks(lib):
    assert B.basq_fp6_bytes(64, 1024) == 64 * 768
    assert B.basq_fp6_bytes(33, 256) == 64 * 192                      # whole 32-row blocks
    assert B.basq_fp6_bytes(5, 100) == 0 and B.basq_fp6_bytes(-1, 128) == 0
    assert lib.basq_pack_fp6(FAKE, 8, 100, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_pack_fp6(None, 8, 128, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_pack_fp6(FAKE, 8, 128, ctypes.c_void_p(0x1008), None) == B.BASQ_EINVAL
    assert lib.basq_pack_fp6(None, 0, 128, None, None) == 0


def test_decode_layout_sizes_and_argument_checks(lib):
    assert B.basq_decode_bytes(4096, 4096) == 4096 * 2048
    assert B.basq_decode_bytes(17, 256) == 32 * 128                        # whole 16-row blocks
    assert B.basq_decode_bytes(16, 96) == 0 and B.basq_decode_bytes(0, 128) == 0
    assert lib.basq_pack_decode(FAKE, 8, 96, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_pack_decode(None, 8, 128, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_pack_decode(FAKE, 0, 128, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_pack_decode(FAKE, 8, 128, ctypes.c_void_p(0x1008), None) == B.BASQ_EINVAL
    # the streaming layout: K % 128, and more than 128 tokens only with the fp6 operands
    gemm = lambda M, K, layout, a6=None, w6=None: lib.basq_w4a4_gemm(
        FAKE, FAKE, M, K, FAKE, 32, layout, FAKE, FAKE, FAKE, None, FAKE, 32, None, a6, w6, None)
    assert gemm(4, 96, B.BASQ_W_DECODE16) == B.BASQ_EINVAL
    assert gemm(129, 256, B.BASQ_W_DECODE16) == B.BASQ_EUNSUPPORTED
    assert "fp6" in B.basq_last_error()
    assert gemm(4, 256, 2) == B.BASQ_EUNSUPPORTED
    ws = ctypes.c_void_p(0x100000)
    assert lib.basq_linear_fused(FAKE, 129, 256, 256, 256, None, None, 0.9, 0.9, 4, 0, FAKE, 32, B.BASQ_W_DECODE16,
                                 FAKE, FAKE, FAKE, None, FAKE, 32, None, ws, 1 << 30, None) == B.BASQ_EUNSUPPORTED


def test_grouped_gemm_argument_checks(lib):
    call = lambda M, K, G, gs=FAKE, a6=None, w6=None: lib.basq_w4a4_gemm_grouped(
        FAKE, FAKE, M, K, G, FAKE, 32, FAKE, FAKE, gs, None, FAKE, 32, a6, w6, None)
    assert call(4, 256, 64) == B.BASQ_EUNSUPPORTED                     # only groups of 128
    assert call(4, 192, 128) == B.BASQ_EINVAL                          # K % 128
    assert call(4, 256, 128, None) == B.BASQ_EINVAL
    assert call(0, 256, 128) == 0                                      # no tokens: nothing launched
    assert call(4, 256, 128, FAKE, FAKE, None) == B.BASQ_EINVAL        # fp6 operands: both or neither
    assert call(4, 256, 128, FAKE, None, FAKE) == B.BASQ_EINVAL
    assert call(4, 256, 128, FAKE, FAKE, ctypes.c_void_p(0x1008)) == B.BASQ_EINVAL
    assert call(0, 256, 128, FAKE, FAKE, FAKE) == 0
    assert lib.basq_group_colsums(FAKE, 8, 192, 128, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_group_colsums(FAKE, 8, 256, 32, FAKE, None) == B.BASQ_EUNSUPPORTED
    assert lib.basq_group_colsums(None, 8, 256, 128, FAKE, None) == B.BASQ_EINVAL


def test_zero_tokens_is_valid_without_a_launch(lib):
    assert lib.basq_rotate_quant(None, 0, 1024, 1024, 1024, None, None, 0.9, 0.9, 4, 0, None, None, None, None, None) == 0
    assert lib.basq_w4a4_gemm(None, None, 0, 1024, FAKE, 16, 0, FAKE, FAKE, FAKE, None, None, 16, None, None, None, None) == 0


def test_offline_helpers_reject_bad_arguments(lib):
    assert lib.basq_rotate_weights(None, 8, 64, 64, 64, FAKE, FAKE, 1 << 20, None) == B.BASQ_EINVAL
    assert lib.basq_rotate_weights(FAKE, 8, 64, 64, 48, FAKE, FAKE, 1 << 20, None) != 0       # 48 is no Hadamard size
    assert lib.basq_rotate_weights(FAKE, 8, 64, 64, 64, FAKE, FAKE, 8 * 64 * 4 - 1, None) == B.BASQ_EWORKSPACE
    assert lib.basq_rotate_weights(FAKE, 0, 64, 64, 64, FAKE, FAKE, 1 << 20, None) == B.BASQ_EINVAL
    assert lib.basq_quantize_weights(None, 8, 64, 64, FAKE, FAKE, FAKE, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_quantize_weights(FAKE, 8, 64, 32, FAKE, FAKE, FAKE, FAKE, None) == B.BASQ_EINVAL
    assert lib.basq_fused_bias(FAKE, 0, 64, FAKE, FAKE, None, None, FAKE, None) == B.BASQ_EINVAL
    prep = lambda **kw: lib.basq_prepare_weights(*[{**dict(Wq=FAKE, N=8, K=128, ws=FAKE, wz=FAKE, b=None, lb=None, wsum=FAKE,
                                                           ob=FAKE, pre=None), **kw}[k]
                                                   for k in ("Wq", "N", "K", "ws", "wz", "b", "lb", "wsum", "ob", "pre")], None)
    assert prep(N=0) == B.BASQ_EINVAL and prep(K=48) == B.BASQ_EINVAL
    assert prep(Wq=None) == B.BASQ_EINVAL and prep(wsum=None) == B.BASQ_EINVAL and prep(ob=None) == B.BASQ_EINVAL
    assert prep(Wq=ctypes.c_void_p(0x1004)) == B.BASQ_EINVAL
    assert prep(K=96, pre=FAKE) == B.BASQ_EINVAL                       # the fp6 operand form needs K % 128 == 0
    assert prep(pre=ctypes.c_void_p(0x1008)) == B.BASQ_EINVAL
    assert lib.basq_calibrate_bias(FAKE, 16, 1024, 1024, 1024, None, FAKE, FAKE, 16 * 1024 * 4 - 1, None) == B.BASQ_EWORKSPACE
    assert lib.basq_calibrate_bias(FAKE, 0, 1024, 1024, 1024, None, FAKE, FAKE, 1 << 20, None) == B.BASQ_EINVAL
    assert lib.basq_hadamard28(None) == B.BASQ_EINVAL


def test_hadamard28_table_matches_oracle(lib):
    """The rotation for 28 * 2^t channels needs the same sign table on both sides; the library
    builds its own from the Paley construction."""
    np.testing.assert_array_equal(B.basq_hadamard28().numpy(), oracle.hadamard_paley28())
