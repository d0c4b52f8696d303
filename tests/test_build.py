"""How the library is compiled, and what the compiler made of it."""
import os
import re
import struct
import subprocess

import pytest

from paper_2506_15689_amd import build


@pytest.mark.parametrize("knows", [True, False])
def test_an_option_that_the_compiler_does_not_know_is_left_out(tmp_path, monkeypatch, capfd, knows):
    option = build.MFMA_VGPR_FLAGS[-1]
    hipcc = tmp_path / "hipcc"
    refuse = "" if knows else f'case "$*" in *{option}*) exit 1;; esac\n'
    hipcc.write_text(f'#!/bin/sh\n{refuse}echo "$*" >> {tmp_path}/calls\n')
    hipcc.chmod(0o755)
    monkeypatch.setenv("HIPCC", str(hipcc))
    monkeypatch.setattr(build, "BUILD", str(tmp_path))
    for src in sorted(build.MFMA_VGPR_SOURCES):
        assert os.path.dirname(build._compile(src)) == str(tmp_path)
    compiled = [line for line in (tmp_path / "calls").read_text().splitlines() if " -c " in line]
    assert [option in line for line in compiled] == [knows] * len(build.MFMA_VGPR_SOURCES)
    assert ("built without it" in capfd.readouterr().err) == (not knows)


def code_objects():
    """The code objects of the built library."""
    if not os.path.exists(build.LIB):
        build.build_lib(verbose=False)
    with open(build.LIB, "rb") as f:
        blob = f.read()
    magic, found = b"__CLANG_OFFLOAD_BUNDLE__", []
    bundle = blob.find(magic)
    while bundle >= 0:
        (entries,), entry = struct.unpack_from("<Q", blob, bundle + len(magic)), bundle + len(magic) + 8
        for _ in range(entries):
            offset, size, id_length = struct.unpack_from("<QQQ", blob, entry)
            if b"gfx950" in blob[entry + 24:entry + 24 + id_length]:
                found.append(blob[bundle + offset:bundle + offset + size])
            entry += 24 + id_length
        bundle = blob.find(magic, bundle + 1)
    return found


def llvm(tool, *args, stdin=None):
    return subprocess.run([f"/opt/rocm/llvm/bin/{tool}", *args], input=stdin, stdout=subprocess.PIPE, check=True).stdout.decode()


def kernel_resources():
    """Name, spilled vector registers and bytes of scratch a lane of every kernel, from its code object's notes."""
    found = []
    for code in code_objects():
        for kernel in llvm("llvm-readelf", "--notes", "-", stdin=code).split(".agpr_count:")[1:]:
            field = lambda key: re.search(rf"^ *\.{key}: +(\S+)", kernel, re.M).group(1)
            found.append((field("name"), int(field("vgpr_spill_count")), int(field("private_segment_fixed_size"))))
    return found


def test_no_tiling_of_the_fp6_gemm_spills():
    """Its waits count the loads and stores in flight: a spilled register's are among them, and one that is fetched again behind a tile's
    last step is a memory latency with nothing beside it."""
    gemms = [k for k in kernel_resources() if "gemm_w4a4_fp6_kernel" in k[0]]
    assert len(gemms) >= 12
    assert [k for k in gemms if k[1] or k[2]] == []


def test_small_layers_rotate_while_their_weights_are_on_their_way(tmp_path):
    """The one-launch layer of few small tokens requests its weights in front of the rotation: no wait for everything in flight between
    a kernel's first load and its barrier, behind which the weights are first used."""
    kernels = 0
    for code in code_objects():
        if b"linear_small_kernel" not in code:
            continue
        (tmp_path / "code").write_bytes(code)
        for text in re.split(r"^[0-9a-f]+ <", llvm("llvm-objdump", "-d", str(tmp_path / "code")), flags=re.M)[1:]:
            if "linear_small_kernel" not in text.split(">", 1)[0]:
                continue
            front = text[text.index("global_load"):text.index("s_barrier")]
            assert front.count("global_load_dwordx4") >= 4 and not re.search(r"s_waitcnt .*vmcnt\(0\)|flat_load", front), text.split(">", 1)[0]
            kernels += 1
    assert kernels == 12
