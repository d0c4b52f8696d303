"""How the library is compiled."""
import os

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
