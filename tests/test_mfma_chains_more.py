"""The convolution-state, bf16 sequence and windowed masked kernels hand no MFMA accumulator from
one MFMA shape to another (the scan of test_mfma_chains.py on their sources)."""
import os

import pytest

from paper_2607_02805_amd import build
from tests.test_mfma_chains import _compile_to_asm, mixed_shape_chains


@pytest.mark.parametrize("src", ["bdlm_mix.hip", "bdlm_seq16.hip", "bdlm_maskw.hip"])
def test_no_accumulator_crosses_mfma_shapes(src, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "k.s")
    _compile_to_asm(src, out)
    asm = open(out).read()
    assert "v_mfma" in asm
    assert mixed_shape_chains(asm) == []
