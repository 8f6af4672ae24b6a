"""The convolution-state kernels hand no MFMA accumulator from one MFMA shape to another
(the scan of test_mfma_chains.py on bdlm_mix.hip)."""
import os

import pytest

from paper_2607_02805_amd import build
from tests.test_mfma_chains import _compile_to_asm, mixed_shape_chains


def test_no_accumulator_crosses_mfma_shapes(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "mix.s")
    _compile_to_asm("bdlm_mix.hip", out)
    asm = open(out).read()
    assert "v_mfma" in asm
    assert mixed_shape_chains(asm) == []
