"""Parameter sets as the C ABI takes them: packed in one call, byte for byte the
structure filled field by field, for plain numbers and for values that only float() takes."""
import ctypes

import numpy as np
import pytest

from paper_1207_2192_amd._lib import LLGParamsC
from paper_1207_2192_amd.api import LLGParams

SETS = [LLGParams(),
        LLGParams(alpha=0.1, c=0.14, hext=(1, 2.5, -3), temp=0.01, dtau=0.04, renorm=True, fd_factor=1),
        LLGParams(alpha=np.float64(0.3), c=np.float32(0.25), hext=np.array([1.0, 2.0, 3.0]), hac=[0.1, 0.2, 0.3],
                  freq=2, phase=-0.5, hpulse=(0.0, 1e-3, 0.0), tpulse=7, wpulse=np.int64(3), tau0=1e5),
        LLGParams(hext=("0.5", 0.0, 0.0), freq="0.25")]


@pytest.mark.parametrize("k", range(len(SETS)))
def test_packed_bytes_equal_the_structure(k):
    assert SETS[k].to_bytes() == bytes(SETS[k].to_c())
    assert len(SETS[k].to_bytes()) == ctypes.sizeof(LLGParamsC)


def test_bad_values_are_still_refused():
    with pytest.raises(TypeError):
        LLGParams(alpha="x").to_bytes()
    with pytest.raises(IndexError):
        LLGParams(hext=(1.0, 2.0)).to_bytes()
