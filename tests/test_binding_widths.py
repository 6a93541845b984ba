"""Operator widths are kept per argument values and types: a call that ctypes refuses stays
refused after one that it takes."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1704_08907_amd", "libaboria_mi355x.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
def test_widths_refuse_what_they_refused():
    from paper_1704_08907_amd import _native as N
    for d, ny in ((1, 1), (2, 2), (3, 3)):
        assert N.op_ny("spring", d) == ny and N.op_ny("count", d) == 1
        with pytest.raises(ctypes.ArgumentError):
            N.op_ny("spring", float(d))
    assert N.op_na("dem_spring") == 1 and N.op_na("spring") == 0
    for bad in ("no such operator", 1):
        with pytest.raises(KeyError):
            N.op_ny(bad, 2)
        with pytest.raises(KeyError):
            N.op_na(bad)
    assert N.op_ny.cache_info().maxsize is not None
