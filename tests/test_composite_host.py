"""Host: the compile-time taps of the composite-filter tables are the taps that es_filter derives."""
import os
import re

import pytest

from paper_2507_02401_amd import _lib

HEADER = os.path.join(os.path.dirname(os.path.abspath(_lib.__file__)), "csrc", "composite.h")


@pytest.mark.parametrize("order", range(1, 9))
def test_compile_time_taps_are_the_derived_taps(lib, order):
    with open(HEADER) as f:
        rows = re.search(r"kDaubechies\[.*?= \{(.*?)\};", f.read(), re.S).group(1)
    rows = [[float(v) for v in r.split(",")] for r in re.findall(r"\{(.*?)\}", rows, re.S)]
    h = (_lib.ctypes.c_double * (2 * order))()
    assert lib.es_filter(order, h) == _lib.ES_OK
    assert rows[order - 1] == list(h)
