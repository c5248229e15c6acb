"""Host: tiles and kernel families of levels whose extents a rule on the number of work-groups alone gets wrong
(measured launches, us, with that rule's choice and with the one expected here), and launches within the
runtime's limit of 2^32 threads."""
import ctypes

import pytest

from paper_2507_02401_amd import _lib

OPS = {"adjoint": _lib.OP_ADJOINT, "apply": _lib.OP_APPLY, "cov": _lib.OP_COV}


def _launches(lib, op, shape, batch, order, levels):
    out, buf, wgs = [], ctypes.create_string_buffer(128), ctypes.c_int64()
    while lib.es_schedule_describe(OPS[op], len(shape), _lib.shape_arg(shape), batch, order, levels, len(out), buf, 128,
                                   ctypes.byref(wgs), None) == _lib.ES_OK:
        out.append((buf.value.decode(), wgs.value))
    return out


@pytest.mark.parametrize("op,shape,batch,order,levels,index,slow,fast", [
    ("adjoint", (976, 36), 750, 5, 2, 1, "t1x16x64", "t1x8x16"),          # rows of 18: 112 / 57
    ("adjoint", (4096, 16), 64, 8, 4, 0, "t1x16x64", "t1x8x16"),          # rows of 16
    ("adjoint", (140, 116, 76), 1, 8, 2, 1, "t2x4x16", "t2x4x8"),         # rows of 38: 43 / 15
    ("apply", (368, 8, 12), 19, 3, 2, 1, "t16x16x32", "t4x8x16"),         # thin axes: 31 / 11
    ("cov", (64, 32, 128), 3, 6, 2, 0, "lp_down_p", "lp_down_3d"),        # planes of 32 rows: 8.5 / 7.1
    ("cov", (208, 104, 20), 13, 5, 2, 0, "lp_down_p", "lp_down_s"),       # planes of 10 columns: 32 / 19
], ids=str)
def test_thin_levels_take_the_faster_tile(lib, op, shape, batch, order, levels, index, slow, fast):
    name = _launches(lib, op, shape, batch, order, levels)[index][0]
    assert slow not in name and fast in name


@pytest.mark.parametrize("op,shape,batch,order,levels", [
    ("cov", (4, 64, 128), 1 << 18, 4, 2),  # planes: 2^24 work-groups of 256 threads
    ("cov", (4, 64, 128), 300000, 4, 2),
    ("cov", (4, 128, 64), 1 << 18, 5, 2),
], ids=str)
def test_launches_hold_fewer_than_2_to_32_threads(lib, op, shape, batch, order, levels):
    for name, wgs in _launches(lib, op, shape, batch, order, levels):
        assert (wgs + 7) // 8 * 8 * 256 < 1 << 32, (name, wgs)
