"""Host: the non-periodic operator's launches against the runtime's limit of 2^32 threads (the checks run before
the first device call; the addresses are never read)."""
import os

import pytest

from paper_2507_02401_amd import _lib


def _status(lib, shape, batch, order, levels, transpose):
    size = lib.es_sym_transpose_workspace_bytes if transpose else lib.es_sym_workspace_bytes
    fn = lib.es_sym_cov_apply_transpose if transpose else lib.es_sym_cov_apply
    need = int(size(len(shape), _lib.shape_arg(shape), batch, order, levels))
    return fn(len(shape), _lib.shape_arg(shape), batch, order, levels, 1.0, 1 << 40, 1 << 44, 1 << 48, need, None)


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="made-up addresses: only where no launch can follow")
@pytest.mark.parametrize("transpose", [False, True])
def test_levels_of_tiny_slices_fall_back_to_the_tile(lib, transpose):
    # 16 taps, slices of 4 x 4: 64 work-groups an instance split, 20 as a tile (48 in the transposed synthesis)
    for batch in (1 << 18, 300000 if transpose else 700000):
        assert _status(lib, (64, 4, 4), batch, 8, 2, transpose) != _lib.ES_EINVAL
    assert _status(lib, (64, 4, 4), 1 << 20, 8, 2, transpose) == _lib.ES_EINVAL  # the tile does not fit either
