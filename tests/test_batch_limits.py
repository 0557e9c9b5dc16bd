"""Batches name a tile or block of a system in 20 bits of a map entry: grids
with more of them are refused before anything is laid out (no GPU needed)."""
import ctypes as C

import pytest

import paper_2506_21932_amd as smg


def size(shape, pattern, prec):
    n = C.c_size_t(0)
    cfg = (smg.Config * 1)(smg.make_config(shape, pattern=pattern, prec=prec, max_coarse=1 << 20))
    return smg.load().smg_batch_workspace_size(1, cfg, C.byref(n)), int(n.value)


@pytest.mark.parametrize("prec", ["fp64", "fp16"])
@pytest.mark.parametrize("shape,pattern,ok", [
    ((8192, 8192, 1), 7, True),        # 2^20 prolongation blocks, 2^19 tiles
    ((8192, 8193, 1), 7, False),       # one row of blocks more
    ((16384, 8192, 1), 7, False),      # 2^20 tiles, twice as many blocks
    ((1, 1048576, 8), 7, True),        # one column of tiles
    ((8388608, 1, 8), 7, True),        # one row of 2^20 tiles
    ((8388609, 1, 8), 7, False),
    ((4194304, 10, 2), 27, True),      # sheared: 2 rows of 2^19 tiles
    ((4194305, 10, 2), 27, False),
    ((512, 512, 512), 27, True),
])
def test_map_entries(shape, pattern, prec, ok):
    st, n = size(shape, pattern, prec)
    if ok:
        assert st == smg.SMG_OK and n > 0
    else:
        assert st == smg.SMG_EINVAL
        assert b"too large for a batch" in smg.load().smg_batch_last_error(None)
