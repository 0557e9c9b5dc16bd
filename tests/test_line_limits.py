"""The line sweep names a tile of K x K columns by its x and y in 15 and 16
bits: grids with more are refused at once (no GPU needed).  K is 512 / nz
(FP32) or 256 / nz (FP64) up to 8, and 1 for columns beyond 128 points."""
import ctypes as C

import pytest

import paper_2506_21932_amd as smg


def size(shape, **kw):
    n = C.c_size_t(0)
    cfg = smg.make_config(shape, smoother="lgs", coarsen="semi_xy", max_coarse=1 << 20, **kw)
    return smg.load().smg_workspace_size(C.byref(cfg), C.byref(n))


@pytest.mark.parametrize("shape,pattern,prec,ok", [
    ((32768, 4, 200), 7, "fp64", True),
    ((32769, 4, 200), 7, "fp64", False),
    ((32769, 4, 128), 7, "fp64", True),      # K = 2
    ((4, 65536, 130), 7, "fp32", True),
    ((4, 65537, 130), 7, "fp32", False),
    ((4, 65534, 130), 27, "fp32", False),    # rows sheared by x
    ((4, 65533, 130), 27, "fp32", True),
    ((262144, 2, 64), 19, "fp32", True),     # K = 8
    ((262145, 2, 64), 19, "fp32", False),
    ((131072, 2, 64), 19, "fp64", True),     # K = 4
    ((131073, 2, 64), 19, "fp64", False),
])
def test_tile_entries(shape, pattern, prec, ok):
    st = size(shape, pattern=pattern, prec=prec)
    assert st == (smg.SMG_OK if ok else smg.SMG_EINVAL)
    if not ok:
        assert b"too large" in smg.load().smg_last_error(None)
