"""Workspace sizes and the limit of smg_setup_noalloc (no GPU needed: the
limit is checked first).  The sizes are those of sweeps on wider tiles that
exchanged values through their outputs; the limit counts the same for any
tile."""
import ctypes as C

import pytest

import paper_2506_21932_amd as smg

SIZES = [
    ((256, 256, 256), dict(pattern=7), 5321.3e6),
    ((256, 256, 256), dict(pattern=27), 12073.9e6),
    ((512, 512, 64), dict(pattern=19, smoother="ilu0", coarsen="semi_xy", max_coarse=8192), 23455.3e6),
    ((512, 512, 64), dict(pattern=19, smoother="lgs", coarsen="semi_xy", max_coarse=8192, prec="fp32"), 7622.6e6),
    ((128, 128, 128), dict(pattern=27, block=3, prec="fp32"), 11434.2e6),
    ((45, 52, 39), dict(pattern=27, block=3), 893.3e6),
    ((1000, 1000, 8), dict(pattern=7, prec="fp16"), 5957.0e6),
    ((20, 20, 20), dict(pattern=7), 18.8e6),
]


@pytest.mark.parametrize("shape,kw,most", SIZES, ids=lambda v: str(v))
def test_no_larger(shape, kw, most):
    assert smg.StructMG.workspace_bytes(shape, **kw) <= most


# the longest grid that the static array takes
LIMITS = [
    ((20, 18, 108), dict(pattern=7)),
    ((20, 18, 269), dict(pattern=7, prec="fp16")),
    ((20, 18, 81), dict(pattern=19, smoother="ilu0", prec="fp32")),
    ((9, 8, 99), dict(pattern=27, block=3, prec="fp32")),
    ((20, 18, 44), dict(pattern=27, prec="fp32", coarsen="auto")),
]


@pytest.mark.parametrize("shape,kw", LIMITS, ids=lambda v: str(v))
def test_noalloc_limit(shape, kw):
    L = smg.load()
    if not no_device():
        pytest.skip("a setup beyond the check would run on this machine's GPU")
    buf = C.create_string_buffer(64)
    for more in (0, 1):
        cfg = smg.make_config((shape[0], shape[1], shape[2] + more), **kw)
        h = C.c_void_p()
        st = L.smg_setup_noalloc(C.byref(cfg), C.cast(buf, C.c_void_p), None, C.byref(h))
        assert st == (smg.SMG_ENOMEM if more else smg.SMG_EDEVICE)


def no_device():
    import torch

    return not torch.cuda.is_available()
