"""The tiled sweep at the sizes where its tiling can go wrong: grids that end
inside, at and just past a tile (8 x 16 columns) and a chunk (16 steps), more
tiles than the persistent grid has workgroups, every pattern, precision and
direction, against the CPU oracle; bit-exact (the order of operations of every
value is fixed).  Sweeps alternate in direction and repeat, so both strip
buffers of the level are used."""
import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2506_21932_amd as smg  # noqa: E402

DEV = torch.device("cuda:0")

SHAPES = [(8, 16, 64), (9, 17, 33), (7, 15, 40), (17, 33, 16), (16, 31, 15), (24, 48, 130), (25, 8, 161), (1, 70, 40),
          (64, 1, 80), (130, 370, 9)]


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("pat", [7, 19, 27])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_sweeps_bitexact(shape, pat, prec):
    A = workloads.random_sgdia(shape, pat, seed=31)
    H = oracle.Hierarchy(shape, pat, A, prec=prec)
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, pattern=pat, prec=prec, device=DEV)
    assert H.nlev >= 2
    off = workloads.offsets(pat)
    what, npt, dt = (0, np.float64, torch.float64) if prec == "fp64" else (5, np.float32, torch.float32)
    Al, rd = H.level_data(0, what), H.level_data(0, what + 1).ravel()
    g = workloads.rng(37)
    for rep in range(3):
        f = g.uniform(-1, 1, size=shape).astype(npt)
        u = g.uniform(-1, 1, size=shape).astype(npt)
        ft, ut = (torch.from_numpy(v).to(DEV) for v in (f, u))
        got = _np(mg.op_presmooth(0, ft, torch.empty(f.size, dtype=dt, device=DEV)))
        assert np.array_equal(got, oracle.gs_sweep(off, Al, rd, f, np.zeros(shape, npt), 1, 1).ravel()), rep
        for _ in range(rep + 1):
            got = _np(mg.op_postsmooth(0, ft, ut, None, torch.empty(f.size, dtype=dt, device=DEV)))
        assert np.array_equal(got, oracle.gs_sweep(off, Al, rd, f, u, -1, 0).ravel()), rep


# 3x3 blocks: tiles of 4 x 8 columns
BLOCK_SHAPES = [(8, 8, 33), (4, 9, 16), (5, 17, 15), (9, 7, 64), (13, 24, 41), (1, 20, 18), (72, 170, 5)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("shape", BLOCK_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_block_sweeps_bitexact(shape, prec):
    A = workloads.random_sgdia(shape, 27, seed=41, block=3)
    H = oracle.Hierarchy(shape, 27, A, block=3, prec=prec)
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, pattern=27, block=3, prec=prec, device=DEV)
    assert H.nlev >= 2
    off = workloads.offsets(27)
    what, npt, dt = (0, np.float64, torch.float64) if prec == "fp64" else (5, np.float32, torch.float32)
    Al, D = H.level_data(0, what), H.level_data(0, what + 1)
    g = workloads.rng(43)
    for rep in range(2):
        f = g.uniform(-1, 1, size=shape + (3,)).astype(npt)
        u = g.uniform(-1, 1, size=shape + (3,)).astype(npt)
        ft, ut = (torch.from_numpy(v.ravel()).to(DEV) for v in (f, u))
        got = _np(mg.op_presmooth(0, ft, torch.empty(f.size, dtype=dt, device=DEV)))
        assert np.array_equal(got, oracle.bgs_sweep(off, Al, D, f, np.zeros_like(f), 1, 1).ravel()), rep
        for _ in range(rep + 1):
            got = _np(mg.op_postsmooth(0, ft, ut, None, torch.empty(f.size, dtype=dt, device=DEV)))
        assert np.array_equal(got, oracle.bgs_sweep(off, Al, D, f, u, -1, 0).ravel()), rep


# line sweep: columns around the block of 8 points, the wave of 64 and the
# longest column of the tiled kernel (128; 129 takes the other one)
LINE_SHAPES = [(9, 17, 64), (8, 8, 128), (5, 30, 127), (17, 9, 129), (33, 40, 16), (20, 19, 8), (1, 9, 65),
               (11, 1, 24), (130, 140, 7)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("pat", [7, 19, 27])
@pytest.mark.parametrize("shape", LINE_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_line_sweeps_bitexact(shape, pat, prec):
    A = workloads.random_sgdia(shape, pat, seed=47, symmetric=False)
    kw = dict(smoother="lgs")
    H = oracle.Hierarchy(shape, pat, A, prec=prec, **kw)
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, pattern=pat, prec=prec, **kw, device=DEV)
    assert H.nlev >= 2
    off = workloads.offsets(pat)
    what, npt, dt = (0, np.float64, torch.float64) if prec == "fp64" else (5, np.float32, torch.float32)
    Al, tr, tc = (H.level_data(0, w).astype(npt) for w in (what, 7, 8))
    g = workloads.rng(53)
    f = g.uniform(-1, 1, size=shape).astype(npt)
    u = g.uniform(-1, 1, size=shape).astype(npt)
    ft, ut = (torch.from_numpy(v).to(DEV) for v in (f, u))
    for _ in range(2):
        got = _np(mg.op_presmooth(0, ft, torch.empty(f.size, dtype=dt, device=DEV)))
        assert np.array_equal(got, oracle.lgs_sweep(off, Al, tr, tc, f, np.zeros(shape, npt), 1, 1).ravel())
        got = _np(mg.op_postsmooth(0, ft, ut, None, torch.empty(f.size, dtype=dt, device=DEV)))
        assert np.array_equal(got, oracle.lgs_sweep(off, Al, tr, tc, f, u, -1, 0).ravel())
