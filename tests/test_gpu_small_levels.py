"""Small levels on both sides of the sizes at which one workgroup sweeps them
instead of tiles, against the CPU oracle; bit-exact (the order of operations
of every value is fixed)."""
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
# hyperplanes (7 points: points) at the limit and one beyond
CASES = [((5, 6, 100), 7), ((7, 10, 43), 7), ((5, 11, 80), 7), ((3, 27, 55), 7), ((15, 12, 30), 7), ((15, 19, 19), 7),
         ((1, 1, 900), 7),
         ((4, 4, 78), 27), ((4, 4, 79), 27), ((2, 2, 90), 27), ((2, 2, 91), 27), ((2, 3, 89), 19), ((2, 3, 90), 19),
         ((10, 10, 35), 19), ((10, 10, 36), 19), ((8, 8, 30), 27), ((8, 8, 31), 27),
         ((10, 10, 26), 27), ((10, 10, 27), 27), ((12, 12, 22), 27), ((12, 12, 23), 27)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("shape,pat", CASES, ids=lambda v: str(v))
def test_sweeps_bitexact(shape, pat, prec):
    A = workloads.random_sgdia(shape, pat, seed=19)
    H = oracle.Hierarchy(shape, pat, A, prec=prec)
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, pattern=pat, prec=prec, device=DEV)
    assert H.nlev >= 2
    off = workloads.offsets(pat)
    what, npt, dt = (0, np.float64, torch.float64) if prec == "fp64" else (5, np.float32, torch.float32)
    Al, rd = H.level_data(0, what), H.level_data(0, what + 1).ravel()
    g = workloads.rng(29)
    f, u = (g.uniform(-1, 1, size=shape).astype(npt) for _ in range(2))
    ft, ut = (torch.from_numpy(v).to(DEV) for v in (f, u))
    for _ in range(2):
        got = mg.op_presmooth(0, ft, torch.empty(f.size, dtype=dt, device=DEV)).cpu().numpy()
        assert np.array_equal(got, oracle.gs_sweep(off, Al, rd, f, np.zeros(shape, npt), 1, 1).ravel())
        got = mg.op_postsmooth(0, ft, ut, None, torch.empty(f.size, dtype=dt, device=DEV)).cpu().numpy()
        assert np.array_equal(got, oracle.gs_sweep(off, Al, rd, f, u, -1, 0).ravel())
