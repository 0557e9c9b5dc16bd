"""ILU(0) factors of grids whose hyperplanes need both workgroup widths of the
factorisation (8 threads up to 8192 points of a hyperplane's band, then 64),
bit-exact against the CPU oracle."""
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


# band of a 7-point mask: (nz + 2) * min(nx, ny + nz - 1) slots at most
@pytest.mark.parametrize("shape,pat", [((17, 21, 19), 7), ((17, 21, 19), 27), ((128, 70, 62), 7), ((129, 70, 62), 7)], ids=lambda v: str(v))
def test_ilu0_factors_bitexact(shape, pat):
    A = workloads.random_sgdia(shape, pat, seed=61, symmetric=False)
    H = oracle.Hierarchy(shape, pat, A, smoother="ilu0")
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, pattern=pat, smoother="ilu0", device=DEV)
    for l in range(H.nlev - 1):
        for what in (2, 3, 4):
            ref = H.level_data(l, what)
            got = mg.export(l, what, torch.empty(ref.shape, dtype=torch.float64, device=DEV))
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), ref), (l, what)
