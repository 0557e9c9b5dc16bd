"""FP64 products and residuals on both sides of the sizes at which a row walks
its slots one after another (launches that fill the chip one to four times,
short of at most 64 of 2048 workgroups), against the CPU oracle.  Bit-exact:
the order of operations of every value is fixed."""
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


def _np(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# 2048, 2001, 1937, 4080, 4111 workgroups
@pytest.mark.parametrize("pat", [7, 19, 27])
@pytest.mark.parametrize("shape", [(64, 64, 128), (64, 63, 127), (64, 61, 127), (127, 64, 128), (97, 65, 167)],
                         ids=lambda s: "x".join(map(str, s)))
def test_product_and_residual(shape, pat):
    A = workloads.random_sgdia(shape, pat, seed=91)
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, pattern=pat, device=DEV)
    g = workloads.rng(92)
    u, f = (g.uniform(-1, 1, size=shape) for _ in range(2))
    ut, ft = (torch.from_numpy(v.ravel()).to(DEV) for v in (u, f))
    au = oracle.spmv(workloads.offsets(pat), A, u)
    assert np.array_equal(_np(mg.op_spmv(0, ut, torch.empty_like(ut))), au.ravel())
    ref = oracle.restrict(f - au, mg.level_info(0)["cmask"])
    got = _np(mg.op_resid_restrict(0, ft, ut, torch.empty(ref.size, dtype=torch.float64, device=DEV)))
    assert np.array_equal(got, ref.ravel())
