"""A batch in which one system is not finite: its values meet the other
systems' only through the workgroups that sweep tiles of both, one after
another, so every other system keeps the bits of its own solve.  More tiles
than workgroups, on grids of one tile each and of several."""
import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2506_21932_amd as smg  # noqa: E402

DEV = torch.device("cuda:0")
KW = dict(coarsen="full", max_coarse=512)
# a few workgroups (set_schedule) take every tile, the spoilt system's between the others'
SHAPES = [(18, 33, 20), (9, 17, 40), (24, 20, 17), (18, 33, 20), (16, 16, 16)]
BAD = 1


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def N(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("value", [np.nan, np.inf], ids=["nan", "inf"])
@pytest.mark.parametrize("pat,prec", [(7, "fp64"), (7, "fp16"), (19, "fp32"), (27, "fp64"), (27, "fp16")])
def test_nonfinite_system_stays_alone(pat, prec, value):
    As = [workloads.random_sgdia(s, pat, seed=60 + k) for k, s in enumerate(SHAPES)]
    B = smg.StructMGBatch([T(A) for A in As], SHAPES, pattern=pat, prec=prec, **KW)
    singles = [smg.StructMG(T(A), s, pattern=pat, prec=prec, **KW) for s, A in zip(SHAPES, As)]
    g = workloads.rng(61)
    rs = [T(g.uniform(-1, 1, size=int(np.prod(s)))) for s in SHAPES]
    ref = [N(m.precondition(r, torch.empty_like(r))) for m, r in zip(singles, rs)]
    rs[BAD][rs[BAD].numel() // 2] = value
    for order, grid in [(0, 1), (1, 1), (0, 2)]:
        B.set_schedule(order, grid)
        zs = [torch.empty_like(r) for r in rs]
        B.precondition(rs, zs)
        assert not np.isfinite(N(zs[BAD])).all()
        for k in range(len(SHAPES)):
            if k != BAD:
                assert np.array_equal(N(zs[k]), ref[k]), f"system {k}, order {order}, grid {grid}"


def test_nonfinite_system_solve():
    As = [workloads.reservoir7(s, seed=70 + k) for k, s in enumerate(SHAPES)]
    B = smg.StructMGBatch([T(A) for A, _ in As], SHAPES, pattern=7, prec="fp32", **KW)
    B.set_schedule(0, 1)
    bs = [T(b.ravel()) for _, b in As]
    xs = [torch.zeros_like(b) for b in bs]
    st, res = B.solve(bs, xs, rtol=1e-9, maxit=100)
    assert st == smg.SMG_OK
    bs[BAD][3] = np.nan
    ys = [torch.zeros_like(b) for b in bs]
    _, bad = B.solve(bs, ys, rtol=1e-9, maxit=100)
    assert bad[BAD]["status"] != smg.SMG_OK
    for k in range(len(SHAPES)):
        if k != BAD:
            assert bad[k]["status"] == smg.SMG_OK and bad[k]["iters"] == res[k]["iters"], (k, bad[k])
            assert np.array_equal(N(xs[k]), N(ys[k])), k
