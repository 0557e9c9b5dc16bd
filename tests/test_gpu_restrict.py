"""Restriction at the sizes where it can go wrong (odd and even ends of every
axis, every set of coarsened axes, scalar and 3x3-block
vectors) against the CPU oracle, and a batch just below and just above the
total size at which its levels run residual and restriction as two launches,
against its systems alone (which run them fused).  Bit-exact: the order of
operations of every value is fixed."""
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


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("semi", [0, 1])
@pytest.mark.parametrize("block", [1, 3])
@pytest.mark.parametrize("shape", [(8, 8, 8), (9, 8, 7), (8, 9, 10), (7, 11, 9), (2, 17, 16), (16, 3, 22)],
                         ids=lambda s: "x".join(map(str, s)))
def test_restrict_bitexact(shape, block, semi, prec):
    if block == 3 and semi:
        pytest.skip("block systems coarsen all axes")
    pat = 27 if block == 3 else 7
    A = workloads.random_sgdia(shape, pat, seed=41, block=block)
    kw = dict(pattern=pat, prec=prec, max_coarse=1024, device=DEV)
    if semi:
        kw.update(coarsen="semi_xy", semi_levels=1)
    mg = smg.StructMG(torch.from_numpy(A).to(DEV), shape, block=block, **kw)
    assert mg.nlev >= 2
    cm = mg.level_info(0)["cmask"]
    npt, dt = (np.float64, torch.float64) if prec == "fp64" else (np.float32, torch.float32)
    tail = (3,) if block == 3 else ()
    rf = workloads.rng(43).uniform(-1, 1, size=shape + tail).astype(npt)
    ref = oracle.restrict(rf, cm, bs=block)
    got = _np(mg.op_restrict(0, torch.from_numpy(rf).to(DEV).ravel(), torch.empty(ref.size, dtype=dt, device=DEV)))
    assert np.array_equal(got, ref.ravel())


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("shapes", [[(41, 43, 37), (37, 41, 43)], [(41, 43, 37), (9, 9, 9), (37, 41, 43)]],
                         ids=["130462", "131191"])
def test_batch_levels_around_the_split(shapes, prec):
    sysl = [workloads.reservoir7(s, seed=70 + k) for k, s in enumerate(shapes)]
    As = [torch.from_numpy(A).to(DEV) for A, _ in sysl]
    B = smg.StructMGBatch(As, shapes, pattern=7, prec=prec, device=DEV)
    g = workloads.rng(71)
    rs = [torch.from_numpy(g.uniform(-1, 1, size=int(np.prod(s)))).to(DEV) for s in shapes]
    ref = [_np(smg.StructMG(A, s, pattern=7, prec=prec, device=DEV).precondition(r, torch.empty_like(r)))
           for A, s, r in zip(As, shapes, rs)]
    for rep in range(2):
        zs = [torch.full_like(r, np.nan) for r in rs]
        B.precondition(rs, zs)
        for k in range(len(shapes)):
            assert np.array_equal(_np(zs[k]), ref[k]), (k, rep)
