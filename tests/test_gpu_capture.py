"""Actions captured into a HIP graph once one of their operator has run: the FP64 and
the FP32 whole-mesh action of an operator share what the first of them prepares, so
either can be captured after an eager call of the other.  Every replay, with eager work
between, equals the eager result bit for bit."""
import numpy as np
import pytest

from oracle import shp_oracle as O
from paper_2604_04644_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def shp():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2604_04644_amd import shp as S
    S.lib()
    return S


@pytest.mark.parametrize("op", ["helmholtz", "laplacian"])
@pytest.mark.parametrize("first", ["fp64", "fp32"])
@pytest.mark.parametrize("P", [4, 10])
def test_capture_after_other_precision(shp, P, first, op):
    print(f"[capture] P={P} {op} after an eager {first} call", flush=True)
    n = 5
    plan = shp.Plan([(s, P, n, "curved") for s in O.SHAPES])
    for b, s in enumerate(O.SHAPES):
        xi, _ = shp.quadrature(s, P + 2)
        plan.set_geometry(b, torch.from_numpy(W.jacobian(W.shape_batch(s, n), xi, curved=True)).cuda())
    x = torch.from_numpy(W.coeffs(1, plan.totals()[0], 300 + P)[0]).cuda()
    x32 = x.float()
    run = {"fp64": lambda out=None: plan.apply(-1, op, x, out=out, lam=0.7),
           "fp32": lambda out=None: plan.apply_prec(op, x32, out=out, lam=0.7)}
    warm = run[first]()
    other = run["fp32" if first == "fp64" else "fp64"]
    out = torch.empty_like(x32 if first == "fp64" else x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        other(out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, other())
        assert torch.equal(warm, run[first]())
