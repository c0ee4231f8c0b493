"""The FP64 matrix-core launches against the thread-per-line tile and the oracle,
at the edges of their tiles (elements per work-group) and block lists.

Both launches do each element's sums in the same order with one rounding per
step, so their results are equal bit for bit; the oracle's bar is the FP64
operators' (1e-12 of the largest value).  Every case prints its name before it
touches the GPU."""
import numpy as np
import pytest

from oracle import shp_oracle as O
from paper_2604_04644_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def shp():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2604_04644_amd import shp as S
    S.lib()
    return S


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def plan_of(shp, blocks, P, pts="gj"):
    """A plan of curved blocks [(shape, n)] and the oracle's Jacobians."""
    plan = shp.Plan([(s, P, n, "curved", pts) for s, n in blocks])
    jo = []
    for b, (s, n) in enumerate(blocks):
        maps = W.shape_batch(s, max(n, 1)).take(np.arange(n))
        xi, _ = shp.quadrature(s, P + 2, pts)
        plan.set_geometry(b, torch.from_numpy(W.jacobian(maps, xi, curved=True)).cuda())
        jo.append(W.jacobian(maps, O.reference_points(s, P + 2, pts), curved=True))
    return plan, jo


@pytest.mark.parametrize("P,n", [(2, 1), (2, 8), (2, 17), (6, 1), (6, 3), (9, 2), (10, 1), (10, 3)])
@pytest.mark.parametrize("shape", O.SHAPES)
def test_helm_block(shp, shape, P, n):
    """One block around the tile's element count, both point sets."""
    for pts in ("gj", "radau"):
        print(f"[mf] block {shape} P={P} n={n} {pts}", flush=True)
        plan, jo = plan_of(shp, [(shape, n)], P, pts)
        for op in ("helmholtz", "laplacian"):
            x = W.coeffs(n, plan.n_modes[0], 20 + P)
            xt = torch.from_numpy(x).cuda()
            plan.set_tiling(0, op, 0, 0, 0)
            y = plan.apply(0, op, xt, lam=0.8).cpu().numpy()
            plan.set_tiling(0, op, 1, 64, 0)
            assert np.array_equal(y, plan.apply(0, op, xt, lam=0.8).cpu().numpy()), op
            ref = O.apply_op(op, shape, P, P + 2, jo[0], x, lam=0.8, pts=pts)
            assert rel(y, ref) <= TOL, op


@pytest.mark.parametrize("P", [2, 6, 10])
@pytest.mark.parametrize("nblk", [3, 16, 17])
def test_helm_mesh(shp, P, nblk):
    """Whole-mesh launches over uneven and empty blocks, up to and past the number
    of blocks that one matrix-core launch takes; with zero velocity the
    advection-diffusion-reaction action is the Helmholtz action."""
    print(f"[mf] mesh P={P} blocks={nblk}", flush=True)
    blocks = [(O.SHAPES[(3 * b) % 4], (0 if b == 1 else 1 + (5 * b) % 11)) for b in range(nblk)]
    plan, _ = plan_of(shp, blocks, P)
    nc, npnt = plan.totals()
    x = torch.from_numpy(W.coeffs(1, nc, 77)[0]).cuda()
    adv = plan.advection_factors(torch.zeros(3, npnt, dtype=torch.float64, device="cuda"))
    y = plan.apply(-1, "helmholtz", x, lam=1.1)
    assert torch.equal(plan.apply_adr(x, adv, lam=1.1), y)
    for b, (s, n) in enumerate(blocks):
        if n:
            co, _ = plan.offsets(b)
            xb = x[co:co + n * plan.n_modes[b]].clone()
            plan.set_tiling(b, "helmholtz", 1, 64, 0)
            assert torch.equal(plan.apply(b, "helmholtz", xb, lam=1.1).reshape(-1), y[co:co + n * plan.n_modes[b]]), b


@pytest.mark.parametrize("P,n", [(2, 11), (6, 3), (9, 2), (10, 2)])
@pytest.mark.parametrize("shape", O.SHAPES)
def test_helm_not_finite(shp, shape, P, n):
    """A NaN, and sums that overflow (the reaction term of a positive constant in one
    element), stay in their element of a tile, and an overflow reaches the same modes,
    with the same infinities and NaN, as in the thread-per-line tile."""
    print(f"[mf] not finite {shape} P={P} n={n}", flush=True)
    plan, _ = plan_of(shp, [(shape, n)], P)
    x = W.coeffs(n, plan.n_modes[0], 40 + P)
    k, rest = n // 2, np.arange(n) != n // 2
    for lam, bad in ((0.8, np.nan), (1e288, 1e20), (1e290, 1e20), (1e292, 1e20), (1e300, 1e20)):
        xb = x.copy()
        if np.isnan(bad):
            xb[k, 1] = bad
        else:
            xb[k] = 0.0
            xb[k, O.vertex_modes(shape, P)[0]] = bad
        xt = torch.from_numpy(xb).cuda()
        plan.set_tiling(0, "helmholtz", 0, 0, 0)
        y = plan.apply(0, "helmholtz", xt, lam=lam).cpu().numpy()
        ok = plan.apply(0, "helmholtz", torch.from_numpy(x).cuda(), lam=lam).cpu().numpy()
        plan.set_tiling(0, "helmholtz", 1, 64, 0)
        line = plan.apply(0, "helmholtz", xt, lam=lam).cpu().numpy()
        assert np.isfinite(ok).all() and np.array_equal(y[rest], ok[rest])
        assert np.array_equal(y, line, equal_nan=True), lam
        assert not (lam < 1.0 or lam == 1e300) or not np.isfinite(y[k]).any()


@pytest.mark.parametrize("P", [2, 6, 9, 10])
def test_adr_mesh(shp, P):
    """Advection-diffusion-reaction with a velocity that differs at every point, against
    the oracle; blocks whose last tile is partial and clamps its velocity reads (P = 2,
    8 elements a tile), and a block smaller than a tile."""
    print(f"[mf] adr P={P}", flush=True)
    blocks = [("tet", 11 if P == 2 else 3), ("hex", 5 if P == 2 else 2), ("pyr", 17 if P == 2 else 2),
              ("prism", 9 if P == 2 else 3)]
    plan, jo = plan_of(shp, blocks, P)
    nc, npnt = plan.totals()
    x = W.coeffs(1, nc, 61 + P)[0]
    vel = W.point_values(1, npnt, 71 + P, ncomp=3).reshape(3, npnt)
    adv = plan.advection_factors(torch.from_numpy(np.ascontiguousarray(vel)).cuda())
    y = plan.apply_adr(torch.from_numpy(x).cuda(), adv, lam=1.3).cpu().numpy()
    for b, (s, n) in enumerate(blocks):
        co, po = plan.offsets(b)
        NP, NQ = plan.n_modes[b], plan.n_points[b]
        ref = O.apply_op("adr", s, P, P + 2, jo[b], x[co:co + n * NP].reshape(n, NP), lam=1.3,
                         vel=vel[:, po:po + n * NQ].reshape(3, n, NQ))
        assert rel(y[co:co + n * NP].reshape(n, NP), ref) <= TOL, s


@pytest.mark.parametrize("n", [2048, 2049])
def test_hex_laplacian_rule(shp, n):
    """Hexahedra at P = 2 on both sides of the size from which their Laplacian runs a thread
    per line: the default launch, the matrix-core shape and a thread-per-line shape have
    the same bits, and the last elements agree with the oracle."""
    print(f"[mf] hex laplacian n={n}", flush=True)
    P = 2
    plan, jo = plan_of(shp, [("hex", n)], P)
    x = W.coeffs(n, plan.n_modes[0], 23)
    xt = torch.from_numpy(x).cuda()
    y = plan.apply(0, "laplacian", xt)
    for shape in ((8, 256, 2), (16, 256, 2), (1, 64, 0)):
        plan.set_tiling(0, "laplacian", *shape)
        assert torch.equal(plan.apply(0, "laplacian", xt), y), shape
    ref = O.apply_op("laplacian", "hex", P, P + 2, jo[0][-9:], x[-9:])
    assert rel(y[-9:].cpu().numpy(), ref) <= TOL
