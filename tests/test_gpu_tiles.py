"""GPU parity at the edges of tiles and launches, against the FP64 oracle: the
eta1-line tile of the transforms and the mass with fewer, as many and more lines
than threads; the diagonal's launches over blocks of mixed orders; iso-parametric
launches over more blocks than one launch takes.  Bar: 1e-12 relative in the max
norm (the results differ from the oracle's by summation order alone)."""
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


def say(msg):
    print(msg, flush=True)


def rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def set_curved(shp, plan, b, maps, shape, P):
    xi, _ = shp.quadrature(shape, P + 2)
    plan.set_geometry(b, torch.from_numpy(W.jacobian(maps, xi, curved=True)).cuda())
    return W.jacobian(maps, O.reference_points(shape, P + 2), curved=True)


@pytest.mark.parametrize("P", [1, 4, 8, 9, 10])
def test_values_tile_edges(shp, P):
    """Two whole tiles and one element over: the default launch (spread to one element
    a work-group), tiles whose lines fill the threads, and tiles of twice the lines
    (a second line per thread) give the same bits."""
    Q2, NT = (P + 2) ** 2, 512 if P >= 9 else 256
    E = NT // Q2
    ne = 2 * E + 1
    for s in O.SHAPES:
        say(f"[tiles] values P={P} {s} n_elem={ne}")
        maps = W.shape_batch(s, ne)
        plan = shp.Plan([(s, P, ne, "curved")])
        jo = set_curved(shp, plan, 0, maps, s, P)
        for k, op in enumerate(("bwd", "iprod", "mass")):
            x = W.point_values(ne, Q2 * (P + 2), 900 + k) if op == "iprod" else W.coeffs(ne, plan.n_modes[0], 900 + k)
            xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
            y = plan.apply(0, op, xt).cpu().numpy()
            ref = O.apply_op(op, s, P, P + 2, jo, x, chunk=4)
            assert rel(y.reshape(ref.shape), ref) <= TOL, (s, op)
            for e in (E, 2 * E):
                plan.set_tiling(0, op, e, NT, 0)
                assert np.array_equal(plan.apply(0, op, xt).cpu().numpy(), y), (s, op, e)


def test_diag_mixed_orders_many_blocks(shp):
    """The diagonal of 21 blocks, 17 of them of one order (more than two launches
    take) and the others of another, from one element up."""
    say("[tiles] diagonal of 21 blocks")
    blocks = [(O.SHAPES[i % 4], 2, 1 + 3 * i, "curved") for i in range(17)]
    blocks += [(s, 3, 5, "curved") for s in O.SHAPES]
    plan = shp.Plan(blocks)
    jo = [set_curved(shp, plan, b, W.shape_batch(s, n), s, P) for b, (s, P, n, _) in enumerate(blocks)]
    d = plan.helmholtz_diag(0.8).cpu().numpy()
    for b, (s, P, n, _) in enumerate(blocks):
        co, _ = plan.offsets(b)
        NP = plan.n_modes[b]
        ref = np.diagonal(O.Element(s, P, P + 2, jo[b]).helmholtz(0.8), axis1=1, axis2=2)
        assert rel(d[co:co + n * NP].reshape(n, NP), ref) <= TOL, (b, s)


@pytest.mark.parametrize("P,sizes", [(1, (17, 18, 19, 37)), (3, (3, 4, 5, 9)), (4, (1, 2, 3, 5)), (9, (1, 1, 2, 1))])
def test_iso_many_blocks(shp, P, sizes):
    """Iso-parametric blocks around a tile's size, 20 of them up to P = 4 (one launch
    takes 16): the whole mesh equals the blocks and the oracle."""
    reps = 5 if P <= 4 else 1
    blocks = [(s, P, n, "isoparam") for _ in range(reps) for s, n in zip(O.SHAPES, sizes)]
    say(f"[tiles] iso P={P} {len(blocks)} blocks")
    plan = shp.Plan(blocks)
    X = []
    for b, (s, _, n, _) in enumerate(blocks):
        idx, vxi = O.vertex_modes(s, P)
        X.append(W.iso_coords(W.shape_batch(s, n), idx, vxi, plan.n_modes[b], 950 + b, curved=True,
                              amp=0.02 if P <= 4 else 0.004))
        plan.set_geometry(b, torch.from_numpy(X[b]).cuda())
    x = W.coeffs(1, plan.totals()[0], 960)[0]
    y = plan.apply(-1, "helmholtz", torch.from_numpy(x).cuda(), lam=1.1).cpu().numpy()
    for b, (s, _, n, _) in enumerate(blocks):
        co, _ = plan.offsets(b)
        NP = plan.n_modes[b]
        xb = np.ascontiguousarray(x[co:co + n * NP].reshape(n, NP))
        yb = plan.apply(b, "helmholtz", torch.from_numpy(xb).cuda(), lam=1.1).cpu().numpy().ravel()
        assert np.array_equal(yb, y[co:co + n * NP]), (b, s)
        ref = O.apply_op("helmholtz", s, P, P + 2, O.isoparametric_jacobian(s, P, P + 2, X[b]), xb, lam=1.1, chunk=2)
        assert rel(yb.reshape(n, NP), ref) <= TOL, (b, s)


def test_streamed_launches(shp):
    """Launches whose streams exceed the Infinity Cache (11.34 million points; affine
    elements, P = 1) read and write past it: the last 29 elements have the bits of a
    launch of their own, and agree with the oracle."""
    P, ne, nb = 1, 420_011, 29
    s, Q3 = "tet", 27
    say(f"[tiles] streamed launches n_elem={ne}")
    maps = W.shape_batch(s, ne)
    last = maps.take(np.arange(ne - nb, ne))
    big, small = shp.Plan([(s, P, ne, "affine")]), shp.Plan([(s, P, nb, "affine")])
    big.set_geometry(0, torch.from_numpy(W.affine_jacobian(maps)).cuda())
    small.set_geometry(0, torch.from_numpy(W.affine_jacobian(last)).cuda())
    for k, op in enumerate(("bwd", "iprod", "mass", "physderiv", "iprod_deriv")):
        if op in ("iprod", "physderiv"):
            x = W.point_values(ne, Q3, 970 + k)
        elif op == "iprod_deriv":
            x = W.point_values(ne, Q3, 970 + k, ncomp=3)
        else:
            x = W.coeffs(ne, 4, 970 + k)
        xb = np.ascontiguousarray(x[:, -nb:] if op == "iprod_deriv" else x[-nb:])
        xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
        yb = small.apply(0, op, torch.from_numpy(xb).cuda()).cpu().numpy()
        ref = O.apply_op(op, s, P, P + 2, W.affine_jacobian(last), xb)
        assert rel(yb.reshape(ref.shape), ref) <= TOL, op
        for blk in (0, -1):
            y = big.apply(blk, op, xt if blk == 0 else xt.reshape((3, -1) if op == "iprod_deriv" else (-1,)))
            y = y.reshape((3, ne, Q3) if op == "physderiv" else (ne, -1)).cpu().numpy()
            tail = y[:, -nb:] if op == "physderiv" else y[-nb:]
            assert np.array_equal(tail.reshape(yb.shape), yb), (op, blk)


def test_iso_past_one_launch(shp):
    """16.8 million tetrahedra of P = 4, one to a work-group of 256 threads, are more
    than one launch takes (2^32 threads): the elements around the cut, and the block
    after them, have the bits of a launch of their own and agree with the oracle."""
    P, cut, half = 4, 2**24 - 1, 15
    n, s = cut + 20, "tet"
    say(f"[tiles] iso past one launch n_elem={n}")
    X = {}
    for b, (t, k) in enumerate((("hex", 5), ("tet", 64))):
        idx, vxi = O.vertex_modes(t, P)
        X[t] = torch.from_numpy(W.iso_coords(W.shape_batch(t, k), idx, vxi, O.num_modes(t, P), 980 + b, curved=True,
                                             amp=0.02)).cuda()
    big = shp.Plan([("hex", P, 5, "isoparam"), (s, P, n, "isoparam")])
    big.set_geometry(0, X["hex"])
    Xt = X[s].repeat(n // 64 + 1, 1, 1)[:n]
    big.set_geometry(1, Xt)
    x = torch.rand(big.totals()[0], dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(7))
    y = big.apply(-1, "helmholtz", x, lam=1.1)
    co, NP = big.offsets(1)[0], big.n_modes[1]
    sel = slice(cut - half, cut + half)
    small = shp.Plan([("hex", P, 5, "isoparam"), (s, P, 2 * half, "isoparam")])
    small.set_geometry(0, X["hex"])
    small.set_geometry(1, Xt[sel].contiguous())
    xs = x[co:].reshape(n, NP)[sel].contiguous()
    ys = small.apply(1, "helmholtz", xs, lam=1.1)
    ref = O.apply_op("helmholtz", s, P, P + 2, O.isoparametric_jacobian(s, P, P + 2, Xt[sel].cpu().numpy()),
                     xs.cpu().numpy(), lam=1.1, chunk=2)
    assert rel(ys.cpu().numpy(), ref) <= TOL
    assert torch.equal(y[co:].reshape(n, NP)[sel], ys)
    assert torch.equal(y[:co], small.apply(0, "helmholtz", x[:co].reshape(5, -1), lam=1.1).reshape(-1))
    assert torch.equal(big.apply(1, "helmholtz", x[co:].reshape(n, NP), lam=1.1).reshape(-1), y[co:])
    del big, Xt, x, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("s,P,ne", [("hex", 2, 175_003), ("prism", 10, 6_501)])
def test_streamed_launches_orders(shp, s, P, ne):
    """As above where the derivatives are streamed as well (from P = 2), and at the last
    order: the last 5 elements of a block and of a whole-mesh launch."""
    nb, Q3, NP = 5, (P + 2) ** 3, O.num_modes(s, P)
    say(f"[tiles] streamed launches {s} P={P} n_elem={ne}")
    maps = W.shape_batch(s, ne)
    last = maps.take(np.arange(ne - nb, ne))
    big, small = shp.Plan([(s, P, ne, "affine")]), shp.Plan([(s, P, nb, "affine")])
    big.set_geometry(0, torch.from_numpy(W.affine_jacobian(maps)).cuda())
    small.set_geometry(0, torch.from_numpy(W.affine_jacobian(last)).cuda())
    g = torch.Generator("cuda").manual_seed(11)
    for op in ("bwd", "iprod", "mass", "physderiv", "iprod_deriv"):
        shape = {"iprod": (ne, Q3), "physderiv": (ne, Q3), "iprod_deriv": (3, ne, Q3)}.get(op, (ne, NP))
        x = 2.0 * torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64) - 1.0
        xb = x[..., -nb:, :].contiguous()
        yb = small.apply(0, op, xb).cpu().numpy()
        ref = O.apply_op(op, s, P, P + 2, W.affine_jacobian(last), xb.cpu().numpy())
        assert rel(yb.reshape(ref.shape), ref) <= TOL, op
        for blk in (0, -1):
            y = big.apply(blk, op, x.reshape(-1) if blk < 0 else x).reshape(
                (3, ne, Q3) if op == "physderiv" else (ne, -1))[..., -nb:, :].cpu().numpy()
            assert np.array_equal(y.reshape(yb.shape), yb), (op, blk)
