"""The 2D stage kernels on a node shared by more elements than they load at
once (seven straight-sided quads around one node, walls outside), and the closure's
training kernel at the edges of its row tiles.

Tolerances: FP64 fields against the oracle 1e-12 (normwise, ten steps), FP32
deviation storage 1e-5, as in the other parity tests. Gradient against FP64
autograd: a sum of n terms of FP32 products through four layers of at most 64
terms, 1e-5 of the largest entry."""
import numpy as np
import pytest

from conftest import nerr
from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _star(N, spokes=7):
    """Quads O, P_k, M_k, P_{k+1} around the origin O; the outer faces are walls."""
    x = (I.gll_points(N) + 1.0) / 2.0
    r, s = np.meshgrid(x, x, indexing="xy")  # r fastest
    r, s = r.reshape(-1, 1), s.reshape(-1, 1)
    ang = 2 * np.pi * np.arange(spokes) / spokes
    P = np.stack([np.cos(ang), np.sin(ang)], -1)
    xyz = []
    for k in range(spokes):
        p, q = P[k], P[(k + 1) % spokes]
        m = 0.8 * (p + q)
        xyz.append(r * (1 - s) * p + s * (1 - r) * q + r * s * m)
    xyz = np.stack(xyz)
    key = np.round(xyz.reshape(-1, 2) * 1e9).astype(np.int64)
    _, gid = np.unique(key, axis=0, return_inverse=True)
    tag = np.tile(np.array([[0, 1, 0, 1]], dtype=np.int32), (spokes, 1))
    return I.Mesh(2, N, xyz, gid.reshape(spokes, -1).astype(np.int64), tag, np.zeros((1, 2)))


@pytest.mark.parametrize("rk", ["ssprk3", "printed4"])
@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("N", [4, 7, 10])
def test_node_of_seven_elements(N, filt, rk):
    import oracle
    from paper_2509_19171_amd import sel

    m = _star(N)
    r, u = I.rest_fields(m.xyz)
    c = I.Case("star", m, 9, 1.0, 0.01, 0.5 * I.stable_dt(m), r, u, 0, g=(1e-3, 5e-4, 0.0), filter=filt, filter_kc=2,
               filter_amp=0.1, rk=rk)
    c.rho, c.u = I.random_state(c, seed=N, amp=0.01)
    o = oracle.from_case(c)
    o.step(10)
    orho, ou = o.moments()
    for prec, tol in (("fp64", 1e-12), ("fp32dev", 1e-5)):
        g = sel.from_case(c, prec)
        g.step(3)  # the calls' ends assemble and filter
        g.step(7)
        rho, v = g.moments()
        eu = float(np.abs(v - ou).max() / max(np.abs(ou).max(), 0.01))
        print(f"[gpu] star N {N} {filt} {rk} {prec}: rho {nerr(rho, orho):.2e} u {eu:.2e}", flush=True)
        assert nerr(rho, orho) < tol and eu < tol


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, 4097, 20000])
def test_gradient_at_tile_edges(n):
    from paper_2509_19171_amd import sel

    g = torch.Generator().manual_seed(n)
    X, y = torch.randn((n, 6), generator=g), torch.rand((n,), generator=g)
    p = torch.from_numpy(I.closure_blob(3, mean=[0.0] * 6, std=[1.0] * 6))
    w = p[12:8845].double().requires_grad_(True)
    W1, b1, W2, b2, W3, b3, w4, b4 = torch.split(w, [384, 64, 4096, 64, 4096, 64, 64, 1])
    h = X.double()
    for W, b, k in ((W1, b1, 6), (W2, b2, 64), (W3, b3, 64)):
        h = torch.tanh(h @ W.view(64, k).T + b)
    loss = ((torch.nn.functional.softplus(h @ w4 + b4) - y.double()) ** 2).mean()
    loss.backward()
    loss = loss.item()
    got, l = sel.mlp_gradient(p.cuda(), X.cuda(), y.cuda())
    ref = w.grad
    assert (got.cpu().double() - ref).abs().max() < 1e-5 * ref.abs().max()
    assert abs(l - loss) < 1e-5 * loss
