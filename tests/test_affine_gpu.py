"""The streaming pass of affine meshes at every compiled 3D order against the
FP64 oracle: parallelepiped elements (no metric term vanishes), walls with a
moving wall, a body force and a force per node, and the same mesh without
walls. The pass splits an element's lines and slots over a workgroup by the
order and the storage, so each order is its own case.

Tolerances, normwise as in the other parity tests: FP64 1e-12 (10 steps and the
single operator), FP32 deviation storage 1e-5 after 10 steps. The comparison
with the general path moves one node by d = 1e-11 of the box, which takes the
mesh off the affine path and its metric by at most N^2 d relative; the fields
may differ by that times 10 steps, N^2 1e-10."""
import copy

import numpy as np
import pytest

from conftest import nerr
from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(N, 27) for N in range(2, 9)] + [(2, 19), (5, 19), (8, 19), (12, 19)]
SHEAR = np.array([[1.0, 0.2, 0.1], [0.0, 1.0, 0.0], [0.15, -0.1, 0.9]])


def _case(N, Q, walls):
    nel = (2, 2, 1) if N >= 8 else (3, 2, 2)
    m = I.box_mesh(3, N, nel, (0, 0, 0), (1, 1, 1.5), (True, not walls, True),
                   wall_tags={1: (1, 2)} if walls else None, wall_u=[[0, 0, 0], [0.02, 0, 0.01]] if walls else None,
                   warp=lambda x: x @ SHEAR.T)
    r, u = I.rest_fields(m.xyz)
    c = I.Case(f"affine_N{N}_q{Q}", m, Q, 1.0, 0.01, 0.5 * I.stable_dt(m), r, u, 0, g=(1e-3, 0.0, 5e-4),
               filter="quad", filter_kc=min(2, N - 1), filter_amp=0.1)
    c.rho, c.u = I.random_state(c, seed=N, amp=0.01)
    return c


def _run(c, prec, F=None, steps=10):
    from paper_2509_19171_amd import sel

    g = sel.from_case(c, prec)
    if F is not None:
        g.set_force(F)
    g.step(steps)
    return g.moments()


def uerr(u, uref):
    return float(np.abs(u - uref).max() / max(np.abs(uref).max(), 0.01))


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("N,Q", SHAPES)
def test_affine_steps(N, Q, walls):
    import oracle

    c = _case(N, Q, walls)
    F = None
    if walls:
        F = 1e-3 * np.random.Generator(np.random.PCG64(5)).standard_normal((int(c.gid.max()) + 1, 3))[c.gid]
    o = oracle.from_case(c)
    if F is not None:
        o.set_force(F)
    o.step(10)
    orho, ou = o.moments()
    for prec, tol in (("fp64", 1e-12), ("fp32dev", 1e-5)):
        rho, u = _run(c, prec, F)
        print(f"[gpu] N {N} Q {Q} walls {walls} {prec}: rho {nerr(rho, orho):.2e} u {uerr(u, ou):.2e}", flush=True)
        assert nerr(rho, orho) < tol and uerr(u, ou) < tol, prec


@pytest.mark.parametrize("N,Q", SHAPES)
def test_affine_rhs(N, Q):
    import oracle
    from paper_2509_19171_amd import sel

    c = _case(N, Q, True)
    rng = np.random.Generator(np.random.PCG64(3))
    _, t, _ = oracle.lattice(3, Q)
    f = (t[None, :] * (1.0 + 1e-2 * rng.standard_normal((int(c.gid.max()) + 1, Q))))[c.gid].transpose(0, 2, 1).copy()
    ref = oracle.from_case(c).rhs(f)
    got = sel.from_case(c, "fp64").apply("rhs", f)
    assert np.abs(got - ref).max() < 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32dev"])
@pytest.mark.parametrize("N,Q", [(4, 27), (7, 27), (8, 19), (12, 19)])
def test_affine_and_general_path_agree(N, Q, prec):
    c = _case(N, Q, True)
    d = copy.deepcopy(c)
    p = int(np.argmax(np.all(np.abs(c.mesh.xyz[0] - c.mesh.xyz[0].mean(0)) < 0.45 * np.ptp(c.mesh.xyz[0], axis=0), axis=-1)))
    d.mesh.xyz[0, p, 0] += 1e-11
    (ra, ua), (rg, ug) = _run(c, prec), _run(d, prec)
    tol = N * N * 1e-10 if prec == "fp64" else 1e-5
    assert nerr(ra, rg) < tol and uerr(ua, ug) < tol
