"""Meshes on both sides of the sizes at which a kernel or its split
changes, against the FP64 oracle: low orders with many shared nodes, affine and
curved (one node moved by 1e-9 of the spacing), with and without the filter.

Tolerances as in the other parity tests: FP64 1e-12 (normwise, velocity
against max(|u|, 0.01)), FP32 deviation storage 1e-5."""
import dataclasses

import numpy as np
import pytest

from conftest import nerr
from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def uerr(u, uref):
    return float(np.abs(u - uref).max() / max(np.abs(uref).max(), 0.01))


def curved(c):
    """The case with one interior node moved, so that its elements are not all affine."""
    x, n1 = c.mesh.xyz.copy(), c.N + 1
    x[0, 1 + n1 + n1 * n1, 0] += 1e-9 * I.min_node_spacing(c.mesh)
    return dataclasses.replace(c, mesh=dataclasses.replace(c.mesh, xyz=x))


def box(N, Q, nel, filt=None, walls=False, coupling="cg"):
    m = I.box_mesh(3, N, nel, (0, 0, 0), (1, 1.1, 0.9), (True, not walls, True), wall_tags={1: (1, 2)} if walls else None,
                   wall_u=[[0, 0, 0], [0.02, 0, 0.01]] if walls else None)
    r, u = I.rest_fields(m.xyz)
    c = I.Case(f"box_N{N}_q{Q}", m, Q, 1.0, 0.01, 0.5 * I.stable_dt(m), r, u, 0, g=(1e-3, 0.0, 5e-4), filter=filt,
               filter_kc=min(2, N - 1), filter_amp=0.1, coupling=coupling)
    c.rho, c.u = I.random_state(c, seed=N, amp=0.01)
    return c


def check(c, steps=2, precs=(("fp64", 1e-12), ("fp32dev", 1e-5)), F=None):
    import oracle
    from paper_2509_19171_amd import sel

    o = oracle.from_case(c)
    if F is not None:
        o.set_force(F)
    o.step(steps)
    orho, ou = o.moments()
    for prec, tol in precs:
        g = sel.from_case(c, prec)
        if F is not None:
            g.set_force(F)
        g.step(steps)
        rho, u = g.moments()
        print(f"[gpu] {c.name} E {c.E} {c.filter} {prec}: rho {nerr(rho, orho):.2e} u {uerr(u, ou):.2e}", flush=True)
        assert nerr(rho, orho) < tol and uerr(u, ou) < tol, prec


# 97 k, 138 k, 138 k and 244 k shared nodes
@pytest.mark.parametrize("Q,nel", [(19, (24, 24, 24)), (19, (27, 27, 27)), (27, (27, 27, 27)), (27, (33, 33, 32))])
def test_assembly_splits(Q, nel):
    check(curved(box(2, Q, nel)))


# the first stage of curved elements: one kernel (small meshes, FP64), the filter
# in it (N <= 3) or ahead of it, against separate passes
@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("N,Q", [(2, 27), (3, 19), (4, 27), (5, 19), (6, 27), (7, 27), (8, 19), (8, 27)])
def test_first_stage_small(N, Q, filt):
    c = curved(box(N, Q, (3, 2, 2) if N < 6 else (2, 2, 1), filt, walls=True))
    check(c, 5)
    check(dataclasses.replace(c, rk="printed4"), 3)


@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("N,Q,nel", [(2, 27, (20, 20, 19)), (3, 27, (15, 15, 15)), (4, 27, (12, 12, 12)), (5, 27, (11, 11, 10)),
                                     (6, 19, (11, 11, 10))])
def test_first_stage_large(N, Q, nel, filt):
    check(curved(box(N, Q, nel, filt, walls=True)))


# affine meshes of low order: streaming pass below a size, general kernels above
# (one case each side), N = 4 the pass again for a state of 128 MB
@pytest.mark.parametrize("N,Q,nel", [(2, 27, (14, 14, 14)), (2, 19, (16, 16, 15)), (3, 19, (11, 11, 11)), (3, 27, (12, 12, 12)),
                                     (4, 27, (9, 9, 9)), (4, 19, (12, 12, 12)), (4, 27, (18, 17, 16))])
def test_affine_low_orders(N, Q, nel):
    check(box(N, Q, nel, "quad", walls=True))
    if nel[0] < 15:
        check(box(N, Q, nel))
        check(box(N, Q, nel, coupling="dg"), 1)
        c = box(N, Q, nel, "quad")
        check(c, 1, F=np.broadcast_to([1e-3, 2e-3, -1e-3], (c.E, c.np_, 3)).copy())
