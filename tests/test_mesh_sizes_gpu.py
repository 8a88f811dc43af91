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


# The benchmark workload at full size off the affine path, as the benchmark's
# headline runs it: whole fields and the integrals after 20 steps. Bounds as for the
# box itself: fields 1e-12 and 1e-5; integrals 1e-11 (the oracle adds 2.1 M node
# terms one after another), FP32 1e-8 (mass, momentum against mass x u0), 1e-6
# (kinetic energy).
def test_full_size_off_the_affine_path():
    import oracle
    from paper_2509_19171_amd import sel

    c = I.off_affine(I.case_tgv3d(steps=0))
    o = oracle.from_case(c)
    o.step(20)
    orho, ou = o.moments()
    ored = o.reduce()
    del o
    for prec, tol, rtol in (("fp64", 1e-12, (1e-11, 1e-12, 1e-11)), ("fp32dev", 1e-5, (1e-8, 1e-8, 1e-6))):
        g = sel.from_case(c, prec)
        g.step(20)
        rho, u = g.moments()
        red = g.reduce()
        print(f"[gpu] {prec}: rho {nerr(rho, orho):.2e} u {uerr(u, ou):.2e} {red} {ored}", flush=True)
        assert nerr(rho, orho) < tol and uerr(u, ou) < tol, prec
        assert red[-1] == 0 and abs(red[0] / ored[0] - 1) < rtol[0] and abs(red[4] / ored[4] - 1) < rtol[2], prec
        assert np.abs(red[1:4] - ored[1:4]).max() < rtol[1] * ored[0] * c.meta["u0"], prec
        del g
        torch.cuda.empty_cache()


# Streaming and filter passes over an element dealt to one workgroup, to some (fewer
# than passes) and to as many as passes: the split follows from the element count.
# Bound: the rounding of the coordinates gives the metric of one of n elements along
# a side a relative error of the order 2^-52 n N^2 / 2; three stages along three
# directions at a time step of half the node spacing carry it to the fields, whose
# variation between nodes is of the size the velocity error is taken against.
@pytest.mark.parametrize("N,Q,nel,walls", [(5, 27, (8, 6, 7), True), (5, 27, (9, 8, 8), True), (5, 27, (11, 10, 10), False),
                                           (6, 19, (8, 7, 6), True), (6, 27, (11, 10, 10), True), (7, 19, (9, 8, 8), True),
                                           (7, 27, (7, 6, 7), False), (8, 19, (8, 7, 6), False), (8, 27, (9, 8, 8), True),
                                           (8, 19, (11, 10, 10), True), (12, 19, (5, 4, 3), True), (12, 19, (7, 6, 7), False)])
def test_pass_splits(N, Q, nel, walls):
    tol = max(1e-12, 9 * 2.0 ** -52 * max(nel) * N * N)
    check(box(N, Q, nel, "quad", walls=walls), precs=(("fp64", tol), ("fp32dev", 1e-5)))


# 97 k, 138 k, 138 k and 244 k shared nodes
@pytest.mark.parametrize("Q,nel", [(19, (24, 24, 24)), (19, (27, 27, 27)), (27, (27, 27, 27)), (27, (33, 33, 32))])
def test_assembly_splits(Q, nel):
    check(I.off_affine(box(2, Q, nel)))


# the first stage of curved elements: one kernel (small meshes, FP64), the filter
# in it (N <= 3) or ahead of it, against separate passes
@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("N,Q", [(2, 27), (3, 19), (4, 27), (5, 19), (6, 27), (7, 27), (8, 19), (8, 27)])
def test_first_stage_small(N, Q, filt):
    c = I.off_affine(box(N, Q, (3, 2, 2) if N < 6 else (2, 2, 1), filt, walls=True))
    check(c, 5)
    check(dataclasses.replace(c, rk="printed4"), 3)


@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("N,Q,nel", [(2, 27, (20, 20, 19)), (3, 27, (15, 15, 15)), (4, 27, (12, 12, 12)), (5, 27, (11, 11, 10)),
                                     (6, 19, (11, 11, 10))])
def test_first_stage_large(N, Q, nel, filt):
    check(I.off_affine(box(N, Q, nel, filt, walls=True)))


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


# density and velocity are sums of the same populations (FP64; |f| < 0.5, 19 terms)
@pytest.mark.parametrize("N,Q,nel", [(12, 19, (2, 2, 2)), (12, 19, (5, 4, 4)), (7, 27, (3, 2, 2)), (2, 27, (5, 5, 4))])
def test_moments_of_the_state(N, Q, nel):
    import oracle
    from paper_2509_19171_amd import sel

    c = box(N, Q, nel, walls=True)
    e = np.asarray(oracle.lattice(3, Q)[0], dtype=float)
    for prec in ("fp64", "fp32dev"):
        sim = sel.from_case(c, prec)
        sim.step(1)
        f = sim.get_f()
        rho, u = sim.moments()
        r = f.sum(1)
        assert np.abs(rho - r).max() < 1e-14 and np.abs(u - np.einsum("eqp,qk->epk", f, e) / r[..., None]).max() < 1e-14


# 2D: one kernel per stage below a size, general kernels above. The step is
# compared with the same step put together from the operators of sel_apply, which
# run the general kernels on the same metric (against the oracle the rounding of
# the coordinates, which grows with the number of elements, would be what shows).
# Bound: a stage adds dt L, sums of at most N + 1 <= 11 products of the order of
# the populations (0.44 in FP64, the deviations of 0.01 in FP32) with dt c D_iq of
# order 1 at this time step, so 11 x 0.44 x 1.1e-16 x a few per stage, four passes:
# 1e-13; FP32 11 x 0.01 x 6e-8 x a few: 1e-7.
def channel(N, nel, filt=None, coupling="cg"):
    c = I.case_poiseuille(nelx=nel[0], nely=nel[1], N=N, curved=True, filt=filt)
    c.rho, c.u = I.random_state(c, seed=N, amp=0.01)
    c.g = (1e-3, -2e-3, 0.0)
    c.coupling = coupling
    return c


def step_from_operators(sim, c):
    """f after one SSPRK3 step (Secs. 2.1, 2.2, 2.2.3), [E][Q][np]."""
    import oracle

    e, t, _ = oracle.lattice(c.dim, c.Q)
    e = np.asarray(e, dtype=float)[:, :c.dim]
    y = sim.apply("collide", sim.get_f())
    rho = y.sum(1, keepdims=True)
    Fs = (3.0 * np.asarray(t) * (e @ np.asarray(c.g)[:c.dim]))[None, :, None] * rho

    def L(f):
        return sim.apply("rhs", f) + Fs

    w = y + c.dt * L(y)
    w = 0.75 * y + 0.25 * (w + c.dt * L(w))
    f = y / 3.0 + 2.0 / 3.0 * (w + c.dt * L(w))
    return sim.apply("filter", f) if c.filter else f


def check_operators(c):
    from paper_2509_19171_amd import sel

    for prec, tol in (("fp64", 1e-13), ("fp32dev", 1e-7)):
        sim = sel.from_case(c, prec)
        ref = step_from_operators(sim, c)
        f0, rho = sim.get_f(), sim.moments()[0]
        sim.step(1)
        err = np.abs(sim.get_f() - ref).max()
        print(f"[gpu] {c.name} N {c.N} E {c.E} {c.coupling} {c.filter} {prec}: f {err:.2e}", flush=True)
        assert err < tol
        # the body force given as a force per node: the same step
        d = dataclasses.replace(c, g=(0.0, 0.0, 0.0))
        sim = sel.from_case(d, prec)
        sim.set_f(f0)
        sim.set_force(rho[..., None] * np.asarray(c.g)[:c.dim])
        sim.step(1)
        err = np.abs(sim.get_f() - ref).max()
        print(f"[gpu]   force per node: f {err:.2e}", flush=True)
        assert err < tol


@pytest.mark.parametrize("coupling", ["cg", "dg"])
def test_2d_sizes(coupling):
    check_operators(channel(8, (45, 44), "quad", coupling))


@pytest.mark.parametrize("N,nel", [(2, (130, 125)), (4, (92, 90)), (5, (75, 72))])
def test_2d_sizes_oracle(N, nel):
    c = channel(N, nel, "quad" if N > 2 else None)
    check(c)
    check(dataclasses.replace(c, rk="printed4", filter=None), 1,
          F=np.broadcast_to([1e-3, -2e-3], (c.E, c.np_, 2)).copy())


@pytest.mark.parametrize("coupling", ["cg", "dg"])
@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("N", [3, 5, 8, 10])
def test_2d_small(N, filt, coupling):
    check_operators(channel(N, (5, 4), filt, coupling))


@pytest.mark.parametrize("filt", [None, "quad"])
@pytest.mark.parametrize("rk", ["ssprk3", "printed4"])
@pytest.mark.parametrize("N", [3, 5, 8])
def test_2d_discontinuous_stages(N, rk, filt):
    check(dataclasses.replace(channel(N, (5, 4), filt, "dg"), rk=rk), 7)


# the closure's increments reach the collision on every path: curved 3D (joined first
# stage), 2D one kernel per stage and general, both couplings. Bounds as for the other
# closure runs (FP32 features and weights on both sides): 1e-8 and 1e-5.
@pytest.mark.parametrize("make", [lambda: I.off_affine(box(3, 27, (3, 2, 2), "quad")), lambda: I.off_affine(box(4, 19, (3, 2, 2))),
                                  lambda: I.off_affine(box(5, 27, (2, 2, 2), "quad", walls=True)),
                                  lambda: I.off_affine(box(7, 19, (2, 1, 2), "quad")), lambda: channel(5, (6, 5), "quad"),
                                  lambda: channel(5, (6, 5), None, "dg"), lambda: channel(8, (45, 44), "quad"),
                                  lambda: channel(8, (45, 44), "quad", "dg")])
def test_closure_on_every_path(make):
    import oracle
    from oracle import closure as C
    from paper_2509_19171_amd import sel

    c = make()
    o = oracle.from_case(c)
    X = C.features(o).reshape(-1, 6)
    blob = I.closure_blob(7, mean=X.mean(0), std=np.abs(X).max(0) + 1e-30, b4=0.5)
    C.step_with_closure(o, C.unpack(blob.astype(np.float64)), 2)
    rho_o, u_o = o.moments()
    for prec, tol in (("fp64", 1e-8), ("fp32dev", 1e-5)):
        g = sel.from_case(c, prec, closure=blob)
        g.step(2)
        rho, u = g.moments()
        plain = sel.from_case(c, prec)
        plain.step(2)
        acts = uerr(plain.moments()[1], u_o)
        print(f"[gpu] {c.name} N {c.N} E {c.E} {prec}: rho {nerr(rho, rho_o):.2e} u {uerr(u, u_o):.2e} acts {acts:.2e}", flush=True)
        assert nerr(rho, rho_o) < tol and uerr(u, u_o) < tol, prec
        assert acts > 10 * uerr(u, u_o)
