"""Calls of sel_step captured in a graph: a state that lies in its first array
again after the captured calls is advanced by every replay. Calls without a
filter leave it there, and so do pairs of calls with one; small 2D meshes with the
continuous coupling return it in every call.

The replayed kernels are those of the eager calls with the same operands, so
the states are compared bit for bit."""
import numpy as np
import pytest

from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def replays(c, calls, prec="fp64"):
    from paper_2509_19171_amd import sel

    eager, stream = sel.from_case(c, prec), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = sel.from_case(c, prec, stream=stream)
        sim.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            for n in calls:
                sim.step(n)
    for k in range(4):
        for n in calls:
            eager.step(n)
        eager.sync()
        with torch.cuda.stream(stream):
            g.replay()
        stream.synchronize()
        torch.zeros(1 << 16, device="cuda").sum().item()  # the program's own work in between
        print(f"[gpu] replay {k} {c.name} {c.filter} {c.rk} {calls} {c.coupling}", flush=True)
        assert np.array_equal(sim.get_f(), eager.get_f()), k


@pytest.mark.parametrize("calls,coupling", [((1,), "cg"), ((1, 1), "cg"), ((2, 3), "cg"), ((1, 1), "dg")])
@pytest.mark.parametrize("rk", ["ssprk3", "printed4"])
@pytest.mark.parametrize("filt", [None, "quad"])
def test_replayed_calls_advance_the_state(filt, rk, calls, coupling):
    c = I.case_tgv2d(nel=4, N=5, filt=filt)
    c.rk, c.coupling = rk, coupling
    replays(c, calls)


@pytest.mark.parametrize("curved", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32dev"])
@pytest.mark.parametrize("N,Q,filt,calls", [(3, 27, "quad", (1, 2)), (3, 27, None, (2,)), (7, 27, "quad", (2, 1)), (5, 19, None, (1,))])
def test_replayed_3d_calls(N, Q, filt, calls, prec, curved):
    c = I.case_tgv3d(nel=2, N=N, Q=Q, steps=0, filt=filt)
    replays(I.off_affine(c) if curved else c, calls, prec)


@pytest.mark.parametrize("coupling", ["cg", "dg"])
def test_replayed_large_2d_calls(coupling):
    c = I.case_tgv2d(nel=46, N=8, filt="quad")
    c.coupling = coupling
    replays(c, (1, 1))
