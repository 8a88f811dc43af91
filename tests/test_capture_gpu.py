"""2D calls of sel_step captured in a graph: a state that lies in its first
array again after the captured calls is advanced by every replay. With the
continuous coupling each call returns it there, filtered or not; with the
discontinuous one a filtered call changes sides, so a pair returns it.

The replayed kernels are those of the eager calls with the same operands, so
the states are compared bit for bit."""
import numpy as np
import pytest

from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("calls,coupling", [((1,), "cg"), ((1, 1), "cg"), ((2, 3), "cg"), ((1, 1), "dg")])
@pytest.mark.parametrize("rk", ["ssprk3", "printed4"])
@pytest.mark.parametrize("filt", [None, "quad"])
def test_replayed_calls_advance_the_state(filt, rk, calls, coupling):
    from paper_2509_19171_amd import sel

    c = I.case_tgv2d(nel=4, N=5, filt=filt)
    c.rk, c.coupling = rk, coupling
    eager, stream = sel.from_case(c, "fp64"), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = sel.from_case(c, "fp64", stream=stream)
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
        print(f"[gpu] replay {k} {filt} {rk} {calls} {coupling}", flush=True)
        assert np.array_equal(sim.get_f(), eager.get_f()), k
