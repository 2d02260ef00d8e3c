"""Graph lengths of a batch: whatever the length, a call of an even number of steps leaves the
state in the buffer it was in, so that work a program captured before goes on from it."""
import numpy as np
import pytest

from paper_1511_00242_amd import inputs as I
from paper_1511_00242_amd import lbfv as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.set_device(0)
    yield


# even and odd graph lengths; calls of no, one and several replays, with and without steps left over
@pytest.mark.parametrize("graph_steps", [2, 3, 5, 7])
def test_captured_steps_follow_calls_that_replay_graphs(graph_steps):
    import torch
    cases = [I.taylor_green(33), I.taylor_green(70), I.cavity(40, stretched=False)]
    calls = (2, 12, 24, 40, 54, 6)
    s = torch.cuda.Stream()
    outs = []
    for captured in (False, True):
        b = L.Batch(cases, stream=s.cuda_stream)
        for i, w in enumerate(cases):
            b.init_equilibrium(i, w.rho, w.ux, w.uy)
        if captured:
            b.set_shape(graph_steps=graph_steps)
            b.step(L.LBFV_DUGKS, 2)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            # (shorter than a graph of the batch: one-step launches)
            with torch.cuda.graph(g, stream=s):
                for _ in range(4):
                    b.step(L.LBFV_DUGKS, 1)
        else:
            b.set_shape(rows=4)
            b.step(L.LBFV_DUGKS, 2)
        for n in calls:
            b.step(L.LBFV_DUGKS, n)
            torch.cuda.synchronize()
            if captured:
                g.replay()
                torch.cuda.synchronize()
            else:
                b.step(L.LBFV_DUGKS, 4)
            outs.append([b.get_f(i) for i in range(len(cases))])
        b.close()
    for k, n in enumerate(calls):
        for i in range(len(cases)):
            assert np.array_equal(outs[k][i], outs[len(calls) + k][i]), (n, i)
