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


# small patches of many steps; a batch that takes two steps per launch
BATCHES = {"small": [I.taylor_green(33), I.taylor_green(70), I.cavity(40, stretched=False)],
           "cavities": [I.cavity(256, stretched=False)] * 8}


# even and odd graph lengths K; calls of one replay with 2, 4, 6 or 8 steps per launch, of several,
# and of none, with and without steps left over
@pytest.mark.parametrize("name", sorted(BATCHES))
@pytest.mark.parametrize("K", [2, 3, 5, 7])
def test_captured_steps_follow_calls_that_replay_graphs(name, K):
    import torch
    cases = BATCHES[name]
    calls = (2, 2 * K, 4 * K, 6 * K, 8 * K, 8 * K + 6, 6)
    s = torch.cuda.Stream()
    outs = []
    for captured in (False, True):
        b = L.Batch(cases, stream=s.cuda_stream, compute=L.LBFV_FP64, storage=L.LBFV_STORE_NATIVE)
        for i, w in enumerate(cases):
            b.init_equilibrium(i, w.rho, w.ux, w.uy)
        if captured:
            b.set_shape(graph_steps=K)
            assert b.get_shape()[0] == K
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


def test_a_graph_length_beyond_every_call():
    """The longest graph length: no call replays a graph, every one goes as single launches."""
    w = I.taylor_green(33)
    outs = []
    for K in (2 ** 31 - 1, 2 ** 30 + 1, 2):
        b = L.Batch([w])
        b.init_equilibrium(0, w.rho, w.ux, w.uy)
        b.set_shape(graph_steps=K)
        b.step(L.LBFV_BKG, 37)
        outs.append(b.get_f(0))
        b.close()
    assert np.array_equal(outs[0], outs[2]) and np.array_equal(outs[1], outs[2])
