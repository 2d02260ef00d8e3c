"""A batch's first steps while the same thread captures work on another stream."""
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


def test_first_steps_of_a_batch_during_a_capture_elsewhere():
    import torch
    cases = [I.taylor_green(40), I.cavity(30, stretched=False)]
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for capture in (True, False):
        b = L.Batch(cases, stream=mine.cuda_stream)
        for i, w in enumerate(cases):
            b.init_equilibrium(i, w.rho, w.ux, w.uy)
        x = torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        if capture:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=other):
                x.add_(1.0)
                b.step(L.LBFV_DUGKS, 9)
            for _ in range(3):
                g.replay()
                torch.cuda.synchronize()
            assert float(x.sum()) == 24.0
        else:
            b.step(L.LBFV_DUGKS, 9)
        outs.append([b.get_f(i) for i in range(len(cases))])
        b.close()
    for f, g in zip(*outs):
        assert np.array_equal(f, g)
