"""Contexts on hipStreamPerThread, a handle that means another stream in each thread: fields large
enough for several copying threads are read behind the steps queued before, and steps run behind
the fields that are set."""
import threading

import numpy as np
import pytest

from paper_1511_00242_amd import inputs as I
from paper_1511_00242_amd import lbfv as L

pytestmark = pytest.mark.gpu

PER_THREAD = 2   # hipStreamPerThread


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.set_device(0)
    yield


def results(stream, nx, ny, steps):
    rho, ux, uy = I.random_state_fields(ny, nx, 7, amp_u=0.02, amp_rho=0.02)
    xf, yf = I.uniform_faces(nx, 0.0, nx / 8.0), I.uniform_faces(ny, 0.0, ny / 8.0)
    out = []
    with L.Context(xf, yf, 0.01, I.cfl_dt(xf, yf, 0.5), bcs=["periodic"] * 4, stream=stream) as ctx:
        ctx.init_equilibrium(rho, ux, uy)
        for _ in range(3):
            ctx.dugks_step(steps)      # several milliseconds are queued when the fields are asked for
            out += ctx.moments()
            f = ctx.get_f()
            out.append(f)
            ctx.dugks_step(1)
            ctx.set_f(f[:, ::-1].copy())
    return out


# 1, 2 and 8 copying threads for the moments
@pytest.mark.parametrize("nx,ny", [(150, 140), (430, 421), (1031, 997)])
def test_fields_follow_the_steps_of_the_callers_thread(nx, ny):
    want = results(None, nx, ny, 150)
    for got, ref in zip(results(PER_THREAD, nx, ny, 150), want):
        assert np.array_equal(got, ref)
    # from a thread other than the main one, whose stream is another again
    box = []

    def work():
        import torch
        torch.cuda.set_device(0)
        box.append(results(PER_THREAD, nx, ny, 150))

    t = threading.Thread(target=work)
    t.start()
    t.join()
    for got, ref in zip(box[0], want):
        assert np.array_equal(got, ref)
