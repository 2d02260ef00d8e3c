"""Fields between host arrays and the state, at the edges of the transfer's chunks and threads:
one chunk, the first size with two threads, ragged last chunks, more chunks than slots."""
import threading

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


def case(nx, ny, seed):
    rho, ux, uy = I.random_state_fields(ny, nx, seed, amp_u=0.05, amp_rho=0.05)
    xf, yf = I.uniform_faces(nx, 0.0, 1.0), I.uniform_faces(ny, 0.0, 1.0)
    return I.Workload("fields", xf, yf, 0.01, I.cfl_dt(xf, yf, 0.5), ["periodic"] * 4, rho, ux, uy)


def check(nx, ny, seed=1):
    w = case(nx, ny, seed)
    f = np.random.default_rng(seed).random((9, ny, nx)) + 0.1
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        # moments of an equilibrium are its fields, to the rounding of nine-term sums
        for got, want in zip(ctx.moments(), (w.rho, w.ux, w.uy)):
            assert np.abs(got - want).max() < 5e-15
        ctx.set_f(f)
        assert np.array_equal(ctx.get_f(), f)
        rho, ux, _ = ctx.moments()
        assert np.abs(rho - f.sum(0)).max() < 1e-14
        assert np.abs(ux - (f[1] - f[3] + f[5] - f[6] - f[7] + f[8]) / f.sum(0)).max() < 1e-14
        drv = [np.random.default_rng(seed + k).random((3, ny, nx)) * 1e-3 for k in range(3)]
        ctx.init_chapman_enskog(w.rho, w.ux, w.uy, *drv)
        return ctx.get_f()


# bytes of f: 9 x 8 per cell; threads from 4 MiB on, 1 MiB chunks
@pytest.mark.parametrize("nx,ny", [(2, 2), (170, 171), (241, 241), (242, 241), (512, 513), (1031, 997)])
def test_fields_round_trip(nx, ny):
    check(nx, ny)


def test_fields_of_several_contexts_at_once_and_batches():
    sizes = [(300, 299), (64, 65), (700, 401), (512, 512)]
    alone = [check(*s, seed=k) for k, s in enumerate(sizes)]
    out = [None] * len(sizes)

    def work(k):
        import torch
        torch.cuda.set_device(0)
        out[k] = check(*sizes[k], seed=k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(alone, out):
        assert b is not None and np.array_equal(a, b)
    cases = [case(nx, ny, k) for k, (nx, ny) in enumerate(sizes)]
    b = L.Batch(cases, compute=L.LBFV_FP64, storage=L.LBFV_STORE_NATIVE)
    for i, (w, f) in enumerate(zip(cases, alone)):
        b.init_equilibrium(i, w.rho, w.ux, w.uy)
        for got, want in zip(b.moments(i), (w.rho, w.ux, w.uy)):
            assert np.abs(got - want).max() < 5e-15
        b.set_f(i, f)
        assert np.array_equal(b.get_f(i), f)
    b.close()
