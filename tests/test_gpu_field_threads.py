"""Fields of one object asked for by several threads at once."""
from concurrent.futures import ThreadPoolExecutor

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


def test_threads_read_and_write_the_cases_of_a_batch():
    # one chunk, and fields that several copying threads share
    cases = [I.taylor_green(n) for n in (24, 130, 301, 470, 90, 24)]
    rng = np.random.default_rng(1)
    states = [rng.random((9, w.ny, w.nx)) + 0.1 for w in cases]
    b = L.Batch(cases, compute=L.LBFV_FP64, storage=L.LBFV_STORE_NATIVE)

    def use(i):
        import torch
        torch.cuda.set_device(0)
        ok = True
        for _ in range(4):
            b.set_f(i, states[i])
            ok = ok and np.array_equal(b.get_f(i), states[i])
            ok = ok and np.abs(b.moments(i)[0] - states[i].sum(0)).max() < 1e-14
        return ok

    with ThreadPoolExecutor(6) as pool:
        assert all(pool.map(use, range(len(cases))))
    b.close()


def test_threads_read_one_context():
    w = I.cavity(300, stretched=False)
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        ctx.dugks_step(20)
        f, m = ctx.get_f(), ctx.moments()

        def use(k):
            import torch
            torch.cuda.set_device(0)
            if k & 1:
                return np.array_equal(ctx.get_f(), f)
            return all(np.array_equal(a, b) for a, b in zip(ctx.moments(), m))

        with ThreadPoolExecutor(4) as pool:
            assert all(pool.map(use, range(24)))
