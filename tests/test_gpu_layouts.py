"""When a context moves its state to another strip layout: launches that a program captured, and
buffers that it owns, go on naming the state; and a shape that is set is the one that runs."""
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


def captured_totals(ctx, s):
    import torch
    out = torch.zeros(4, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.totals_device(out.data_ptr())

    def replay():
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        return out.cpu().numpy()[:3].copy()
    return replay


def set_rows(ctx):
    ctx.set_tile(24, 4)


def set_pairs(ctx):
    ctx.set_wave_pairs(True)


# chains of four (56 columns) and pairs (60 columns) unasked
@pytest.mark.parametrize("sides", [False, True])
@pytest.mark.parametrize("shape", [set_rows, set_pairs])
def test_captured_totals_after_a_long_call_and_a_shape(sides, shape):
    import torch
    w = I.cavity(520, stretched=False) if sides else I.taylor_green(450)
    s = torch.cuda.Stream()
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0, stream=s.cuda_stream) as ctx:
        ctx.init_equilibrium(w.rho, w.ux * 30, w.uy * 30 + 0.01)
        ctx.dugks_step(40)
        totals = captured_totals(ctx, s)
        for k in (2, 64, 100):
            ctx.dugks_step(k)
            assert np.array_equal(totals(), ctx.totals()), k
            if k == 2:
                shape(ctx)
                assert np.array_equal(totals(), ctx.totals())


def test_captured_steps_after_a_shape_on_a_moved_layout():
    """A shape set after a long call, then steps captured, then long calls again."""
    import torch
    w = I.taylor_green(450)
    s = torch.cuda.Stream()
    outs = []
    for captured in (True, False):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0, stream=s.cuda_stream) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            if not captured:
                ctx.set_tile(24, 4)
                ctx.dugks_step(40 + 4 + 64 + 4)
            else:
                ctx.dugks_step(40)
                ctx.set_tile(24, 4)
                torch.cuda.synchronize()
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g, stream=s):
                    ctx.dugks_step(4)
                g.replay()
                torch.cuda.synchronize()
                ctx.dugks_step(64)
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
            outs.append(ctx.get_f())
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("sides", [False, True])
def test_bound_buffers_can_be_saved_and_restored(sides):
    """A program that owns the two buffers saves the state by copying them and puts it back after
    an even number of steps; no call that it makes asks for another layout."""
    import torch
    w = I.cavity(520, stretched=False) if sides else I.taylor_green(450)
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
        a, b = ctx.bind_torch_buffers()
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        ctx.dugks_step(4)
        f0 = ctx.get_f()
        torch.cuda.synchronize()
        kept = a.clone(), b.clone()
        ctx.dugks_step(40)
        f1 = ctx.get_f()
        torch.cuda.synchronize()
        a.copy_(kept[0])
        b.copy_(kept[1])
        torch.cuda.synchronize()
        assert np.array_equal(ctx.get_f(), f0)
        ctx.dugks_step(40)
        assert np.array_equal(ctx.get_f(), f1)


def kernels_of(call):
    """Names of the kernels that a call runs, graph replays included."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return {e.name for e in p.events()}


def test_the_time_block_that_is_set_is_the_one_that_runs():
    """After a long call in which a context with sides took pairs of waves by itself, two steps per
    launch asked for without pairs run on one wave per item, in graph replays too."""
    w = I.cavity(520, stretched=False)
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        unasked = kernels_of(lambda: ctx.dugks_step(128))
        ctx.set_time_block(2)
        assert not ctx.get_wave_pairs()
        asked = kernels_of(lambda: ctx.dugks_step(128))
    steps = lambda names: sorted(n for n in names if "step2b" in n)   # noqa: E731
    print(unasked, asked, flush=True)
    assert steps(unasked) and all("step2bp" in n for n in steps(unasked))
    assert steps(asked) and not any("step2bp" in n for n in steps(asked))


def test_a_call_of_no_steps_moves_nothing():
    w = I.taylor_green(450)
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        ctx.dugks_step(32)
        ctx.set_tile(8, 4)
        moved = lambda n: any("relayout" in k for k in kernels_of(lambda: ctx.dugks_step(n)))   # noqa: E731
        assert not moved(0)
        assert moved(1) and not moved(1)
