"""The patch form (several steps per launch, one cell per lane) against the march of one step
per launch: the same bits, on meshes at the edges of its tiles, for every kind of side, scheme
and storage.  A context that sets no launch shape takes the patch form on these meshes; one
that sets a row height marches."""
import os
import sys

import numpy as np
import pytest

from paper_1511_00242_amd import inputs as I
from paper_1511_00242_amd import lbfv as L

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_gpu_parity import ALL_SCHEMES, _mixed_workload, _periodic_workload, _side_sets  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.set_device(0)
    yield


FORMS = {"f64": (L.LBFV_FP64, L.LBFV_STORE_NATIVE), "f32": (L.LBFV_FP32, L.LBFV_STORE_DEV_FP32),
         "bf16": (L.LBFV_FP32, L.LBFV_STORE_DEV_BF16), "f16": (L.LBFV_FP32, L.LBFV_STORE_DEV_FP16)}


def workloads(nx, ny):
    yield _periodic_workload(nx, ny, 5)
    for k, sides in enumerate(_side_sets(nx)):
        w = _mixed_workload(nx, ny)
        yield I.Workload(f"sides{k}_{nx}x{ny}", w.xf, w.yf, w.tau, w.dt, sides, w.rho, w.ux, w.uy)


def advance(w, form, march, u0, plan):
    compute, storage = FORMS[form]
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, compute=compute, storage=storage, check_every=7) as ctx:
        if u0:
            ctx.set_reference_velocity(*u0)
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        if march:
            ctx.set_tile(3, 2)
        for scheme, n in plan:
            ctx.step(scheme, n)
        return ctx.get_f()


# one cell beyond the ghost rows, halos that wrap a short axis, one patch and several per
# axis, patches one cell shorter than their neighbours, a strip seam inside a patch
@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 9), (9, 8), (17, 2), (33, 64), (63, 5), (130, 37)])
@pytest.mark.parametrize("form", sorted(FORMS))
def test_patches_equal_one_step_marches(form, nx, ny):
    for w in workloads(nx, ny):
        schemes = [s for s, _ in ALL_SCHEMES]
        # every number of leftover steps, a check due inside a call, alternating schemes
        plan = [(s, n) for n, s in enumerate(schemes, 1)] + [(schemes[0], 23), (schemes[1], 10)]
        a, b = (advance(w, form, march, None, plan) for march in (True, False))
        assert np.all(np.isfinite(a)), w.name
        assert np.array_equal(a, b), (w.name, np.abs(a - b).max())


def test_patches_with_a_reference_velocity_and_graphs():
    w = I.boundary_layer(100, 70)
    for scheme in (L.LBFV_DUGKS, L.LBFV_BKG):
        a, b = (advance(w, "f32", march, (0.1, 0.0), [(scheme, 5)]) for march in (True, False))
        assert np.array_equal(a, b)
    w = I.taylor_green(20)
    outs = []
    for march in (True, False):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            if march:
                ctx.set_tile(4, 1)
            for n in (301, 300):      # graph replays from either buffer
                ctx.dugks_step(n)
                outs.append(ctx.get_f())
    assert np.array_equal(outs[0], outs[2]) and np.array_equal(outs[1], outs[3])


def test_sides_changed_between_steps_and_autotuned_patches(tmp_path):
    """New kinds of sides need other patches; the autotuner's choice, cached or not, keeps the
    bits and leaves march controls that a program may hand to another context."""
    w = _periodic_workload(40, 30, 9)
    outs = []
    for march in (True, False):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            if march:
                ctx.set_tile(5, 1)
            ctx.bkg_step(9)
            ctx.set_sides([("wall", 0.0, 0.01), ("outflow", 1), "periodic", "periodic"])
            ctx.bkg_step(9)
            ctx.set_sides([("wall", 0.0, 0.01), ("outflow", 0), ("inflow", 1.0, 0.01, 0.0), "symmetry"])
            ctx.bkg_step(8)
            outs.append(ctx.get_f())
    assert np.array_equal(outs[0], outs[1])
    cache = str(tmp_path / "tune.txt")
    for _ in range(2):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            ctx.autotune(L.LBFV_DUGKS, 30, cache)
            shape = (ctx.get_tile(), ctx.get_time_block(), ctx.get_wave_pairs())
            ctx.dugks_step(50)
            f = ctx.get_f()
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            ctx.set_time_block(shape[1])
            ctx.set_tile(*shape[0])
            ctx.set_wave_pairs(shape[2])
            ctx.dugks_step(50)
            assert np.array_equal(ctx.get_f(), f)


def test_captured_steps_replay():
    """Steps captured into a program's own graph: an even number of them advances the state at
    every replay, as one-step launches always did."""
    import torch
    w = I.taylor_green(32)
    s = torch.cuda.Stream()
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0, stream=s.cuda_stream) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        ctx.dugks_step(2)             # uploads what the steps need
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.dugks_step(4)
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
        f = ctx.get_f()
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        ctx.set_tile(4, 1)
        ctx.dugks_step(2 + 12)
        assert np.array_equal(ctx.get_f(), f)


@pytest.mark.parametrize("form", sorted(FORMS))
def test_batch_patches_equal_one_step_marches(form):
    """The batched patch form on uneven meshes and sides, in a batch with and without
    non-periodic sides, through graph replays and leftover steps; and after the autotuner."""
    compute, storage = FORMS[form]
    sided = [w for nx, ny in ((9, 8), (33, 64), (70, 21)) for w in workloads(nx, ny)
             if not any(isinstance(b, tuple) and b[0] == "wall_from" for b in w.bcs)]
    for cases in (sided, [_periodic_workload(nx, ny, 3) for nx, ny in ((9, 9), (64, 10), (130, 37))]):
        for scheme in (L.LBFV_DUGKS, L.LBFV_BKG):
            outs = []
            for how in ("march", "patch", "tuned"):
                b = L.Batch(cases, compute=compute, storage=storage)
                for i, w in enumerate(cases):
                    b.init_equilibrium(i, w.rho, w.ux, w.uy)
                b.set_shape(graph_steps=3)
                if how == "march":
                    b.set_shape(rows=5)
                elif how == "tuned":
                    b.autotune(scheme, 4)
                    if storage in (L.LBFV_STORE_DEV_BF16, L.LBFV_STORE_DEV_FP16) and b.get_time_block() == 2:
                        b.close()   # two steps between roundings: other values by design
                        continue
                for n in (1, 29, 6):
                    b.step(scheme, n)
                outs.append([b.get_f(i) for i in range(len(cases))])
                b.close()
            for other in outs[1:]:
                for w, f, g in zip(cases, outs[0], other):
                    assert np.all(np.isfinite(f)) and np.array_equal(f, g), w.name


@pytest.mark.parametrize("form,sides,nx,ny", [("f64", None, 420, 410), ("f64", 3, 520, 510),
                                              ("f32", None, 601, 590), ("f32", 5, 730, 720)])
def test_unasked_marches_of_several_steps_equal_one_step_marches(form, sides, nx, ny):
    """The smallest meshes on which a context without a shape moves to several steps per launch
    in its long calls: short calls before and after, leftover steps, a switch of scheme, and a
    shape set later."""
    w = _periodic_workload(nx, ny, 5)
    if sides is not None:
        w.bcs = _side_sets(nx)[sides]
    compute, storage = FORMS[form]
    plan = [(L.LBFV_DUGKS, 3), (L.LBFV_DUGKS, 37), (L.LBFV_DUGKS, 2), (L.LBFV_BKG, 18), (L.LBFV_BKG, 1)]
    outs = []
    for march in (True, False):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, compute=compute, storage=storage, check_every=10) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            if march:
                ctx.set_tile(24, 4)
            for scheme, n in plan:
                ctx.step(scheme, n)
            if not march:
                assert ctx.get_time_block() == 1
                ctx.set_tile(24, 4)
            ctx.dugks_step(5)
            outs.append(ctx.get_f())
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("n", [32, 420])
def test_captured_totals_follow_steps(n):
    """lbfv_totals_device captured once and replayed between calls of an even number of steps: the
    state stays in the buffer and the layout that the captured launches name."""
    import torch
    w = I.taylor_green(n)
    s = torch.cuda.Stream()
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0, stream=s.cuda_stream) as ctx:
        ctx.init_equilibrium(w.rho, w.ux * 30, w.uy * 30 + 0.01)
        ctx.dugks_step(2)
        out = torch.zeros(4, dtype=torch.float64, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.totals_device(out.data_ptr())
        for k in (2, 4, 64, 100, 300):
            ctx.dugks_step(k)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy()[:3], ctx.totals()), k
