"""Calls of a few steps on meshes that take patches in longer ones: one step is marched where that
is faster, and calls that mix patches and marches keep the bits and the buffer."""
import os
import sys

import numpy as np
import pytest

from paper_1511_00242_amd import inputs as I
from paper_1511_00242_amd import lbfv as L

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_gpu_layouts import kernels_of  # noqa: E402

pytestmark = pytest.mark.gpu

FORMS = {"f64": (L.LBFV_FP64, L.LBFV_STORE_NATIVE), "f32": (L.LBFV_FP32, L.LBFV_STORE_DEV_FP32),
         "f16": (L.LBFV_FP32, L.LBFV_STORE_DEV_FP16)}


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.set_device(0)
    yield


def steps_run(call):
    return {n for n in kernels_of(call) if "patch" in n or "step" in n or "lbfv::batch" in n}


@pytest.mark.parametrize("form,scheme,n", [("f64", L.LBFV_BKG, 620), ("f32", L.LBFV_BKG, 700),
                                           ("f32", L.LBFV_DUGKS, 900), ("f16", L.LBFV_BKG, 1000)])
def test_single_steps_of_larger_meshes_are_marched(form, scheme, n):
    w = I.taylor_green(n)
    compute, storage = FORMS[form]
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, compute=compute, storage=storage, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        one, five = (steps_run(lambda: ctx.step(scheme, k)) for k in (1, 9))
        assert one and not any("patch" in k for k in one), one
        assert any("patch" in k for k in five), five


def test_single_steps_of_larger_batches_are_marched():
    cases = [I.taylor_green(512)] * 2
    b = L.Batch(cases)
    for i, w in enumerate(cases):
        b.init_equilibrium(i, w.rho, w.ux, w.uy)
    one, nine = (steps_run(lambda: b.step(L.LBFV_DUGKS, k)) for k in (1, 9))
    b.close()
    assert one and not any("patch" in k for k in one), one
    assert any("patch" in k for k in nine), nine


# just above the sizes from which single steps are marched
@pytest.mark.parametrize("form,kind,n", [("f64", "vortex", 600), ("f32", "vortex", 820), ("f32", "cavity", 820),
                                         ("f16", "vortex", 820)])
def test_short_calls_keep_the_bits(form, kind, n):
    w = I.cavity(n, stretched=False) if kind == "cavity" else I.taylor_green(n)
    compute, storage = FORMS[form]
    outs = []
    for march in (True, False):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, compute=compute, storage=storage, check_every=4) as ctx:
            ctx.init_equilibrium(w.rho, w.ux * 10 + 0.01, w.uy * 10)
            if march:
                ctx.set_tile(16, 4)
            for k in (1, 2, 3, 4, 5, 8, 11):
                ctx.step(L.LBFV_DUGKS if k & 1 else L.LBFV_BKG, k)
            outs.append(ctx.get_f())
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("form", ["f64", "f32"])
def test_short_calls_of_batches_keep_the_bits(form):
    compute, storage = FORMS[form]
    cases = [I.taylor_green(512), I.cavity(300, stretched=False), I.taylor_green(64)]
    for scheme in (L.LBFV_DUGKS, L.LBFV_BKG):
        outs = []
        for march in (True, False):
            b = L.Batch(cases, compute=compute, storage=storage)
            for i, w in enumerate(cases):
                b.init_equilibrium(i, w.rho, w.ux * 10 + 0.01, w.uy * 10)
            b.set_shape(graph_steps=3)
            if march:
                b.set_shape(rows=5)
            for k in (1, 2, 3, 4, 5, 8, 11, 29):
                b.step(scheme, k)
            outs.append([b.get_f(i) for i in range(len(cases))])
            b.close()
        for f, g in zip(*outs):
            assert np.array_equal(f, g)


def test_heights_of_one_step_follow_the_layout():
    """After a long call the strips are narrower and more: the row blocks of one-step launches
    still fill one round of resident waves, and no part of a second one."""
    w = I.taylor_green(2100)
    items = []
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        for strip in (62, 56):
            rows = ctx.get_tile()[0]
            items.append(-(-w.nx // strip) * -(-w.ny // rows))
            ctx.dugks_step(32)
    print(items)
    assert items[1] <= items[0] * 1.03


@pytest.mark.parametrize("kind,few", [("vortex", 2), ("cavity", 3)])
def test_single_steps_move_the_state_back(kind, few):
    """Calls too short for launches of several steps, many in a row after a long one: the state
    goes back to the strips of one-step launches, and to the others in the next long call.  A
    program that holds captured work keeps the layout."""
    import torch
    w = I.cavity(1100, stretched=False) if kind == "cavity" else I.taylor_green(1100)
    moved = lambda call: any("relayout" in k for k in kernels_of(call))   # noqa: E731
    outs = []
    for how in ("march", "auto", "captured"):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
            ctx.init_equilibrium(w.rho, w.ux, w.uy)
            if how == "march":
                ctx.set_tile(24, 4)
                ctx.dugks_step(32 + 12 * few + 32 + 1 + 4)
                outs.append(ctx.get_f())
                continue
            assert moved(lambda: ctx.dugks_step(32))
            if how == "captured":
                out = torch.zeros(4, dtype=torch.float64, device="cuda")
                ctx.totals_device(out.data_ptr())
            back = [moved(lambda: ctx.dugks_step(few)) for _ in range(12)]
            assert back.count(True) == (how == "auto") and not any(back[:8 // few])
            assert moved(lambda: ctx.dugks_step(32)) == (how == "auto")
            assert not moved(lambda: ctx.dugks_step(1)) and not moved(lambda: ctx.dugks_step(4))
            outs.append(ctx.get_f())
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("form,n,low,high", [("f64", 300, 8, 12), ("f64", 8, 1, 8), ("f32", 300, 3, 12),
                                             ("f32", 4096, 32, 100), ("f16", 3000, 32, 100)])
def test_default_heights_of_chains(form, n, low, high):
    """Four steps per launch without a height: on a small mesh not so low that chains share a CU for
    little, nor, on a large one in FP32 arithmetic, so high that a launch is one round of tall blocks."""
    xf, yf = I.uniform_faces(n), I.uniform_faces(n)
    compute, storage = FORMS[form]
    with L.Context(xf, yf, 0.01, I.cfl_dt(xf, yf, 0.5), bcs=["periodic"] * 4, compute=compute, storage=storage) as ctx:
        ctx.set_time_block(4)
        rows = ctx.get_tile()[0]
    print(form, n, rows)
    assert low <= rows <= high


def launches_of(call):
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return sum("patch_kernel" in e.name or "patch_ptr_kernel" in e.name for e in p.events())


def test_tuned_patches_take_the_fewest_launches():
    """A form that the autotuner picked has no buffer to end in, as its marches have none, unless a
    program holds captured work; then calls keep the parity of their steps."""
    import torch
    w = I.taylor_green(64)
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        assert launches_of(lambda: ctx.dugks_step(2)) == 2
        ctx.autotune(L.LBFV_DUGKS, 20)
        assert launches_of(lambda: ctx.dugks_step(2)) == 1
        out = torch.zeros(4, dtype=torch.float64, device="cuda")
        ctx.totals_device(out.data_ptr())
        assert launches_of(lambda: ctx.dugks_step(2)) == 2
        f = ctx.get_f()
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0) as ctx:
        ctx.init_equilibrium(w.rho, w.ux, w.uy)
        ctx.set_tile(4, 1)
        ctx.dugks_step(6)
        assert np.array_equal(ctx.get_f(), f)
