"""Wall segments on meshes that are periodic in x: the segment ends at the seam, where the cells
on its two sides see different ghost rows.  Every launch form a context may take has to give the
bits of one-step launches there, and the oracle's result."""
import os
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_1511_00242_amd import inputs as I
from paper_1511_00242_amd import lbfv as L

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from test_gpu_parity import ALL_SCHEMES, TOL64, oracle_case, perturbed_state, rel  # noqa: E402

pytestmark = pytest.mark.gpu

FORMS = {"f64": (L.LBFV_FP64, L.LBFV_STORE_NATIVE), "f32": (L.LBFV_FP32, L.LBFV_STORE_DEV_FP32),
         "f16": (L.LBFV_FP32, L.LBFV_STORE_DEV_FP16)}


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    torch.cuda.set_device(0)
    yield


def seam_sides(nx):
    """symmetry, a wall or an inflow ahead of the segment; a segment from the first cell, inside
    the mesh and of the last cell alone; on one y side or on both"""
    p = "periodic"
    return [
        [p, p, ("wall_from", nx // 3, 0.05, 0.0, "symmetry"), ("wall", 0.01, 0.0)],
        [p, p, ("wall", 0.0, 0.0), ("wall_from", 0, 0.05, 0.0, ("wall", -0.02, 0.0))],
        [p, p, ("wall_from", nx - 1, 0.05, 0.01, ("inflow", 1.0, 0.02, 0.0)),
         ("wall_from", nx // 2, -0.03, 0.0, ("outflow", 0))],
    ]


def workload(nx, ny, sides):
    xf = I.tanh_faces(nx, 0.8, 0.0, nx / 8.0) if nx < 200 else I.uniform_faces(nx, 0.0, nx / 8.0)
    yf = I.uniform_faces(ny, 0.0, ny / 8.0)
    rho, ux, uy = I.random_state_fields(ny, nx, nx * 31 + ny, amp_u=0.04, amp_rho=0.02)
    return I.Workload("seam", xf, yf, 0.01, I.cfl_dt(xf, yf, 0.5), sides, rho, ux, uy)


def advance(w, form, f0, plan, shape):
    compute, storage = FORMS[form]
    with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, compute=compute, storage=storage, check_every=7) as ctx:
        ctx.set_f(f0)
        shape(ctx)
        for scheme, n in plan:
            ctx.step(scheme, n)
        return ctx.get_f()


def one_step(ctx):
    ctx.set_tile(3, 2)


def two_steps(ctx):
    ctx.set_time_block(2)


def pairs(ctx):
    ctx.set_time_block(2)
    ctx.set_tile(5, 1)
    ctx.set_wave_pairs(True)


def unasked(ctx):
    pass


def tuned(ctx):
    ctx.autotune(L.LBFV_DUGKS, 4)


@pytest.mark.parametrize("nx,ny", [(2, 3), (24, 16), (63, 9), (130, 37)])
def test_segments_at_a_periodic_seam(nx, ny):
    for k, sides in enumerate(seam_sides(nx)):
        w = workload(nx, ny, sides)
        ora = oracle_case(w, 1)
        f0 = perturbed_state(ora, w, 5 + k)
        for scheme, oscheme in ALL_SCHEMES:
            want = advance(w, "f64", f0, [(scheme, 9)], one_step)
            if scheme in (L.LBFV_DUGKS, L.LBFV_BKG):
                assert rel(want, ora.run(f0, oscheme, 9)) < TOL64, (k, scheme)
            for shape in (unasked, two_steps, pairs):
                assert np.array_equal(want, advance(w, "f64", f0, [(scheme, 9)], shape)), (k, scheme, shape.__name__)
        for form in ("f32", "f16"):
            want = advance(w, form, f0, [(L.LBFV_DUGKS, 5), (L.LBFV_BKG, 4)], one_step)
            for shape in (unasked, two_steps, pairs):
                got = advance(w, form, f0, [(L.LBFV_DUGKS, 5), (L.LBFV_BKG, 4)], shape)
                assert np.array_equal(want, got), (k, form, shape.__name__)


def test_the_tuned_shape_at_a_periodic_seam():
    w = workload(100, 40, seam_sides(100)[0])
    f0 = perturbed_state(oracle_case(w, 1), w, 3)
    plan = [(L.LBFV_DUGKS, 12)]
    assert np.array_equal(advance(w, "f64", f0, plan, one_step), advance(w, "f64", f0, plan, tuned))


def test_a_large_mesh_with_a_segment_at_the_seam():
    """A mesh that takes several steps per launch unasked; the segment is set between calls."""
    w = workload(520, 500, ["periodic", "periodic", "symmetry", ("wall", 0.0, 0.0)])
    f0 = perturbed_state(oracle_case(w, 1), w, 3)
    outs = []
    for march in (True, False):
        with L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs) as ctx:
            ctx.set_f(f0)
            if march:
                ctx.set_tile(24, 4)
            ctx.dugks_step(20)
            ctx.set_sides(seam_sides(w.nx)[0])
            ctx.dugks_step(37)
            outs.append(ctx.get_f())
    assert np.all(np.isfinite(outs[0])) and np.array_equal(outs[0], outs[1])
