"""Row blocks of their own height for the strips at the x sides (a pair of waves per item): the
bits of one-step launches whatever the height asked for."""
import numpy as np
import pytest

from paper_1511_00242_amd import inputs as I
from paper_1511_00242_amd import lbfv as L

pytestmark = pytest.mark.gpu

STEPS = 10


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    torch.cuda.init()


def _run(w, scheme, precision, pairs, rows):
    with_type = dict(compute=L.LBFV_FP32, storage=L.LBFV_STORE_DEV_FP32) if precision == "f32" else {}
    ctx = L.Context(w.xf, w.yf, w.tau, w.dt, bcs=w.bcs, check_every=0, **with_type)
    ctx.init_equilibrium(w.rho, w.ux, w.uy)
    if pairs:
        ctx.set_time_block(2)
    ctx.set_tile(rows, 1)
    ctx.set_wave_pairs(pairs)
    ctx.step(scheme, STEPS)
    f = ctx.get_f()
    ctx.close()
    return f


# 120: two strips (no blocks of their own); 121: three, the last of one column; 181; walls on every
# side, or inflow, outflow and a symmetry plane with a wall segment
@pytest.mark.parametrize("scheme,precision", [(L.LBFV_DUGKS, "f64"), (L.LBFV_BKG, "f64"), (L.LBFV_DUGKS, "f32")])
@pytest.mark.parametrize("w", [I.cavity(120), I.cavity(121), I.cavity(181), I.boundary_layer(240, 97)],
                         ids=["cavity120", "cavity121", "cavity181", "layer240x97"])
def test_side_blocks_give_the_bits_of_single_steps(w, scheme, precision):
    one = _run(w, scheme, precision, 0, 8)
    assert np.isfinite(one).all()
    for rows in (1, 2, 5, 8, 19, w.ny - 1, w.ny):
        assert np.array_equal(one, _run(w, scheme, precision, 1, rows)), rows
