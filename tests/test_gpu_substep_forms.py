"""GPU: the sweeps that form the RK3 register from the two state sets, and the
divergence sweep of the 19-point method, at the sizes and time steps where they
could go wrong.

Tolerances: FP64 within 1e-12 of the oracle (as every FP64 parity test); a time
step too small for any increment leaves the state as it is, bit for bit.
"""
import numpy as np
import pytest

import synthetic_inputs as si

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fd6():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible ROCm GPU")
    import paper_1707_08900_amd as p
    return p


def make(fd6, w, precision, variant="55p", layout="soa", dt=None):
    box = fd6.Box(w.shape, precision, variant, layout=layout)
    box.set_params(w.nu, w.cs, w.dx, w.dy, w.dz, w.dt if dt is None else dt)
    box.init_fields(w.fields)
    return box


# the divergence sweep's tile is 64 x 8: one tile exactly, one cell short of it
# and past it, two tiles, fewer planes than a z stencil's span
@pytest.mark.parametrize("shape", [(6, 8, 64), (7, 7, 63), (12, 9, 65), (6, 16, 128),
                                   (17, 15, 127), (20, 17, 129)])
def test_19p_at_the_edges_of_the_divergence_tile(fd6, orc, shape):
    w = si.noise_box(shape, seed=31)
    box = make(fd6, w, "fp64", "19p")
    box.step(2)
    out = box.get_fields()
    box.close()
    ref = orc.rk3(w.fields, w.nu, w.cs, w.dx, w.dy, w.dz, w.dt, "19p", 2)
    for a, b in zip(out, ref):
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))


@pytest.mark.parametrize("precision,dt", [("fp32", 1e-30), ("fp32", 1e-39), ("fp32", 1e-60),
                                          ("fp64", 1e-300), ("fp64", 1e-310),
                                          ("fp32_acc64", 1e-39)])
@pytest.mark.parametrize("variant", ["55p", "19p"])
def test_vanishing_time_steps_leave_the_state(fd6, precision, dt, variant):
    """1 / dt enters the form of the register: it must not overflow into NaN
    where the step itself is harmless."""
    w = si.noise_box((9, 10, 40), seed=32)
    w.fields = [np.where(np.abs(f) < 1e-6, 1e-3, f) for f in w.fields]
    box = make(fd6, w, precision, variant, dt=dt)
    before = box.get_fields()
    box.step(3)
    for a, b in zip(box.get_fields(), before):
        assert np.array_equal(a, b)
    box.close()


@pytest.mark.parametrize("layout", ["soa", "aos"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_acc64"])
def test_the_right_hand_side_leaves_a_run_alone(fd6, precision, layout):
    """The hook between steps changes no later state (the register is formed
    from the state sets, which it may not touch)."""
    w = si.noise_box((14, 19, 70), seed=33)
    a, b = (make(fd6, w, precision, layout=layout) for _ in range(2))
    for s in range(3):
        a.step(1)
        b.rhs()
        b.step(1)
        b.rhs()
    for x, y in zip(a.get_fields(), b.get_fields()):
        assert np.array_equal(x, y)
    a.close()
    b.close()
