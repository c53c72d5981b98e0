"""GPU: the sweeps that form the RK3 register from the two state sets, and the
divergence sweep of the 19-point method, the shapes the library chooses by itself
and the one-pass transfers, at the sizes and time steps where they
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


# Edges where the unset shape's rule turns: one narrow tile and one cell more, a
# wide tile's last column nearly empty, fewer planes than one chunk of 8, chunks
# down to one plane, a box with more tiles than the device holds at once, and one of
# whole columns in several rounds (wide ones from substep 2 on in the FP32 array of
# structures).
@pytest.mark.parametrize("shape", [(6, 8, 32), (7, 9, 33), (13, 75, 65), (32, 32, 32),
                                   (41, 50, 150), (18, 300, 420), (8, 264, 1056)])
@pytest.mark.parametrize("precision,variant,layout", [
    ("fp32", "55p", "aos"), ("fp32", "55p", "soa"), ("fp32", "19p", "soa"),
    ("fp64", "55p", "aos"), ("fp64", "19p", "soa"), ("fp32_acc64", "55p", "aos")])
def test_a_shape_left_to_the_library_gives_the_same_state(fd6, shape, precision, variant, layout):
    """Bit for bit the state of shape 1 in chunks of 8 planes, plain, with the
    diagnostics in the last sweep, with only the chunk set, and replayed; the
    diagnostics to 1e-12 (their FP64 partial sums are grouped by tile)."""
    import torch
    w = si.noise_box(shape, seed=34)
    boxes = [make(fd6, w, precision, variant, layout) for _ in range(4)]
    boxes[0].set_tile(1)
    boxes[0].set_zchunk(8)
    boxes[2].set_zchunk(9)
    boxes[3].set_graph(True)
    out = []
    for b in boxes:
        d = torch.zeros(5, dtype=torch.float64, device="cuda:0")
        b.step(1)
        b.step_reduce(1, d)
        out.append((b.get_fields(), d.cpu().numpy()))
        b.close()
    for f, d in out[1:]:
        for x, y in zip(f, out[0][0]):
            assert np.array_equal(x, y)
        assert np.all(np.abs(d - out[0][1]) <= 1e-12 * np.abs(out[0][1]).max())


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shapes", [[(6, 6, 6)], [(33, 7, 40), (8, 9, 10)],
                                    [(48, 48, 48), (96, 96, 96), (32, 32, 32)]])
def test_an_ensemble_left_to_the_library_gives_the_same_state(fd6, shapes, precision):
    """Chunks fitted to the boxes against whole boxes of shape 1."""
    out = []
    for fixed in (False, True):
        b = fd6.Batch(shapes, precision)
        ws = [si.noise_box(s, seed=35 + i) for i, s in enumerate(shapes)]
        b.set_params([(w.nu, w.cs, w.dx, w.dy, w.dz, w.dt) for w in ws])
        for i, w in enumerate(ws):
            b.init_fields(i, w.fields)
        if fixed:
            b.set_schedule(1, 0)
        b.step(2)
        out.append([b.get_fields(i) for i in range(len(shapes))])
        b.close()
    for x, y in zip(*out):
        assert all(np.array_equal(p, q) for p, q in zip(x, y))


# a wave takes a row, 64 points at a time, 4 rows to a workgroup
@pytest.mark.parametrize("shape", [(6, 6, 6), (7, 9, 63), (6, 11, 64), (9, 7, 65), (6, 13, 200)])
@pytest.mark.parametrize("layout", ["soa", "aos"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_acc64"])
def test_device_transfers_match_host_transfers(fd6, shape, layout, precision):
    """In from the device, out to the host and the other way: the same numbers,
    rounded to the state's type once."""
    import torch
    w = si.noise_box(shape, seed=36)
    a = fd6.Box(shape, precision, layout=layout)
    b = fd6.Box(shape, precision, layout=layout)
    for x in (a, b):
        x.set_params(w.nu, w.cs, w.dx, w.dy, w.dz, w.dt)
    a.init_fields([torch.from_numpy(np.ascontiguousarray(f)).to("cuda:0") for f in w.fields])
    b.init_fields(w.fields)
    kind = np.float64 if precision == "fp64" else np.float32
    for x, y, z in zip(a.get_fields(), b.get_fields_device(), w.fields):
        ref = np.asarray(z).astype(kind).astype(np.float64)
        assert np.array_equal(x, ref) and np.array_equal(y.cpu().numpy(), ref)
    a.close()
    b.close()
