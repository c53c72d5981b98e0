"""GPU: combinations of schedule settings that share state between launches."""
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


def make(fd6, w, precision="fp32", variant="55p", layout="soa"):
    box = fd6.Box(w.shape, precision, variant, layout=layout)
    box.set_params(w.nu, w.cs, w.dx, w.dy, w.dz, w.dt)
    box.init_fields(w.fields)
    return box


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("fused_first", [False, True])
def test_fused_substeps_with_the_direct_kernels(fd6, fused_first, graph):
    """Shape 0 asked for beside the fused substeps, in either order: bit for bit
    the plain steps of shape 0, with and without diagnostics and replayed."""
    import torch
    w = si.noise_box((14, 19, 37), seed=41)
    ref, box = make(fd6, w), make(fd6, w)
    ref.set_tile(0)
    if fused_first:
        box.set_fused_substeps(True)
    box.set_tile(0)
    box.set_fused_substeps(True)
    box.set_graph(graph)
    d = [torch.zeros(5, dtype=torch.float64, device="cuda:0") for _ in range(2)]
    for b, x in ((ref, d[0]), (box, d[1])):
        b.step(3)
        b.step_reduce(2, x)
    for a, b in zip(ref.get_fields(), box.get_fields()):
        assert np.array_equal(a, b)
    assert torch.equal(d[0], d[1])
    ref.close()
    box.close()


# whole columns in several rounds (a tile of its own for substeps 2 and 3 with a
# force), a ragged box, a narrow one
@pytest.mark.parametrize("shape", [(8, 264, 1056), (41, 50, 150), (40, 9, 20)])
@pytest.mark.parametrize("precision,variant,layout", [
    ("fp32", "55p", "aos"), ("fp32", "55p", "soa"), ("fp32", "19p", "soa"),
    ("fp64", "55p", "soa"), ("fp64", "19p", "soa"), ("fp32_acc64", "55p", "soa")])
@pytest.mark.parametrize("forced", [False, True])
def test_the_librarys_shape_with_and_without_a_force(fd6, shape, precision, variant, layout,
                                                     forced):
    """Bit for bit the state of shape 1 in chunks of 8 planes, plain steps and steps
    with diagnostics; these to 1e-12 (FP64 partial sums grouped by tile)."""
    import torch
    w = si.noise_box(shape, seed=42)
    out = []
    for fixed in (False, True):
        b = make(fd6, w, precision, variant, layout)
        if forced:
            b.set_forcing({"k": (1.0, 0.0, 2.0), "e": (0.0, 1.0, 0.0), "f0": 0.02, "phase": 0.4})
        if fixed:
            b.set_tile(1)
            b.set_zchunk(8)
        d = torch.zeros(5, dtype=torch.float64, device="cuda:0")
        b.step(1)
        b.step_reduce(1, d)
        out.append((b.get_fields(), d.cpu().numpy()))
        b.close()
    for x, y in zip(out[0][0], out[1][0]):
        assert np.array_equal(x, y)
    assert np.all(np.abs(out[0][1] - out[1][1]) <= 1e-12 * np.abs(out[1][1]).max())


@pytest.mark.parametrize("precision", ["fp32", "fp64", "fp32_acc64"])
@pytest.mark.parametrize("shapes", [[(6, 6, 6)], [(33, 7, 40), (8, 9, 10)],
                                    [(48, 48, 48), (96, 96, 96), (32, 32, 32)]])
def test_an_ensemble_of_structures_left_to_the_library(fd6, shapes, precision):
    """Chunks fitted to the boxes, array of structures, against whole boxes of shape 1."""
    out = []
    for fixed in (False, True):
        b = fd6.Batch(shapes, precision, layout="aos")
        ws = [si.noise_box(s, seed=43 + i) for i, s in enumerate(shapes)]
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


# z: time step times the viscous eigenvalue of the grid-scale mode; the scheme is stable
# to 2.51
@pytest.mark.parametrize("z", [0.1, 0.6, 1.0, 2.4])
def test_rounding_error_of_the_formed_register_up_to_the_diffusive_limit(fd6, orc, z):
    """FP32 error of one step against the direct kernel's, which keeps the register in
    memory.  Of the errors e1, e2, e3 of the substeps' stored states, on a mode of
    eigenvalue -x per step, the sweeps leave (1/2 + x^2/2) e1, (0.32 - 8/15 x) e2, e3, the
    kept register (1 - 5/6 x + x^2/2) e1, (1 - 8/15 x) e2, e3: the ratio may not pass the
    worst mode's, with a tenth for 24000 values and the register's own rounding."""
    shape, h, nu = (24, 28, 36), 0.1, 1e-2
    dt = z / (nu * 4.0 * 6.0444 / h ** 2)
    rng = np.random.default_rng(4)
    f = [(1e-3 * rng.normal(size=shape)).astype(np.float32).astype(np.float64) for _ in range(4)]
    ref = orc.rk3(f, nu, 1e-3, h, h, h, dt, "55p", 1)
    err = []
    for tile in (0, None):
        box = fd6.Box(shape, "fp32")
        box.set_params(nu, 1e-3, h, h, h, dt)
        if tile is not None:
            box.set_tile(tile)
        box.init_fields(f)
        box.step(1)
        err.append(np.sqrt(np.mean([np.mean((a - b) ** 2)
                                    for a, b in zip(box.get_fields()[1:], ref[1:])])))
        box.close()
    x = np.linspace(0.0, z, 200)
    swept = (0.5 + x * x / 2) ** 2 + (0.32 - 8 / 15 * x) ** 2 + 1
    kept = (1 - 5 / 6 * x + x * x / 2) ** 2 + (1 - 8 / 15 * x) ** 2 + 1
    assert err[1] <= 1.1 * np.sqrt((swept / kept).max()) * err[0]


@pytest.mark.parametrize("precision", ["fp32", "fp64", "fp32_acc64"])
def test_an_ensemble_of_equal_and_unequal_time_steps(fd6, precision):
    """Each box with its own time step, equal to its neighbour's or not: bit for bit
    its single-box run."""
    w = si.noise_box((9, 10, 40), seed=44)
    dts = [w.dt, w.dt, 0.7 * w.dt, w.dt, 0.7 * w.dt, 0.7 * w.dt]
    b = fd6.Batch([w.shape] * len(dts), precision)
    b.set_params([(w.nu, w.cs, w.dx, w.dy, w.dz, dt) for dt in dts])
    for i in range(len(dts)):
        b.init_fields(i, w.fields)
    b.step(2)
    for i, dt in enumerate(dts):
        box = fd6.Box(w.shape, precision)
        box.set_params(w.nu, w.cs, w.dx, w.dy, w.dz, dt)
        box.init_fields(w.fields)
        box.step(2)
        for x, y in zip(b.get_fields(i), box.get_fields()):
            assert np.array_equal(x, y), (i, dt)
        box.close()
    b.close()
