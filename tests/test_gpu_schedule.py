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
