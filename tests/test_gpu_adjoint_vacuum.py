"""A cell without pressure: its sound speed is zero and the speed's derivative infinite, but Rusanov's flux takes the
other side's wave speed, so J v and J^T w stay finite and are each other's transpose.

One cell of p = 0 in a flow at rest (gamma = 2, so that E = 0 gives p = 0 exactly); the tolerance is that of two roundings of one sum of
products with normwise errors of a few hundred roundings of 2^-53: 1e-13 of ||w|| ||J v||."""
import sys

import numpy as np
import pytest
import torch

import rok_inputs as ri
from tests._util import t64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


@pytest.mark.parametrize("shape,cell", [((18, 17), (5, 4)), ((18, 17), (16, 0)), ((33, 20), (15, 16))])
@pytest.mark.parametrize("recon", ["first", "muscl"])
def test_cell_without_pressure(dev, shape, cell, recon):
    print("[case] adjoint, cell without pressure", shape, cell, recon, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(shape, (0.0, 0.0), (1.0, 1.0), "euler", recon, gamma=2.0)
    rng = np.random.default_rng(8)
    y = np.zeros((4, shape[1], shape[0]))
    y[0] = rng.uniform(0.8, 1.2, y[0].shape)
    y[3] = rng.uniform(0.8, 1.2, y[0].shape)
    y[3, cell[1], cell[0]] = 0.0
    y = y.reshape(-1)
    v, w = ri.random_direction(y.size, 51), ri.random_direction(y.size, 52)
    R = Rok(pb, "fp64")
    yd, vd, wd = (torch.tensor(a, device=dev) for a in (y, v, w))
    Jv, g = R.jvp(yd, vd, "tangent").cpu(), R.vjp(yd, wd).cpu()
    assert bool(torch.isfinite(Jv).all()) and bool(torch.isfinite(g).all())
    assert abs(float(torch.dot(t64(w), Jv) - torch.dot(g, t64(v)))) <= 1e-13 * float(torch.linalg.norm(Jv))
