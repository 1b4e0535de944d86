"""Adjoint products round like correctly rounded quotients: on a flow at rest whose every intermediate is a binary
fraction of a few bits, J^T w is exact.

gamma = 2, rho = 49, u = 0, E = p = 24.5: the sound speed is sqrt(2 * 24.5 / 49) = 1, the flux Jacobian's entries are
0 and 1 ((E + p) / rho = 1), and with dx = 1 and whole numbers for w every term of J^T w is a multiple of 1/4 below
2^10.  A quotient by 49 is exact there; a product with the rounded 1/49 is not (49 * fl(1/49) != 1)."""
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


def exact_product(shape, w):
    """J^T w for Rusanov's flux at the state above, a = 1: face fluxes (A (U_L + U_R) - (U_R - U_L)) / 2 (all exact)."""
    D = len(shape)
    W = w.reshape((D + 2,) + tuple(reversed(shape)))
    g = np.zeros_like(W)
    for d in range(D):
        A = np.zeros((D + 2, D + 2))
        A[0, 1 + d] = A[1 + d, D + 1] = A[D + 1, 1 + d] = 1.0
        ax = D - d                       # axis of direction d in (variable, [z,] y, x)
        Fb = np.roll(W, -1, ax) - W      # adjoint of the face above each cell (dx = 1)
        ATF = np.einsum("ij,i...->j...", A, Fb)
        g += 0.5 * (ATF + Fb) + np.roll(0.5 * (ATF - Fb), 1, ax)
    return g.reshape(-1)


@pytest.mark.parametrize("shape", [(19, 18), (40, 7), (5, 4, 3), (16, 16, 5)])
@pytest.mark.parametrize("recon", ["first", "muscl"])
def test_exact_at_rest(dev, shape, recon):
    print("[case] adjoint rounding", shape, recon, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    D = len(shape)
    pb = ri.problem(shape, (0.0,) * D, tuple(float(n) for n in shape), "euler", recon, gamma=2.0)
    y = np.zeros((D + 2, int(np.prod(shape))))
    y[0], y[D + 1] = 49.0, 24.5
    y = y.reshape(-1)
    w = np.random.default_rng(3).integers(-9, 10, y.size).astype(np.float64)
    R = Rok(pb, "fp64")
    yd, wd = torch.tensor(y, device=dev), torch.tensor(w, device=dev)
    assert torch.equal(R.vjp(yd, wd).cpu(), t64(exact_product(shape, w)))
    assert torch.equal(R.vjp(yd, wd, v=torch.zeros_like(yd))[0].cpu(), t64(exact_product(shape, w)))
