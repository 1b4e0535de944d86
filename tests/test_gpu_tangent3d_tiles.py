"""The 3-D tile kernel's tangents at the edges of the 16 x 4 x 4 tiles (one cell past, one short, grids
narrower than the stencil), whose faces of all directions are taken together, and the column-marching kernel where a
column's ranges have two planes and one: against the oracle."""
import sys

import pytest
import torch

import rok_inputs as ri
from oracle import fv
from tests._util import oracle_problem, relerr, t64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


def _case(dev, shape, physics, recon, flux, suth):
    print("[case]", shape, physics, recon, flux, suth, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(shape, (0.0, 0.0, 0.0), (1.0, 0.9, 1.2), physics, recon, flux=flux,
                    mu=0.05 if physics == "ns" else 0.0, sutherland=suth, t_ref=0.8)
    y, v = ri.smooth_random_state(pb, seed=8, amplitude=0.15), ri.random_direction(5 * shape[0] * shape[1] * shape[2], 9)
    return oracle_problem(pb), Rok(pb, "fp64"), t64(y), t64(v)


# a few hundred roundings of 2^-53 in sums that do not cancel, as in the other tangent tests
@pytest.mark.parametrize("shape", [(16, 4, 4), (17, 5, 3), (15, 3, 9), (1, 2, 3), (33, 8, 5)])
@pytest.mark.parametrize("physics,recon,flux,suth", [("euler", "first", "rusanov", 0.0), ("euler", "muscl", "roe", 0.0),
                                                     ("ns", "muscl", "rusanov", 0.4), ("ns", "first", "roe", 0.0)])
def test_tangent_tile_edges(dev, shape, physics, recon, flux, suth):
    P, R, y, v = _case(dev, shape, physics, recon, flux, suth)
    out = R.jvp(y.to(dev), v.to(dev), "tangent").cpu()
    assert relerr(out, fv.jvp_exact(P, y, v)) <= 1e-12


@pytest.mark.parametrize("shape", [(48, 48, 99), (16, 16, 7)])
def test_column_ranges_bitwise(dev, shape):
    P, R, y, v = _case(dev, shape, "ns", "muscl", "rusanov", 0.0)
    F, eps = fv.residual(P, y), 1.7e-7
    assert torch.equal(R.residual(y.to(dev)).cpu(), F)
    assert torch.equal(R.jvp(y.to(dev), v.to(dev), "fd", fy=F.to(dev), eps=eps).cpu(), fv.jvp_fd(P, y, F, v, eps))
