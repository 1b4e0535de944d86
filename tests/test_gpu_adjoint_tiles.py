"""Adjoint products on 2-D Cartesian grids at the edges of the 16 x 16 tiles (one cell past, one short, grids
narrower than the stencil, whose halo wraps several times), against the oracle's reverse and
forward-over-reverse differentiation: 1e-12, the bound of the other adjoint tests (a few hundred roundings of
2^-53 in sums that do not cancel)."""
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


@pytest.mark.parametrize("shape", [(16, 16), (17, 15), (33, 31), (1, 5), (3, 2), (48, 17)])
@pytest.mark.parametrize("physics,recon,flux,suth", [("euler", "first", "rusanov", 0.0), ("euler", "muscl", "roe", 0.0),
                                                     ("ns", "first", "roe", 0.4), ("ns", "muscl", "rusanov", 0.4),
                                                     ("ns", "muscl", "rusanov", 0.0)])
def test_tile_edges(dev, shape, physics, recon, flux, suth):
    print("[case] adjoint tile", shape, physics, recon, flux, suth, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(shape, (0.0, 0.0), (1.0, 1.3), physics, recon, flux=flux, mu=0.02 if physics == "ns" else 0.0,
                    sutherland=suth, t_ref=0.7)
    y = ri.smooth_random_state(pb, seed=6, amplitude=0.15)
    v, w = ri.random_direction(y.size, 106), ri.random_direction(y.size, 206)
    P = oracle_problem(pb)
    R = Rok(pb, "fp64")
    yd, vd, wd = (torch.tensor(a, device=dev) for a in (y, v, w))
    assert relerr(R.vjp(yd, wd).cpu(), fv.vjp(P, t64(y), t64(w))) <= 1e-12
    base = torch.tensor(v, device=dev)
    g1, g2 = R.vjp(yd, wd, v=vd, accumulate_into=base.clone(), accumulate_into2=base.clone())
    assert relerr(g1.cpu(), t64(v) + fv.vjp(P, t64(y), t64(w))) <= 1e-12
    assert relerr(g2.cpu(), t64(v) + fv.vjp_second(P, t64(y), t64(v), t64(w))) <= 1e-12
