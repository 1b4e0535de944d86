"""Adjoint products on 2-D Cartesian grids on both sides of the choice between tiles and cells (thin grids of one
tile more than CUs, and of exactly that many; first-order Roe flux, Euler's second-order adjoint), against the
oracle: 1e-12, the bound of the other adjoint tests (a few hundred roundings of 2^-53)."""
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


@pytest.mark.parametrize("shape", [(4097, 2), (3, 4099), (4096, 1), (4200, 6), (19, 23)])
@pytest.mark.parametrize("physics,recon,flux,suth", [("euler", "first", "rusanov", 0.0), ("euler", "first", "roe", 0.0),
                                                     ("euler", "muscl", "rusanov", 0.0), ("ns", "first", "roe", 0.4),
                                                     ("ns", "first", "rusanov", 0.4), ("ns", "muscl", "roe", 0.0)])
def test_tiles_and_cells(dev, shape, physics, recon, flux, suth):
    print("[case] adjoint route", shape, physics, recon, flux, suth, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(shape, (0.0, 0.0), (1.0, 1.3), physics, recon, flux=flux, mu=1e-4 if physics == "ns" else 0.0,
                    sutherland=suth, t_ref=0.7)
    y = ri.smooth_random_state(pb, seed=16, amplitude=0.15)
    v, w = ri.random_direction(y.size, 116), ri.random_direction(y.size, 216)
    P = oracle_problem(pb)
    R = Rok(pb, "fp64")
    yd, vd, wd = (torch.tensor(a, device=dev) for a in (y, v, w))
    ref, ref2 = fv.vjp(P, t64(y), t64(w)), fv.vjp_second(P, t64(y), t64(v), t64(w))
    assert relerr(R.vjp(yd, wd).cpu(), ref) <= 1e-12
    g1, g2 = R.vjp(yd, wd, v=vd)
    assert relerr(g1.cpu(), ref) <= 1e-12
    assert relerr(g2.cpu(), ref2) <= 1e-12
