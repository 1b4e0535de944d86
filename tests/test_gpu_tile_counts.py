"""Residuals, FD products and tangents on the two sides of the number of tiles from which a tile no longer has a
CU to itself (256 tiles of 16 x 16, 32 x 8 or 16 x 4 x 4 cells), against the oracle: the same bits, tangents 1e-12; FP32 residuals and
tangents 2e-5 (a few hundred roundings of 2^-24)."""
import sys

import pytest
import torch

import rok_inputs as ri
from oracle import fv
from tests._util import oracle_problem, relerr, t64
from tests.test_gpu_curvilinear import _ogrid_ns_setup, _ogrid_setup

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


def _check(dev, P, g, y):
    F, v, eps = fv.residual(P, y), t64(ri.random_direction(P.size, seed=3)), 1.7e-7
    out = g.residual(y.to(dev)).cpu()
    assert torch.equal(out, F), relerr(out, F)
    assert torch.equal(g.jvp(y.to(dev), v.to(dev), "fd", fy=F.to(dev), eps=eps).cpu(), fv.jvp_fd(P, y, F, v, eps))
    assert relerr(g.jvp(y.to(dev), v.to(dev), "exact").cpu(), fv.jvp_exact(P, y, v)) <= 1e-12


@pytest.mark.parametrize("shape", [(256, 256), (256, 257), (257, 248), (15, 4096), (17, 4096)])
@pytest.mark.parametrize("physics,recon,flux", [("ns", "muscl", "rusanov"), ("euler", "first", "roe")])
def test_cartesian(dev, shape, physics, recon, flux):
    print("[case] tiles", shape, physics, recon, flux, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(shape, (0.0, 0.0), (1.0, 1.2), physics, recon, flux=flux, mu=0.05 if physics == "ns" else 0.0)
    _check(dev, oracle_problem(pb), Rok(pb, "fp64"), t64(ri.smooth_random_state(pb, seed=4, amplitude=0.15)))


@pytest.mark.parametrize("shape", [(256, 256), (272, 256)])
@pytest.mark.parametrize("ns", [False, True])
def test_ogrid(dev, shape, ns):
    print("[case] ogrid tiles", shape, ns, flush=True)
    sys.stdout.flush()
    P, g, y = _ogrid_ns_setup(*shape, "muscl", "roe", 0.0) if ns else _ogrid_setup(*shape, "muscl", "rusanov")
    _check(dev, P, g, y)


@pytest.mark.parametrize("shape", [(61, 16, 64), (61, 17, 64), (5, 130, 31)])
@pytest.mark.parametrize("physics,recon,flux", [("ns", "muscl", "rusanov"), ("euler", "first", "roe")])
def test_3d(dev, shape, physics, recon, flux):
    print("[case] 3-D tiles", shape, physics, recon, flux, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(shape, (0.0, 0.0, 0.0), (1.0, 1.2, 0.9), physics, recon, flux=flux,
                    mu=0.05 if physics == "ns" else 0.0)
    P, y = oracle_problem(pb), t64(ri.smooth_random_state(pb, seed=4, amplitude=0.15))
    _check(dev, P, Rok(pb, "fp64"), y)
    g, v = Rok(pb, "fp32"), t64(ri.random_direction(P.size, seed=3))
    assert relerr(g.residual(y.to(dev)).cpu().double(), fv.residual(P, y)) <= 2e-5
    assert relerr(g.jvp(y.to(dev), v.to(dev), "exact").cpu().double(), fv.jvp_exact(P, y, v)) <= 2e-5
