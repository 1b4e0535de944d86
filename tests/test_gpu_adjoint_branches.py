"""The 2-D adjoint product is the transpose of the library's own tangent also where a limiter or a wave speed sits
on its switch: both differentiate the branch that the residual takes, which rounding decides there.

Flows whose velocity or pressure is uniform or piecewise linear, so that slopes are equal or pure rounding noise
(96 x 64: 24576 unknowns).  <w, J v> and <J^T w, v> are two roundings of one number; each is a sum of products in
which J v and J^T w carry normwise errors of a few hundred roundings of 2^-53, so they agree to 1e-13 of
||w|| ||J v||.  Against the oracle's reverse differentiation, 1e-12: the bound of the other adjoint tests."""
import sys

import numpy as np
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


def pack(pb, rho, vel, p):
    ke = sum(u * u for u in vel)
    return np.stack([rho, *(rho * u for u in vel), p / (pb["gamma"] - 1.0) + 0.5 * rho * ke]).reshape(-1)


def state(pb, flow):
    (nx, ny), one = pb["n"], np.ones(tuple(reversed(pb["n"])))
    X, Y = (np.arange(nx) + 0.5)[None, :] / nx * one, (np.arange(ny) + 0.5)[:, None] / ny * one
    if flow == "density wave":
        return pack(pb, 1.0 + 0.3 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y), [0.3 * one, 0.7 * one], one / 1.4)
    if flow == "linear shear":
        return pack(pb, 1.3 * one, [np.abs(Y - 0.5), 0.2 * one], one)
    if flow == "linear both":
        return pack(pb, 1.3 * one, [np.abs(Y - 0.5), np.abs(X - 0.5)], one)
    return pack(pb, 1.3 * one, [np.tanh(10.0 * (Y - 0.5)), 0.1 * one], one)   # shear layer


@pytest.mark.parametrize("flow", ["density wave", "linear shear", "linear both", "shear layer"])
@pytest.mark.parametrize("physics,recon,flux", [("euler", "muscl", "rusanov"), ("euler", "first", "rusanov"),
                                                ("euler", "muscl", "roe"), ("ns", "muscl", "rusanov")])
def test_transpose_at_switches(dev, flow, physics, recon, flux):
    print("[case] adjoint at switches", flow, physics, recon, flux, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem((96, 64), (0.0, 0.0), (1.0, 1.0), physics, recon, flux=flux, mu=0.01 if physics == "ns" else 0.0)
    y = state(pb, flow)
    v, w = ri.random_direction(y.size, 41), ri.random_direction(y.size, 42)
    R = Rok(pb, "fp64")
    yd, vd, wd = (torch.tensor(a, device=dev) for a in (y, v, w))
    Jv = R.jvp(yd, vd, "tangent").cpu()
    g = R.vjp(yd, wd).cpu()
    g2 = R.vjp(yd, wd, v=vd)[0].cpu()
    lhs = torch.dot(t64(w), Jv)
    bound = 1e-13 * float(torch.linalg.norm(Jv))
    assert abs(float(lhs - torch.dot(g, t64(v)))) <= bound
    assert abs(float(lhs - torch.dot(g2, t64(v)))) <= bound
    assert relerr(g, fv.vjp(oracle_problem(pb), t64(y), t64(w))) <= 1e-12
