"""The recovery of large stages (vectors above 4194304 elements, whose lanes hold several results back and store them together)
against the step written in torch on the device: ragged ends, more compiled columns than basis vectors (M = 7 of 8,
13 of 16), no basis, a stage whose successor takes no stage terms, and the last stage.

The basis and H come from rok_arnoldi and the stage residuals from rok_residual; projections, reduced solve, recoveries and
the update are torch's, in 64 bits.  The two steps differ by the rounding of sums of at most 4 M + 8 products per
element of sizes up to max |y| and by the basis' last bits: 1e-12 of max |y| in every element, the library's bound
between its orthogonalisations."""
import sys

import pytest
import torch

import rok_inputs as ri

pytestmark = pytest.mark.gpu

# stage 1 starts from k_0; stage 2 from y alone, so stage 1's recovery writes no stage input
TABLEAU = {"s": 3, "gamma": 0.4, "alpha": [[0, 0, 0], [0.5, 0, 0], [0, 0, 0]],
           "gam": [[0, 0, 0], [-0.2, 0, 0], [0.1, 0.3, 0]], "b": [0.25, 0.5, 0.25]}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


def reference(R, y, h, tab, M):
    """The step of the tableau with the library's f, V and H, everything else in torch."""
    F0 = R.residual(y)
    if M:
        V, H, meff = R.arnoldi(y, F0, M, "tangent")
        V, H = V[:meff], H[:meff, :meff]
        A = torch.eye(meff, dtype=torch.float64, device=y.device) - h * tab["gamma"] * H
    ks, lams = [], []
    for i in range(tab["s"]):
        Y = y.clone()
        for j in range(i):
            Y += tab["alpha"][i][j] * ks[j]
        F = F0 if i == 0 else R.residual(Y)
        k = h * F
        if M:
            phi = V @ F
            rhs = h * phi
            for j in range(i):
                rhs = rhs + h * tab["gam"][i][j] * (H @ lams[j])
            lams.append(torch.linalg.solve(A, rhs))
            k = (lams[-1] - h * phi) @ V + k
        ks.append(k)
    out = y.clone()
    for b, k in zip(tab["b"], ks):
        out += b * k
    return out


@pytest.mark.parametrize("n", [(1024, 1025), (1201, 1103), (1448, 1449)])
@pytest.mark.parametrize("M", [0, 1, 2, 7, 13])
def test_against_torch(dev, n, M):
    print("[case] recovery", n, M, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    pb = ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", "first")
    y = ri.smooth_random_state(pb, seed=31, amplitude=0.1)
    h = ri.cfl_step(pb, y, 1.0)
    R = Rok(pb, "fp64")
    yd = torch.tensor(y, device=dev)
    for tab in (TABLEAU, ri.rok4_tableau()):
        out = R.step(yd, h, tab, M, "tangent", out=torch.full_like(yd, float("nan")))
        assert float((out - reference(R, yd, h, tab, M)).abs().max()) <= 1e-12 * float(yd.abs().max())
