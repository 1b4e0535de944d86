"""The reduced (Krylov-space) solve at the edges of its compiled widths: M = 1, 2, 7, 24, 25, 33 and 64 columns,
on a vector shorter than one reduction block, one of a few blocks, and one past 256 blocks.  Finite-difference steps
against the oracle's bit for bit (pivoting, both substitutions and every sum keep the textbook order); the
transposed solve through the step adjoint against the oracle's gradient (1e-10, the bound of the other step
gradients)."""
import sys

import pytest
import torch

import rok_inputs as ri
from oracle import rok, rok_ad
from tests._util import oracle_problem, relerr, t64

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


def _case(n):
    pb = ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", "first")
    return pb, ri.smooth_random_state(pb, seed=21)


@pytest.mark.parametrize("n,M", [((7, 8), M) for M in (1, 2, 7, 24, 25)] + [((12, 10), M) for M in (33, 64)] +
                         [((150, 130), M) for M in (7, 24)])
def test_fd_step_bitwise(dev, n, M):
    from paper_1607_06834_amd import Rok
    pb, y0 = _case(n)
    say("reduced solve", n, "N", y0.size, "M", M)
    tab, h = ri.rok4_tableau(), ri.cfl_step(pb, y0, 1.5)
    f, mv = rok.fv_system(oracle_problem(pb), "fd")
    ref = rok.rok_step(f, mv, tab, M, h, t64(y0))
    R = Rok(pb, "fp64")
    got = R.step(torch.tensor(y0, device=dev), h, tab, M, mode="fd").cpu()
    assert R.last_status()[1] == M
    assert torch.equal(got, ref)


@pytest.mark.parametrize("n,M", [((7, 8), 1), ((7, 8), 25), ((12, 10), 33)])
def test_step_adjoint(dev, n, M):
    from paper_1607_06834_amd import Rok
    pb, y0 = _case(n)
    say("reduced reverse", n, M)
    P, tab, h = oracle_problem(pb), ri.rok4_tableau(), ri.cfl_step(pb, y0, 1.5)
    c = ri.random_direction(y0.size, 5)
    ref = rok_ad.gradient(lambda z: torch.dot(t64(c), rok_ad.rok_step(P, tab, M, h, z)), t64(y0))
    g = Rok(pb, "fp64").step_vjp(torch.tensor(y0, device=dev), torch.tensor(c, device=dev), h, tab, M).cpu()
    say("  relerr", relerr(g, ref))
    assert relerr(g, ref) <= 1e-10
