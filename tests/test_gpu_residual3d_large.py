"""The column-marching 3-D residual and FD product on the two sides of the size where a vector's variables reach
past 2^32 bytes (the accesses' offsets then move into their base): a tall grid that repeats a
state of 16 planes has that state's residual in every repetition, bit for bit the oracle's on the 16 planes."""
import sys

import pytest
import torch

import rok_inputs as ri
from oracle import fv
from tests._util import oracle_problem, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("repeats", [2**15 - 1, 2**15])
def test_variables_around_four_gigabytes(repeats):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    print("[case] tall column", repeats, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok, load_library
    load_library()
    dev = torch.device("cuda", 0)

    def pb(n):   # the same spacing 1.25 / 16 for any n (both products are exact)
        return ri.problem((16, 16, 16 * n), (0.0, 0.0, 0.0), (1.0, 0.9, 1.25 * n), "ns", "muscl", mu=0.05)

    P = oracle_problem(pb(1))
    y = t64(ri.smooth_random_state(pb(1), seed=14, amplitude=0.2))
    v = t64(ri.random_direction(P.size, seed=15))
    F, eps = fv.residual(P, y), 1.7e-7
    D = fv.jvp_fd(P, y, F, v, eps)

    def tall(x):
        return x.to(dev).view(5, 1, -1).expand(5, repeats, -1).contiguous().view(-1)

    def same(x, ref):
        return bool((x.view(5, repeats, -1) == ref.to(dev).view(5, 1, -1)).all())

    R = Rok(pb(repeats), "fp64")
    Y = tall(y)
    FY = R.residual(Y)
    assert same(FY, F)
    assert same(R.jvp(Y, tall(v), "fd", fy=FY, eps=eps), D)
