"""A slope that the limiter drops takes its tangent with it, whatever that holds: in a sawtooth flow every cell is an
extremum, every slope is zero and (J v)_c depends on v in c and the cells next to it alone, so an infinite or
not-a-number entry of v leaves every other cell of J v finite."""
import sys

import numpy as np
import pytest
import torch

import rok_inputs as ri

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


@pytest.mark.parametrize("shape", [(18, 20), (48, 34), (18, 12, 10)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_dropped_tangents(dev, shape, precision, bad):
    print("[case] limited tangents", shape, precision, bad, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok
    D = len(shape)
    pb = ri.problem(shape, (0.0,) * D, (1.0,) * D, "euler", "muscl")
    grid = tuple(reversed(shape))
    saw = 1.0 - 2.0 * (np.indices(grid).sum(0) % 2)
    rho, vel, p = 1.0 + 0.1 * saw, [0.2 * (d + 1) + 0.05 * saw for d in range(D)], 1.0 + 0.1 * saw
    ke = sum(u * u for u in vel)
    y = np.stack([rho, *(rho * u for u in vel), p / 0.4 + 0.5 * rho * ke]).reshape(-1)
    v = np.random.default_rng(2).uniform(-1.0, 1.0, (D + 2,) + grid)
    at = tuple(n // 2 for n in grid)
    v[(0,) + at] = bad
    R = Rok(pb, precision)
    Jv = R.jvp(torch.tensor(y, device=dev), torch.tensor(v.reshape(-1), device=dev), "tangent").cpu().double()
    finite = torch.isfinite(Jv).reshape((D + 2,) + grid).all(0).numpy()
    distance = sum(np.abs(x - a) for x, a in zip(np.indices(grid), at))
    assert finite[distance > 1].all()
    assert not finite[at]
