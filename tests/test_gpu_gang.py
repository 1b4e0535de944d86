"""Gram-Schmidt columns whose 256 blocks do not all find room on the device in time: the blocks that are in
do the whole column, with the same bits; so does the column after it, whose blocks all come."""
import sys

import pytest
import torch

import rok_inputs as ri

pytestmark = pytest.mark.gpu

BARRIER = 8


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


def _make(n):
    from paper_1607_06834_amd import Rok
    pb = ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", "first")
    return Rok(pb, "fp64"), ri.smooth_random_state(pb, seed=21, amplitude=0.1), ri.cfl_step(pb, ri.smooth_random_state(
        pb, seed=21, amplitude=0.1), 2.0)


def _hold(R, blocks):
    from paper_1607_06834_amd import rok
    assert rok._lib.rok_set_gang_hold(R._ctx, blocks) == 0


def _columns(R, V, J, M, holds):
    """The columns from v_0 = V[0] and the products J, under the given holds: (V, H)."""
    V2 = torch.zeros_like(V)
    V2[0] = V[0]
    H = torch.zeros(M + 1, M, dtype=torch.float64, device=V.device)
    ws = R.mgs_workspace(M)
    for j in range(M):
        _hold(R, holds[j % len(holds)])
        R.mgs_column(V2, j, J[j].clone(), H, ws, V2[j + 1] if j + 1 < M else None)
    _hold(R, 0)
    torch.cuda.synchronize()
    return V2, H, R.last_status()[0]


# one, two, eight (ragged) and sixteen elements per thread; few, half and all but one of the blocks, and closed and
# complete gangs in turn
@pytest.mark.parametrize("n", [(129, 128), (257, 256), (701, 701), (1000, 1000)])
@pytest.mark.parametrize("holds", [(1,), (3,), (128,), (255,), (0, 5, 0, 200, 9, 0, 0), (3, 3, 0, 254, 0, 0, 1)])
def test_forward_columns(dev, n, holds):
    say("gang", n, holds)
    R, y, _ = _make(n)
    yd = torch.tensor(y, device=dev)
    M = 8
    gen = torch.Generator(device="cpu").manual_seed(5)
    V = torch.zeros(M, R.N, dtype=torch.float64, device=dev)
    V[0] = torch.tensor(ri.random_direction(R.N, 23), device=dev)
    V[0] /= V[0].norm()
    J = torch.rand(M, R.N, dtype=torch.float64, generator=gen).to(dev)
    ref = _columns(R, V, J, M, (0,))
    out = _columns(R, V, J, M, holds)
    assert torch.equal(ref[0], out[0]) and torch.equal(ref[1], out[1])
    assert not (ref[2] | out[2]) & BARRIER


@pytest.mark.parametrize("n", [(129, 128), (701, 701)])
@pytest.mark.parametrize("hold", [1, 77, 255])
def test_reverse_columns(dev, n, hold):
    say("gang reverse", n, hold)
    R, y, h = _make(n)
    yd = torch.tensor(y, device=dev)
    w = torch.tensor(ri.random_direction(y.size, 22), device=dev)
    tab = ri.rok4_tableau()
    y1, ref = R.step(yd, h, tab, 4, "tangent"), R.step_vjp(yd, w, h, tab, 4)
    _hold(R, hold)
    z1, out = R.step(yd, h, tab, 4, "tangent"), R.step_vjp(yd, w, h, tab, 4)
    _hold(R, 0)
    assert torch.equal(y1, z1) and torch.equal(ref, out)
    assert torch.equal(ref, R.step_vjp(yd, w, h, tab, 4))
