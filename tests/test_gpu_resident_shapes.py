"""The resident Gram-Schmidt kernels at the edges of their grid shapes (one
block, eight blocks, 256 blocks; 1 to 16 elements per thread), against the
pass-by-pass kernels: the same sums in the same order, so the same bits."""
import sys

import numpy as np
import pytest
import torch

import rok_inputs as ri

pytestmark = pytest.mark.gpu

NONFINITE, BARRIER = 1, 8


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


def gpu(pb, mgs="auto"):
    from paper_1607_06834_amd import Rok
    return Rok(pb, "fp64", mgs)


def _problem(n):
    return ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", "first")


# grids with N = 4 n0 n1 at, just below and just past the sizes where the shape changes
EDGES = [(1, 7), (16, 16), (257, 1), (32, 16), (513, 1), (32, 32), (41, 25), (64, 32), (683, 3), (64, 64), (241, 17),
         (128, 64), (2731, 3), (128, 128), (16385, 1), (256, 256), (65537, 1)]


@pytest.mark.parametrize("n", EDGES)
def test_columns_and_reverse_bitwise(dev, n):
    """V and H of 6 exact-product columns, and the step adjoint (the reverse of the columns)."""
    pb = _problem(n)
    y0 = ri.smooth_random_state(pb, seed=9)
    say("shape edge", n, "N", y0.size)
    y = torch.tensor(y0, device=dev)
    c = torch.tensor(ri.random_direction(y0.size, 4), device=dev)
    tab, h = ri.rok4_tableau(), ri.cfl_step(pb, y0, 0.5)
    M = min(6, y0.size)
    a, b = gpu(pb), gpu(pb, "pass")
    assert a.arnoldi_path(M) == "resident"
    fy = a.residual(y)
    Va, Ha, ma = a.arnoldi(y, fy, M, "tangent")
    Vb, Hb, mb = b.arnoldi(y, fy, M, "tangent")
    assert a.last_arnoldi_flags() & BARRIER == 0
    assert ma == mb and torch.equal(Va, Vb) and torch.equal(Ha, Hb)
    ga, gb = a.step_vjp(y, c, h, tab, M), b.step_vjp(y, c, h, tab, M)
    assert a.last_status()[0] & BARRIER == 0
    assert torch.isfinite(ga).all() and torch.equal(ga, gb)


@pytest.mark.parametrize("n", [(32, 32), (128, 64), (300, 300)])
def test_columns_repeated_on_one_workspace(dev, n):
    """The exchange continues over any sequence of column calls on one prepared workspace."""
    pb = _problem(n)
    N, M = ri.size(pb), 5
    say("repeated columns", n, "N", N)
    rng = np.random.default_rng(3)
    V = torch.tensor(rng.standard_normal((M, N)) / np.sqrt(N), device=dev)
    w = torch.tensor(rng.standard_normal(N), device=dev)

    def columns(mgs):
        g = gpu(pb, mgs)
        H = torch.zeros(M + 1, M, dtype=torch.float64, device=dev)
        ws = g.mgs_workspace(M)
        out = []
        for j in (0, 3, 3, 4, 1, 2, 0):
            vn = torch.zeros(N, dtype=torch.float64, device=dev)
            g.mgs_column(V, j, w.clone(), H, ws, vnext=vn)
            out.append(vn)
        assert g.last_status()[0] == 0
        return torch.stack(out), H

    (va, Ha), (vb, Hb) = columns("auto"), columns("pass")
    assert torch.equal(va, vb) and torch.equal(Ha, Hb)


@pytest.mark.parametrize("n", [(32, 32), (128, 64), (300, 300)])
@pytest.mark.parametrize("bits", [0x7ff8000000000000, 0x7ff4000000000ea5])
def test_nan_passes_through_the_exchange(dev, n, bits):
    """A NaN in w, of the exchange's own empty mark too, gives NaN coefficients and no failed exchange."""
    pb = _problem(n)
    N, M = ri.size(pb), 4
    say("nan", n, hex(bits))
    w = torch.ones(N, dtype=torch.float64, device=dev)
    w.view(torch.int64)[N // 2] = bits
    V = torch.full((M, N), 1.0 / np.sqrt(N), dtype=torch.float64, device=dev)
    g = gpu(pb)
    H = torch.zeros(M + 1, M, dtype=torch.float64, device=dev)
    g.mgs_column(V, 2, w, H, g.mgs_workspace(M), vnext=torch.empty(N, dtype=torch.float64, device=dev))
    flags = g.last_status()[0]
    assert flags & NONFINITE and not flags & BARRIER
    assert torch.isnan(H[:4, 2]).all()
