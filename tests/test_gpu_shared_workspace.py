"""A product with the default increment in a Gram-Schmidt column's workspace: rok_jvp uses the smallest layout
(rok_workspace_bytes(ctx, 0, 0)) at its start, which must leave what the column's exchange keeps there alone.

One column against one vector (M = 1, the layout closest to the smallest one): h_00 = <v_0, w> in the library's
fixed order, the same bits with and without the product before it."""
import ctypes
import sys

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


# one block, eight blocks, 256 blocks, pass by pass (one-reduce above the resident sizes)
@pytest.mark.parametrize("n", [(40, 40), (64, 100), (129, 128), (701, 701), (1030, 1030)])
@pytest.mark.parametrize("M", [1, 2, 5])
def test_product_between_columns(dev, n, M):
    print("[case] shared workspace", n, M, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok, rok
    pb = ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", "first")
    R = Rok(pb, "fp64")
    yd = torch.tensor(ri.smooth_random_state(pb, seed=7, amplitude=0.1), device=dev)
    f, p = R.residual(yd), lambda t: ctypes.c_void_p(t.data_ptr())
    v0 = torch.tensor(ri.random_direction(R.N, 8), device=dev)

    def columns(shared):
        V, H = torch.zeros(M, R.N, dtype=torch.float64, device=dev), torch.zeros(M + 1, M, dtype=torch.float64, device=dev)
        V[0] = v0
        ws = R.mgs_workspace(M)
        for j in range(M):
            w = torch.empty_like(yd)
            work = ws if shared else R.workspace(0, 0)
            assert rok._lib.rok_jvp(R._ctx, p(yd), p(f), p(V[j]), p(w), rok.JVP_FD, 0.0, p(work), work.numel(),
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
            R.mgs_column(V, j, w, H, ws, V[j + 1] if j + 1 < M else None)
        return V, H

    V, H = columns(False)
    V2, H2 = columns(True)
    assert bool(H.isfinite().all()) and float(H.abs().max()) > 0.0
    assert torch.equal(H, H2) and torch.equal(V, V2)
