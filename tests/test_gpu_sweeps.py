"""The one-reduce form's update sweep where its lanes hold a whole number of elements in LDS, one row more, one row less and a
ragged end, for narrow and wide columns, against modified Gram-Schmidt in torch on the device."""
import sys

import pytest
import torch

import rok_inputs as ri

pytestmark = pytest.mark.gpu


# N = 4 n0 n1; a lane of 262144 holds 16 elements at a time
@pytest.mark.parametrize("n", [(1024, 1024), (1024, 1025), (1024, 1023), (1448, 1449), (16, 16)])
@pytest.mark.parametrize("j", [0, 1, 5, 15, 19, 22])
def test_update_sweep(n, j):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    print("[case] update sweep", n, j, flush=True)
    sys.stdout.flush()
    from paper_1607_06834_amd import Rok, load_library
    load_library()
    dev, M = torch.device("cuda", 0), 24
    R = Rok(ri.problem(n, (0.0, 0.0), (1.0, 1.0), "euler", "first"), "fp64", "one_reduce")
    gen = torch.Generator(device=dev).manual_seed(7 + j)
    V = torch.zeros(M, R.N, dtype=torch.float64, device=dev)
    H = torch.zeros(M + 1, M, dtype=torch.float64, device=dev)
    ws = R.mgs_workspace(M)
    V[0].normal_(generator=gen)
    V[0] /= V[0].norm()
    for c in range(j + 1):   # the columns before set up the Gram rows
        w = torch.empty(R.N, dtype=torch.float64, device=dev).normal_(generator=gen)
        ref = w.clone()
        R.mgs_column(V, c, w, H, ws, V[c + 1])
    h = torch.zeros(j + 2, dtype=torch.float64, device=dev)
    for i in range(j + 1):
        h[i] = V[i] @ ref
        ref -= h[i] * V[i]
    h[j + 1] = ref.norm()
    # entries of h are sums of N products of size |w| / sqrt(N) whose roundings add up to a few 2^-53 |w|
    assert (H[:j + 2, j] - h).abs().max() <= 1e-13 * h[j + 1]
    assert (V[j + 1] - ref / h[j + 1]).norm() <= 1e-12
