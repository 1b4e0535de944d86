"""Which way a Gram-Schmidt column of 256 blocks goes, and that it gives the same bits whatever else the device does.

A closed gang updates the work vector in memory, the complete resident kernel leaves it as it was: that tells the
two ways apart."""
import sys

import pytest
import torch

import rok_inputs as ri

pytestmark = pytest.mark.gpu

BARRIER = 8
M = 6


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1607_06834_amd import load_library
    load_library()
    return torch.device("cuda", 0)


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def problem(n):
    from paper_1607_06834_amd import Rok
    pb = ri.problem(n, (-5.0, -5.0), (5.0, 5.0), "euler", "first")
    y = ri.smooth_random_state(pb, seed=21, amplitude=0.1)
    return Rok(pb, "fp64"), y, ri.cfl_step(pb, y, 2.0)


def columns(R, dev, before=lambda: None, hold=0):
    """(V, H, whether each column's work vector was changed, status)."""
    from paper_1607_06834_amd import rok
    gen = torch.Generator(device="cpu").manual_seed(5)
    J = torch.rand(M, R.N, dtype=torch.float64, generator=gen).to(dev)
    V = torch.zeros(M, R.N, dtype=torch.float64, device=dev)
    V[0] = torch.tensor(ri.random_direction(R.N, 23), device=dev)
    V[0] /= V[0].norm()
    H = torch.zeros(M + 1, M, dtype=torch.float64, device=dev)
    ws = R.mgs_workspace(M)
    W = [J[j].clone() for j in range(M)]
    assert rok._lib.rok_set_gang_hold(R._ctx, hold) == 0
    torch.cuda.synchronize()
    before()
    for j in range(M):
        R.mgs_column(V, j, W[j], H, ws, V[j + 1] if j + 1 < M else None)
    assert rok._lib.rok_set_gang_hold(R._ctx, 0) == 0
    torch.cuda.synchronize()
    return V, H, [not torch.equal(W[j], J[j]) for j in range(M)], R.last_status()[0]


# one, two, eight and sixteen elements per thread
@pytest.mark.parametrize("n", [(129, 128), (257, 256), (701, 701), (1000, 1000)])
@pytest.mark.parametrize("hold", [0, 1, 9, 254, 255, 256])
def test_held_blocks_close_the_gang(dev, n, hold):
    say("gang path", n, hold)
    R = problem(n)[0]
    V, H, changed, _ = columns(R, dev)
    assert changed == [False] * M
    V2, H2, changed, status = columns(R, dev, hold=hold)
    assert changed == [0 < hold < 256] * M
    assert torch.equal(V, V2) and torch.equal(H, H2) and not status & BARRIER


@pytest.mark.parametrize("n", [(129, 128), (1000, 1000)])
def test_waits_for_running_kernels(dev, n):
    """A product of 64-bit matrices on another stream holds the CUs for several milliseconds; nothing else waits, so
    the columns wait for it (20 ms at most) and run complete."""
    say("gang behind a running kernel", n)
    R = problem(n)[0]
    V, H, _, _ = columns(R, dev)
    a = torch.rand(4096, 8192, dtype=torch.float64, device=dev)
    side, c = torch.cuda.Stream(), torch.empty(4096, 4096, dtype=torch.float64, device=dev)
    torch.mm(a, a.t(), out=c)   # (workspaces and kernels are there before the streams run together)

    def busy():
        with torch.cuda.stream(side):
            torch.mm(a, a.t(), out=c)

    V2, H2, changed, status = columns(R, dev, before=busy)
    assert changed == [False] * M
    assert torch.equal(V, V2) and torch.equal(H, H2) and not status & BARRIER


# one block, eight blocks and 256 blocks a column, alone and against each other
@pytest.mark.parametrize("sizes", [((40, 40), (40, 40)), ((64, 100), (64, 100)), ((129, 128), (129, 128)),
                                   ((64, 100), (300, 300)), ((701, 701), (40, 40)), ((1000, 1000), (64, 100)),
                                   ((1000, 1000), (701, 701))])
def test_two_streams(dev, sizes):
    say("two streams", sizes)
    tab, steps = ri.rok4_tableau(), 3
    probs = [problem(n) for n in sizes]
    ys = [torch.tensor(p[1], device=dev) for p in probs]

    def march(i, out):
        y = ys[i]
        for k in range(steps):
            y = probs[i][0].step(y, probs[i][2], tab, M, "tangent", out=out[k])
        return y

    outs = [[torch.empty_like(y) for _ in range(steps)] for y in ys]
    refs = []
    for i in range(2):
        march(i, outs[i])
        torch.cuda.synchronize()
        refs.append([o.clone() for o in outs[i]])
        for o in outs[i]:
            o.zero_()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for k in range(steps):      # both streams get their launches in turn
        for i in range(2):
            R, _, h = probs[i]
            with torch.cuda.stream(streams[i]):
                R.step(ys[i] if k == 0 else outs[i][k - 1], h, tab, M, "tangent", out=outs[i][k])
    torch.cuda.synchronize()
    for i in range(2):
        for a, b in zip(refs[i], outs[i]):
            assert torch.equal(a, b)
        assert not probs[i][0].last_status()[0] & BARRIER
