"""Level sweeps of the solve: block sizes around the 16-wide tiles and the
padded sizes, right-hand sides around the columns per pass, ragged chains,
every launch shape.

The solution is checked against the FP64 oracle's relative residual (1e-12,
the bound of the FP64 path; 1e-10 after refinement), and against itself bit
for bit: the launch shape, the other columns of a call and the columns per
pass do not enter a column's arithmetic."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu
SHAPE, FORWARD, BACKWARD = 6, 1, 2


@pytest.fixture(scope="module")
def btc():
    from paper_2601_03754_amd import btc as b
    b.lib()
    keys = [(SHAPE, p, n) for p in (0, 1) for n in (8, 16, 32, 64, 96, 128)]
    keys += [(op, p, n) for op in (FORWARD, BACKWARD) for p in (0, 1) for n in (8, 16, 32, 64, 96, 128)]
    before = [b.btc_tune_get(op, p, n, 0) for op, p, n in keys]
    yield b
    for (op, p, n), v in zip(keys, before):
        b.btc_tune_set(op, p, n, 0, v)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("N,n,m", [(1, 1, 1), (2, 15, 5), (3, 16, 4), (5, 17, 16), (9, 31, 17), (33, 33, 3),
                                   (37, 64, 21), (21, 65, 8), (70, 95, 5), (12, 97, 9), (19, 128, 1), (6, 127, 10),
                                   (4100, 7, 2), (3001, 20, 1)])
@pytest.mark.parametrize("precision", [0, 1])
def test_shapes_and_columns(btc, N, n, m, precision):
    pr = inputs.block_tridiag(N, n, seed=N + n + m, nrhs=m)
    f = btc.Factor(dev(pr.D), dev(pr.E), precision=precision)
    B = dev(pr.B)
    out = {}
    for shape in (0, 1, 2):
        for cols in (0, 1):
            btc.btc_tune_set(SHAPE, precision, n, 0, shape)
            btc.btc_tune_set(FORWARD, precision, n, 0, cols)
            btc.btc_tune_set(BACKWARD, precision, n, 0, cols)
            for rep in range(2):  # the synchronisation words are reused
                out[shape, cols, rep] = f.solve(B).cpu().numpy()
    X = out[0, 0, 0]
    assert oracle.relres(pr.D, pr.E, X, pr.B) <= (1e-12 if precision == 0 else 1e-10)
    for k, v in out.items():
        assert np.array_equal(X, v), k
    if precision == 0:
        for q in {0, m // 2, m - 1}:
            alone = f.solve(dev(pr.B[:, :, q:q + 1])).cpu().numpy()
            assert np.array_equal(alone[:, :, 0], X[:, :, q]), q
    f.close()


def test_solves_of_one_handle_on_two_streams(btc):
    """Overlapping solves take workspaces (and synchronisation words) of
    their own."""
    pr = inputs.block_tridiag(900, 40, seed=3, nrhs=3)
    f = btc.Factor(dev(pr.D), dev(pr.E))
    Bs = [dev(pr.B * (k + 1)) for k in range(8)]
    want = [f.solve(b).cpu().numpy() for b in Bs]
    streams = [torch.cuda.Stream() for _ in range(2)]
    Xs = [torch.empty_like(b) for b in Bs]
    torch.cuda.synchronize()
    for k, b in enumerate(Bs):
        f.solve(b, Xs[k], stream=streams[k % 2])
    torch.cuda.synchronize()
    for x, w in zip(Xs, want):
        assert np.array_equal(x.cpu().numpy(), w)
    f.close()
