"""The one-workgroup-per-node factor kernel (n <= 64) at the edges of its tiles
and 4-column steps, on short ragged chains (nodes without a right or left
neighbour, without one or both deferred updates).

FP64 factors against the oracle's blocks and every solution's FP64 residual,
to the bounds of the other factor tests (factor and residual 1e-12 FP64,
residual 1e-10 refined)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 9, 12, 13, 16, 17, 20, 21, 29, 32, 33, 36, 37, 48, 49, 61, 64])
def test_node_step_edges(n, precision):
    from paper_2601_03754_amd import btc

    for N in (1, 2, 3, 5, 6, 7, 12, 23):
        pr = inputs.block_tridiag(N, n, seed=100 * N + n)
        f = btc.Factor(dev(pr.D), dev(pr.E), precision=precision)
        X = f.solve(dev(pr.B))
        torch.cuda.synchronize()
        assert f.info == 0
        if precision == 0:
            Ld, Rb, Tb, info = oracle.factor_nd(pr.D, pr.E)
            scale = max(np.abs(Ld).max(), 1.0)
            for g, o in zip(f.export(), (Ld, Rb, Tb)):
                assert np.abs(g - o).max() <= 1e-12 * scale, (N, n)
        assert oracle.relres(pr.D, pr.E, X.cpu().numpy(), pr.B) <= (1e-12 if precision == 0 else 1e-10), (N, n)
        f.close()


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n", [2, 8, 16, 27, 32, 40, 64])
def test_node_step_breakdown(n, precision):
    """A block that is not positive definite is reported, and only it: in the
    first, an inner and the last 4-column step of its factorization."""
    from paper_2601_03754_amd import btc

    for k in sorted({0, n // 2, n - 1}):
        pr = inputs.block_tridiag(6, n, seed=n)
        D = pr.D.copy()
        D[2, k, k] = -1.0
        f = btc.Factor(dev(D), dev(pr.E), precision=precision)
        torch.cuda.synchronize()
        assert f.info == 3
        f.close()
