"""The tip of an arrow matrix at the sizes where its factorization, its solve
and the tall-skinny product change tiles or kernels: against the FP64 oracle to
the bounds of the other arrow tests (1e-12 factor and residual), and the failing
column of an indefinite tip in the first, an inner and the last column."""
import numpy as np
import pytest
import torch

import oracle
from oracle import structures as st
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("N", [1, 23, 150])
@pytest.mark.parametrize("m", [1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 96, 97, 127, 128])
def test_tip_sizes(m, N):
    from paper_2601_03754_amd import btc

    n, q = 7, 3
    pr = inputs.arrow(N, n, m, seed=m + N, nrhs=q)
    a = btc.Arrow(dev(pr.D), dev(pr.E), dev(pr.F), dev(pr.C))
    X = a.solve(dev(pr.B))
    torch.cuda.synchronize()
    assert a.info == (0, 0)
    fac = st.arrow_factor(pr.D, pr.E, pr.F, pr.C)
    Ls, _ = a.export()
    assert np.abs(Ls - fac["Ls"]).max() <= 1e-12 * np.abs(fac["Ls"]).max()
    Xg = X.cpu().numpy()
    K = N * n
    x1, x2 = Xg[:K], Xg[K:]
    C = np.tril(pr.C) + np.tril(pr.C, -1).T
    r1 = oracle.residual(pr.D, pr.E, x1.reshape(N, n, q), pr.B[:K].reshape(N, n, q)).reshape(K, q) - pr.F @ x2
    r2 = pr.B[K:] - pr.F.T @ x1 - C @ x2
    r = np.sqrt((r1 ** 2).sum(0) + (r2 ** 2).sum(0)) / np.linalg.norm(pr.B, axis=0)
    assert r.max() <= 1e-12
    for k in sorted({0, m // 2, m - 1}):
        C = pr.C.copy()
        C[k, k] = -1e3
        a.refactor(dev(pr.D), dev(pr.E), dev(pr.F), dev(C))
        torch.cuda.synchronize()
        assert a.info == (0, k + 1)
    a.close()
