"""Sweeps and residual of blocks whose tile rows are fewer than their padded
size has (n 33..48, 65..80): one workgroup has a wavefront per tile row, and the
results are those of a batch that pads them to a larger neighbour, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,larger", [(33, 49), (40, 64), (48, 50), (65, 81), (72, 96), (80, 90)])
@pytest.mark.parametrize("m", [1, 4, 9])
def test_padding_does_not_enter(n, larger, m, precision):
    from paper_2601_03754_amd import btc

    prs = [inputs.block_tridiag(N, k, seed=N + k, nrhs=m) for N, k in ((37, n), (11, larger))]
    Ds, Es, Bs = ([dev(getattr(p, a)) for p in prs] for a in "DEB")
    r = btc.Runner()
    hs = [btc.btc_create(p.N, p.n, precision) for p in prs]
    Xs = [torch.empty_like(b) for b in Bs]
    r.factor_batched(hs, Ds, Es)
    info = r.solve_batched(hs, Bs, Xs, m, want_info=True)
    f = btc.Factor(Ds[0], Es[0], precision=precision)
    X, alone = f.solve(Bs[0], want_info=True)
    X = X.cpu().numpy()
    assert np.array_equal(X, Xs[0].cpu().numpy())
    if precision:
        assert info[0]["relres"] == alone["relres"] and info[0]["steps"] == alone["steps"]
    # the FP64 residual of the solve's report, formed by the same kernels
    rel = oracle.relres(prs[0].D, prs[0].E, X, prs[0].B)
    assert rel <= (1e-12 if precision == 0 else 1e-10)
    assert alone["relres"] <= 2 * rel + 1e-15
    f.close()
    for h in hs:
        btc.btc_destroy(h)
    r.close()
