"""More right-hand sides than 32-bit offsets within a tile row reach (16 rows of
more than 2^23 columns): every column solved, against the residual in torch."""
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


def test_solve_of_more_than_2_23_columns():
    from paper_2601_03754_amd import btc

    N, n, m = 2, 16, (1 << 23) + 3
    pr = inputs.block_tridiag(N, n, seed=6)
    D, E = (torch.from_numpy(a).to("cuda:0") for a in (pr.D, pr.E))
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1)
    B = torch.randn(N, n, m, dtype=torch.float64, device="cuda:0", generator=g)
    f = btc.Factor(D, E)
    X = torch.full_like(B, float("nan"))
    f.solve(B, X)
    torch.cuda.synchronize()
    r0 = B[0] - D[0] @ X[0] - E[0].T.contiguous() @ X[1]
    r1 = B[1] - D[1] @ X[1] - E[0] @ X[0]
    rel = ((r0.square().sum(0) + r1.square().sum(0)) / (B[0].square().sum(0) + B[1].square().sum(0))).sqrt()
    assert float(rel.max()) <= 1e-12  # (NaN fails)
    # and the bits of a narrow solve
    for q in (0, 4, (1 << 22) + 1, m - 5, m - 1):
        one = f.solve(B[:, :, q:q + 1].contiguous())
        assert torch.equal(one[:, :, 0], X[:, :, q]), q
    f.close()
    assert oracle.relres(pr.D, pr.E, X[:, :, -2:].cpu().numpy(), B[:, :, -2:].cpu().numpy()) <= 1e-12
