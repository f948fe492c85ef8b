"""The block updates of the tiled factor at the node count where they go from
one workgroup per tile to one per node.

Both forms accumulate in the same order, so an instance below the count must
get the same bits from a batch above it; both are checked against the FP64
oracle to the bounds of the other factor tests (1e-12 FP64, 1e-10 refined)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [33, 50, 64, 65, 81, 96, 97, 127, 128])
def test_update_by_tile_and_by_node(n, precision):
    from paper_2601_03754_amd import btc

    tol = 1e-12 if precision == 0 else 1e-10
    # level 0 of N blocks eliminates about N / 2 of them: 190 .. 193 by themselves
    prs = [inputs.block_tridiag(N, n, seed=N + n) for N in (381, 383, 385, 2, 131)]
    hs = [btc.btc_create(p.N, p.n, precision) for p in prs]
    Ds, Es = [dev(p.D) for p in prs], [dev(p.E) for p in prs]
    r = btc.Runner()
    r.factor_batched(hs, Ds, Es)
    r.sync()
    for k, p in enumerate(prs):
        f = btc.Factor(Ds[k], Es[k], precision=precision)
        X = f.solve(dev(p.B))
        torch.cuda.synchronize()
        assert oracle.relres(p.D, p.E, X.cpu().numpy(), p.B) <= tol
        blocks = f.export()
        f.close()
        for a, b in zip(btc.btc_export_factor(hs[k], p.N, p.n), blocks):
            assert np.array_equal(a, b), (p.N, p.n)
        btc.btc_destroy(hs[k])
    r.close()
