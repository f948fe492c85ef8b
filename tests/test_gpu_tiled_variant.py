"""The tile-parallel level step at padded size 64, which runs where the tune
table asks for it (variant 0 there), on both sides of the node counts at which
its kernels change: the update by tile or by node (192), the pivot and strips
with one or four wavefronts a strip (256).

All forms accumulate in the same order, so an instance below the counts must
get the same bits from a batch above them; both are checked against the FP64
oracle to the bounds of the other factor tests (1e-12 FP64, 1e-10 refined)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu
FACTOR, TILED = 0, 0


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("n", [33, 50, 64])
def test_tiled_step_alone_and_in_a_batch(n, precision):
    from paper_2601_03754_amd import btc

    tol = 1e-12 if precision == 0 else 1e-10
    before = [btc.btc_tune_get(FACTOR, precision, n, lvl) for lvl in (0, 1)]
    prs = [inputs.block_tridiag(N, n, seed=N + n) for N in (381, 385, 2, 131, 515)]
    Ds, Es = [dev(p.D) for p in prs], [dev(p.E) for p in prs]
    try:
        for lvl in (0, 1):
            btc.btc_tune_set(FACTOR, precision, n, lvl, TILED)
        hs = [btc.btc_create(p.N, p.n, precision) for p in prs]
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
        # the step that ran is the tile-parallel one, whose kernels are timed
        # each for itself: pivot and strips, update
        r.profile(FACTOR)
        h = btc.btc_create(385, n, precision)
        r.factor_batched([h], [Ds[1]], [Es[1]])
        r.sync()
        assert {s["part"] for s in r.profile_read()} >= {2, 3}
        btc.btc_destroy(h)
        r.close()
    finally:
        for lvl in (0, 1):
            btc.btc_tune_set(FACTOR, precision, n, lvl, before[lvl])
