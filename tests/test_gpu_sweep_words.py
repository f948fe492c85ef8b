"""The synchronisation words of the shared sweep launches: part of a handle's
workspace (and of btc_footprint_bytes), and cleared also where the first solve
of a workspace is captured into a graph."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def btc():
    from paper_2601_03754_amd import btc as b
    b.lib()
    return b


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


class Sizes:
    """torch's caching allocator behind the library's hook, noting sizes."""

    def __init__(self, btc):
        self.btc, self.sizes = btc, []
        self._a = btc._ALLOC_FN(self._alloc)
        self._f = btc._FREE_FN(btc._torch_free)

    def _alloc(self, size, stream, ctx):
        self.sizes.append(size)
        return self.btc._torch_alloc(size, stream, ctx)

    def __enter__(self):
        assert self.btc.lib().btc_set_allocator(self._a, self._f, None) == 0
        return self

    def __exit__(self, *exc):
        self.btc.btc_set_allocator(True)


@pytest.mark.parametrize("precision", [0, 1, 2])
@pytest.mark.parametrize("N,n,m", [(1, 3, 1), (40, 8, 2), (3000, 5, 1), (70, 100, 3)])
def test_footprint_counts_everything_a_solve_takes(btc, precision, N, n, m):
    pr = inputs.block_tridiag(N, n, seed=N + n, nrhs=m)
    with Sizes(btc) as a:
        f = btc.Factor(dev(pr.D), dev(pr.E), precision=precision)
        factor = len(a.sizes)
        X = f.solve(dev(pr.B))
        torch.cuda.synchronize()
        assert len(a.sizes) == factor + 1  # the workspace, nothing beside it
        f.solve(dev(pr.B), X)
        torch.cuda.synchronize()
        assert len(a.sizes) == factor + 1
        assert sum(a.sizes) == btc.btc_footprint_bytes(N, n, precision, m)
        f.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("hook", [True, False])
def test_first_solve_captured(btc, precision, hook):
    """A handle whose workspace the runner has allocated: the first solve of its
    own is captured, then solves inside and outside the graph alternate."""
    pr = inputs.block_tridiag(300, 20, seed=4, nrhs=2)
    D, E, B = dev(pr.D), dev(pr.E), dev(pr.B)
    X, Xg = torch.empty_like(B), torch.empty_like(B)
    btc.btc_set_allocator(hook)
    try:
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            h = btc.btc_create(300, 20, precision)
            r = btc.Runner(stream=st)
            r.factor_batched([h], [D], [E])
            r.solve_batched([h], [B], [X])
            r.sync()
            want = X.cpu().numpy()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st):
                btc.btc_solve(h, B, Xg, stream=st)
            for k in range(3):
                X.fill_(float("nan"))
                btc.btc_solve(h, B, X, stream=st)
                assert np.array_equal(X.cpu().numpy(), want), k
                Xg.fill_(float("nan"))
                g.replay()
                assert np.array_equal(Xg.cpu().numpy(), want), k
            torch.cuda.synchronize()
            btc.btc_destroy(h)
            r.close()
            del g
    finally:
        btc.btc_set_allocator(True)
    assert oracle.relres(pr.D, pr.E, want, pr.B) <= (1e-12 if precision == 0 else 1e-10)
