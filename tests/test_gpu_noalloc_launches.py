"""btc_solve_noalloc runs the launches of btc_solve: the levels of few nodes
share one launch in each direction."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,n,m", [(2, 8, 1), (16, 8, 1), (3000, 16, 2), (2100, 100, 1)])
def test_same_launches_as_solve(N, n, m, precision):
    from paper_2601_03754_amd import btc

    L = btc.lib()
    L.btc_solve_noalloc.restype = ctypes.c_int
    L.btc_solve_noalloc.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64,
                                    ctypes.c_void_p, ctypes.c_void_p]
    pr = inputs.block_tridiag(N, n, seed=N + n, nrhs=m)
    B = dev(pr.B)
    f = btc.Factor(dev(pr.D), dev(pr.E), precision=precision)

    def noalloc(X):
        assert L.btc_solve_noalloc(f.handle, B.data_ptr(), X.data_ptr(), m,
                                   torch.cuda.current_stream().cuda_stream, None) == 0

    counts, out = [], []
    for solve in (lambda X: f.solve(B, X), noalloc):
        X = torch.empty_like(B)
        btc.btc_profile(f.handle, True)
        for _ in range(40):  # more calls than sets of synchronisation words
            solve(X)
        torch.cuda.synchronize()
        counts.append([btc.btc_profile_read(f.handle, ph)[1].tolist() for ph in (1, 2)])
        out.append(X.cpu().numpy())
    btc.btc_profile(f.handle, False)
    f.close()
    assert counts[0] == counts[1]
    assert np.array_equal(out[0], out[1])
    assert oracle.relres(pr.D, pr.E, out[1], pr.B) <= (1e-12 if precision == 0 else 1e-10)
