"""Rounding of the FP64 path: the solve's componentwise backward error on
ill-conditioned blocks, and Schur sums of products far below the block they
are subtracted from."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def ill_conditioned(N, n, digits, seed):
    """D_i = Q diag(1 .. 10^-digits) Q^T, E_i = 0.4 D_{i+1}^(1/2) V D_i^(1/2) with
    V orthogonal: positive definite, every pivot block of condition about
    10^digits."""
    rng = np.random.default_rng(seed)
    lam = np.logspace(0, -digits, n)
    orth = lambda: np.linalg.qr(rng.standard_normal((n, n)))[0]
    D, H = np.zeros((N, n, n)), []
    for i in range(N):
        q = orth()
        D[i] = (q * lam) @ q.T
        D[i] = (D[i] + D[i].T) / 2
        H.append((q * np.sqrt(lam)) @ q.T)
    E = np.stack([0.4 * H[i + 1] @ orth() @ H[i] for i in range(N - 1)])
    return D, E, rng.standard_normal((N, n, 2))


def backward_error(D, E, B, X):
    """max |b - Psi x| / (|Psi| |x| + |b|) by component, in extended precision."""
    D, E, B, X = (a.astype(np.longdouble) for a in (D, E, B, X))
    r, den = B - D @ X, np.abs(D) @ np.abs(X) + np.abs(B)
    Et = E.transpose(0, 2, 1)
    r[1:] -= E @ X[:-1]
    r[:-1] -= Et @ X[1:]
    den[1:] += np.abs(E) @ np.abs(X[:-1])
    den[:-1] += np.abs(Et) @ np.abs(X[1:])
    return float((np.abs(r) / den).max())


@pytest.mark.parametrize("digits", [6, 9, 11])
@pytest.mark.parametrize("n", [4, 5, 8, 11, 16, 17, 24, 33, 64, 96, 128])
def test_backward_error_of_ill_conditioned_blocks(n, digits):
    """A backward stable solve: an element of the factor is a sum of at most
    (2 levels + 1) n products, and Cholesky's bound is three times that many
    unit roundoffs."""
    from paper_2601_03754_amd import btc

    N = 11 if n <= 24 else 5
    D, E, B = ill_conditioned(N, n, digits, 100 * n + digits)
    f = btc.Factor(dev(D), dev(E))
    X = f.solve(dev(B)).cpu().numpy()
    assert f.info == 0
    f.close()
    levels = N.bit_length()
    assert backward_error(D, E, B, X) <= 3 * (2 * levels + 1) * n * U


# the Schur sum of block k is formed by: the separator update of its left
# neighbour, its own deferred update, the deferred update its left neighbour
# applies for it
@pytest.mark.parametrize("N,coupling,k", [(2, 1, 2), (3, 2, 2), (5, 4, 4)])
@pytest.mark.parametrize("n", [48, 64])
def test_schur_sums_of_small_products(n, N, coupling, k):
    """D_i = I and one coupling block of entries 2^-28: S_k = I - n 2^-56, whose
    first element is representable.  Subtracted one at a time (or four) the
    products of 2^-56 would each be lost against 1.  L_11^2 then is 1 - n 2^-56
    to the four roundoffs of a square of a square root."""
    from paper_2601_03754_amd import btc

    D = np.broadcast_to(np.eye(n), (N, n, n)).copy()
    E = np.zeros((N - 1, n, n))
    E[coupling - 1] = 2.0 ** -28
    f = btc.Factor(dev(D), dev(E))
    L = f.export()[0][k - 1]
    f.close()
    S = np.longdouble(1) - np.longdouble(n) * np.longdouble(2) ** -56
    assert abs(np.longdouble(L[0, 0]) ** 2 - S) <= 4.5 * U
