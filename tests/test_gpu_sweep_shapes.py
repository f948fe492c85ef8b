"""Launch shapes of the sweeps in calls of many nodes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2601_03754_amd import inputs

pytestmark = pytest.mark.gpu
SHAPE, FORWARD, BACKWARD = 6, 1, 2


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("precision", [0, 1])
def test_wide_levels_of_a_batch_keep_launches_of_their_own(precision):
    """Shape 2 starts the shared launch one level lower than shape 0; the levels
    below still have a launch each (kind 0 / 1 of the launch profile, the
    shared one kind 2 / 3), and the results stay the same."""
    from paper_2601_03754_amd import btc

    N, n = 140001, 5
    pr = inputs.block_tridiag(N, n, seed=5)
    D, E, B = dev(pr.D), dev(pr.E), dev(pr.B)
    before = btc.btc_tune_get(SHAPE, precision, n, 0)
    launches, out = {}, {}
    try:
        for shape in (0, 1, 2):
            btc.btc_tune_set(SHAPE, precision, n, 0, shape)
            r = btc.Runner()
            h = btc.btc_create(N, n, precision)
            X = torch.empty_like(B)
            r.factor_batched([h], [D], [E])
            r.profile(FORWARD)
            r.solve_batched([h], [B], [X])
            stats = r.profile_read()
            rounds = 1 if precision == 0 else 5
            launches[shape] = {k: sum(s["launches"] for s in stats if s["op"] == FORWARD and s["kind"] == k) / rounds
                               for k in (precision, 2 + precision)}
            out[shape] = X.cpu().numpy()
            btc.btc_destroy(h)
            r.close()
    finally:
        btc.btc_tune_set(SHAPE, precision, n, 0, before)
    levels = N.bit_length()
    own = {s: launches[s][precision] for s in launches}
    shared = {s: launches[s][2 + precision] for s in launches}
    assert (own[1], shared[1]) == (levels, 0)
    assert shared[0] == shared[2] == 1 and own[2] == own[0] - 1 >= 1
    assert oracle.relres(pr.D, pr.E, out[0], pr.B) <= (1e-12 if precision == 0 else 1e-10)
    for s in (1, 2):
        assert np.array_equal(out[s], out[0])


@pytest.mark.parametrize("large", [700, 2600])
def test_refinements_that_end_in_different_rounds(large):
    """A shared launch of few nodes, and one of many (which first asks whether
    any instance still has work): an instance that needs several corrections
    beside ones that are done after the first, each as if alone."""
    from paper_2601_03754_amd import btc

    n = 12
    prs = [inputs.block_tridiag(large, n, seed=1), inputs.block_tridiag(40, n, c=0.1, seed=2, margin=True),
           inputs.block_tridiag(90, n, seed=3)]
    Ds, Es, Bs = ([dev(getattr(p, a)) for p in prs] for a in "DEB")
    precision = btc.BTC_BF16_IR
    r = btc.Runner()
    hs = [btc.btc_create(p.N, n, precision) for p in prs]
    Xs = [torch.empty_like(b) for b in Bs]
    r.factor_batched(hs, Ds, Es)
    info = r.solve_batched(hs, Bs, Xs, 1, want_info=True)
    steps = []
    for k, p in enumerate(prs):
        f = btc.Factor(Ds[k], Es[k], precision=precision)
        X, alone = f.solve(Bs[k], want_info=True)
        assert np.array_equal(X.cpu().numpy(), Xs[k].cpu().numpy()), k
        assert info[k]["steps"] == alone["steps"] and info[k]["converged"]
        steps.append(alone["steps"])
        f.close()
    assert steps[1] > max(steps[0], steps[2])
    for h in hs:
        btc.btc_destroy(h)
    r.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_served_ranges_share_only_small_levels(precision):
    """A server in level ranges: one tick of a whole long sweep would hold up
    every other request of its lane, so only levels of a few nodes (up to 32)
    share a launch (kind 2 / 3 of the launch profile); the rest run level by level."""
    from paper_2601_03754_amd import btc

    N, n = 1000, 12
    pr = inputs.block_tridiag(N, n, seed=3)
    D, E, B = dev(pr.D), dev(pr.E), dev(pr.B)
    X = torch.empty_like(B)
    srv = btc.Server(precision=precision, sweep_ranges=True)
    c = srv.add_client(N, n)
    for r in srv.runner_handles():
        btc.runner_profile(r, FORWARD, -1)
    srv.submit(c, B, X, A=(D, E))
    done = []
    while not done:
        srv.step()
        done = srv.poll()
    torch.cuda.synchronize()
    stats = [s for r in srv.runner_handles() for s in btc.runner_profile_read(r)]
    own = [s for s in stats if s["kind"] == precision]
    shared = [s for s in stats if s["kind"] == 2 + precision]
    srv.close()
    assert sum(s["launches"] for s in own) >= 5 and sum(s["launches"] for s in shared) >= 1
    assert all(s["items"] <= 64 * s["launches"] for s in shared)  # N >> l nodes from level l up
    assert oracle.relres(pr.D, pr.E, X.cpu().numpy(), pr.B) <= (1e-12 if precision == 0 else 1e-10)
