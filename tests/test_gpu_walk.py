"""GPU: the level walk's groups of 64 entries, its lowering stack and its slots
at their edges, against the walk of every leaf by itself: the same pairs, and
forces within the parity bar of the FP64 solve (1e-12 of the largest).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def torch():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


@pytest.fixture(scope="module")
def P(torch):
    import paper_2602_05804_amd as P

    return P


@pytest.mark.parametrize("theta", [0.25, 0.8])
@pytest.mark.parametrize("h", [1e-4, 0.05, 0.6])  # short P2P lists, mixed, whole subtrees
@pytest.mark.parametrize("n,leaf_size", [(1, 16), (2, 1), (65, 1), (129, 1), (257, 2), (1500, 1),
                                         (4100, 8), (9000, 32)])
def test_level_walk_equals_leaf_walk(torch, P, n, leaf_size, h, theta):
    print(f"case: walk n {n} leaf {leaf_size} h {h} theta {theta}", flush=True)
    g = np.random.default_rng(n + leaf_size)
    x = g.standard_normal((n, 3)) * np.exp(g.standard_normal((n, 1)))
    hs = np.full(n, h) * np.exp(0.5 * g.standard_normal(n))
    arrs = [torch.from_numpy(a).cuda() for a in (x, g.random(n) + 0.5, hs)]
    got = []
    for walk in ("level", "leaf"):
        s = P.Solver(walk=walk, leaf_size=leaf_size)
        for _ in range(2):  # first with the slots of a new state, then with those it chose
            acc, pot = s.solve(*arrs, theta=theta)[:2]
        st = s.stats()
        got.append((acc.cpu().numpy(), pot.cpu().numpy(),
                    [st[k] for k in ("num_nodes", "n_m2l", "n_p2p_pairs")]))
    assert got[0][2] == got[1][2]
    for k in range(2):
        assert np.abs(got[0][k] - got[1][k]).max() <= TOL * max(np.abs(got[1][k]).max(), 1e-300)
