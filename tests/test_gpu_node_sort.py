"""GPU: the node sorts (by depth, by list length) where the tree has at most 2^18
nodes and the particles would have room for more: small leaves from 2^17
particles on, and many tiny systems.  Tree against the oracle's, whole numbers
compared exactly; the solve of sampled particles against the oracle's at 1e-12
relative per particle, as in test_gpu_parity.py.
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


@pytest.mark.parametrize("n,leaf_size", [(131073, 4), (150000, 5), (150000, 6), (200000, 2),
                                         (200000, 3), (300000, 4), (450000, 5)])
def test_small_leaves(torch, P, orc, n, leaf_size):
    print(f"case: node sorts n {n} leaf {leaf_size}", flush=True)
    g = np.random.default_rng(n + leaf_size)
    x = g.standard_normal((n, 3))
    m = g.random(n) + 0.5
    h = np.full(n, 0.01)
    t = orc.Tree(x, m, h, leaf_size=leaf_size)
    s = P.Solver(leaf_size=leaf_size)
    args = [torch.from_numpy(a).cuda() for a in (x, m, h)]
    for _ in range(2):
        acc, pot = s.solve(*args, theta=0.8)
    got = s.tree()
    assert len(got["lo"]) == t.num_nodes
    assert np.array_equal(got["perm"], t.perm())
    o = t.nodes()
    a = sorted(zip(got["lo"], got["cnt"]))
    assert a == sorted(zip(o["lo"], o["hi"] - o["lo"]))
    assert s.stats()["max_depth"] == t.max_depth
    ids = np.sort(g.permutation(n)[:300])
    oa, op, _ = t.solve(theta=0.8, targets=ids)
    acc, pot = acc.cpu().numpy()[ids], pot.cpu().numpy()[ids]
    nb = np.linalg.norm(oa, axis=1)
    e = np.linalg.norm(acc - oa, axis=1)
    assert (e / np.maximum(nb, 1e-6 * np.sqrt((nb ** 2).mean()))).max() < TOL
    assert (np.abs(pot - op) / np.abs(op)).max() < TOL
    s.close()


def test_many_pairs(torch, P):
    """70000 systems of two particles: as many nodes as particles."""
    print("case: node sorts, 70000 systems of two", flush=True)
    k = 70000
    g = np.random.default_rng(5)
    x = g.standard_normal((k, 2, 3))
    m = g.random((k, 2)) + 0.5
    h = np.full((k, 2), 1e-6)
    xd, md, hd = (torch.from_numpy(a).cuda() for a in (x, m, h))
    s = P.Solver(include_self_potential=False)
    for _ in range(2):
        out = s.solve_batch(list(zip(xd, md, hd)), theta=0.5)
    acc = torch.stack([a for a, _ in out]).cpu().numpy()
    pot = torch.stack([p for _, p in out]).cpu().numpy()
    d = x[:, 0] - x[:, 1]
    r = np.linalg.norm(d, axis=1)
    for i, sign in ((0, -1.0), (1, 1.0)):
        want = sign * (m[:, 1 - i] / r ** 3)[:, None] * d
        assert np.abs(acc[:, i] - want).max(axis=1).max() <= TOL * np.abs(want).max()
        assert (np.linalg.norm(acc[:, i] - want, axis=1) / np.linalg.norm(want, axis=1)).max() < TOL
        assert (np.abs(pot[:, i] + m[:, 1 - i] / r) / (m[:, 1 - i] / r)).max() < TOL
    s.close()
