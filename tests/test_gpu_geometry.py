"""GPU: masses, centres, sizes and moments of the nodes at the edges of the
launches that make them: a tree of one leaf, of one block's subtree (512
internal nodes), of one more, of many subtrees, unbalanced ones; nodes of 64
and 65 particles and of 2048 and 2049 (the chunks of the sizes).

Masses, centres, largest h and sizes are made by the same operations in the
same order here and there: compared exactly.  The second moments against sums
over the particles: within 1e-13 of sum m |b|^2 (a few hundred roundings of
2^-53 each).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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


def make(n, kind):
    g = np.random.default_rng(n)
    x = g.standard_normal((n, 3))
    if kind == "chain":  # scales down to 2^-18: a tree with long arms
        x *= 2.0 ** -g.integers(0, 19, (n, 1))
    return x, g.random(n) + 0.5, g.random(n) * 0.01 + 1e-4


@pytest.mark.parametrize("kind", ["ball", "chain"])
@pytest.mark.parametrize("n,leaf_size", [(7, 8), (9, 8), (65, 1), (513, 1), (514, 1), (2049, 1),
                                         (2050, 16), (5000, 1), (30000, 2), (150000, 8)])
def test_node_geometry(torch, P, n, leaf_size, kind):
    print(f"case: geometry n {n} leaf {leaf_size} {kind}", flush=True)
    x, m, h = make(n, kind)
    s = P.Solver(leaf_size=leaf_size)
    s.solve(*[torch.from_numpy(a).cuda() for a in (x, m, h)], theta=0.9, order=2)
    t = s.tree(order=2)
    xs, ms, hs = (a[t["perm"]] for a in (x, m, h))
    inner = np.flatnonzero(t["child"] >= 0)
    a = t["child"][inner]
    ma, mb = t["mass"][a], t["mass"][a + 1]
    assert np.array_equal(t["mass"][inner], ma + mb)
    want = (ma[:, None] * t["s"][a] + mb[:, None] * t["s"][a + 1]) / (ma + mb)[:, None]
    assert np.array_equal(t["s"][inner], want)
    assert np.array_equal(t["hmax"][inner], np.maximum(t["hmax"][a], t["hmax"][a + 1]))
    nodes = np.arange(len(t["lo"]))
    big = nodes[t["cnt"] > 40]
    few = np.random.default_rng(1).permutation(nodes[t["cnt"] <= 40])[:300]
    for v in np.concatenate([big[:600], big[-600:], few]):
        lo, c = t["lo"][v], t["cnt"][v]
        b = xs[lo:lo + c] - t["s"][v]
        d2 = b[:, 0] * b[:, 0] + b[:, 1] * b[:, 1] + b[:, 2] * b[:, 2]
        assert t["l"][v] == np.sqrt(d2.max())
        if c <= leaf_size:
            assert t["hmax"][v] == hs[lo:lo + c].max()
        mm = ms[lo:lo + c]
        q = [(mm * b[:, i] * b[:, j]).sum() * (0.5 if i == j else 1.0)
             for i, j in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]
        assert np.abs(t["Q"][v][4:10] - q).max() <= 1e-13 * max((mm * d2).sum(), 1e-300)
