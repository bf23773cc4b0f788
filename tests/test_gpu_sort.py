"""GPU: the particle and node orderings at the edges of the sorts: one block
in LDS up to 4096 elements, tiles of 1024 up to 2^18, tiles of 4096 above;
equal keys keep the caller's order.  Whole numbers: compared exactly.
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


def spread3(v):
    v = v.astype(np.uint64)
    for sh, mask in ((32, 0x1f00000000ffff), (16, 0x1f0000ff0000ff), (8, 0x100f00f00f00f00f),
                     (4, 0x10c30c30c30c30c3), (2, 0x1249249249249249)):
        v = (v | (v << np.uint64(sh))) & np.uint64(mask)
    return v


def morton(x):
    lo = x.min(0)
    ext = (x.max(0) - lo).max()
    if ext == 0.0:
        return np.zeros(len(x), np.uint64)
    c = np.minimum(np.floor((x - lo) * (2097152.0 / ext)), 2097151.0)
    a, b, d = (spread3(c[:, k]) for k in range(3))
    return (a << np.uint64(2)) | (b << np.uint64(1)) | d


def make(n, kind, seed):
    g = np.random.default_rng(seed)
    if kind == "clumps":  # many equal keys: sites drawn again and again
        x = g.standard_normal((max(1, n // 5), 3))[g.integers(0, max(1, n // 5), n)]
    elif kind == "line":  # digits of one axis only
        x = np.zeros((n, 3))
        x[:, 1] = g.random(n)
    else:
        x = g.standard_normal((n, 3)) ** 3
    return x, g.random(n) + 0.5, g.random(n) * 0.01 + 1e-4


def dev(torch, *arrs):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]


@pytest.mark.parametrize("kind", ["cubed", "clumps", "line"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1025, 4095, 4096, 4097, 12289,
                               (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 4097])
def test_particle_order(torch, P, n, kind):
    print(f"case: order n {n} {kind}", flush=True)
    x, m, h = make(n, kind, n)
    s = P.Solver()
    s.solve(*dev(torch, x, m, h), theta=0.9, order=1)
    t = s.tree(order=1)
    key = morton(x)
    perm = np.argsort(key, kind="stable")
    assert np.array_equal(t["perm"], perm)
    assert np.array_equal(t["keys"], key[perm])


@pytest.mark.parametrize("sizes", [[1, 1], [1, 700, 3], [300] * 255, [40] * 256, [40] * 257,
                                   [3000, 2, 3000], [200000, 1, 70000]])
def test_batch_order(torch, P, sizes):
    """Each system sorted by itself, in one and in two digits of its number."""
    print(f"case: batch order {len(sizes)} systems", flush=True)
    sysl = [make(n, "clumps" if k % 2 else "cubed", k) for k, n in enumerate(sizes)]
    s = P.Solver()
    s.solve_batch([tuple(dev(torch, *a)) for a in sysl], theta=0.9, order=1)
    t = s.tree(order=1)
    at = 0
    for x, _, _ in sysl:
        key = morton(x)
        perm = np.argsort(key, kind="stable")
        assert np.array_equal(t["perm"][at:at + len(x)], perm + at)
        assert np.array_equal(t["keys"][at:at + len(x)], key[perm])
        at += len(x)
