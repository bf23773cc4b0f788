"""GPU: the range of lengths that a solve takes.

Lengths (positions and softening lengths) times 2^k: every operation of the FP64
solve is homogeneous in them and a power of two rounds nothing, so accelerations
are 2^-2k and potentials 2^-k times those at k = 0, bit for bit, as long as
nothing leaves the range of FP64.  The largest derivative met is of degree
order + 1, of the size of r^-(order + 2): at order 4 and |k| = 160 about 2^960.
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


@pytest.mark.parametrize("far", ["shared", "leaf"])
@pytest.mark.parametrize("order", [0, 1, 2, 3, 4])
def test_powers_of_two_in_the_lengths(torch, P, order, far):
    print(f"case: lengths times 2^k, order {order} far {far}", flush=True)
    g = np.random.default_rng(order)
    n = 3000
    x, m, h = (torch.from_numpy(a).cuda()
               for a in (g.standard_normal((n, 3)), g.random(n) + 0.5, np.full(n, 0.05)))
    s = P.Solver(far=far)
    acc0, pot0 = (t.clone() for t in s.solve(x, m, h, theta=0.7, order=order))
    assert s.stats()["n_m2l_unique"] > 1000
    for k in (-160, -120, -100, -60, -1, 60, 100, 120, 160):
        f = 2.0 ** k
        acc, pot = s.solve(x * f, m, h * f, theta=0.7, order=order)
        assert torch.equal(acc * f * f, acc0), k
        assert torch.equal(pot * f, pot0), k


def escaped(far):
    """A small system, one particle of it so far away that it acts on nothing."""
    g = np.random.default_rng(11)
    n = 300
    x = g.standard_normal((n, 3))
    x[7] = (far, 0.0, 0.0)
    return x, g.random(n) + 0.5, np.full(n, 0.3)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32c", 1e-4)])
@pytest.mark.parametrize("far", [1e100, 1e150, 1e160, 1e300])
def test_solve_with_an_escaped_particle(torch, P, orc, far, precision, tol):
    """|r|^2 overflows from 1e154 on.  The others as without it (an opening angle
    at which they meet each other directly); bars as in test_gpu_parity.py."""
    print(f"case: solve, a particle at {far} {precision}", flush=True)
    x, m, h = escaped(far)
    keep = np.arange(len(m)) != 7
    oa, op = orc.direct(x[keep], m[keep], h[keep])
    for order in (0, 3, 4):
        s = P.Solver()
        acc, pot = (t.cpu().numpy() for t in s.solve(
            *(torch.from_numpy(a).cuda() for a in (x, m, h)), theta=0.05, order=order,
            precision=precision))
        assert (np.linalg.norm(acc[keep] - oa, axis=1) / np.linalg.norm(oa, axis=1)).max() <= tol
        assert (np.abs(pot[keep] - op) / np.abs(op)).max() <= tol
        assert np.abs(acc[7]).max() <= 1e-190  # (its own: the others' mass / far^2 at most)
        assert abs(pot[7] + 1.4 * m[7] / h[7]) <= 1e-12 * 1.4 * m[7] / h[7]


@pytest.mark.parametrize("far", [1e100, 1e150, 1e160, 1e300])
def test_direct_with_an_escaped_particle(torch, P, orc, far):
    print(f"case: direct, a particle at {far}", flush=True)
    x, m, h = escaped(far)
    keep = np.arange(len(m)) != 7
    oa, op = orc.direct(x[keep], m[keep], h[keep])
    args = [torch.from_numpy(a).cuda() for a in (x, m, h)]
    h_all = torch.full_like(args[2], 1e160)  # (every |r|^2 below 4 h^2, which overflows)
    for hs, da, dp in ((args[2], oa, op), (h_all, None, None)):
        acc, pot = (t.cpu().numpy() for t in P.Solver().direct(args[0], args[1], hs))
        assert np.isfinite(acc).all() and np.isfinite(pot).all()
        if da is None:
            continue
        assert (np.linalg.norm(acc[keep] - da, axis=1) / np.linalg.norm(da, axis=1)).max() <= 1e-12
        assert (np.abs(pot[keep] - dp) / np.abs(dp)).max() <= 1e-12
        assert np.abs(acc[7]).max() <= 1e-190
