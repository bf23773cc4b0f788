"""GPU: the shared far field's node order and source records at their edges.

Bar as in test_gpu_parity.py: 1e-12 relative per particle against the oracle.
"""
import numpy as np
import pytest

import workloads

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


# trees of a few nodes, of one and of several windows, and on both sides of the
# size (8192 nodes) from which long lists come first; every record length
@pytest.mark.parametrize("n,leaf_size,order,theta", [
    (11, 10, 3, 0.5), (64, 1, 3, 0.7), (300, 10, 0, 0.6), (300, 10, 4, 0.6),
    (4000, 1, 3, 0.6), (4200, 1, 3, 0.6), (4200, 1, 4, 0.7), (20000, 8, 1, 0.6),
    (20000, 8, 2, 0.5), (40000, 10, 3, 0.4)])
def test_order_and_record_edges(torch, P, orc, n, leaf_size, order, theta):
    print(f"case: far field n={n} leaf {leaf_size} order {order} theta {theta}", flush=True)
    x, m, h = workloads.plummer(n, seed=80 + n)
    h = h * 0.1  # (the opening angle decides: long M2L lists)
    oa, op = orc.sfmm_solve(x, m, h, theta=theta, order=order, leaf_size=leaf_size)
    s = P.Solver(leaf_size=leaf_size)
    xd, md, hd = (torch.from_numpy(a).cuda() for a in (x, m, h))
    acc, pot = s.solve(xd, md, hd, theta=theta, order=order)
    torch.cuda.synchronize()
    nb = np.linalg.norm(oa, axis=1)
    e = np.linalg.norm(acc.cpu().numpy() - oa, axis=1)
    assert (e / np.maximum(nb, 1e-6 * np.sqrt((nb ** 2).mean()))).max() < TOL
    assert (np.abs(pot.cpu().numpy() - op) / np.abs(op)).max() < TOL
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
@pytest.mark.parametrize("n", [4095, 4096, 20000, 1 << 19, (1 << 19) + 1])
def test_near_beside_far_by_size(torch, P, monkeypatch, n, precision):
    """The sizes at which the P2P kernel takes a second stream: the same sums, so
    the same bits, as one after the other; a second solve reuses the buffers."""
    print(f"case: near beside far n {n} {precision}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, 3, dtype=torch.float64, device="cuda", generator=g)
    m = torch.rand(n, dtype=torch.float64, device="cuda", generator=g) + 0.5
    h = torch.full((n,), 1.2 * n ** (-1.0 / 3.0), dtype=torch.float64, device="cuda")
    got = []
    for ov in (None, "0"):
        if ov is None:
            monkeypatch.delenv("SFMM_OVERLAP", raising=False)
        else:
            monkeypatch.setenv("SFMM_OVERLAP", ov)
        s = P.Solver()
        for scale in (1.0, 0.5):
            acc, pot = s.solve(x * scale, m, h * scale, theta=0.8, precision=precision)[:2]
            got.append((acc.clone(), pot.clone()))
    for k in range(2):
        assert torch.equal(got[k][0], got[2 + k][0]) and torch.equal(got[k][1], got[2 + k][1])
