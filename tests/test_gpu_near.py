"""GPU: the P2P work items and the wave kernel's passes at their edges.

Bars as in test_gpu_parity.py: 1e-12 relative per particle against the
oracle in FP64, and bit-identical results of a system alone and in a batch.
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


def dev(torch, *arrs):
    return [torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in arrs]


@pytest.mark.parametrize("leaf_size", [1, 7, 8, 9, 10, 15, 16, 17, 31, 32])
@pytest.mark.parametrize("n", [63, 64, 65, 255, 257, 513])
def test_pass_and_run_edges(torch, P, orc, leaf_size, n):
    """Target counts around the pass size of 8 and source counts around a group
    of 64 and a run of 256: every particle inside the others' kernels (so each
    leaf meets all n sources, and every pair but the self pair is queued)."""
    print(f"case: P2P edges n={n} leaf {leaf_size}", flush=True)
    x, m, h = workloads.plummer(n, seed=40 + n)
    h = np.full(n, 1e3)
    da, dp = orc.direct(x, m, h)
    s = P.Solver(leaf_size=leaf_size)
    acc, pot = s.solve(*dev(torch, x, m, h), theta=0.9)
    torch.cuda.synchronize()
    st = s.stats()
    assert st["n_p2p_pairs"] == n * (n - 1) == st["n_p2p_soft_pairs"]
    e = np.linalg.norm(acc.cpu().numpy() - da, axis=1)
    assert (e / np.linalg.norm(da, axis=1)).max() < TOL
    assert (np.abs(pot.cpu().numpy() - dp) / np.abs(dp)).max() < TOL
    s.close()


@pytest.mark.parametrize("near_kernel", [0, 13])
def test_run_length_follows_the_system(torch, P, near_kernel):
    """Sizes on both sides of every change of the run length: a system gets the
    same bits alone and in a batch, whose total size is another."""
    print(f"case: P2P run lengths, shape {near_kernel}", flush=True)
    sizes = [2048, 2049, 16384, 16385, 131072, 131073]
    systems = [tuple(dev(torch, *workloads.plummer(k, seed=60 + i))) for i, k in enumerate(sizes)]
    s = P.Solver(near_kernel=near_kernel)
    batch = [(a.clone(), p.clone()) for a, p in s.solve_batch(systems, theta=0.6)]
    for (a, p), system in zip(batch, systems):
        a1, p1 = s.solve(*system, theta=0.6)
        torch.cuda.synchronize()
        assert torch.equal(a, a1) and torch.equal(p, p1)
    s.close()
