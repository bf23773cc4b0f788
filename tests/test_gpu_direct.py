"""GPU: the direct sum at the edges of its groups of 4 sources, of 64 targets and
of its queue of softened pairs (none, some, every pair inside a kernel, a few
targets that reach everything), against the CPU oracle's direct sum; bar as for
the FP64 solve, 1e-12 per target relative to its sum of magnitudes.
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


@pytest.mark.parametrize("kind", ["none", "some", "all", "few"])
@pytest.mark.parametrize("n,nt", [(1, None), (2, None), (3, None), (5, 4), (63, None), (64, None),
                                  (65, 130), (127, 1), (257, 64), (700, 65), (2000, None)])
def test_direct_edges(torch, orc, n, nt, kind):
    import paper_2602_05804_amd as P

    print(f"case: direct n {n} targets {nt} {kind}", flush=True)
    g = np.random.default_rng(n)
    x = g.standard_normal((n, 3))
    if n > 4:
        x[n // 2] = x[0]  # a pair at one place
    m = g.random(n) + 0.5
    h = {"none": 1e-9, "some": 0.1, "all": 50.0, "few": 1e-3}[kind] * (1.0 + g.random(n))
    if kind == "few":
        h[::37] = 20.0
    tg = None if nt is None else g.integers(0, n, nt)  # (targets may repeat)
    s = P.Solver()
    args = [torch.from_numpy(a).cuda() for a in (x, m, h)]
    acc, pot = s.direct(*args, targets=None if tg is None else torch.from_numpy(tg).cuda())
    again, _ = s.direct(*args, targets=None if tg is None else torch.from_numpy(tg).cuda())
    assert torch.equal(acc, again)
    ids = np.arange(n) if tg is None else tg
    oa, op = orc.direct(x, m, h, targets=ids.astype(np.int64))
    acc, pot = acc.cpu().numpy(), pot.cpu().numpy()
    scale = np.maximum(np.linalg.norm(oa, axis=1), np.abs(op))  # (unit lengths)
    scale = np.maximum(scale, 1e-300)
    assert (np.linalg.norm(acc - oa, axis=1) / scale).max() <= TOL
    assert (np.abs(pot - op) / np.maximum(np.abs(op), 1e-300)).max() <= TOL


@pytest.mark.parametrize("n,nt", [(3, None), (64, None), (67, 33), (130, None), (1500, 70)])
@pytest.mark.parametrize("first", [0, 1, 2, 3, 4])
def test_chunks_met_in_place(torch, orc, n, nt, first):
    """Chunks of which `first` of the four sources looked at reach every target and
    the others few, on both sides of the share from which all are met in place."""
    import paper_2602_05804_amd as P

    print(f"case: direct in place n {n} targets {nt} first {first}", flush=True)
    g = np.random.default_rng(n + first)
    x = g.standard_normal((n, 3))
    m = g.random(n) + 0.5
    h = np.full(n, 1e-3)
    h[np.isin(np.arange(n) % 64, [0, 16, 32, 48][:first])] = 20.0
    h[::50] = 1e-110  # (and some point masses)
    tg = None if nt is None else g.integers(0, n, nt)
    s = P.Solver(include_self_potential=False)
    acc, pot = s.direct(*(torch.from_numpy(a).cuda() for a in (x, m, h)),
                        targets=None if tg is None else torch.from_numpy(tg).cuda())
    ids = np.arange(n) if tg is None else tg
    oa, op = orc.direct(x, m, h, targets=ids.astype(np.int64), include_self=False)
    scale = np.maximum(np.linalg.norm(oa, axis=1), np.abs(op))  # (unit lengths)
    assert (np.linalg.norm(acc.cpu().numpy() - oa, axis=1) / scale).max() <= TOL
    assert (np.abs(pot.cpu().numpy() - op) / np.abs(op)).max() <= TOL


@pytest.mark.parametrize("nt", [1, 2, 65])
@pytest.mark.parametrize("n", [64 * 256, 64 * 256 + 1, 64 * 257 + 5, 64 * 600])
def test_few_targets(torch, orc, n, nt):
    """256 chunks and more: one thread, then one wave a target."""
    import paper_2602_05804_amd as P

    print(f"case: direct n {n} targets {nt}", flush=True)
    g = np.random.default_rng(n)
    x, m, h = g.standard_normal((n, 3)), g.random(n) + 0.5, np.full(n, 0.02)
    tg = g.integers(0, n, nt)
    s = P.Solver()
    args = [torch.from_numpy(a).cuda() for a in (x, m, h)]
    acc, pot = s.direct(*args, targets=torch.from_numpy(tg).cuda())
    again, _ = s.direct(*args, targets=torch.from_numpy(tg).cuda())
    assert torch.equal(acc, again)
    oa, op = orc.direct(x, m, h, targets=tg.astype(np.int64))
    assert (np.linalg.norm(acc.cpu().numpy() - oa, axis=1) / np.linalg.norm(oa, axis=1)).max() <= TOL
    assert (np.abs(pot.cpu().numpy() - op) / np.abs(op)).max() <= TOL
    with pytest.raises(P.SfmmError):
        s.direct(*args, targets=torch.tensor([n]).cuda())
