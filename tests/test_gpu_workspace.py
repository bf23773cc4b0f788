"""GPU: device memory a context holds per particle.  Node records are the largest
part of what grows with the tree; they are sized by the nodes there are (0.3 a
particle at leaf size 10), not by the two a particle there could be.

Bars: 2950 and 3050 bytes a particle (FP64, FP32C) at 20000 particles in a cube;
records for 2n nodes take 3390 and 3490.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bar", [("fp64", 2950), ("fp32c", 3050)])
def test_bytes_per_particle(precision, bar):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2602_05804_amd as P

    print(f"case: workspace {precision}", flush=True)
    n = 20000
    g = torch.Generator(device="cuda").manual_seed(0)
    x = torch.rand((n, 3), dtype=torch.float64, device="cuda", generator=g)
    m = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    h = torch.full((n,), 0.05, dtype=torch.float64, device="cuda")
    s = P.Solver()
    for _ in range(3):
        s.solve(x, m, h, precision=precision)
    torch.cuda.synchronize()
    assert s.workspace_bytes() / n <= bar
