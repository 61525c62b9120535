"""The z-marching residual restriction where its tiles and chunks end: grids
below, at and above the tiles of 16 x 8 and 32 x 8 coarse columns, against the
per-node gather (equal bits), with values that must not spread from the boundary."""
import numpy as np
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu
MARCH = (2, 3, 4, 7, 8, 9, 10, 11)


def run(n, v, f, u):
    nc = (n + 1) // 2
    before = Q.tune_get_rr(n)
    try:
        Q.tune_set_rr(n, v)
        out = [torch.full((nc,) * 3, 3.0, dtype=torch.float64, device="cuda") for _ in range(3)]
        Q.k_residual_restrict(f, u, 1.0 / (n - 1), *out)
        return [o.cpu().numpy() for o in out]
    finally:
        Q.tune_set_rr(n, before)


@pytest.mark.parametrize("n", [5, 9, 17, 33, 65, 129])
def test_equals_the_gather_with_large_boundary_values(n):
    """Right-hand sides on the faces and iterates on the edges and corners enter
    no interior residual: NaN there changes nothing."""
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    f, u = (torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    face = torch.zeros((n,) * 3, dtype=torch.int32, device="cuda")
    for d in range(3):
        for e in (0, n - 1):
            face.select(d, e).add_(1)
    f[face > 0] = float("nan")
    u[face > 1] = float("nan")
    ref = run(n, 0, f, u)
    assert np.isfinite(ref[0]).all()
    for v in MARCH:
        for a, b in zip(ref, run(n, v, f, u)):
            assert np.array_equal(a, b), v
