"""The two-sweep march masks nothing on its way in: values on the grid's edges and
corners, and right-hand sides on its faces, enter no interior node's update."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 9, 33, 65, 129])
def test_values_that_no_update_reads(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    h, nc = 1.0 / (n - 1), (n + 1) // 2
    f, u = (torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    uc = torch.zeros((nc,) * 3, dtype=torch.float64, device="cuda")
    uc[1:-1, 1:-1, 1:-1] = 1.5
    faces = torch.zeros((n,) * 3, dtype=torch.int32, device="cuda")
    for d in range(3):
        for e in (0, n - 1):
            faces.select(d, e).add_(1)
    fbad, ubad = f.clone(), u.clone()
    fbad[faces > 0] = float("nan")
    ubad[faces > 1] = float("inf")
    inner = (slice(1, -1),) * 3
    before = Q.tune_get_fused(n)
    try:
        for v in (8, 9, 10):
            for kc in (0, 4, 8):
                Q.tune_set_fused(n, v, kc)
                for c in (None, uc):
                    want, got = torch.zeros_like(u), torch.zeros_like(u)
                    Q.k_rbgs_double_sweep(f, u, want, h, uc=c)
                    Q.k_rbgs_double_sweep(fbad, ubad, got, h, uc=c)
                    assert torch.isfinite(got).all() and torch.equal(got[inner], want[inner]), (v, kc)
    finally:
        Q.tune_set_fused(n, *before)
