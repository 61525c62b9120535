"""The residual restriction at 513^3, where a march of whole columns fills the
chip: every index a saved table can hold gives the per-node gather's bits, and no
march is much slower than the fastest."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu
MARCH = (2, 3, 4, 7, 8, 9, 10, 11)


def test_every_march_at_513():
    n, nc = 513, 257
    g = torch.Generator(device="cuda").manual_seed(n)
    f, u = (torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    before, got, us = Q.tune_get_rr(n), {}, {}
    try:
        for v in (0,) + MARCH:
            Q.tune_set_rr(n, v)
            out = [torch.full((nc,) * 3, 3.0, dtype=torch.float64, device="cuda") for _ in range(3)]
            best = float("inf")
            for _ in range(5):
                e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                e0.record()
                for _ in range(3):
                    Q.k_residual_restrict(f, u, 1.0 / (n - 1), *out)
                e1.record()
                e1.synchronize()
                best = min(best, 1e3 * e0.elapsed_time(e1) / 3)
            got[v], us[v] = out, best
    finally:
        Q.tune_set_rr(n, before)
    for v in MARCH:
        assert all(torch.equal(a, b) for a, b in zip(got[0], got[v])), v
        assert us[v] <= 1.25 * min(us.values()), (v, us)     # a narrow tile reads 1.41 nodes per node, a wide one 1.33
