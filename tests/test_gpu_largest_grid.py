"""The default shapes at 1025^3, where no launch table has entries: the bits of
two single sweeps, and of the per-node gather."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu
N = 1025


def grid(g, n=N):
    return torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g)


def test_two_sweeps():
    g = torch.Generator(device="cuda").manual_seed(N)
    f, u, h = grid(g), grid(g), 1.0 / (N - 1)
    uc = torch.zeros((513,) * 3, dtype=torch.float64, device="cuda")
    uc[1:-1, 1:-1, 1:-1] = torch.randn((511,) * 3, dtype=torch.float64, device="cuda", generator=g)
    for c in (None, uc):
        a, b = u.clone(), u.clone()
        if c is not None:
            Q.k_prolong_add(c, a)
        Q.k_rbgs_sweep(f, a, b, h)
        Q.k_rbgs_sweep(f, b, a, h)
        b.copy_(u)
        Q.k_rbgs_double_sweep(f, u, b, h, uc=c)
        assert torch.equal(a, b), c is not None


def test_restriction():
    g = torch.Generator(device="cuda").manual_seed(N + 1)
    f, u, h = grid(g), grid(g), 1.0 / (N - 1)
    before, out = Q.tune_get_rr(N), []
    try:
        for v in (0, before):
            Q.tune_set_rr(N, v)
            out.append([torch.full((513,) * 3, 3.0, dtype=torch.float64, device="cuda") for _ in range(3)])
            Q.k_residual_restrict(f, u, h, *out[-1])
    finally:
        Q.tune_set_rr(N, before)
    assert before == 7 and all(torch.equal(a, b) for a, b in zip(*out))
