"""Interpolation (without the addition) on both sides of the size from which a
thread takes a coarse cell: the trilinear expression's bits inside, faces left alone."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def refine(a, d):
    n = a.shape[d]
    out = torch.empty([2 * n - 1 if e == d else m for e, m in enumerate(a.shape)], dtype=a.dtype, device=a.device)
    out.narrow(d, 0, 2 * n - 1).index_copy_(d, torch.arange(0, 2 * n - 1, 2, device=a.device), a)
    out.index_copy_(d, torch.arange(1, 2 * n - 1, 2, device=a.device), 0.5 * a.narrow(d, 0, n - 1) + 0.5 * a.narrow(d, 1, n - 1))
    return out


@pytest.mark.parametrize("nc", [3, 65, 129])
def test_interpolation_equals_the_expression(nc):
    n = 2 * nc - 1
    g = torch.Generator(device="cuda").manual_seed(nc)
    uc = torch.randn((nc,) * 3, dtype=torch.float64, device="cuda", generator=g)
    u = torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g)
    want = u.clone()
    inner = (slice(1, -1),) * 3
    want[inner] = refine(refine(refine(uc, 2), 1), 0)[inner]
    Q.k_interp(uc, u)
    assert torch.equal(u, want)
