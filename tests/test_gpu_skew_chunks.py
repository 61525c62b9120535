"""The skewed two-sweep march on chunks of a column: every chunk boundary gives
the bits of two single sweeps, with the coarse-grid correction those of a
prolong-add and two sweeps, and from a zero iterate those of a zeroed array."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


# one chunk and several, chunks that end beside the far face or hold one plane there, odd sizes (rounded up)
@pytest.mark.parametrize("n,kchunks", [(5, (4,)), (9, (4, 5, 6)), (17, (4, 8, 14)), (33, (4, 6, 10, 30)),
                                       (65, (4, 12, 44, 62)), (129, (8, 10, 42)), (257, (52, 64))])
def test_chunks_keep_the_bits(n, kchunks):
    g = torch.Generator(device="cuda").manual_seed(n)
    h, nc = 1.0 / (n - 1), (n + 1) // 2

    def zero_faces(a):
        a[0] = a[-1] = a[:, 0] = a[:, -1] = a[:, :, 0] = a[:, :, -1] = 0.0
        return a

    f = torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g)
    u = torch.randn((n,) * 3, dtype=torch.float64, device="cuda", generator=g)
    uc = zero_faces(torch.randn((nc,) * 3, dtype=torch.float64, device="cuda", generator=g))

    def two(a):
        b, c = a.clone(), a.clone()
        Q.k_rbgs_sweep(f, a, b, h)
        Q.k_rbgs_sweep(f, b, c, h)
        return c

    p = u.clone()
    Q.k_prolong_add(uc, p)
    want = two(u), two(p), two(torch.zeros_like(u))
    before = Q.tune_get_fused(n)
    try:
        for v in (8, 9, 10):
            for kc in kchunks:
                Q.tune_set_fused(n, v, kc)
                for src, c, ref in ((u, None, want[0]), (u, uc, want[1]), (None, None, want[2])):
                    out = u.clone() if src is not None else torch.zeros_like(u)
                    out[1:-1, 1:-1, 1:-1] = -7.0
                    Q.k_rbgs_double_sweep(f, src, out, h, uc=c)
                    assert torch.equal(out, ref), (v, kc, c is not None, src is None)
    finally:
        Q.tune_set_fused(n, *before)
