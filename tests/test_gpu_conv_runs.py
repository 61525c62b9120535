"""The stride-1 convolution on runs of tiles: several tiles per workgroup, tiles
that end at the grid's faces, one to three blocks of output channels per
workgroup, weights kept in registers or read ahead."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


# (65, 32 -> 16) has 1445 tiles for 768 workgroups; (81, 16 -> 48) and (97, 8 -> 16) several per workgroup too
@pytest.mark.parametrize("n,cin,cout", [(3, 8, 16), (17, 16, 32), (33, 48, 16), (33, 32, 96), (65, 32, 16), (65, 16, 16),
                                        (81, 16, 48), (97, 8, 16), (35, 96, 32), (19, 8, 96)])
def test_tiles_match_fp64(n, cin, cout):
    g = torch.Generator(device="cuda").manual_seed(n + cin + cout)
    x = torch.randn(n ** 3 * cin, generator=g, device="cuda").to(torch.bfloat16)
    kpad = (27 * cin + 31) // 32 * 32
    w = torch.full((cout, kpad), float("nan"), device="cuda", dtype=torch.bfloat16)   # the padding is not read as weights
    w[:, :27 * cin] = (torch.randn(cout, 27 * cin, generator=g, device="cuda") / (27 * cin) ** 0.5).to(torch.bfloat16)
    b = torch.randn(cout, generator=g, device="cuda")
    y = Q.k_conv3d_fwd(x, n, cin, w, cout, b, 1, False).double().reshape(n, n, n, cout)
    p = torch.nn.functional.pad(x.double().reshape(n, n, n, cin), (0, 0, 1, 1, 1, 1, 1, 1))
    ref = b.double().expand(n, n, n, cout).clone()
    mag = b.double().abs().expand(n, n, n, cout).clone()
    for t in range(27):
        v = p[t // 9:t // 9 + n, t // 3 % 3:t // 3 % 3 + n, t % 3:t % 3 + n].reshape(-1, cin)
        wt = w[:, t * cin:(t + 1) * cin].double().t().contiguous()
        ref += (v @ wt).reshape(n, n, n, cout)
        mag += (v.abs() @ wt.abs()).reshape(n, n, n, cout)
    # one rounding to 8 bits, and FP32 sums of 27 cin products (2^-23 of the sum of magnitudes per addition at most,
    # one addition per 32 products and the products' own sum inside an MFMA)
    tol = 2.0 ** -8 * ref.abs() + 2.0 ** -23 * (kpad // 32 + 32) * mag
    assert bool(((y - ref).abs() <= tol).all())
