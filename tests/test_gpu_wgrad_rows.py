"""The weight gradient of a convolution: the LDS-transposed kernel takes aligned
tensors, the gathering one any alignment, with the same chain of MFMAs per
weight, so the two agree bit for bit; both agree with the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def _shifted(t, by=4):
    """The same values 2 * by bytes past a 16-byte boundary."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")
    buf[by:].copy_(t)
    return buf[by:]


# one chunk and less, ends of rows inside a fragment, channel groups of 8, splits that end in the middle of a chunk
@pytest.mark.parametrize("n,cin,cout,stride", [(3, 8, 16, 1), (3, 8, 16, 2), (5, 24, 16, 1), (7, 16, 32, 2),
                                               (17, 8, 16, 1), (17, 40, 48, 2), (19, 16, 16, 1), (33, 48, 64, 1),
                                               (33, 32, 96, 2), (35, 64, 128, 1)])
def test_rows_equal_gather(n, cin, cout, stride):
    g = torch.Generator(device="cuda").manual_seed(n * 1000 + cin + cout)
    no = (n + 1) // 2 if stride == 2 else n
    x = torch.randn(n ** 3 * cin, generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randn(no ** 3 * cout, generator=g, device="cuda").to(torch.bfloat16)
    assert x.data_ptr() % 16 == 0 and _shifted(x).data_ptr() % 16 == 8
    rows = Q.k_conv3d_wgrad(n, cin, x, cout, dy, stride)
    assert torch.equal(rows, Q.k_conv3d_wgrad(n, cin, _shifted(x), cout, dy, stride))
    assert torch.equal(rows, Q.k_conv3d_wgrad(n, cin, x, cout, _shifted(dy), stride))
    ref = O.conv3d_wgrad(x.double().cpu().numpy().reshape(-1, cin), dy.double().cpu().numpy().reshape(-1, cout), cout, stride)
    got = rows.cpu().numpy().reshape(cout, -1)
    # no^3 products of unit variance: partial sums of about sqrt(no^3), each rounded to 24 bits, add up to
    # 2^-24 no^3 if every rounding had the same sign; 8 times that leaves room for the values' tails
    assert np.abs(got[:, :27 * cin] - ref.reshape(cout, 27 * cin)).max() <= 2.0 ** -21 * no ** 3
    assert not got[:, 27 * cin:].any()
