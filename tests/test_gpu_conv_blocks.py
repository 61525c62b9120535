"""The stride-1 convolution from 32 input channels up: one to four blocks of 16
output channels per workgroup by the size of the grid, one tile or a run."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def _draw(n, cin, cout):
    g = torch.Generator(device="cuda").manual_seed(n + cin + cout)
    kpad = (27 * cin + 31) // 32 * 32
    x = torch.randn(n ** 3 * cin, generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn(cout, kpad, generator=g, device="cuda") / (27 * cin) ** 0.5).to(torch.bfloat16)
    return x, w, torch.randn(cout, generator=g, device="cuda")


# Sizes at which the number of blocks changes: from 98 tiles (25^3) to 2197 (49^3 has 676, 65^3 1445).  An output
# channel's sums do not depend on the channels beside it, so each slice of 16 is the 16-channel convolution's, in
# every bit.
@pytest.mark.parametrize("n", [3, 17, 25, 33, 41, 49, 65])
@pytest.mark.parametrize("cin,cout", [(32, 32), (32, 48), (32, 64), (48, 32), (48, 48), (48, 64), (64, 48), (64, 64),
                                      (96, 64), (32, 96), (32, 128)])
def test_blocks_are_the_single_blocks(n, cin, cout):
    x, w, b = _draw(n, cin, cout)
    y = Q.k_conv3d_fwd(x, n, cin, w, cout, b, 1, True).reshape(-1, cout)
    for k in range(0, cout, 16):
        one = Q.k_conv3d_fwd(x, n, cin, w[k:k + 16].contiguous(), 16, b[k:k + 16].contiguous(), 1, True)
        assert torch.equal(y[:, k:k + 16], one.reshape(-1, 16)), k


# Twice the output channels is at most twice the work, less the staging that the blocks share; a block of 16 per
# workgroup, each staging the tile again, had taken 2.17 and 2.12 times the time.
@pytest.mark.parametrize("cin,narrow,wide", [(32, 32, 64), (48, 32, 64)])
def test_wide_outputs_share_their_tiles(cin, narrow, wide):
    def best(cout):
        x, w, b = _draw(97, cin, cout)
        times = []
        for _ in range(12):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(4):
                Q.k_conv3d_fwd(x, 97, cin, w, cout, b, 1, True)
            ev[1].record()
            ev[1].synchronize()
            times.append(ev[0].elapsed_time(ev[1]))
        return min(times)

    assert best(wide) <= 2.0 * best(narrow)
