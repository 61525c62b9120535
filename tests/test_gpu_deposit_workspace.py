"""The workspace of large deposits: counts that creep up share one, and a call
that needs a larger one neither waits for the stream nor disturbs the deposit
before it."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def disk(count, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, y, z = (torch.randn(count, generator=g, device="cuda", dtype=torch.float64) * s for s in (15.0, 15.0, 0.5))
    return x, y, z, torch.rand(count, generator=g, device="cuda", dtype=torch.float64) + 0.5


def test_creeping_counts_share_a_workspace():
    p = disk(1 << 19, 1)
    ctx = Q.Context(Q.Config(n=129, box_side=[100.0]))
    bare, seen = ctx.device_bytes, []
    for count in list(range(250000, 262144, 2000)) + [262144, 262145, 400000, 1 << 19, 300000]:
        ctx.deposit(*(a[:count] for a in p), 1e6)
        seen.append(ctx.device_bytes)
    assert bare < seen[0] and len(set(seen)) == 2, seen     # 2^18 and 2^19 particles
    ctx.close()


def test_growth_waits_for_nothing():
    small, large = disk(250000, 2), disk(2500000, 3)
    s = torch.cuda.Stream()
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    b = torch.empty_like(a)
    done = torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        ctx = Q.Context(Q.Config(n=129, box_side=[100.0]), stream=s)
        ctx.deposit(*large, 1e7)
        want = ctx.get_field(0, Q.FIELD_RHO_FIXED)
        ctx.close()
        ctx = Q.Context(Q.Config(n=129, box_side=[100.0]), stream=s)
        torch.mm(a, a, out=b)
        s.synchronize()
        for _ in range(100):                 # about 0.1 s of work
            torch.mm(a, a, out=b)
        ctx.deposit(*small, 1e6, count_outside=False)
        done.record(s)
        ctx.deposit(*large, 1e7, count_outside=False)
        assert not done.query()
        got = ctx.get_field(0, Q.FIELD_RHO_FIXED)
    s.synchronize()
    assert torch.equal(got, want)
    ctx.close()
