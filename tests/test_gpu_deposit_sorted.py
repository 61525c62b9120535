"""The deposit that sorts particles by cell tile: the same integers as the
oracle's deposit, for particles on tile faces, box faces and outside, in slices,
and (by the window form) under stream capture."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _particles(n, sides, count, seed):
    """A thin disk, particles on cell and tile faces of every box, and some outside the outermost."""
    g = np.random.default_rng(seed)
    x, y = g.normal(0.0, sides[-1] * 0.4, (2, count))
    z = g.normal(0.0, sides[-1] * 0.02, count)
    m = g.uniform(0.5, 2.0, count)
    k = count // 10
    L = np.array(sides)[g.integers(0, len(sides), k)]
    for a in (x, y, z):
        a[:k] = (g.integers(0, (n - 1) // 8 + 1, k) * 8) * (L / (n - 1)) - 0.5 * L
    x[k:k + 50] = sides[0] * g.uniform(0.5, 3.0, 50)
    return x, y, z, m


@pytest.mark.parametrize("n,sides,count", [(129, [100.0], 250000), (129, [400.0, 200.0, 100.0, 50.0], 300001),
                                           (257, [120.0], 250001), (257, [64.0 * 2.0 ** -b for b in range(11)], 260003)])
def test_same_integers_as_the_oracle(n, sides, count):
    x, y, z, m = _particles(n, sides, count, n + len(sides))
    M = float(m.sum())
    ctx = Q.Context(Q.Config(n=n, box_side=sides))
    outside = ctx.deposit(_dev(x), _dev(y), _dev(z), _dev(m), M)
    shift = O.fixed_shift(M)
    for b, L in enumerate(sides):
        q, inside = O.cic_deposit(n, L, x, y, z, m, shift)
        assert np.array_equal(ctx.get_field(b, Q.FIELD_RHO_FIXED).cpu().numpy(), q), b
        if b == 0:
            assert outside == count - inside
    ctx.close()


def test_slices_and_a_smaller_deposit_after_a_larger_one():
    count, cut = (1 << 26) + 12345, 300000
    g = torch.Generator(device="cuda").manual_seed(5)
    x, y = (torch.randn(count, generator=g, device="cuda", dtype=torch.float64) * 9.0 for _ in range(2))
    z = torch.randn(count, generator=g, device="cuda", dtype=torch.float64) * 0.4
    m = torch.ones_like(x)
    ctx = Q.Context(Q.Config(n=129, box_side=[60.0], fixed_shift=30))
    out = [ctx.deposit(x, y, z, m, float(count))]
    whole = ctx.get_field(0, Q.FIELD_RHO_FIXED)
    parts = torch.zeros_like(whole)
    for s in (slice(0, cut), slice(cut, count)):
        out.append(ctx.deposit(x[s], y[s], z[s], m[s], float(count)))
        parts += ctx.get_field(0, Q.FIELD_RHO_FIXED)
    assert torch.equal(whole, parts) and out[0] == out[1] + out[2] and out[0] > 0
    ctx.close()


def test_first_workspace_beside_another_capture():
    x, y, z, m = (_dev(a) for a in _particles(129, [100.0], 260000, 4))
    M = float(m.sum().item())
    ctx = Q.Context(Q.Config(n=129, box_side=[100.0]), stream=torch.cuda.Stream())
    with torch.cuda.stream(ctx.stream):
        torch.cuda.synchronize()
        a = torch.zeros(1000, device="cuda")
        other, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=other):
            a += 1.0
            with torch.cuda.stream(ctx.stream):
                ctx.deposit(x, y, z, m, M, count_outside=False)
        q = ctx.get_field(0, Q.FIELD_RHO_FIXED)
    graph.replay()
    torch.cuda.synchronize()
    assert float(a[0]) == 1.0
    ref = O.cic_deposit(129, 100.0, x.cpu().numpy(), y.cpu().numpy(), z.cpu().numpy(), m.cpu().numpy(), O.fixed_shift(M))
    assert np.array_equal(q.cpu().numpy(), ref[0])
    ctx.close()


def test_capture_keeps_no_workspace():
    x, y, z, m = (_dev(a) for a in _particles(129, [100.0], 300000, 3))
    M = float(m.sum().item())
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = Q.Context(Q.Config(n=129, box_side=[100.0]), stream=s)
        ctx.deposit(x, y, z, m, M, count_outside=False)
        want = ctx.get_field(0, Q.FIELD_RHO_FIXED)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        ctx.deposit(x, y, z, m, M, count_outside=False)
    for _ in range(3):
        with torch.cuda.stream(s):      # a larger deposit replaces the workspace between replays
            big = [torch.cat([a, a]) for a in (x, y, z, m)]
            ctx.deposit(*big, 2.0 * M, count_outside=False)
        s.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            got = ctx.get_field(0, Q.FIELD_RHO_FIXED)
        s.synchronize()
        assert torch.equal(got, want)
    ctx.close()
