"""Large deposits choose between the window and the sorted form from a sample of
the particles: the integers do not depend on the choice, and no distribution
takes much longer than the window form alone, which a captured deposit records."""
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def particles(kind, n, sides, count, seed=7):
    """A thin disk, one that fills the outermost box, and one a few cells wide; some particles outside."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def r():
        return torch.randn(count, generator=g, device="cuda", dtype=torch.float64)

    def u():
        return torch.rand(count, generator=g, device="cuda", dtype=torch.float64) - 0.5

    h = sides[-1] / (n - 1)
    if kind == "disk":
        x, y, z = r() * sides[-1] * 0.2, r() * sides[-1] * 0.2, r() * sides[-1] * 0.005
    elif kind == "uniform":
        x, y, z = (u() * sides[0] for _ in range(3))
    else:
        x, y, z = r() * 4.0 * h, r() * 4.0 * h, r() * 0.7 * h
    x[::1009] = sides[0]
    return x, y, z, torch.rand(count, generator=g, device="cuda", dtype=torch.float64) + 0.5


def forms(n, sides, p, reps=1, calls=1):
    """Grids, particles outside, and the shortest time of a call (us), of the chosen form and of the window form."""
    s = torch.cuda.Stream()
    M = float(p[3].sum().item())
    torch.cuda.synchronize()
    out = []
    with torch.cuda.stream(s):
        ctx = Q.Context(Q.Config(n=n, box_side=sides), stream=s)
        outside = ctx.deposit(*p, M)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        ctx.deposit(*p, M, count_outside=False)
    with torch.cuda.stream(s):
        for call in (lambda: ctx.deposit(*p, M, count_outside=False), graph.replay):
            best = float("inf")
            for _ in range(reps):
                e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                call()
                e0.record()
                for _ in range(calls):
                    call()
                e1.record()
                e1.synchronize()
                best = min(best, 1e3 * e0.elapsed_time(e1) / calls)
            out.append(([ctx.get_field(b, Q.FIELD_RHO_FIXED) for b in range(len(sides))], best))
    s.synchronize()
    ctx.close()
    return outside, out[0], out[1]


# with and without a sample, one box and several, both sizes of the histogram, shares with a remainder
@pytest.mark.parametrize("kind", ["disk", "uniform", "compact"])
@pytest.mark.parametrize("n,sides,count", [(129, [100.0], 999999), (129, [100.0], 1000001), (129, [80.0, 40.0, 20.0], 1000001),
                                           (257, [64.0 * 2.0 ** -b for b in range(5)], 1000001), (513, [100.0], 250001)])
def test_same_integers(n, sides, count, kind):
    p = particles(kind, n, sides, count)
    outside, (chosen, _), (window, _) = forms(n, sides, p)
    half = 0.5 * sides[0]
    gone = sum(((a < -half) | (a >= half)).int() for a in p[:3]) > 0
    assert outside == int(gone.sum().item()) > 0
    for a, b in zip(chosen, window):
        assert torch.equal(a, b)


# A call may cost a fifth more than the window form (what the fitted costs are
# off by) and 15 us (the launches that end at once, and the gaps a graph lacks).
@pytest.mark.parametrize("n,sides,count,kind", [(129, [100.0], 10000000, "compact"), (129, [100.0], 10000000, "disk"),
                                                (257, [100.0], 10000000, "compact"), (513, [100.0], 250000, "uniform"),
                                                (513, [100.0, 50.0], 250000, "uniform")])
def test_no_set_is_slower_than_the_window(n, sides, count, kind):
    _, (_, chosen), (_, window) = forms(n, sides, particles(kind, n, sides, count), reps=5, calls=5)
    assert chosen <= 1.2 * window + 15.0, (chosen, window)
