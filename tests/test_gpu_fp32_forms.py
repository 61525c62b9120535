"""The FP32 forms of the multigrid's kernels, bit for bit.  Mixed solves of two
refinement steps, stopped there whatever the residual, carry every FP32 value
into the potential: with the two-sweep march, the marching restriction and the
prolongation of their own launch they give the bits of single sweeps, the
per-node gather and the correction folded into a sweep.  The coarse tail gives
those of its schedule written out in numpy."""
import json

import numpy as np
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu
L_BOX = 60.0


def particles(seed=11, count=20000):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, y, z = (torch.randn(count, generator=g, device="cuda", dtype=torch.float64) * s for s in (6.0, 5.0, 0.7))
    return x + 0.3, y, z, torch.rand(count, generator=g, device="cuda", dtype=torch.float64) * 1e6


def newton(n, p, **kw):
    ctx = Q.Context(Q.Config(n=n, box_side=[L_BOX], precision=Q.QUMOND_MIXED, ncycle_fmg=1, **kw))
    ctx.deposit(*p, float(p[3].sum().item()))
    info = ctx.solve_newton(allow_not_converged=True)
    out = ctx.get_field(0, Q.FIELD_PHI_N), ctx.get_field(0, Q.FIELD_RHS), info
    ctx.close()
    return out


class Forms:
    """FP32 shapes of the levels up to n; the tables as they were on leaving."""

    def __init__(self, n, path):
        self.levels = [m for m in (33, 65, 129, 257, 513) if m <= n]
        self.path = str(path)
        self.saved = [(m, Q.tune_get_fused(m, True), Q.tune_get_rr(m, True), Q.tune_get_split(m, True)) for m in self.levels]

    def use(self, two, rr, split, m=None):
        for k in self.levels if m is None else [m]:
            if two:
                Q.tune_set_fused(k, *two, fp32=True)
            Q.tune_set_rr(k, rr, fp32=True)
            Q.tune_set_split(k, split, fp32=True)
            with open(self.path, "w") as f:      # the one switch that only a table holds
                json.dump({"smoother": [{"n": k, "fp32": 1, "corr_variant": -1, "corr_kchunk": 0},
                                        {"n": k, "fp32": 1, "use_fused": 1 if two else 0}]}, f)
            Q.tune_load(self.path)

    def __enter__(self):
        return self

    def __exit__(self, *a):
        for m, two, rr, split in self.saved:
            self.use(two, rr, split, m)


# two-sweep shapes and chunks, restrictions, with the correction inside the sweep or by its own launch; at 513^3 the
# FP32 restriction has its chunk seam (two chunks of 128 planes)
@pytest.mark.parametrize("n,forms", [
    (65, [((8, 0), 7, 0), ((9, 4), 2, 0), ((10, 6), 3, 1), ((8, 30), 9, 1), ((9, 62), 4, 0)]),
    (129, [((8, 8), 2, 0), ((9, 16), 7, 1), ((10, 42), 9, 0), ((10, 0), 4, 1)]),
    (257, [((8, 64), 7, 0), ((9, 52), 2, 1), ((10, 0), 9, 1), ((8, 0), 4, 0)]),
    (513, [((8, 0), 7, 0), ((8, 64), 7, 1), ((10, 32), 2, 0)])])
def test_mixed_solves_give_the_same_bits(n, forms, tmp_path):
    p = particles()
    with Forms(n, tmp_path / "t.json") as shapes:
        shapes.use(None, 0, 0)
        want, _, info = newton(n, p, tol_rel=1e-300, max_vcycles=2)
        assert info["refine_iters"][0] == 2
        for form in forms:
            shapes.use(*form)
            assert torch.equal(newton(n, p, tol_rel=1e-300, max_vcycles=2)[0], want), form


def test_stacked_problems_of_257_give_the_bits_of_each_alone(tmp_path):
    parts = [particles(s) for s in (21, 22, 23)]

    def run(which):
        b = Q.Batch(Q.BatchConfig(box_side=L_BOX, refine_iters=2, max_extra=0, ncycle_fmg=1), [257] * len(which), [5.0])
        for q, w in enumerate(which):
            b.set_particles(q, *parts[w], float(parts[w][3].sum().item()))
        b.run(use_graph=False, allow_not_converged=True)
        out = [b.get_field(q, Q.FIELD_PHI) for q in range(len(which))]
        b.close()
        return out

    with Forms(257, tmp_path / "t.json") as shapes:
        for split in (0, 1):
            shapes.use((8, 64), 7, split)
            for a, w in zip(run([0, 1, 2]), range(3)):
                assert torch.equal(a, run([w])[0]), (split, w)


# ------------------------------------- the FP32 FMG in single torch operations

F = np.float32
IN = (slice(1, -1),) * 3


def neighbours(u):
    """Sum of the six neighbours of the interior nodes, x first; arrays are [k, j, i]."""
    c = slice(1, -1)
    return u[c, c, :-2] + u[c, c, 2:] + u[c, :-2, c] + u[c, 2:, c] + u[:-2, c, c] + u[2:, c, c]


def sweep(u, f, hh):
    i = torch.arange(1, u.shape[0] - 1, device=u.device)
    parity = (i[:, None, None] + i[None, :, None] + i[None, None, :]) % 2
    for colour in (0, 1):
        v = (neighbours(u) - f[IN] * float(hh)) * float(F(1) / F(6))
        u[IN] = torch.where(parity == colour, v, u[IN])


def weighted(v):
    n = v.shape[0]
    acc = torch.zeros(((n - 3) // 2,) * 3, dtype=v.dtype, device=v.device)
    w = (0.25, 0.5, 0.25)
    for c in (-1, 0, 1):
        for b in (-1, 0, 1):
            for a in (-1, 0, 1):
                x = v[2 + c:n - 2 + c:2, 2 + b:n - 2 + b:2, 2 + a:n - 2 + a:2]
                acc = acc + x * (w[a + 1] * w[b + 1] * w[c + 1])
    out = torch.zeros(((n + 1) // 2,) * 3, dtype=v.dtype, device=v.device)
    out[IN] = acc
    return out


def refined(u):
    for d in (2, 1, 0):
        n = u.shape[d]
        v = torch.empty([2 * m - 1 if e == d else m for e, m in enumerate(u.shape)], dtype=u.dtype, device=u.device)
        at = [slice(None)] * 3
        at[d] = slice(0, None, 2)
        v[tuple(at)] = u
        at[d] = slice(1, None, 2)
        v[tuple(at)] = u.narrow(d, 0, n - 1) * 0.5 + u.narrow(d, 1, n - 1) * 0.5
        u = v
    return u


def exact(u, f):
    d = u.double()
    s = d[1, 1, 0] + d[1, 1, 2] + d[1, 0, 1] + d[1, 2, 1] + d[0, 1, 1] + d[2, 1, 1]
    u[1, 1, 1] = ((s - (L_BOX / 2.0) ** 2 * f[1, 1, 1].double()) / 6.0).float()


def steps(n, top):
    """h^2 and 1 / h^2 of a level; those from 17^3 down come from the largest of them, by powers of two."""
    if n > 17:
        h = L_BOX / (n - 1)
        return F(h * h), F(1.0 / (h * h))
    h = F(L_BOX) / F(top - 1)
    r = F(((top - 1) // (n - 1)) ** 2)
    return h * h * r, F(1) / (h * h) * (F(1) / r)


def vcycle(u, f, top):
    if u.shape[0] == 3:
        return exact(u, f)
    hh, ih = steps(u.shape[0], top)
    for _ in range(2):
        sweep(u, f, hh)
    r = torch.zeros_like(u)
    r[IN] = f[IN] - (neighbours(u) - u[IN] * 6.0) * float(ih)
    c = torch.zeros(((u.shape[0] + 1) // 2,) * 3, dtype=u.dtype, device=u.device)
    vcycle(c, weighted(r), top)
    u[IN] += refined(c)[IN]
    for _ in range(2):
        sweep(u, f, hh)


@pytest.mark.parametrize("n", [5, 9, 17, 33, 65, 129, 257])
def test_fmg_against_single_operations(n):
    """tol_rel = 0 leaves the FP32 FMG's iterate, widened."""
    phi, rhs, info = newton(n, particles(5), tol_rel=0.0)
    f = [rhs.float()]
    assert info["refine_iters"][0] == 0 and float(f[0].abs().max()) > 0
    u = phi.float()
    u[IN] = 0
    while f[-1].shape[0] > 3:
        f.append(weighted(f[-1]))
    for up in range(len(f) - 1, -1, -1):
        level = u[::2 ** up, ::2 ** up, ::2 ** up].clone()
        if level.shape[0] == 3:
            exact(level, f[up])
        else:
            level[IN] = refined(coarse)[IN]
            vcycle(level, f[up], min(n, 17))
        coarse = level
    assert torch.equal(phi[IN], coarse[IN].double())
