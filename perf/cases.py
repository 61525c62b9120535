"""The work a program has this package do, as cases that can be timed and checked.

A case is a dict of plain values.  ``prepare`` makes what the program holds before
the call (particles on the GPU, a context, a batch or a network), ``run`` makes
one pass through the package's public entry points, ``work`` counts what the
path cannot do without, and ``exact`` gives the same outputs in 64 bits from
plain torch: the multigrid solves by a sine transform that inverts the 7-point
Laplacian directly, everything else from its definition.

Particles follow the two-component exponential disk (stars 5e10 Msun, R_d = 3
kpc, sech^2 height 0.3 kpc; gas 1e10 Msun, 6 kpc, 0.15 kpc) or the razor-thin
Kuzmin disk (1e10 Msun) that the tests and the benchmark use.
"""
import math
import os

import torch

from paper_1201_3185_amd import qumond as Q

HERE = os.path.dirname(os.path.abspath(Q.__file__))
G, A0 = 4.300917270e-6, 3600.0
DEV = "cuda"
LAYERS = [(8, 16, 1, 2), (16, 16, 1, 16), (16, 32, 2, 16), (32, 32, 1, 32), (32, 64, 2, 32), (64, 64, 1, 64),
          (64, 64, 2, 64), (64, 64, 1, 64), (128, 64, 1, 128), (96, 32, 1, 96), (48, 16, 1, 48)]


def listed():
    return [
        # the curve of a solved model, 60 radii and 16 azimuths: the smallest call, once per model of a fit
        {"name": "curve_65", "kind": "curves", "n": 65, "nbox": 1, "side": 100.0, "radii": 60, "naz": 16},
        # one small model from particles to forces: a 65^3 box, 1e5 particles of a thin Kuzmin disk
        {"name": "kuzmin_65", "kind": "step", "n": 65, "nbox": 1, "side": 100.0, "particles": 100000,
         "disk": "kuzmin", "mixed": False, "tol": 1e-10, "ncycle": 6, "monopole": True, "nu_n": 1.0},
        # an N-body step in four nested 129^3 boxes with 1e6 particles
        {"name": "nested_129", "kind": "step", "n": 129, "nbox": 4, "side": 400.0, "particles": 1000000,
         "disk": "two", "mixed": False, "tol": 1e-10, "ncycle": 6, "monopole": True, "nu_n": 1.0},
        # the nesting of the accuracy runs: eleven 257^3 boxes from 4096 to 4 kpc, zero outer potential, 2e7 particles
        {"name": "paper_257", "kind": "step", "n": 257, "nbox": 11, "side": 4096.0, "particles": 20000000,
         "disk": "two", "mixed": False, "tol": 1e-10, "ncycle": 6, "monopole": False, "nu_n": 1.0},
        # the largest single grid, 513^3 with 1e7 particles, FP64 to 1e-10
        {"name": "disk_513", "kind": "step", "n": 513, "nbox": 1, "side": 120.0, "particles": 10000000,
         "disk": "two", "mixed": False, "tol": 1e-10, "ncycle": 6, "monopole": True, "nu_n": 1.0},
        # the same to 1e-6 in mixed precision
        {"name": "mixed_513", "kind": "step", "n": 513, "nbox": 1, "side": 120.0, "particles": 10000000,
         "disk": "two", "mixed": True, "tol": 1e-6, "ncycle": 2, "monopole": True, "nu_n": 1.0},
        # one batch of a rotation-curve fit: disks of 129^3 and 257^3 grids, 2e5 to 2e6 particles each
        {"name": "fit_batch", "kind": "batch", "n129": 7, "n257": 9, "side": 120.0, "radii": 60},
        # mass assignment alone, an odd count of particles on three nested 257^3 grids
        {"name": "deposit_257", "kind": "deposit", "n": 257, "nbox": 3, "side": 200.0, "particles": 4000001,
         "disk": "two"},
        # forces alone, at tracers inside and outside two nested 257^3 boxes
        {"name": "gather_257", "kind": "gather", "n": 257, "nbox": 2, "side": 120.0, "particles": 4000003, "which": 1},
        # one convolution of the network's second level: forward, input gradient, weight gradient
        {"name": "conv_65", "kind": "conv", "n": 65, "cin": 32, "cout": 32, "stride": 1},
        # the learned guess of a 129^3 box
        {"name": "infer_129", "kind": "infer", "n": 129},
        # one training step on a 129^3 sample
        {"name": "train_129", "kind": "train", "n": 129},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "batch", "deposit", "gather", "curves", "conv", "conv", "infer", "train"])
    c = {"kind": kind}
    if kind in ("step", "deposit", "gather", "curves"):
        c["n"] = rng.choice([33, 65, 129, 257] if kind == "step" else [17, 33, 65, 129, 257])
        c["nbox"] = rng.randint(1, {17: 6, 33: 6, 65: 6, 129: 5, 257: 3}[c["n"]])
        c["side"] = round(rng.uniform(60.0, 120.0), 2) * 2 ** (c["nbox"] - 1)
    if kind == "step":
        c["particles"] = _log(rng, 2e4, 5e6)
        c["disk"] = rng.choice(["two", "kuzmin"])
        c["mixed"] = rng.random() < 0.4
        c["tol"] = rng.choice([1e-6, 1e-7]) if c["mixed"] else rng.choice([1e-10, 1e-10, 1e-8])
        c["ncycle"] = 2 if c["mixed"] else rng.choice([2, 6, 6])
        c["monopole"] = rng.random() < 0.75
        c["nu_n"] = rng.choice([1.0, 1.0, 1.0, 2.0])
    elif kind == "batch":
        c["n129"], c["n257"] = rng.randint(1, 8), rng.randint(0, 4)
        c["side"] = round(rng.uniform(100.0, 140.0), 2)
        c["radii"] = rng.randint(20, 200)
    elif kind == "deposit":
        c["particles"] = _log(rng, 1e4, 1.2e7)
        c["disk"] = rng.choice(["two", "two", "kuzmin"])
    elif kind == "gather":
        c["particles"], c["which"] = _log(rng, 1e4, 1.2e7), rng.choice([0, 1, 2])
    elif kind == "curves":
        c["radii"], c["naz"] = _log(rng, 10, 400), rng.choice([16, 32, 64])
    elif kind == "conv":
        c["n"] = 2 * _log(rng, 8, 48) + 1
        c["cin"], c["cout"] = rng.choice([(16, 16), (16, 32), (32, 32), (32, 64), (64, 64), (48, 16), (96, 32), (128, 64)])
        c["stride"] = rng.choice([1, 1, 2])
    else:
        c["n"] = rng.choice([17, 33, 65])
        if kind == "infer":
            c["side"] = round(rng.uniform(100.0, 140.0), 2)
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 12011)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64).clamp_(1e-12, 1.0 - 1e-12)


def _particles(disk, n, g, scale=1.0, ml=1.0, zs=0.3, zg=0.15, a=3.0):
    """x, y, z, m and the total mass; the radius of an exponential disk is the sum of two exponential deviates."""
    phi = 2.0 * math.pi * _rand(g, n)
    if disk == "kuzmin":     # its plane 0.1 kpc above the grid's, so that the vertical force is not zero by symmetry
        R = a * torch.sqrt((1.0 - _rand(g, n)) ** -2 - 1.0)
        M = 1e10
        return R * torch.cos(phi), R * torch.sin(phi), torch.full_like(R, 0.1), torch.full_like(R, M / n), M
    stars = torch.arange(n, device=DEV) < (n + 1) // 2
    Rd = torch.where(stars, 3.0 * scale, 6.0 * scale)
    R = -Rd * torch.log(_rand(g, n) * _rand(g, n))
    z = torch.where(stars, zs, zg) * torch.atanh(2.0 * _rand(g, n) - 1.0)
    ns = (n + 1) // 2
    Ms, Mg = ml * 5e10 * scale ** 2, 1e10 * scale ** 2
    m = torch.where(stars, Ms / ns, Mg / max(n - ns, 1)).to(torch.float64)
    return R * torch.cos(phi), R * torch.sin(phi), z, m, float(Ms + (Mg if n > ns else 0.0))


def _sides(c):
    return [c["side"] / 2 ** b for b in range(c["nbox"])]


def _axis(n, L):
    return torch.arange(n, device=DEV, dtype=torch.float64) * (L / (n - 1)) - 0.5 * L


def _disk_potential(n, L, M=6e10, a=3.0, b=0.3):
    """-GM / sqrt(R^2 + (a + sqrt(z^2 + b^2))^2), the potential of a flattened disk."""
    t = _axis(n, L)
    z = (a + torch.sqrt(t * t + b * b)) ** 2
    return -G * M / torch.sqrt(t[None, None, :] ** 2 + t[None, :, None] ** 2 + z[:, None, None])


def _field(c, b, seed):
    """A potential with a disk and a few lumps, so that no symmetry hides an error."""
    n, L = c["n"], _sides(c)[b]
    g = torch.Generator().manual_seed(int(seed) + 17)
    p = _disk_potential(n, L)
    t = _axis(n, L)
    for _ in range(3):
        o = (torch.rand(3, generator=g, dtype=torch.float64) - 0.5) * 0.3 * _sides(c)[-1]
        r2 = (t[None, None, :] - float(o[0])) ** 2 + (t[None, :, None] - float(o[1])) ** 2 + \
             (t[:, None, None] - float(o[2])) ** 2
        p -= G * 2e9 / torch.sqrt(r2 + 4.0)
    return p


def _tracers(c, seed):
    g = _gen(seed)
    x, y, z, _, _ = _particles("two", c["particles"], g)
    s = 0.35 * c["side"] / 20.0      # a few of them beyond the outermost box
    return x * s, y * s, z * s


def _batch_disks(c, seed):
    g = torch.Generator().manual_seed(int(seed) + 31)
    ns = [129] * c["n129"] + [257] * c["n257"]
    out = []
    for p, n in enumerate(ns):
        u = torch.rand(5, generator=g, dtype=torch.float64).tolist()
        out.append(dict(n=n, particles=int(2e5 * 10 ** u[0]) | 1, scale=0.8 + 0.4 * u[1], ml=0.3 + 0.9 * u[2],
                        zs=0.1 + 0.5 * u[3], zg=0.05 + 0.45 * u[4], seed=int(seed) * 1000 + p))
    return out


def _batch_particles(d):
    return _particles("two", d["particles"], _gen(d["seed"]), d["scale"], d["ml"], d["zs"], d["zg"])


def _bf16(g, n, scale):
    return (torch.randn(n, generator=g, device=DEV, dtype=torch.float32) * scale).to(torch.bfloat16)


def _kpad(cin):
    return (27 * cin + 31) // 32 * 32


def _conv_inputs(c, seed):
    g = _gen(seed)
    n, cin, cout = c["n"], c["cin"], c["cout"]
    no = (n + 1) // 2 if c["stride"] == 2 else n
    x = _bf16(g, n ** 3 * cin, 1.0).relu_()
    w = torch.zeros(cout, _kpad(cin), device=DEV, dtype=torch.bfloat16)
    w[:, :27 * cin] = _bf16(g, cout * 27 * cin, math.sqrt(2.0 / (27 * cin))).reshape(cout, -1)
    b = torch.randn(cout, generator=g, device=DEV, dtype=torch.float32) * 0.1
    dy = _bf16(g, no ** 3 * cout, 1.0)
    return x, w, b, dy


def _net_params(seed):
    """He-normal weights of the eleven convolutions and the head, in the network's parameter order."""
    g = torch.Generator().manual_seed(int(seed) + 43)
    out = []
    for cin, cout, _, fan in LAYERS:
        w = torch.zeros(cout, _kpad(cin))
        w[:, :27 * cin].reshape(cout, 27, cin)[:, :, :fan] = \
            torch.randn(cout, 27, fan, generator=g) * math.sqrt(2.0 / (27 * fan))
        out += [w.reshape(-1), torch.randn(cout, generator=g) * 0.02]
    out += [torch.randn(16, generator=g) * 0.25, torch.zeros(1)]
    return torch.cat(out).numpy()


def _net_fields(c, seed):
    n, L = c["n"], c.get("side", 120.0)
    phin = _field({"n": n, "nbox": 1, "side": L}, 0, seed)
    return phin, _source64(phin, L / (n - 1)), L


def _scales(L, M=6e10):
    r = 0.5 * L
    y = G * M / (r * r * A0)
    return G * M / r, G * M / r * (0.5 + 0.5 * math.sqrt(1.0 + 4.0 / y))


def _train_inputs(c, seed):
    n, g = c["n"], _gen(seed)
    t = torch.linspace(-1.0, 1.0, n, device=DEV, dtype=torch.float64)
    k = torch.rand(8, generator=g, device=DEV, dtype=torch.float64) * 6.0
    wave = torch.sin(k[0] * t[None, None, :] + k[1]) * torch.cos(k[2] * t[None, :, None] + k[3]) * \
        torch.cos(k[4] * t[:, None, None] + k[5])
    bump = torch.exp(-8.0 * (t[None, None, :] ** 2 + t[None, :, None] ** 2 + 6.0 * t[:, None, None] ** 2))
    x = torch.stack([0.3 * wave + bump, 0.5 * bump * (1.0 + wave)], dim=-1).to(torch.bfloat16)
    return x.reshape(-1).contiguous(), (0.4 * wave + 0.8 * bump).to(torch.float32).reshape(-1).contiguous()


# ------------------------------------------------------------- the package

_tuned = False


def _tables():
    """The shipped launch shapes of this GPU, as the benchmark and the large runs install them."""
    global _tuned
    if not _tuned:
        Q.tune_load(os.path.join(HERE, "launch_shapes_mi355x.json"))
        _tuned = True


def _config(c):
    return Q.Config(n=c["n"], box_side=_sides(c), precision=Q.QUMOND_MIXED if c.get("mixed") else Q.QUMOND_FP64,
                    tol_rel=c.get("tol", 1e-10), ncycle_fmg=c.get("ncycle", 6), nu_n=c.get("nu_n", 1.0),
                    outer_bc=Q.QUMOND_BC_MONOPOLE if c.get("monopole", True) else Q.QUMOND_BC_ZERO)


def prepare(case, seed):
    c, k = case, case["kind"]
    _tables()
    if k in ("step", "deposit"):
        return {"c": c, "ctx": Q.Context(_config(c)), "p": _particles(c["disk"], c["particles"], _gen(seed))}
    if k in ("gather", "curves"):
        ctx = Q.Context(_config(c))
        x = torch.ones(1, device=DEV, dtype=torch.float64)
        ctx.deposit(x, x, x, x, 6.6e10, count_outside=False)      # states the total mass of the monopole beyond the boxes
        for b in range(c["nbox"]):
            p = _field(c, b, seed)
            ctx.set_field(b, Q.FIELD_PHI_N, p)
            ctx.set_field(b, Q.FIELD_PHI, p)
        torch.cuda.synchronize()
        if k == "gather":
            return {"c": c, "ctx": ctx, "x": _tracers(c, seed)}
        return {"c": c, "ctx": ctx, "R": _radii(c, seed)}
    if k == "batch":
        disks = _batch_disks(c, seed)
        b = Q.Batch(Q.BatchConfig(box_side=c["side"], refine_iters=3, tol_rel=1e-6, autotune=True),
                    [d["n"] for d in disks], _batch_radii(c))
        for p, d in enumerate(disks):
            x, y, z, m, M = _batch_particles(d)
            b.set_particles(p, x, y, z, m, M)
        return {"c": c, "batch": b}
    if k == "conv":
        return {"c": c, "in": _conv_inputs(c, seed)}
    net = Q.UNet(n=c["n"])
    net.set_params(_net_params(seed))
    if k == "train":
        return {"c": c, "net": net, "in": _train_inputs(c, seed)}
    phin, S, L = _net_fields(c, seed)
    return {"c": c, "net": net, "phin": phin.contiguous(), "S": S.contiguous(), "L": L}


def run(state):
    c = state["c"]
    k = c["kind"]
    if k == "step":
        ctx, (x, y, z, m, M) = state["ctx"], state["p"]
        ctx.deposit(x, y, z, m, M, count_outside=False)
        ctx.solve()
        return ctx.gather_forces(x, y, z, 1, with_box=False)[:3]
    if k == "deposit":
        ctx, (x, y, z, m, M) = state["ctx"], state["p"]
        out = ctx.deposit(x, y, z, m, M, count_outside=True)
        return {"outside": out, "q": [ctx.get_field(b, Q.FIELD_RHO_FIXED) for b in range(c["nbox"])],
                "rhs": ctx.get_field(c["nbox"] - 1, Q.FIELD_RHS)}
    if k == "gather":
        return state["ctx"].gather_forces(*state["x"], c["which"])
    if k == "curves":
        ctx, R = state["ctx"], state["R"]
        return ctx.rotation_curve(R, c["naz"], 1), ctx.sigma_z(R, 0.3, 0.3, c["naz"], 1)
    if k == "batch":
        b = state["batch"]
        b.run(use_graph=True)
        return b.rotation_curves(False), b.rotation_curves(True)
    if k == "conv":
        x, w, b, dy = state["in"]
        n, cin, cout, s = c["n"], c["cin"], c["cout"], c["stride"]
        return {"y": Q.k_conv3d_fwd(x, n, cin, w, cout, b, s, True), "dx": Q.k_conv3d_dgrad(n, cin, cout, w, dy, s),
                "dw": Q.k_conv3d_wgrad(n, cin, x, cout, dy, s)}
    net = state["net"]
    if k == "train":
        loss = net.train_step(*state["in"], lr=1e-3)
        return {"loss": loss, "grads": net.get_grads()}
    c_phin, c_out = _scales(state["L"])
    return net.infer(state["phin"], state["S"], state["L"] / (c["n"] - 1), c_phin, c_out, GM=G * 6e10, a0=A0, soft=3.0)


# -------------------------------------------------------------------- work

def _solve_work(n, ncycle, esize):
    """FMG with ncycle V(2,2) cycles per level: in each cycle of a level the pre- and the post-smoothing pass read u and
    f and write u once; about 50 operations per node and cycle (four sweeps, residual, transfers)."""
    by = fl = 0.0
    J = (n - 1).bit_length() - 1
    for top in range(1, J + 1):
        for l in range(1, top + 1):
            N = float((1 << l) + 1) ** 3
            by += ncycle * 6 * esize * N
            fl += ncycle * 50 * N
    return by, fl


def _conv_flops(n, layers):
    size = [n, (n + 1) // 2, (n + 3) // 4, (n + 7) // 8]
    at = [0, 0, 1, 1, 2, 2, 3, 3, 2, 1, 0]
    return sum(2.0 * 27 * fan * cout * size[l] ** 3 for (_, cout, _, fan), l in zip(layers, at))


def work(case):
    c, k = case, case["kind"]
    if k in ("step", "batch"):
        probs = [(c["n"], c["nbox"], c["particles"])] if k == "step" else \
            [(n, 1, 6e5) for n in [129] * c["n129"] + [257] * c["n257"]]
        by = fl = 0.0
        for n, nbox, np_ in probs:
            mixed = k == "batch" or c["mixed"]
            sb, sf = _solve_work(n, 2 if mixed else c["ncycle"], 4 if mixed else 8)
            by += nbox * (2 * sb + 32.0 * n ** 3) + 56.0 * np_
            fl += nbox * (2 * sf + 100.0 * n ** 3) + 200.0 * np_
        return {"bytes": by, "flops": fl}
    if k == "deposit":
        return {"bytes": 32.0 * c["particles"] + 16.0 * c["nbox"] * c["n"] ** 3, "flops": 40.0 * c["particles"] * c["nbox"]}
    if k == "gather":
        return {"bytes": 49.0 * c["particles"] + 8.0 * c["nbox"] * c["n"] ** 3, "flops": 130.0 * c["particles"]}
    if k == "curves":
        pts = 3.0 * c["radii"] * c["naz"]
        return {"bytes": 32 * 8 * pts, "flops": 130.0 * pts}
    if k == "conv":
        no = (c["n"] + 1) // 2 if c["stride"] == 2 else c["n"]
        xb, yb = 2.0 * c["cin"] * c["n"] ** 3, 2.0 * c["cout"] * no ** 3
        return {"bytes": 3 * xb + 3 * yb, "flops": 3 * 2.0 * 27 * c["cin"] * c["cout"] * no ** 3}
    n = c["n"]
    if k == "infer":
        return {"bytes": 24.0 * n ** 3, "flops": _conv_flops(n, LAYERS)}
    return {"bytes": 8.0 * n ** 3 + 6e6, "flops": 3 * _conv_flops(n, LAYERS)}


# --------------------------------------------------------- 64-bit references

def _cic(n, L, x, y, z, m):
    u = [(t + 0.5 * L) * ((n - 1) / L) for t in (x, y, z)]
    ok = (u[0] >= 0) & (u[0] < n - 1) & (u[1] >= 0) & (u[1] < n - 1) & (u[2] >= 0) & (u[2] < n - 1)
    u = [t[ok] for t in u]
    m = m[ok]
    i = [torch.floor(t) for t in u]
    f = [t - s for t, s in zip(u, i)]
    cell, order = torch.sort((i[0] + n * (i[1] + n * i[2])).long())
    f, m = [t[order] for t in f], m[order]
    rho = torch.zeros(n ** 3, device=DEV, dtype=torch.float64)
    if not cell.numel():
        return rho.reshape(n, n, n)
    cell, count = torch.unique_consecutive(cell, return_counts=True)
    last = torch.cumsum(count, 0) - 1
    for cz in (0, 1):        # sums over the particles of a cell as differences of one running sum: no add meets another
        for cy in (0, 1):
            for cx in (0, 1):
                w = (f[0] if cx else 1 - f[0]) * (f[1] if cy else 1 - f[1]) * (f[2] if cz else 1 - f[2])
                s = torch.cumsum(w * m, 0)[last]
                s[1:] -= s[:-1].clone()
                rho[cell + (cx + n * (cy + n * cz))] += s
    return rho.reshape(n, n, n)


def _dst(a, dim):
    """Type-I sine transform over `dim` (odd extension and a real FFT), in slabs."""
    a = a.transpose(dim, -1)
    m = a.shape[-1]
    out = torch.empty_like(a, memory_format=torch.contiguous_format)
    for s in range(0, a.shape[0], 64):
        v = a[s:s + 64].contiguous()
        e = torch.zeros(*v.shape[:-1], 2 * (m + 1), device=v.device, dtype=v.dtype)
        e[..., 1:m + 1] = v
        e[..., m + 2:] = -v.flip(-1)
        out[s:s + 64] = -torch.fft.rfft(e).imag[..., 1:m + 1]
    return out.transpose(dim, -1)


def _poisson(u, f, h):
    """Interior of u from the 7-point equation with u's boundary values."""
    n = u.shape[0]
    r = f.clone()
    r[1] -= u[0] / h ** 2
    r[n - 2] -= u[n - 1] / h ** 2
    r[:, 1] -= u[:, 0] / h ** 2
    r[:, n - 2] -= u[:, n - 1] / h ** 2
    r[:, :, 1] -= u[:, :, 0] / h ** 2
    r[:, :, n - 2] -= u[:, :, n - 1] / h ** 2
    a = r[1:-1, 1:-1, 1:-1].contiguous()
    for d in range(3):
        a = _dst(a, d)
    t = torch.arange(1, n - 1, device=DEV, dtype=torch.float64) * (math.pi / (2 * (n - 1)))
    e = -4.0 / h ** 2 * torch.sin(t) ** 2
    a = a / (e[:, None, None] + e[None, :, None] + e[None, None, :])
    for d in range(3):
        a = _dst(a, d)
    u[1:-1, 1:-1, 1:-1] = a / (2.0 * (n - 1)) ** 3
    return u


def _source64(P, h, a0=A0):
    """Divergence of nu(|g| / a0) g with nu(y) = (1 + sqrt(1 + 4 / y)) / 2 through the faces of each interior node."""
    n = P.shape[0]
    S = torch.zeros_like(P)
    inner = slice(1, n - 1)
    for d in range(3):
        q = P.transpose(d, 0)
        gn = (q[1:, inner, inner] - q[:-1, inner, inner]) / h
        g2 = gn * gn
        for a in (1, 2):
            lo, hi = [slice(None), inner, inner], [slice(None), inner, inner]
            lo[a], hi[a] = slice(0, n - 2), slice(2, n)
            t = q[tuple(hi)] - q[tuple(lo)]
            t = (t[1:] + t[:-1]) / (4 * h)
            g2 = g2 + t * t
        g = torch.sqrt(g2)
        F = torch.where(g > 0, 0.5 * gn * (1 + torch.sqrt(1 + 4 * a0 / g.clamp_min(1e-300))), torch.zeros_like(gn))
        S.transpose(d, 0)[1:-1, inner, inner] += (F[1:] - F[:-1]) / h
    return S


def _point_phi(r, GM, mond):
    if not mond:
        return -GM / r
    return -GM / (2 * r) - math.sqrt(GM) * torch.sqrt(GM + 4 * A0 * r * r) / (2 * r) + \
        math.sqrt(GM * A0) * torch.asinh(2 * r * math.sqrt(A0 / GM))


def _boundary(n, L, value):
    u = torch.zeros(n, n, n, device=DEV, dtype=torch.float64)
    if value is not None:
        t = _axis(n, L)
        for d in range(3):
            for s in (0, n - 1):
                r = torch.sqrt(t[:, None] ** 2 + t[None, :] ** 2 + 0.25 * L * L)
                u.select(d, s).copy_(value(r))
    return u


def _inner_boundary(uc):
    """Boundary of a box of half the side, from the coarser box of the same points by trilinear interpolation."""
    n = uc.shape[0]
    q = (n - 1) // 4
    a = uc[q:n - q, q:n - q, q:n - q] if n % 4 == 1 else None
    for d in range(3):
        s = a.transpose(d, 0)
        m = s.shape[0]
        e = torch.empty(2 * m - 1, *s.shape[1:], device=DEV, dtype=torch.float64)
        e[0::2] = s
        e[1::2] = 0.5 * (s[1:] + s[:-1])
        a = e.transpose(d, 0)
    u = a.clone().contiguous()
    u[1:-1, 1:-1, 1:-1] = 0.0
    return u


def _solved64(c, sides, x, y, z, m, M, monopole=True):
    """Newtonian and QUMOND potentials of every box."""
    pn, pq = [], []
    for b, L in enumerate(sides):
        n = c["n"]
        h = L / (n - 1)
        f = _cic(n, L, x, y, z, m) * (4 * math.pi * G / h ** 3)
        for mond, chain in ((False, pn), (True, pq)):
            u = _inner_boundary(chain[-1]) if b else \
                _boundary(n, L, (lambda r: _point_phi(r, G * M, mond)) if monopole else None)
            chain.append(_poisson(u, f if not mond else _source64(pn[b], h), h))
        del f
    return pn, pq


def _grad(P, d, h):
    q = P.transpose(d, 0)
    g = torch.empty_like(q)
    g[1:-1] = (q[2:] - q[:-2]) / (2 * h)
    g[0] = (-3 * q[0] + 4 * q[1] - q[2]) / (2 * h)
    g[-1] = (3 * q[-1] - 4 * q[-2] + q[-3]) / (2 * h)
    return -g.transpose(d, 0)


def _gather64(fields, sides, x, y, z, which, GM, frac=0.2):
    n, nb = fields[0].shape[0], len(sides)
    R, az = torch.sqrt(x * x + y * y), z.abs()
    sel = torch.full(x.shape, -1, device=DEV, dtype=torch.long)
    for b in range(nb):
        L = sides[nb - 1 - b]
        sel = torch.where((sel < 0) & (R < frac * L) & (az < frac * L), nb - 1 - b, sel)
    for b, L in enumerate(sides):
        u = [(t + 0.5 * L) * ((n - 1) / L) for t in (x, y, z)]
        sel = torch.where((sel < 0) & (u[0] >= 0) & (u[0] < n - 1) & (u[1] >= 0) & (u[1] < n - 1) & (u[2] >= 0) &
                          (u[2] < n - 1), b, sel)
    acc = [torch.zeros_like(x) for _ in range(3)]
    for b, L in enumerate(sides):
        at = (sel == b).nonzero().squeeze(1)
        if not at.numel():
            continue
        u = [(t[at] + 0.5 * L) * ((n - 1) / L) for t in (x, y, z)]
        i = [torch.floor(t) for t in u]
        f = [t - s for t, s in zip(u, i)]
        base = (i[0] + n * (i[1] + n * i[2])).long()
        for d in range(3):
            g = _grad(fields[b], 2 - d, L / (n - 1)).reshape(-1)
            s = torch.zeros_like(u[0])
            for k in range(8):
                cx, cy, cz = k & 1, (k >> 1) & 1, k >> 2
                w = (f[0] if cx else 1 - f[0]) * (f[1] if cy else 1 - f[1]) * (f[2] if cz else 1 - f[2])
                s += w * g[base + (cx + n * (cy + n * cz))]
            acc[d][at] = s
    out = sel < 0
    r = torch.sqrt(x * x + y * y + z * z)
    gN = GM / r ** 2
    gm = (gN * (0.5 + 0.5 * torch.sqrt(1 + 4 * A0 / gN)) if which == 1 else gN) / r
    acc = [torch.where(out, -gm * t, a) for t, a in zip((x, y, z), acc)]
    if which == 2:
        g = torch.sqrt(acc[0] ** 2 + acc[1] ** 2 + acc[2] ** 2)
        nu = torch.where(g > 0, 0.5 + 0.5 * torch.sqrt(1 + 4 * A0 / g.clamp_min(1e-300)), torch.ones_like(g))
        acc = [a * nu for a in acc]
    return acc


def _curve64(fields, sides, R, naz, GM, mond=True):
    ph = torch.arange(naz, device=DEV, dtype=torch.float64) * (2 * math.pi / naz)
    x, y = (R[:, None] * torch.cos(ph)).reshape(-1), (R[:, None] * torch.sin(ph)).reshape(-1)
    a = _gather64(fields, sides, x, y, torch.zeros_like(x), 1 if mond else 0, GM)
    return (-(x * a[0] + y * a[1])).reshape(-1, naz).mean(1)


def _sigma64(fields, sides, R, naz, GM, z, z0):
    ph = torch.arange(naz, device=DEV, dtype=torch.float64) * (2 * math.pi / naz)
    x, y = (R[:, None] * torch.cos(ph)).reshape(-1), (R[:, None] * torch.sin(ph)).reshape(-1)
    up = _gather64(fields, sides, x, y, torch.full_like(x, z), 1, GM)[2]
    dn = _gather64(fields, sides, x, y, torch.full_like(x, -z), 1, GM)[2]
    return ((dn - up) * 0.5 * z0 / (2 * math.tanh(z / z0))).reshape(-1, naz).mean(1)


def _radii(c, seed):
    return torch.linspace(0.3, 0.45 * c["side"], c["radii"], device=DEV, dtype=torch.float64) * (1.0 + 1e-3 * (seed % 7))


def _batch_radii(c):
    return [0.5 * (k + 1) * 30.0 / (0.5 * c["radii"]) for k in range(c["radii"])]


def _taps(x, stride):
    """The 27 shifted views of a zero-padded [z, y, x, c] tensor, tap = dx + 3 dy + 9 dz."""
    n = x.shape[0]
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    no = (n - 1) // stride + 1
    e = stride * (no - 1) + 1
    for t in range(27):
        i, j, k = t % 3, (t // 3) % 3, t // 9
        yield t, p[k:k + e:stride, j:j + e:stride, i:i + e:stride]


class _Conv64(torch.autograd.Function):
    """conv(x) with weights [cout, 27, cin]."""

    @staticmethod
    def forward(ctx, x, w, b, stride):
        ctx.save_for_backward(x, w)
        ctx.stride = stride
        y = 0.0
        for t, v in _taps(x, stride):
            y = y + v.reshape(-1, x.shape[-1]) @ w[:, t].t().contiguous()
        no = (x.shape[0] - 1) // stride + 1
        return (y + b).reshape(no, no, no, -1)

    @staticmethod
    def backward(ctx, g):
        x, w = ctx.saved_tensors
        n, s = x.shape[0], ctx.stride
        g2 = g.reshape(-1, g.shape[-1]).contiguous()
        dw = torch.zeros_like(w)
        dx = torch.zeros(n + 2, n + 2, n + 2, x.shape[-1], device=x.device, dtype=x.dtype)
        e = s * (g.shape[0] - 1) + 1
        for t, v in _taps(x, s):
            dw[:, t] = g2.t().contiguous() @ v.reshape(-1, x.shape[-1]).contiguous()
            i, j, k = t % 3, (t // 3) % 3, t // 9
            dx[k:k + e:s, j:j + e:s, i:i + e:s] += (g2 @ w[:, t].contiguous()).reshape(*g.shape[:3], -1)
        return dx[1:-1, 1:-1, 1:-1], dw, g2.sum(0), None


def _up64(x):
    for d in range(3):
        s = x.transpose(d, 0)
        m = torch.zeros(2 * s.shape[0] - 1, *s.shape[1:], device=x.device, dtype=x.dtype)
        m[0::2] = s
        m[1::2] = 0.5 * (s[1:] + s[:-1])
        x = m.transpose(d, 0)
    return x


def _net64(params, x, grad):
    """Output [z, y, x] of the network for the two input channels, and its parameters as leaves."""
    flat = torch.from_numpy(params).double().to(DEV)
    W, off = [], 0
    for cin, cout, _, fan in LAYERS:
        k = _kpad(cin)
        w = flat[off:off + cout * k].reshape(cout, k)[:, :27 * cin].reshape(cout, 27, cin)[:, :, :fan].clone()
        off += cout * k
        W.append((w.requires_grad_(grad), flat[off:off + cout].clone().requires_grad_(grad)))
        off += cout
    head = (flat[off:off + 16].clone().requires_grad_(grad), flat[off + 16].clone().requires_grad_(grad))

    def conv(l, v):
        return torch.relu(_Conv64.apply(v, W[l][0], W[l][1], LAYERS[l][2]))

    s0 = conv(1, conv(0, x))
    s1 = conv(3, conv(2, s0))
    s2 = conv(5, conv(4, s1))
    b3 = conv(7, conv(6, s2))
    d2 = conv(8, torch.cat([_up64(b3), s2], -1))
    d1 = conv(9, torch.cat([_up64(d2), s1], -1))
    d0 = conv(10, torch.cat([_up64(d1), s0], -1))
    return d0 @ head[0] + head[1], W, head


def exact(case, seed):
    c, k = case, case["kind"]
    if c.get("nu_n", 1.0) != 1.0:
        return None      # no closed form for the outer potential of the other functions
    if k == "step":
        x, y, z, m, M = _particles(c["disk"], c["particles"], _gen(seed))
        _, pq = _solved64(c, _sides(c), x, y, z, m, M, c["monopole"])
        return tuple(_gather64(pq, _sides(c), x, y, z, 1, G * M))
    if k == "deposit":
        x, y, z, m, M = _particles(c["disk"], c["particles"], _gen(seed))
        L = _sides(c)[-1]
        return {"outside": None, "q": [None] * c["nbox"],
                "rhs": _cic(c["n"], L, x, y, z, m) * (4 * math.pi * G / (L / (c["n"] - 1)) ** 3)}
    if k in ("gather", "curves"):
        fields, sides, GM = [_field(c, b, seed) for b in range(c["nbox"])], _sides(c), G * 6.6e10
        if k == "gather":
            return tuple(_gather64(fields, sides, *_tracers(c, seed), c["which"], GM)) + (None,)
        R = _radii(c, seed)
        return _curve64(fields, sides, R, c["naz"], GM), _sigma64(fields, sides, R, c["naz"], GM, 0.3, 0.3)
    if k == "batch":
        R = torch.tensor(_batch_radii(c), device=DEV, dtype=torch.float64)
        cn, cq = [], []
        for d in _batch_disks(c, seed):
            x, y, z, m, M = _batch_particles(d)
            pn, pq = _solved64({"n": d["n"]}, [c["side"]], x, y, z, m, M)
            cn.append(_curve64(pn, [c["side"]], R, 16, G * M, False))
            cq.append(_curve64(pq, [c["side"]], R, 16, G * M, True))
        return torch.stack(cn), torch.stack(cq)
    if k == "conv":
        x, w, b, dy = _conv_inputs(c, seed)
        n, cin, cout, s = c["n"], c["cin"], c["cout"], c["stride"]
        no = (n + 1) // 2 if s == 2 else n
        xd = x.double().reshape(n, n, n, cin).requires_grad_(True)
        wd = w.double()[:, :27 * cin].reshape(cout, 27, cin).clone().requires_grad_(True)
        y = _Conv64.apply(xd, wd, b.double(), s)
        y.backward(dy.double().reshape(no, no, no, cout))
        dw = torch.zeros(cout, _kpad(cin), device=DEV, dtype=torch.float64)
        dw[:, :27 * cin] = wd.grad.reshape(cout, -1)
        return {"y": torch.relu(y.detach()).reshape(-1), "dx": xd.grad.reshape(-1), "dw": dw.reshape(-1)}
    n = c["n"]
    if k == "infer":
        phin, S, L = _net_fields(c, seed)
        c_phin, c_out = _scales(L)
        t = _axis(n, L)
        r = torch.sqrt(t[None, None, :] ** 2 + t[None, :, None] ** 2 + t[:, None, None] ** 2 + 9.0)
        x = torch.stack([(phin - _point_phi(r, G * 6e10, False)) / c_phin, S * (L / (n - 1)) ** 2 / c_out], -1)
        with torch.no_grad():
            y, _, _ = _net64(_net_params(seed), x, False)
        return (_point_phi(r, G * 6e10, True) + c_out * y).reshape(-1)
    x, target = _train_inputs(c, seed)
    y, W, head = _net64(_net_params(seed), x.double().reshape(n, n, n, 2), True)
    loss = ((y - target.double().reshape(n, n, n))[1:-1, 1:-1, 1:-1] ** 2).mean()
    loss.backward()
    out = []
    for (cin, cout, _, fan), (w, b) in zip(LAYERS, W):
        g = torch.zeros(cout, _kpad(cin), device=DEV, dtype=torch.float64)
        full = torch.zeros(cout, 27, cin, device=DEV, dtype=torch.float64)
        full[:, :, :fan] = w.grad
        g[:, :27 * cin] = full.reshape(cout, -1)
        out += [g.reshape(-1), b.grad]
    out += [head[0].grad, head[1].grad.reshape(1)]
    return {"loss": float(loss), "grads": torch.cat(out)}
