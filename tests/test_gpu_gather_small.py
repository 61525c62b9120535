"""Forces on the smallest grids: 5^3, where one form serves all cells, and 9^3,
where the inner cells have one of their own."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 9])
def test_forces_of_every_cell(n):
    L = 10.0
    h = L / (n - 1)
    rng = np.random.default_rng(n)
    p = [torch.as_tensor(rng.normal(size=5000) * s).cuda() for s in (1.5, 1.5, 0.4)]
    ctx = Q.Context(Q.Config(n=n, box_side=[L]))
    ctx.deposit(*p, torch.full_like(p[0], 1e6), 5e9)
    ctx.solve_newton()
    phi = ctx.get_field(0, Q.FIELD_PHI_N).cpu().numpy().reshape(n, n, n)
    pts = rng.uniform(-L / 2, L / 2, (3, 64 * (n - 1) ** 3))      # 64 points a cell on average
    *a, used = ctx.gather_forces(*(torch.as_tensor(c).cuda() for c in pts), 0)
    ref = O.gather([phi], [L], *pts, M=5e9, mond=False)
    assert np.array_equal(used.cpu().numpy(), ref[3])
    # eight weighted differences of three values of at most 4 |phi| / 2h each, some 16 roundings
    tol = 16 * 2.0 ** -53 * 8 * np.abs(phi).max() / (2 * h)
    for g, r in zip(a, ref):
        assert np.abs(g.cpu().numpy() - r).max() <= tol
    ctx.close()
