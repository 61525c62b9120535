"""The coarse tail's modes on every top level, with boundary
values on the far faces as on the low ones: FMG and V-cycles against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu


def problem(n, far_only):
    rng = np.random.default_rng(n + far_only)
    f = rng.standard_normal((n,) * 3)
    u = np.zeros((n,) * 3)
    for d in range(3):
        for e in ((n - 1,) if far_only else (0, n - 1)):
            face = [slice(None)] * 3
            face[d] = e
            u[tuple(face)] = rng.standard_normal((n, n))
    return f, u


@pytest.mark.parametrize("far_only", [0, 1])
@pytest.mark.parametrize("n", [5, 9, 17, 33])
def test_against_the_oracle(n, far_only):
    """Same operations as the oracle: rounding of a few hundred additions of
    values of order one, 1e-12, on every node (33^3 enters the tail from u = 0)."""
    f, u = problem(n, far_only)
    for ncycle, reps in ((1, 0), (2, 3)):
        d = torch.from_numpy(u).cuda()
        Q.k_fmg(torch.from_numpy(f).cuda(), d, 2.5, ncycle=ncycle, max_extra=0, tol=0.0)
        ref = u.copy()
        O.fmg(f, ref, 2.5, ncycle=ncycle, max_extra=0, tol=0.0)
        if reps:
            Q.k_vcycles(torch.from_numpy(f).cuda(), d, 2.5, reps)
            O.vcycles(f, ref, 2.5, reps)
        got = d.cpu().numpy()
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
        edge = np.ones((n,) * 3, dtype=bool)
        edge[1:-1, 1:-1, 1:-1] = False
        assert np.array_equal(got[edge], u[edge])
