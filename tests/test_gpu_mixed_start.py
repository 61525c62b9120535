"""The first refinement step of a mixed solve takes its scale from the size of
the right-hand side and of the boundary values, before the FP32 FMG."""
import numpy as np
import pytest
import torch

from paper_1201_3185_amd import qumond as Q

pytestmark = pytest.mark.gpu
L_BOX = 50.0


def solve(n, g, particles=True, precision=Q.QUMOND_MIXED, tol=1e-9, max_vcycles=30):
    rng = np.random.default_rng(n)
    s = 0.2 * L_BOX if particles else 0.0
    pos = [torch.as_tensor(rng.normal(0.0, 1.0, 4000) * 0.1 * s, device="cuda") for _ in range(3)]
    if not particles:
        pos[0] = pos[0] + 2.0 * L_BOX       # all outside: f = 0, boundary values only
    m = torch.full((4000,), 1e10 / 4000, device="cuda", dtype=torch.float64)
    ctx = Q.Context(Q.Config(n=n, box_side=[L_BOX], G=g, precision=precision, ncycle_fmg=2, tol_rel=tol,
                             max_vcycles=max_vcycles))
    ctx.deposit(*pos, m, 1e10)
    info = ctx.solve_newton()
    phi = ctx.get_field(0, Q.FIELD_PHI_N).cpu().numpy()
    ctx.close()
    return phi, info


@pytest.mark.parametrize("n", [9, 17, 33, 65])
def test_units_of_another_power_of_two_give_the_same_bits(n):
    """Every operation of the Newtonian solve commutes with a power of two, the
    scale of the first step included, so G times 2^-40 gives Phi times 2^-40."""
    g = Q.Config(n=n, box_side=[L_BOX]).G
    a, ia = solve(n, g)
    b, ib = solve(n, g * 2.0 ** -40)
    assert ia["refine_iters"][0] >= 1 and ia["refine_iters"] == ib["refine_iters"]
    assert np.array_equal(a * 2.0 ** -40, b)


@pytest.mark.parametrize("n", [17, 65])
def test_boundary_values_alone_scale_the_first_step(n):
    """No mass inside: the scale comes from the boundary values.  A residual r in
    the 2-norm of 1e-11 of the boundary terms, at most 1e-11 sqrt(6) n max|Phi| /
    h^2, leaves an error below n^2 h^2 / 8 times that: n^3 1e-11 max|Phi| bounds
    the two solves' difference."""
    g = Q.Config(n=n, box_side=[L_BOX]).G * 2.0 ** -40
    a, ia = solve(n, g, particles=False, tol=1e-11)
    b, _ = solve(n, g, particles=False, tol=1e-11, precision=Q.QUMOND_FP64)
    assert ia["converged"][0] == 1 and ia["refine_iters"][0] >= 1
    assert np.abs(a - b).max() <= 1e-11 * n ** 3 * np.abs(b).max()


def test_no_refinement_asked_for():
    """tol_rel = 0 leaves the FP32 FMG's iterate: FP32 accuracy of |Phi|."""
    g = Q.Config(n=33, box_side=[L_BOX]).G
    a, ia = solve(33, g, tol=0.0)
    b, _ = solve(33, g, precision=Q.QUMOND_FP64)
    assert ia["refine_iters"][0] == 0
    assert np.abs(a - b).max() <= 5e-3 * np.abs(b).max()
