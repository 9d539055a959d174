"""The last two pre-smoothing sweeps with the restriction of their residual in
the same launch: a cycle against the same cycle stage by stage (each stage is
pinned to the oracle by its own tests), and the FP32 correction cycles against
FP64 ones.

The tolerance: rounding of a residual, eps |d| |u| with |d| = 2 sum 1/h^2,
reaches the solution through 1 / lambda_min = 1 / (pi^2 sum 1/L^2), a relative
eps 0.2 (n - 1)^2 on n^3 nodes of a cube, and there are a few such terms."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402


@pytest.fixture(scope="module")
def S():
    from paper_1307_6720_amd import solver

    return solver


def setup(S, dims, lengths, precision):
    g = synth.make_grid(*dims, *lengths)
    plan = S.Plan(g, precision)
    model = synth.make_model(g, 0.3, 0.4, 0.2 * lengths[2])
    rng = np.random.default_rng(11)
    P = torch.zeros(plan.shape, dtype=torch.float64, device="cuda")
    P[0] = torch.from_numpy(rng.standard_normal(plan.shape[1:])).cuda()
    P[:, 0] = P[:, -1] = 0
    P[:, :, 0] = P[:, :, -1] = 0
    return plan, model, P


def tol(dims, eps):
    return 8.0 * eps * max(1.0, 0.2 * (max(dims) - 1) ** 2)


def cycle(plan, model, u, f, level, bottom):
    """One V(2,2) cycle on level `level`, stage by stage."""
    zero = level > 0
    if level == bottom:
        plan.stage_bottom(model, 3, u, f)
        return
    plan.stage_smooth(model, 3, level, u, f, 2, zero_guess=zero)
    fc = torch.zeros(plan.level_shape(3, level + 1), dtype=torch.float64, device="cuda")
    plan.stage_restrict(model, 3, level, u, f, fc)
    ec = torch.zeros_like(fc)
    cycle(plan, model, ec, fc, level + 1, bottom)
    plan.stage_correct_smooth(model, 3, level, u, f, ec, nsweeps=2)


# one window per row and several, remainders in y and z, steps that keep z
# (the last two: dz = 4 dx and dz = 2 dx)
GRIDS = [((33, 33, 33), (1.0, 1.0, 1.0)), ((65, 65, 65), (1.0, 1.0, 1.0)), ((129, 65, 33), (2.0, 1.0, 0.5)),
         ((65, 257, 65), (0.25, 1.0, 0.25)), ((257, 129, 129), (2.0, 1.0, 1.0)), ((513, 65, 65), (4.0, 0.5, 0.5)),
         ((129, 129, 33), (1.0, 1.0, 1.0)), ((257, 129, 65), (2.0, 1.0, 1.0))]


@pytest.mark.parametrize("dims,lengths", GRIDS)
def test_a_cycle_equals_its_stages(S, dims, lengths):
    plan, model, P = setup(S, dims, lengths, 1)
    u = P.clone()
    plan.solve_interior(model, P, S.make_opts(rtol=0.0, max_cycles=1), raise_on_error=False)
    cycle(plan, model, u, None, 0, plan.bottom_level(3))
    diff = (P - u).abs().max().item()
    assert diff <= tol(dims, 2.0**-53) * P.abs().max().item()


@pytest.mark.parametrize("dims,lengths", GRIDS)
@pytest.mark.parametrize("cycles", [1, 3])
def test_correction_cycles_in_fp32(S, dims, lengths, cycles):
    plan, model, P = setup(S, dims, lengths, 3)
    u = P.clone()
    plan.solve_interior(model, P, S.make_opts(precision=2, rtol=0.0, max_cycles=1, inner_cycles=cycles),
                        raise_on_error=False)
    plan.solve_interior(model, u, S.make_opts(rtol=0.0, max_cycles=cycles), raise_on_error=False)
    diff = (P - u).abs().max().item()
    assert diff <= tol(dims, 2.0**-24) * u.abs().max().item()


# one tile and several, remainders in x and y, the largest with two levels above
# the bottom
@pytest.mark.parametrize("dims,lengths", [((65, 129, 9), (1.0, 2.0, 1.0)), ((129, 129, 9), (1.0, 1.0, 1.0)),
                                          ((257, 65, 9), (4.0, 1.0, 1.0)), ((257, 257, 9), (1.0, 1.0, 1.0))])
def test_a_cycle_of_the_boundary_problem_equals_its_stages(S, dims, lengths):
    g = synth.make_grid(*dims, *lengths)
    plan = S.Plan(g, 1)
    nx, ny, _ = dims
    rng = np.random.default_rng(12)
    bz0 = torch.from_numpy(rng.standard_normal((ny, nx))).cuda()
    P = torch.zeros(plan.shape, dtype=torch.float64, device="cuda")
    plan.solve_boundary(bz0, P, S.make_opts(rtol=0.0, max_cycles=1), raise_on_error=False)
    # equation (11): the Laplacian of P on the base is -Bz0 (P = 0 on its edges)
    bottom = plan.bottom_level(2)

    def down(u, f, level):
        if level == bottom:
            plan.stage_bottom(None, 2, u, f)
            return
        plan.stage_smooth(None, 2, level, u, f, 2, zero_guess=level > 0)
        fc = torch.zeros(plan.level_shape(2, level + 1), dtype=torch.float64, device="cuda")
        plan.stage_restrict(None, 2, level, u, f, fc)
        ec = torch.zeros_like(fc)
        down(ec, fc, level + 1)
        plan.stage_correct_smooth(None, 2, level, u, f, ec, nsweeps=2)

    u = torch.zeros((ny, nx), dtype=torch.float64, device="cuda")
    down(u, -bz0, 0)
    diff = (P[0] - u).abs().max().item()
    assert u.abs().max().item() > 0 and diff <= tol((nx, ny), 2.0**-53) * u.abs().max().item()
