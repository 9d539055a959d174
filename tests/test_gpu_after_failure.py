"""A solve on a plan whose last solve overflowed: what that one left in the
plan's arrays must not reach the next, whatever sweeps either of them takes."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402


@pytest.fixture(scope="module")
def S():
    from paper_1307_6720_amd import solver

    return solver


# a level's first sweep is one of a pair or a single one from zero, its last
# ones a pair in either of the level's two buffers or a single one
@pytest.mark.parametrize("then", [(1, 1), (1, 2), (1, 4), (2, 2), (3, 2), (3, 4)])
@pytest.mark.parametrize("failed", [(2, 2), (3, 4)])
def test_a_solve_after_an_overflow_equals_one_on_a_new_plan(S, failed, then):
    g = synth.make_grid(65, 33, 65, 2.0, 1.0, 2.0)
    model = synth.make_model(g, 0.3, 0.4, 0.4)
    P = torch.zeros((65, 33, 65), dtype=torch.float64, device="cuda")
    P[0, 1:-1, 1:-1] = torch.from_numpy(np.random.default_rng(4).standard_normal((31, 63))).cuda()
    plans = [S.Plan(g, 2) for _ in range(2)]
    assert plans[0].bottom_level(3) > 1
    bad = 1e60 * P  # a residual past the range of FP32, with a finite norm
    info = plans[0].solve_interior(model, bad, S.make_opts(2, nu1=failed[0], nu2=failed[1]),
                                   raise_on_error=False)
    assert info.status != 0
    got = [P.clone() for _ in plans]
    for plan, u in zip(plans, got):
        plan.solve_interior(model, u, S.make_opts(2, nu1=then[0], nu2=then[1]))
    assert torch.equal(*got)
