"""Two red-black sweeps in one launch against the same two sweeps launched one
by one (each sweep is pinned to the oracle by the stage tests): the values are
the same expressions of the same inputs, so they agree bit for bit."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402


@pytest.fixture(scope="module")
def S():
    from paper_1307_6720_amd import solver

    return solver


# one window per row (nx - 1 = 2^k lanes' worth), windows overlapping in x
# (513) and in y, chunks in z with a remainder, long rows of few lanes
DIMS = [(9, 9, 9), (17, 9, 33), (9, 65, 17), (33, 33, 33), (65, 129, 33), (129, 65, 65), (257, 33, 9), (513, 17, 9),
        (513, 129, 17), (1025, 65, 17), (33, 257, 17)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("precision", [1, 2])
def test_two_sweeps_in_one_launch_equal_two_launches(S, dims, precision):
    lengths = [n - 1.0 for n in dims]  # equal spacings
    g = synth.make_grid(*dims, *lengths)
    plan = S.Plan(g, precision)
    model = synth.make_model(g, 0.01, 0.5, 0.2 * lengths[2])
    dtype = torch.float64 if precision == 1 else torch.float32
    rng = np.random.default_rng(5)
    for level in range(plan.bottom_level(3)):
        shape = plan.level_shape(3, level)
        f = torch.from_numpy(rng.standard_normal(shape)).to("cuda", dtype)
        one = torch.zeros(shape, dtype=dtype, device="cuda")
        two = torch.zeros(shape, dtype=dtype, device="cuda")
        plan.stage_smooth(model, 3, level, two, f, 2, precision, zero_guess=True)
        plan.stage_smooth(model, 3, level, one, f, 1, precision, zero_guess=True)
        plan.stage_smooth(model, 3, level, one, f, 1, precision)
        assert torch.equal(one, two), f"level {level} {shape}"


@pytest.mark.parametrize("dims", [(9, 9, 9), (17, 9, 33), (33, 33, 33), (65, 129, 33), (129, 65, 65), (257, 33, 9),
                                  (33, 257, 17)])
def test_two_sweeps_with_boundary_data_equal_two_launches(S, dims):
    lengths = [n - 1.0 for n in dims]
    g = synth.make_grid(*dims, *lengths)
    plan = S.Plan(g, 1)
    model = synth.make_model(g, 0.01, 0.5, 0.2 * lengths[2])
    rng = np.random.default_rng(6)
    two = torch.from_numpy(rng.standard_normal(plan.shape)).to("cuda")
    one = two.clone()
    plan.stage_smooth(model, 3, 0, two, None, 2)
    plan.stage_smooth(model, 3, 0, one, None, 1)
    plan.stage_smooth(model, 3, 0, one, None, 1)
    assert torch.equal(one, two)


# windows of sixteen lanes per row, several of them in x and in y, of four,
# eight and twelve waves; the last marches through more planes than a wave has lanes
@pytest.mark.parametrize("dims", [(257, 129, 65), (129, 65, 65), (513, 65, 33), (257, 257, 129), (513, 257, 65),
                                  (513, 513, 257)])
@pytest.mark.parametrize("precision", [1, 2])
def test_two_sweeps_in_windows_of_sixteen_lanes(S, dims, precision):
    lengths = [n - 1.0 for n in dims]
    g = synth.make_grid(*dims, *lengths)
    plan = S.Plan(g, precision)
    model = synth.make_model(g, 0.01, 0.5, 0.2 * lengths[2])
    dtype = torch.float64 if precision == 1 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(8)
    f = torch.randn(plan.shape, generator=gen, dtype=dtype, device="cuda")
    rhs = [f, None] if precision == 1 else [f]
    for q in rhs:
        two = torch.randn(plan.shape, generator=gen, dtype=dtype, device="cuda")
        if q is not None:  # the boundary nodes of a correction are zero
            for axis in range(3):
                two.select(axis, 0).zero_()
                two.select(axis, -1).zero_()
        one = two.clone()
        plan.stage_smooth(model, 3, 0, two, q, 2, precision)
        plan.stage_smooth(model, 3, 0, one, q, 1, precision)
        plan.stage_smooth(model, 3, 0, one, q, 1, precision)
        assert torch.equal(one, two)


def test_two_fp32_sweeps_without_a_right_hand_side(S):
    g = synth.make_grid(33, 17, 33, 32.0, 16.0, 32.0)
    plan = S.Plan(g, 2)
    model = synth.make_model(g, 0.01, 0.5, 6.0)
    two = torch.from_numpy(np.random.default_rng(7).standard_normal(plan.shape)).to("cuda", torch.float32)
    one = two.clone()
    plan.stage_smooth(model, 3, 0, two, None, 2, 2)
    plan.stage_smooth(model, 3, 0, one, None, 1, 2)
    plan.stage_smooth(model, 3, 0, one, None, 1, 2)
    assert torch.equal(one, two)
