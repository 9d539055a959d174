"""Stage entry points: a right-hand side has no meaning on boundary nodes, so
whatever its array holds there is not used, however many sweeps a launch takes."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402


@pytest.fixture(scope="module")
def S():
    from paper_1307_6720_amd import solver

    return solver


@pytest.mark.parametrize("dims", [(9, 9, 9), (65, 33, 65), (513, 33, 17)])
@pytest.mark.parametrize("nsweeps", [1, 2, 3])
@pytest.mark.parametrize("precision", [1, 2])
def test_boundary_values_of_a_right_hand_side_are_not_used(S, precision, nsweeps, dims):
    g = synth.make_grid(*dims, *[n - 1.0 for n in dims])
    model = synth.make_model(g, 0.01, 0.4, 0.2 * (dims[2] - 1))
    plan = S.Plan(g, precision)
    dtype = torch.float64 if precision == 1 else torch.float32
    inner = (slice(1, -1),) * 3
    f = torch.zeros(plan.shape, dtype=dtype, device="cuda")
    f[inner] = torch.from_numpy(np.random.default_rng(9).standard_normal(f[inner].shape)).to("cuda", dtype)
    h = torch.full_like(f, float("nan"))
    h[inner] = f[inner]
    for zero in (True, False):
        u = torch.zeros_like(f) if zero else torch.ones_like(f)
        got = [plan.stage_smooth(model, 3, 0, u.clone(), q, nsweeps, precision, zero_guess=zero) for q in (f, h)]
        assert torch.equal(*got) and got[0][inner].abs().max().item() > 0
