"""The general solve with other sweep counts than two: pairs of sweeps in one
pass, what an odd count leaves over, the copy back when the cycle ends in the
ping-pong partner, and levels whose steps keep z or keep x and y; against the
oracle's cycles with the same counts."""

import numpy as np
import pytest

import synth
from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1307_6720_amd import PLAN_GENERAL, PREC_FP64, _lib  # noqa: E402
from paper_1307_6720_amd.solver import Plan, make_opts  # noqa: E402

GRIDS = [((33, 33, 33), (1.0, 1.0, 1.0)), ((129, 65, 33), (1.0, 0.5, 0.25)), ((65, 33, 17), (1.0, 1.0, 1.0)),
         ((9, 9, 65), (1.0, 1.0, 1.0)), ((9, 129, 9), (0.0625, 1.0, 0.0625)), ((5, 5, 5), (1.0, 1.0, 1.0))]
COUNTS = [(1, 1), (1, 2), (2, 1), (2, 2), (3, 4)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def close(got, want):
    assert np.abs(got - want).max() < 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("nu", COUNTS)
@pytest.mark.parametrize("dims,lengths", GRIDS, ids=lambda v: "x".join(map(str, v)))
def test_box(dims, lengths, nu):
    shape = dims[::-1]
    a, b, c, u = synth.general_problem(shape, lengths, 21)
    want, st, *_ = ref.gen_mg(u, a, b, c, rtol=-1.0, max_cycles=2, nu1=nu[0], nu2=nu[1], lengths=lengths)
    assert st == ref.OK
    plan = Plan(synth.make_grid(*dims, *lengths), PREC_FP64 | PLAN_GENERAL)
    ud = dev(u)
    for _ in range(2):  # the second call starts cold again, on used work arrays
        info = plan.solve_general(dev(a), dev(b), dev(c), ud, make_opts(rtol=1e-300, max_cycles=2, nu1=nu[0], nu2=nu[1]),
                                  raise_on_error=False)
        assert info.cycles == 2
        close(ud.cpu().numpy(), want)


@pytest.mark.parametrize("nu", COUNTS)
@pytest.mark.parametrize("dims", [(33, 17, 65), (257, 33, 129), (9, 5, 9)], ids=lambda v: "x".join(map(str, v)))
def test_face(dims, nu):
    """The (x, z) face y = 0."""
    lengths = [float(n - 1) / 64 for n in dims]
    shape = (dims[2], dims[0])
    flen = (lengths[0], lengths[2])
    a, b, c, u = synth.general_problem(shape, flen, 22)
    want, st, *_ = ref.gen_mg(u, a, b, c, rtol=-1.0, max_cycles=2, nu1=nu[0], nu2=nu[1], lengths=flen, planar=True)
    assert st == ref.OK
    plan = Plan(synth.make_grid(*dims, *lengths), PREC_FP64 | PLAN_GENERAL)
    P = np.random.default_rng(3).standard_normal(dims[::-1])
    P[:, 0, :] = u
    Pd = dev(P)
    info = plan.solve_face(_lib.FACE_YLO, dev(a), dev(b), dev(c), Pd,
                           make_opts(rtol=1e-300, max_cycles=2, nu1=nu[0], nu2=nu[1]), raise_on_error=False)
    assert info.cycles == 2
    close(Pd[:, 0, :].cpu().numpy(), want)


def test_warm_start_continues():
    """Two cycles from a warm start after two equal four from a cold one."""
    dims, lengths = (65, 33, 33), (1.0, 0.5, 0.5)
    a, b, c, u = synth.general_problem(dims[::-1], lengths, 23)
    plan = Plan(synth.make_grid(*dims, *lengths), PREC_FP64 | PLAN_GENERAL)
    A, B, C = dev(a), dev(b), dev(c)
    four, two = dev(u), dev(u)
    plan.solve_general(A, B, C, four, make_opts(rtol=1e-300, max_cycles=4), raise_on_error=False)
    plan.solve_general(A, B, C, two, make_opts(rtol=1e-300, max_cycles=2), raise_on_error=False)
    plan.solve_general(A, B, C, two, make_opts(rtol=1e-300, max_cycles=2, warm_start=True), raise_on_error=False)
    assert torch.equal(four, two)
