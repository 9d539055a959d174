"""The cycles' launch of two sweeps, in every tiling, against the launches of
one sweep, one residual norm and one restriction (which the stage tests pin to
the oracle): every value is the same expression of the same inputs, so they
agree bit for bit.  The norm is a sum of non-negative terms in another order: a
thread adds up to a few thousand of them, so it is within 4096 rounding errors."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from paper_1307_6720_amd import _lib  # noqa: E402

NORM_TOL = 4096 * 2.0**-53
# waves per workgroup, planes of loads in flight, rows of sixteen lanes, most planes per workgroup
VARIANTS = [(12, 1, False, 128), (4, 3, False, 44), (8, 3, False, 44), (12, 1, True, 128), (4, 3, True, 44),
            (8, 3, True, 128)]


@pytest.fixture(scope="module")
def S():
    from paper_1307_6720_amd import solver

    return solver


def fits(variant, dims, precision, over, ext):
    """Whether the level's rows and rims allow the variant's windows."""
    waves, _, row, _ = VARIANTS[variant]
    v = 2 if precision == 1 else 4
    mx, my = dims[0] - 1 + ext, dims[1] - 1 + ext
    lanes = 16 if row else min(64, (mx - 1) // v + 1)
    lanes = 1 << (lanes - 1).bit_length()
    rows = 2 * waves * (64 // lanes)
    return not (row and lanes * v > mx) and not (rows <= over and rows < my)


def rand(shape, dtype, seed, zero_faces=True):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.randn(shape, generator=gen, dtype=dtype, device="cuda")
    if zero_faces:
        for axis in range(3):
            u.select(axis, 0).zero_()
            u.select(axis, -1).zero_()
    return u


def same(a, b):
    inner = (slice(1, -1),) * 3
    return torch.equal(a[inner], b[inner])


# one window per row and several, remainders in y and z, marches through more planes than a wave has
# lanes, steps that keep z (dz = 4 dx); the last two are the sizes whose windows a solve of 257^3
# and of 513 x 513 x 257 takes
GRIDS = [((17, 9, 33), 1), ((65, 129, 33), 1), ((129, 65, 65), 1), ((257, 129, 17), 1), ((513, 65, 33), 1),
         ((1025, 65, 17), 1), ((129, 257, 65), 4), ((65, 65, 257), 1), ((257, 257, 257), 1), ((513, 513, 257), 1)]


@pytest.mark.parametrize("variant", range(-1, len(VARIANTS)))
@pytest.mark.parametrize("precision", [1, 2])
@pytest.mark.parametrize("dims,dz", GRIDS)
def test_two_sweeps_equal_single_launches(S, dims, dz, precision, variant):
    nx, ny, nz = dims
    lengths = (nx - 1.0, ny - 1.0, dz * (nz - 1.0))
    g = synth.make_grid(nx, ny, nz, *lengths)
    plan = S.Plan(g, precision)
    model = synth.make_model(g, 0.01, 0.5, 0.2 * lengths[2])
    dtype = torch.float64 if precision == 1 else torch.float32
    shape, coarse = plan.shape, plan.level_shape(3, 1)
    u, f, ec = rand(shape, dtype, 1), rand(shape, dtype, 2), rand(coarse, dtype, 3)
    most = VARIANTS[variant][3] if variant >= 0 else 0
    # the chosen number of planes, the most, and one with a remainder
    planes = list(dict.fromkeys((0, min(most, 2 * (nz // 2)), min(most, 26))))
    run = dict(precision=precision, variant=variant)

    def single(zero=False, data=None, e=None):
        w = torch.zeros_like(u) if zero else (u if data is None else data).clone()
        q = f if data is None else None
        if e is None:
            plan.stage_smooth(model, 3, 0, w, q, 1, precision, zero_guess=zero)
        else:
            plan.stage_correct_smooth(model, 3, 0, w, q, e, precision)
        return plan.stage_smooth(model, 3, 0, w, q, 1, precision)

    def fused(start, q, kz, e=None, rest=False, **kw):
        out = torch.zeros_like(u)
        fc = torch.zeros(coarse, dtype=dtype, device="cuda") if rest else None
        plan.stage_two_sweeps(model, 0, start, q, out, e, fc, kz=kz, **run, **kw)
        return out, fc

    def check(want, start, q, over=8, ext=0, **kw):
        kinds = planes if variant < 0 or fits(variant, dims, precision, over, ext) else []
        if variant >= 0 and not kinds:
            with pytest.raises(S.MHSError) as err:
                fused(start, q, 0, **kw)
            assert err.value.code == _lib.ERR_UNSUPPORTED
        for kz in kinds:
            got, fc = fused(start, q, kz, **kw)
            assert same(got, want), f"planes {kz} {kw.keys()}"
            if fc is not None:
                ref = plan.stage_restrict(model, 3, 0, want, q, torch.zeros_like(fc), precision)
                assert same(fc, ref) and ref.abs().max().item() > 0, f"restriction, planes {kz}"

    want, from_zero = single(), single(zero=True)
    check(want, u, f)
    check(from_zero, None, f)
    check(want, u, f, over=12, rest=True)
    check(from_zero, None, f, over=12, rest=True)
    check(single(e=ec), u, f, e=ec)
    if precision == 1:
        for faces in (False, True):
            d = rand(shape, dtype, 4, zero_faces=False)
            if not faces:
                d[:, 0] = d[:, -1] = 0
                d[:, :, 0] = d[:, :, -1] = 0
            kw = dict(ext=2 if faces else 0, faces_given=faces)
            check(single(data=d), d, None, **kw)
            check(single(data=d, e=ec), d, None, e=ec, **kw)
            if variant < 0 or fits(variant, dims, precision, 8, kw["ext"]):
                try:
                    norm = plan.stage_two_sweeps(model, 0, d, None, torch.zeros_like(d), faces_given=faces, norm=True,
                                                 **run)
                except S.MHSError as err:  # more workgroups than the plan keeps sums for
                    assert variant >= 0 and err.code == _lib.ERR_WORKSPACE
                else:
                    assert norm == pytest.approx(plan.stage_residual_norm(model, 3, 0, d), rel=NORM_TOL)


def test_every_tiling_is_compared(S):
    plan = S.Plan(synth.make_grid(33, 33, 33, 1.0, 1.0, 1.0), 1)
    model = synth.make_model(plan.grid, 0.01, 0.5, 0.2)
    u = rand(plan.shape, torch.float64, 1)
    for variant in (len(VARIANTS), -2):
        with pytest.raises(S.MHSError) as err:
            plan.stage_two_sweeps(model, 0, u, u, torch.zeros_like(u), variant=variant)
        assert err.value.code == _lib.ERR_INVALID_ARG
    # and no more planes than its table of coefficients holds
    for variant, (_, _, _, most) in enumerate(VARIANTS):
        with pytest.raises(S.MHSError) as err:
            plan.stage_two_sweeps(model, 0, u, u, torch.zeros_like(u), variant=variant, kz=most + 1)
        assert err.value.code == _lib.ERR_INVALID_ARG


@pytest.mark.parametrize("wrong", ["in place", "no f in FP32", "norm with f", "ec and fc", "zero and ec", "odd planes"])
def test_other_combinations_are_refused(S, wrong):
    plan = S.Plan(synth.make_grid(33, 33, 33, 1.0, 1.0, 1.0), 3)
    model = synth.make_model(plan.grid, 0.01, 0.5, 0.2)
    precision = 2 if wrong == "no f in FP32" else 1
    dtype = torch.float32 if precision == 2 else torch.float64
    u, out = rand(plan.shape, dtype, 1), torch.zeros(plan.shape, dtype=dtype, device="cuda")
    ec = torch.zeros(plan.level_shape(3, 1), dtype=dtype, device="cuda")
    args = {"in place": (u, u, u), "no f in FP32": (u, None, out), "norm with f": (u, u, out),
            "ec and fc": (u, u, out, ec, ec.clone()), "zero and ec": (None, u, out, ec),
            "odd planes": (u, u, out, None, ec)}[wrong]
    with pytest.raises(S.MHSError) as err:
        plan.stage_two_sweeps(model, 0, *args, precision=precision, norm=wrong == "norm with f",
                              kz=9 if wrong == "odd planes" else 0)
    assert err.value.code == _lib.ERR_INVALID_ARG
