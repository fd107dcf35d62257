"""The ways a solve's inner steps are split over lanes and waves change no bit
of any output: each split is compared with the one-lane group (or the other
split) on the same instances, at horizons around the chunk edges."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2602_19699_amd import inputs as I

from gpu_helpers import gpu_solve, oracle_opts, rel

pytestmark = pytest.mark.gpu

PM, P3 = I.SYS_POINT_MASS, I.SYS_PLANAR3
FIELDS = ("X", "U", "J", "iters", "status", "Vbar", "Vx", "xK", "cost_trace", "work", "jtrace")
EDGES = np.array([1, 2, 3, 15, 16, 17, 31, 32, 33, 47, 7, 1, 16], np.int32)


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2602_19699_amd import cbic
    assert torch.cuda.is_available()
    c = cbic.Context(0)
    yield c
    c.close()


def _equal(a, b, fields=FIELDS, what=""):
    for k in fields:
        np.testing.assert_array_equal(a[k], b[k], err_msg=f"{what} field {k}")


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("form", [{}, {"u_max": 4.0}, {"regularization": 1}], ids=["clip", "bound", "lm"])
def test_arm_column_lanes_match_one_lane(ctx, prec, form):
    # 16 lanes: a lane per column of the Riccati step; 1 lane: the whole step.
    # A non-finite instance and an odd batch (a part-filled last wave) ride along.
    p, x0 = I.planar3_params(0), I.planar3_x0(len(EDGES), 77)
    x0[5, 4] = np.nan
    o = dict(T=EDGES, precision=prec, max_iter=8, trace=True, **form)
    ref = gpu_solve(ctx, P3, p, x0, 47, group_lanes=1, **o)
    got = gpu_solve(ctx, P3, p, x0, 47, group_lanes=16, **o)
    # the work counters count what the lanes of a group read and write together
    _equal(ref, got, [k for k in FIELDS if k != "work"], f"{form}")
    np.testing.assert_array_equal(ref["work"][:, 0], got["work"][:, 0])


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("kind", [PM, P3], ids=["pm", "arm"])
@pytest.mark.parametrize("B,trials", [(4097, 8), (8193, 4), (16385, 2), (32769, 1)])
def test_default_widths_match_narrow_groups(ctx, kind, prec, B, trials):
    # the library's own choice of lanes for a large batch keeps that batch's
    # line-search rounds: every output and the work counters equal those of a
    # group as wide as its rounds
    p = I.point_mass_params(0) if kind == PM else I.planar3_params(0)
    x0 = I.point_mass_x0(B, 5) if kind == PM else I.planar3_x0(B, 5)
    o = dict(T=I.horizons(B, 1, 19, 6), precision=prec, max_iter=3, trace=True)
    _equal(gpu_solve(ctx, kind, p, x0, 19, group_lanes=trials, **o), gpu_solve(ctx, kind, p, x0, 19, **o))


@pytest.mark.parametrize("kind", [PM, P3], ids=["pm", "arm"])
@pytest.mark.parametrize("trials", [1, 3, 5, 11])
def test_trial_budget_of_any_size(ctx, kind, trials):
    # a last line-search round with fewer trials than lanes
    p = I.point_mass_params(0) if kind == PM else I.planar3_params(0)
    x0 = I.point_mass_x0(40, 5) if kind == PM else I.planar3_x0(40, 5)
    o = dict(T=I.horizons(40, 1, 50, 6), max_iter=6, ls_max_trials=trials, trace=True)
    ref = gpu_solve(ctx, kind, p, x0, 50, group_lanes=1, **o)
    for g in (2, 4, 8, 16):
        _equal(ref, gpu_solve(ctx, kind, p, x0, 50, group_lanes=g, **o), [k for k in FIELDS if k != "work"], f"{g}")


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("form", [{}, {"u_max": 6.0}, {"regularization": 1}], ids=["clip", "bound", "lm"])
def test_quadruped_chunk_edges(ctx, prec, form):
    # horizons around the sweep's 12-step chunks of derivative blocks, a bad
    # and a non-finite instance among them, against the FP64 oracle
    T = np.array([1, 2, 11, 12, 13, 23, 24, 25, 36, 37, 0, 5], np.int32)
    p = I.quad_params(0)
    x0 = I.quad_x0(len(T), p, 91)
    x0[11, 20] = np.nan
    o = dict(max_iter=6, stop_mode=1, rtol=1e-10 if prec == 0 else 1e-4, **form)
    g = gpu_solve(ctx, I.SYS_QUAD_SYNTH, p, x0, 37, T=T, precision=prec, **o)
    r = orc.solve_batch(I.SYS_QUAD_SYNTH, p, x0[:10], 37, T=T[:10],
                        opts=oracle_opts(**{**o, "rtol": 1e-10}))
    assert np.all(rel(g["J"][:10], r.J) <= (1e-9 if prec == 0 else 1e-4))
    assert g["status"][10] == 32 and g["status"][11] == 8
    for wg in (1, 2):  # either schedule
        _equal(g, gpu_solve(ctx, I.SYS_QUAD_SYNTH, p, x0, 37, T=T, precision=prec, wg_per_cu=wg, **o),
               [k for k in FIELDS if g[k] is not None], f"wg_per_cu={wg}")


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("u_max", [0.5, 3.0, 10.0, 30.0])
def test_two_control_bound_from_rarely_to_always_active(ctx, prec, u_max):
    # the in-line courses of the two-control box QP and its loop (released
    # bounds): against the oracle, and every group width alike
    p, x0 = I.point_mass_params(0), I.point_mass_x0(200, 12)
    T = I.horizons(200, 1, 60, 13)
    o = dict(u_max=u_max, max_iter=25, stop_mode=1, rtol=1e-10 if prec == 0 else 1e-7)
    g = gpu_solve(ctx, PM, p, x0, 60, T=T, precision=prec, **o)
    r = orc.solve_batch(PM, p, x0, 60, T=T, opts=oracle_opts(**{**o, "rtol": 1e-10}))
    assert np.all(rel(g["J"], r.J) <= (1e-9 if prec == 0 else 1e-4))
    assert np.all(np.abs(g["U"]) <= u_max)
    for gl in (1, 4):
        _equal(g, gpu_solve(ctx, PM, p, x0, 60, T=T, precision=prec, group_lanes=gl, **o),
               ["X", "U", "J", "iters", "status", "Vbar", "Vx"], f"{gl}")


@pytest.mark.parametrize("lanes", [1, 16])
def test_arm_angles_past_the_short_range(ctx, lanes):
    # angles around 2^30, where the FP64 sine and cosine change course, and far
    # past it; one angle at a time, so that the absolute angles are exact sums.
    # A step's velocities are dt M^-1 (tau - b): errors of a few ulp, grown by
    # the mass matrix's condition (below 1e3)
    p = I.planar3_params(0)
    a = np.array([2.0**30 - 0.5, 2.0**30, 2.0**30 + 0.5, -(2.0**30) - 0.5, 1e12, 3e15])
    x0 = np.zeros((3 * len(a), 6))
    for j in range(3):
        x0[j * len(a):(j + 1) * len(a), j] = a
    x0[:, 3:] = [0.3, -0.4, 0.5]
    U0 = np.tile([1.0, -2.0, 0.5], (len(x0), 2, 1))
    got = gpu_solve(ctx, P3, p, x0, 2, U0=U0, group_lanes=lanes, precision=0, max_iter=0)
    want = np.stack([orc.dyn(P3, p, x0[b], U0[b, 0]) for b in range(len(x0))])
    v = want[:, 3:]
    assert np.max(np.abs(got["X"][:, 1, 3:] - v)) <= 1e3 * 8 * np.finfo(float).eps * np.max(np.abs(v))
    one = gpu_solve(ctx, P3, p, x0, 2, U0=U0, group_lanes=1, precision=0, max_iter=2, trace=True)
    _equal(one, gpu_solve(ctx, P3, p, x0, 2, U0=U0, group_lanes=lanes, precision=0, max_iter=2, trace=True),
           [k for k in FIELDS if k != "work"])
