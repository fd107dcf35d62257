"""Line-search rounds that do not fill a group: last rounds with fewer trials
than lanes, and groups wider than their rounds, in every form of a solve."""
import numpy as np
import pytest

from paper_2602_19699_amd import inputs as I

from gpu_helpers import gpu_solve

pytestmark = pytest.mark.gpu

FIELDS = ("X", "U", "J", "iters", "status", "Vbar", "Vx", "xK", "cost_trace", "work", "jtrace")


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
@pytest.mark.parametrize("n,m", [(2, 1), (4, 2), (6, 3)])
@pytest.mark.parametrize("trials", [1, 3, 11, 16])
def test_lq_trial_budget_of_any_size(ctx, n, m, trials, prec):
    # a linear-quadratic solve is at its optimum after one step: the second
    # iteration's line search finds no decrease and runs through its budget,
    # the last round with fewer trials than lanes
    p, x0 = I.lq_random(n, m, 0), I.lq_x0(37, n)
    o = dict(T=I.horizons(37, 1, 40, 6), precision=prec, max_iter=4, ls_max_trials=trials, trace=True)
    ref = gpu_solve(ctx, I.SYS_LQ, p, x0, 40, group_lanes=1, **o)
    assert np.all(ref["work"][:, 0] >= 2)
    for g in (2, 4, 8, 16):
        _equal(ref, gpu_solve(ctx, I.SYS_LQ, p, x0, 40, group_lanes=g, **o), [k for k in FIELDS if k != "work"], f"{g}")


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("kind", [I.SYS_POINT_MASS, I.SYS_PLANAR3], ids=["pm", "arm"])
@pytest.mark.parametrize("form", [{}, {"u_max": 4.0}, {"regularization": 1}, {"iters_per_launch": 2},
                                  {"ls_max_trials": 5}, {"stop_mode": 1, "rtol": 1e-4}, {"max_iter": 40}],
                         ids=["clip", "bound", "lm", "launches", "odd_trials", "stop", "budget"])
@pytest.mark.parametrize("ragged", [False, True], ids=["one", "ragged"])
@pytest.mark.parametrize("B,trials", [(4097, 8), (8193, 4), (16385, 2)])
def test_own_choice_matches_narrow_groups(ctx, kind, prec, form, ragged, B, trials):
    # whatever lanes the library takes for a large batch, of one horizon or of
    # several, every output and the work counters equal those of groups as wide
    # as the batch's line-search rounds
    p = I.point_mass_params(0) if kind == I.SYS_POINT_MASS else I.planar3_params(0)
    x0 = I.point_mass_x0(B, 5) if kind == I.SYS_POINT_MASS else I.planar3_x0(B, 5)
    o = {**dict(T=I.horizons(B, 1, 19, 6) if ragged else None, precision=prec, max_iter=3, trace=True), **form}
    _equal(gpu_solve(ctx, kind, p, x0, 19, group_lanes=trials, **o), gpu_solve(ctx, kind, p, x0, 19, **o))


def test_a_tuned_solve_is_no_slower_than_an_untuned_one(ctx):
    # ragged arm batches beyond 8192 instances: the library's own choice (16
    # lanes, 4 trials per round) takes 0.85 times the best width or less; a
    # solve after tuning keeps it and its results
    import torch
    from paper_2602_19699_amd import cbic
    B, T = 12000, 40
    sysm = cbic.System(ctx, I.SYS_PLANAR3, I.planar3_params(0))
    x0, Td = torch.as_tensor(I.planar3_x0(B, 5), device="cuda"), torch.as_tensor(I.horizons(B, 8, T, 6), device="cuda")
    o = cbic.Options(precision=1, max_iter=6)

    def solve():
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        out = cbic.solve_batch(ctx, sysm, x0, T, T=Td, opts=o)
        e1.record()
        torch.cuda.synchronize()
        return out, e0.elapsed_time(e1)

    before = min((solve() for _ in range(5)), key=lambda r: r[1])
    lanes, ms = cbic.autotune(ctx, sysm, x0, T, T=Td, opts=o)
    after, _ = solve()
    assert lanes in (1, 2, 4, 8, 16) and ms <= 1.1 * before[1]
    for k in ("X", "U", "J", "iters", "status", "Vbar", "Vx"):
        assert torch.equal(getattr(before[0], k), getattr(after, k)), k
    sysm.close()
