"""The two kernels of the actor rollout, a network per wave or spread over the
waves of a block, give the same bits: batches large enough for the first
against the same instances in calls small enough for the second."""
import numpy as np
import pytest

from paper_2602_19699_amd import inputs as I

pytestmark = pytest.mark.gpu

SYSTEMS = {"pm": (I.SYS_POINT_MASS, I.point_mass_params(0), 4, 2, I.point_mass_x0),
           "arm": (I.SYS_PLANAR3, I.planar3_params(0), 6, 3, I.planar3_x0),
           "lq21": (I.SYS_LQ, I.lq_random(2, 1, 0), 2, 1, lambda B, s: I.lq_x0(B, 2, s)),
           "lq63": (I.SYS_LQ, I.lq_random(6, 3, 0), 6, 3, lambda B, s: I.lq_x0(B, 6, s))}


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2602_19699_amd import cbic
    assert torch.cuda.is_available()
    c = cbic.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("depth", [1, 2, 3, 4])
@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("name", list(SYSTEMS))
@pytest.mark.parametrize("ragged", [False, True], ids=["one", "ragged"])
def test_large_batches_match_small_calls(ctx, name, width, depth, ragged):
    import torch
    from paper_2602_19699_amd import cbic
    kind, p, n, m, draw = SYSTEMS[name]
    B, Tm, part = (70001 if ragged else 16381), 7, 4000
    x0 = draw(B, 3)
    x0[11, 0] = np.nan
    T = I.horizons(B, 1, Tm, seed=5)
    T[[3, 7]] = [0, Tm + 1]  # outside 1..T_max: zero rows
    g = cbic.Mlp(n + 1, width, depth, m, torch.as_tensor(I.mlp_params(n + 1, width, depth, m, seed=depth), device="cuda"),
                 depth % 3, 1, 3.0)
    x, Td = torch.as_tensor(x0, device="cuda"), torch.as_tensor(T, device="cuda") if ragged else None
    sysm = cbic.System(ctx, kind, p)
    U, X = cbic.actor_rollout(ctx, sysm, g, x, Tm, T=Td, states=True)
    for b in list(range(0, B, 4 * part)) + [B - 1]:  # (every fourth part, and the last instance)
        e = min(B, b + part)
        u, s = cbic.actor_rollout(ctx, sysm, g, x[b:e], Tm, T=None if Td is None else Td[b:e], states=True)
        np.testing.assert_array_equal(U[b:e].cpu().numpy(), u.cpu().numpy(), err_msg=f"controls from {b}")
        np.testing.assert_array_equal(X[b:e].cpu().numpy(), s.cpu().numpy(), err_msg=f"states from {b}")
    sysm.close()
