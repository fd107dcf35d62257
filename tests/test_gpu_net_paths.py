"""The paths a network call can take (weights in registers or in shared memory,
one wave per tile or a wave per 16 neurons) at the edges of their ranges."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2602_19699_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 2e-5  # FP32 rounding through at most five layers of fan-in <= 64 (see test_gpu_nets.py)


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2602_19699_amd import cbic
    assert torch.cuda.is_available()
    c = cbic.Context(0)
    yield c
    c.close()


def _net(in_dim, width, depth, out_dim, seed, act=0, out_act=0, scale=1.0):
    import torch
    from paper_2602_19699_amd import cbic
    params = I.mlp_params(in_dim, width, depth, out_dim, seed=seed)
    return (cbic.Mlp(in_dim, width, depth, out_dim, torch.as_tensor(params, device="cuda"), act, out_act, scale),
            orc.Net(in_dim, width, depth, out_dim, act, out_act, scale, params))


@pytest.mark.parametrize("in_dim", [4, 5, 8, 9])
@pytest.mark.parametrize("depth", [1, 2, 3])
@pytest.mark.parametrize("width", [32, 64])
def test_forward_at_path_edges(ctx, in_dim, depth, width):
    import torch
    from paper_2602_19699_amd import cbic
    rng = np.random.default_rng(in_dim + 10 * depth)
    for B, out_dim, act in ((1, 1, 0), (15, 16, 1), (17, 5, 2), (65, 3, 0), (60001, 2, 1)):
        g, o = _net(in_dim, width, depth, out_dim, seed=B + depth, act=act)
        x = rng.normal(size=(B, in_dim)).astype(np.float32)
        y = cbic.mlp_forward(ctx, g, torch.as_tensor(x, device="cuda")).cpu().numpy()
        k = np.unique(np.r_[0:min(B, 40), max(0, B - 40):B])
        r = orc.mlp_forward(o, x[k].astype(np.float64))
        assert np.all(np.abs(y[k] - r) <= TOL * (1 + np.abs(r))), (B, out_dim, act)


@pytest.mark.parametrize("depth", [1, 2, 3, 4])
@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("kind", ["pm", "arm", "lq21"])
def test_actor_controls_are_the_networks(ctx, kind, width, depth):
    # every control of a rollout equals, bit for bit, the network's output for
    # that step's state and time (another kernel, the same products in order)
    import torch
    from paper_2602_19699_amd import cbic
    kd, p, n, m, x0 = {"pm": (I.SYS_POINT_MASS, I.point_mass_params(0), 4, 2, I.point_mass_x0(33, 3)),
                       "arm": (I.SYS_PLANAR3, I.planar3_params(0), 6, 3, I.planar3_x0(33, 3)),
                       "lq21": (I.SYS_LQ, I.lq_random(2, 1, 0), 2, 1, I.lq_x0(33, 2))}[kind]
    Tm = 19
    sysm = cbic.System(ctx, kd, p)
    g, _ = _net(n + 1, width, depth, m, seed=depth, act=depth % 3, out_act=1, scale=3.0)
    for B in (1, 16, 33):
        T = I.horizons(B, 1, Tm, seed=B)
        U, X = cbic.actor_rollout(ctx, sysm, g, torch.as_tensor(x0[:B], device="cuda"), Tm,
                                  T=torch.as_tensor(T, device="cuda"), states=True)
        U, X = U.cpu().numpy(), X.cpu().numpy()
        k = np.arange(Tm)[None]
        tau = (Tm - T[:, None] + k).astype(np.float32) * (np.float32(1) / np.float32(Tm))
        rows = np.concatenate([X[:, :Tm].astype(np.float32), tau[..., None]], 2).reshape(-1, n + 1)
        y = cbic.mlp_forward(ctx, g, torch.as_tensor(rows, device="cuda")).cpu().numpy().reshape(B, Tm, m)
        live = (k < T[:, None])[..., None]
        np.testing.assert_array_equal(U, np.where(live, y, 0).astype(np.float64))
    sysm.close()


@pytest.mark.parametrize("Bc,N", [(1, 1), (1023, 1022), (16384, 1), (16384, 16384), (16385, 5000), (18432, 18432),
                                  (18433, 2049), (600001, 3)])
@pytest.mark.parametrize("levels", [0, 3], ids=["distinct", "ties"])
def test_selection_at_path_edges(ctx, Bc, N, levels):
    # one workgroup up to 16384 keys, blocks of 2048 beyond; `levels` states
    # only: long runs of equal scores
    import torch
    from paper_2602_19699_amd import cbic
    g, _ = _net(5, 32, 1, 1, seed=9)
    x, T, Tm = I.bic_candidates("pm16k", Bc, seed=Bc)
    if levels:
        x, T = np.tile(x[:levels], (Bc // levels + 1, 1))[:Bc], np.full(Bc, 7, np.int32)
    s, sel, xs, Ts = cbic.bic_select(ctx, g, torch.as_tensor(x, device="cuda"), torch.as_tensor(T, device="cuda"), Tm, N,
                                     gather=True)
    s, sel, xs, Ts = (v.cpu().numpy() for v in (s, sel, xs, Ts))
    want = np.sort(np.lexsort((np.arange(Bc), -s))[:N])
    np.testing.assert_array_equal(sel, want)
    np.testing.assert_array_equal(xs, x[want])
    np.testing.assert_array_equal(Ts, T[want])
