"""Calls on one context are ordered one after the other also when they are given
different streams, whatever path a call takes."""
import numpy as np
import pytest

from paper_2602_19699_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2602_19699_amd import cbic
    assert torch.cuda.is_available()
    c = cbic.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("B", [100, 200], ids=["one_workgroup", "whole_chip"])
def test_selection_waits_for_the_solve_before_it(ctx, B):
    # the candidates are the states that a solve on another stream, some
    # milliseconds long, is still to write
    import torch
    from paper_2602_19699_amd import cbic
    T = 100
    sysm = cbic.System(ctx, I.SYS_PLANAR3, I.planar3_params(0))
    g = cbic.Mlp(6, 64, 2, 1, torch.as_tensor(I.mlp_params(6, 64, 2, 1, seed=3), device="cuda"))
    x0 = torch.as_tensor(I.planar3_x0(B, 4), device="cuda")
    out = cbic.Outputs.allocate(B, T, 6, 3, x0.device)
    out.X.zero_()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    cbic.solve_batch(ctx, sysm, x0, T, opts=cbic.Options(max_iter=30), out=out, stream=s1.cuda_stream)
    score, sel, xs, _ = cbic.bic_select(ctx, g, out.X.view(-1, 6), None, 0, 50, gather=True, stream=s2.cuda_stream)
    torch.cuda.synchronize()
    want = cbic.bic_select(ctx, g, out.X.view(-1, 6), None, 0, 50, gather=True)
    torch.cuda.synchronize()
    for a, b in zip((score, sel, xs), want):
        assert torch.equal(a, b)
    sysm.close()


@pytest.mark.parametrize("Bc", [3000, 20000], ids=["one_workgroup", "whole_chip"])
def test_solve_waits_for_the_selection_before_it(ctx, Bc):
    # the selection starts only when its stream's earlier work, some
    # milliseconds, has ended; the solve on another stream takes its states
    import torch
    from paper_2602_19699_amd import cbic
    N, Tm = 64, 20
    x, T, _ = I.bic_candidates("pm16k", Bc)
    x, T = torch.as_tensor(x, device="cuda"), torch.as_tensor(np.minimum(T, Tm).astype(np.int32), device="cuda")
    sysm = cbic.System(ctx, I.SYS_POINT_MASS, I.point_mass_params(0))
    g = cbic.Mlp(5, 64, 2, 1, torch.as_tensor(I.mlp_params(5, 64, 2, 1, seed=5), device="cuda"))
    o = cbic.Options(max_iter=5)
    ref = cbic.bic_select(ctx, g, x, T, Tm, N, gather=True)
    want = cbic.solve_batch(ctx, sysm, ref[2], Tm, T=ref[3], opts=o)
    torch.cuda.synchronize()
    # the caching allocator hands the next outputs fresh memory that holds neither
    hold = [torch.zeros_like(v) for v in ref]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s1):
        for _ in range(20):
            a = torch.tanh(a @ a)
    got = cbic.bic_select(ctx, g, x, T, Tm, N, gather=True, stream=s1.cuda_stream)
    out = cbic.solve_batch(ctx, sysm, got[2], Tm, T=got[3], opts=o, stream=s2.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(got[1], ref[1]) and len(hold) == 4
    for k in ("X", "U", "J", "iters", "status"):
        assert torch.equal(getattr(out, k), getattr(want, k)), k
    sysm.close()


def test_captured_selection_stands_alone(ctx):
    # a selection of one workgroup can be captured on a stream of its own though
    # the context's previous call ran on another, and later calls do not wait on it
    import torch
    from paper_2602_19699_amd import cbic
    N, Tm = 64, 100
    x, T, _ = I.bic_candidates("pm16k", 3000)
    x, T = torch.as_tensor(x, device="cuda"), torch.as_tensor(T, device="cuda")
    g = cbic.Mlp(5, 64, 2, 1, torch.as_tensor(I.mlp_params(5, 64, 2, 1, seed=5), device="cuda"))
    want = cbic.bic_select(ctx, g, x, T, Tm, N, gather=True)
    torch.cuda.synchronize()
    graph, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=s):
        got = cbic.bic_select(ctx, g, x, T, Tm, N, gather=True)
    for _ in range(3):
        graph.replay()
        again = cbic.bic_select(ctx, g, x, T, Tm, N, gather=True)
        torch.cuda.synchronize()
        for a, b, c in zip(got, want, again):
            assert torch.equal(a, b) and torch.equal(c, b)


def test_many_selections_and_solves_over_three_streams(ctx):
    # one chain of calls, each on the next stream: a selection from the states of
    # the solve before it, a solve from the states selected, and so on
    import torch
    from paper_2602_19699_amd import cbic
    N, Tm = 96, 12
    sysm = cbic.System(ctx, I.SYS_POINT_MASS, I.point_mass_params(0))
    g = cbic.Mlp(4, 32, 2, 1, torch.as_tensor(I.mlp_params(4, 32, 2, 1, seed=7), device="cuda"))
    x0 = torch.as_tensor(I.point_mass_x0(N, 8), device="cuda")
    o = cbic.Options(max_iter=4)

    def chain(streams):
        xs, outs = x0, []
        for k in range(12):
            s = [streams[(2 * k + i) % len(streams)].cuda_stream for i in range(2)]
            out = cbic.solve_batch(ctx, sysm, xs, Tm, opts=o, stream=s[0])
            _, _, xs, _ = cbic.bic_select(ctx, g, out.X.view(-1, 4), None, 0, N, gather=True, stream=s[1])
            outs += [out.J, xs, out]
        torch.cuda.synchronize()
        return [v for v in outs if torch.is_tensor(v)]

    one = chain([torch.cuda.Stream()])
    for _ in range(3):
        for a, b in zip(one, chain([torch.cuda.Stream() for _ in range(3)])):
            assert torch.equal(a, b)
    sysm.close()
