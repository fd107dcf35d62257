"""Network calls at the largest sizes that a 32-bit count takes: tile and block
numbers must not wrap."""
import numpy as np
import pytest

from paper_2602_19699_amd import inputs as I

pytestmark = pytest.mark.gpu

MOST = 2**31 - 1


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2602_19699_amd import cbic
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of free device memory")
    c = cbic.Context(0)
    yield c
    c.close()
    torch.cuda.empty_cache()


def test_forward_of_the_most_rows(ctx):
    # a wave's next tile lies past 2^31 rows for the last waves of the grid
    import torch
    from paper_2602_19699_amd import cbic
    g = cbic.Mlp(5, 32, 1, 1, torch.as_tensor(I.mlp_params(5, 32, 1, 1, seed=3), device="cuda"))
    x = torch.zeros((MOST, 5), device="cuda")
    x[-1000:] = torch.as_tensor(np.random.default_rng(1).normal(size=(1000, 5)).astype(np.float32))
    print("forward", x.shape, flush=True)
    y = cbic.mlp_forward(ctx, g, x)
    assert torch.equal(y[-1000:], cbic.mlp_forward(ctx, g, x[-1000:]))
    zero = cbic.mlp_forward(ctx, g, x[:1])
    assert bool((y[:-1000] == zero).all())


def test_selection_from_the_most_candidates(ctx):
    import torch
    from paper_2602_19699_amd import cbic
    torch.cuda.empty_cache()
    g = cbic.Mlp(5, 32, 1, 1, torch.as_tensor(I.mlp_params(5, 32, 1, 1, seed=4), device="cuda"))
    x = torch.zeros((MOST, 4), dtype=torch.float64, device="cuda")
    T = torch.full((MOST,), 7, dtype=torch.int32, device="cuda")
    at = np.array([5, MOST // 2, MOST - 3, MOST - 1])
    for i, v in zip(at, np.random.default_rng(2).normal(size=(4, 4))):
        x[int(i)] = torch.as_tensor(v, device="cuda")
    rows = np.r_[0, 1, 2, at]  # more of the equal ones than are selected, and the others
    few, _ = cbic.bic_select(ctx, g, torch.stack([x[int(i)] for i in rows]), T[:7], 9, 0)
    want = np.sort(rows[np.lexsort((rows, -few.cpu().numpy()))[:3]])
    print("select", x.shape, flush=True)
    s, sel = cbic.bic_select(ctx, g, x, T, 9, 3)
    assert torch.equal(torch.stack([s[int(i)] for i in rows]), few)
    np.testing.assert_array_equal(sel.cpu().numpy(), want)
