"""Tall-skinny products at the edges of their split: two rows a thread, 512 a
block, columns in groups of four (the columns past k are read but not used)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 19, 63, 64])
@pytest.mark.parametrize("n", [1, 2, 3, 511, 512, 513, 1025, 600_001])
def test_rows_and_columns(n, k):
    import paper_1309_5571_amd as dm

    print(f"gemv edges n={n} k={k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1000 * k + n % 997)
    # the columns start at odd multiples of 8 bytes, k + 1 columns are there
    # and the one after the last is not a number
    buf = torch.randn((k + 1) * (n + 2) + 1, dtype=torch.float64, device="cuda", generator=g)
    V = buf[1:].view(k + 1, n + 2)[:, :n]
    V[k] = float("nan")
    V[k - 1, n - 1] = float("inf")  # a value of the last column that must not reach the others
    x = torch.randn(n + 1, dtype=torch.float64, device="cuda", generator=g)[1:]
    s = dm.gemv_t(V[:k], x)
    Vh, xh = V[:k].cpu().numpy(), x.cpu().numpy()
    got = s.cpu().numpy()
    assert got[k - 1] == np.copysign(np.inf, xh[n - 1])
    # any order of n products and n - 1 additions: n u sum |V| |x|, u = 2^-53
    assert np.all(np.abs(got[:-1] - Vh[:-1] @ xh) <= n * 2.0 ** -53 * (np.abs(Vh[:-1]) @ np.abs(xh)))

    c = torch.randn(k, dtype=torch.float64, device="cuda", generator=g)
    y0 = torch.randn(n + 1, dtype=torch.float64, device="cuda", generator=g)[1:]
    ch, yh = c.cpu().numpy(), y0.cpu().numpy()
    for beta in (0.0, 1.5):
        y = torch.full_like(y0, float("nan")) if beta == 0.0 else y0.clone()
        dm.gemv_n(V[:k], c, y, beta=beta)
        got = y.cpu().numpy()
        assert got[n - 1] == np.copysign(np.inf, ch[k - 1])
        ref = (beta * yh if beta else 0.0) + ch @ np.where(np.isinf(Vh), 0.0, Vh)
        bound = (k + 2) * 2.0 ** -53 * (beta * np.abs(yh) + np.abs(ch) @ np.where(np.isinf(Vh), 0.0, np.abs(Vh)))
        assert np.all(np.abs(got - ref)[:-1] <= bound[:-1])
