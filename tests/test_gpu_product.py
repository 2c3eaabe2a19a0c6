"""The products of the density matrices and of the renormalized operators at the
edges of their tiles (32 x 32, a 16 x 16 quarter per wavefront; panels of 32 along the
contraction, two of them on their way) against FP64 NumPy.  Tolerance: (K + 2) u sum |a| |b| for a sum of K
products in any order, u = 2^-53, twice for two products in turn."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.mark.parametrize("rows,cols", [(1, 1), (2, 15), (15, 16), (16, 17), (17, 31), (33, 64), (65, 79), (80, 129)])
@pytest.mark.parametrize("diag", [0, 1])
def test_renormalize_edges(rows, cols, diag):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1309_5571_amd as dm

    print(f"renormalize {rows} x {cols} diag={diag}", flush=True)
    if diag:
        cols = rows
    rng = np.random.default_rng(100 * rows + cols)
    kd, ks = max(1, rows - 1), max(1, (2 * cols) // 3)
    o = rng.standard_normal(rows if diag else rows * cols)
    ud, us = rng.standard_normal((rows, rows)), rng.standard_normal((cols, cols))
    # operands at odd multiples of 8 bytes
    data = torch.from_numpy(np.concatenate([[0.0], o])).cuda()
    u = torch.from_numpy(np.concatenate([[0.0], ud.reshape(-1), us.reshape(-1)])).cuda()
    got = dm.renormalize(data, u, [(1, 1, 1 + rows * rows, 1, rows, cols, kd, ks, diag)], 1 + kd * ks).cpu().numpy()
    O = np.diag(o) if diag else o.reshape(rows, cols)
    ref = ud[:, :kd].T @ O @ us[:, :ks]
    bound = 2 * (rows + cols + 4) * U64 * (np.abs(ud[:, :kd]).T @ np.abs(O) @ np.abs(us[:, :ks]))
    assert np.all(np.abs(got[1:].reshape(kd, ks) - ref) <= bound)
