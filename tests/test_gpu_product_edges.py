"""The products of the density matrices and of the renormalized operators at the
edges of their 32 x 32 tiles and of the panels of 32 along the contraction, against
FP64 NumPy.  Tolerance: (K + 2) u sum |a| |b| for a sum of K products in any order,
u = 2^-53, twice for two products in turn."""
import numpy as np
import pytest
import torch

from gen.workloads import Operator, Problem, Space

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("rows,cols", [(31, 32), (32, 33), (33, 31), (63, 64), (64, 65), (65, 97), (97, 63)])
def test_renormalize(rows, cols):
    import paper_1309_5571_amd as dm

    print(f"renormalize {rows} x {cols}", flush=True)
    rng = np.random.default_rng(100 * rows + cols)
    o, ud, us = (rng.standard_normal(s) for s in ((rows, cols), (rows, rows), (cols, cols)))
    dev = lambda *x: torch.from_numpy(np.concatenate([v.reshape(-1) for v in x])).cuda()
    got = dm.renormalize(dev(o), dev(ud, us), [(0, 0, rows * rows, 0, rows, cols, rows, cols, 0)], rows * cols)
    bound = 2 * (rows + cols + 4) * U64 * (np.abs(ud).T @ np.abs(o) @ np.abs(us))
    assert np.all(np.abs(got.cpu().numpy().reshape(rows, cols) - ud.T @ o @ us) <= bound)


@pytest.mark.parametrize("dl,dr", [(31, 32), (32, 33), (33, 31), (63, 64), (64, 65), (65, 97), (97, 63)])
def test_density(dl, dr):
    import paper_1309_5571_amd as dm

    print(f"density {dl} x {dr}", flush=True)
    rng = np.random.default_rng(100 * dl + dr)
    L, R = Space([[0]], [dl]), Space([[0]], [dr])
    p = Problem(L, R, [0], [Operator("identity")], [Operator("identity")], [(0, 0)], [1.0])
    x = rng.standard_normal((dl, dr))
    left, right = dm.Plan(p).density(torch.from_numpy(x.reshape(-1)).cuda())
    for got, a in ((left, x), (right, x.T)):
        n, k = a.shape
        bound = (k + 2) * U64 * (np.abs(a) @ np.abs(a).T)
        assert np.all(np.abs(got.cpu().numpy().reshape(n, n) - a @ a.T) <= bound)
