"""Tile tables whose small blocks get the larger tiles: legal (bounds ascend, tiles
are 16 or 32 in any order), and every block of a plan can then have 16 x 16 tiles
while an intermediate of a two-sided term falls into the class of 32 x 32 ones.

Tolerance: a sum of FP64 products, at most a few hundred terms of comparable size:
normwise K u ~ 1e-13, so 1e-12 as for every FP64 projection."""
import numpy as np
import pytest

from gen.workloads import Operator, Problem, Space
from oracle import projection

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("a,b", [(18, 70), (17, 65), (20, 96)])
def test_intermediates_of_the_wider_class(a, b):
    """Blocks a x b and b x a under (20 -> 32, else 16): the two-sided term from
    one to the other takes X B^T of a x a (b above 64: not fused)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1309_5571_amd as dm

    print(f"tile table {a} x {b}", flush=True)
    rng = np.random.default_rng(a)
    L, R = Space([[0], [1]], [a, b]), Space([[-1], [0]], [a, b])

    def shift(sp, src, dst):
        return Operator("dense", src=[src], dst=[dst], blocks=[rng.standard_normal((sp.dims[dst], sp.dims[src]))])

    p = Problem(L, R, [0], [shift(L, 0, 1), shift(L, 1, 0)], [shift(R, 1, 0), shift(R, 0, 1)], [(0, 0), (1, 1)],
                rng.standard_normal(2))
    plan = dm.Plan(p, tiles=((20, 1 << 30), (32, 16)))
    dev = lambda x: torch.from_numpy(x).cuda()
    X, g = rng.standard_normal((5, plan.n)), rng.standard_normal(plan.n)
    ref = [projection.project_sectors(p, x) for x in X]
    close = lambda got, want: np.linalg.norm(got - want) <= 1e-12 * np.linalg.norm(want)
    assert close(plan.project_raw(dev(X[0])).cpu().numpy(), ref[0])
    Y = plan.project_block(dev(X)).cpu().numpy()  # four vectors in one launch, then one
    assert all(close(y, r) for y, r in zip(Y, ref))
    gpsi, gcoef = (t.cpu().numpy() for t in plan.backward_raw(dev(X[0]), dev(g)))
    assert close(gpsi, projection.project_adjoint_sectors(p, g))
    assert close(gcoef, projection.coef_gradient(p, X[0], g))


def test_mixed_batch():
    """One large member and many small ones: more than 320 tiles of 64 x 64 by their
    number, but the work of far fewer (the plan keeps the smaller tiles); every member
    against its own oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gen
    import paper_1309_5571_amd as dm

    probs = [gen.heisenberg_synthetic(m, seed=600 + m) for m in range(32, 62)] + [gen.heisenberg_synthetic(700, seed=9)]
    plan = dm.Plan(probs, tiles=None)
    x = np.random.default_rng(4).standard_normal(plan.n)
    y = plan.project_raw(torch.from_numpy(x).cuda()).cpu().numpy()
    mo = plan.member_off
    for i, p in enumerate(probs):
        ref = projection.project_sectors(p, x[mo[i]:mo[i + 1]])
        assert np.linalg.norm(y[mo[i]:mo[i + 1]] - ref) <= 1e-12 * np.linalg.norm(ref), i
