"""Adjoint and coefficient gradient, above all of plans whose tiles are all 16 x 16: block
orders around 1, 4, 16, 36 (one piece of a contraction) and 64 (widest intermediate
that is fused), copy segments, tiles without a segment, more segments than the
packed descriptors, and the outputs each asked for alone.

Tolerance: sums of FP64 products, at most a few hundred terms of comparable size:
normwise K u ~ 1e-13, so 1e-12 as for every FP64 projection."""
import numpy as np
import pytest

import gen
from gen.workloads import Operator, Problem, Space
from oracle import l11r, projection

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = [(1, 2, 15), (16, 17, 31), (4, 36, 37), (48, 63, 64), (65, 1, 40), (3, 5, 70), (33, 66, 16)]
A16 = ((1 << 30,), (16,))


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _problem(ldims, rdims, seed, copies=1):
    """Operators that keep and shift the label, diagonal factors, identities;
    `copies` of the terms with coefficients of their own."""
    rng = np.random.default_rng(seed)
    L, R = Space([[-1], [0], [1]], ldims), Space([[-1], [0], [1]], rdims)

    def ops(sp):
        def dense(shift):
            pairs = [(s, s + shift) for s in range(3) if 0 <= s + shift < 3]
            return Operator("dense", src=[a for a, _ in pairs], dst=[b for _, b in pairs],
                            blocks=[rng.standard_normal((sp.dims[b], sp.dims[a])) for a, b in pairs])
        return [Operator("identity"), dense(0), dense(1), dense(-1), Operator("diag", diag=rng.standard_normal(sp.m))]

    terms = [(1, 0), (0, 1), (2, 3), (3, 2), (1, 4), (4, 1), (4, 4), (1, 1)] * copies
    return Problem(L, R, [0], ops(L), ops(R), terms, rng.standard_normal(len(terms)))


def _check(dm, p, plan, seed, adjoint, gradient):
    rng = np.random.default_rng(seed)
    psi, g = rng.standard_normal(plan.n), rng.standard_normal(plan.n)
    dpsi, dg = torch.from_numpy(psi).cuda(), torch.from_numpy(g).cuda()
    gpsi, gcoef = plan.backward_raw(dpsi, dg)
    alone, _ = plan.backward_raw(dpsi, dg, want_coef=False)
    _, coef_alone = plan.backward_raw(dpsi, dg, want_psi=False)
    assert torch.equal(gpsi, alone) and torch.equal(gcoef, coef_alone)
    ref = adjoint(p, g)
    assert np.linalg.norm(gpsi.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
    ref = gradient(p, psi, g)
    assert np.max(np.abs(gcoef.cpu().numpy() - ref)) <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("copies", [1, 3])
@pytest.mark.parametrize("e", range(len(EDGES)))
def test_edges(e, copies):
    import paper_1309_5571_amd as dm

    print(f"fused adjoint {EDGES[e]} x {EDGES[-1 - e]} copies={copies}", flush=True)
    p = _problem(EDGES[e], EDGES[-1 - e], 60 + e, copies)
    if e == 0 and copies == 1:  # only diagonal terms reach some of the tiles
        p.terms, p.coef = p.terms[[2, 6]], p.coef[[2, 6]]
    _check(dm, p, dm.Plan(p, tiles=A16), e, projection.project_adjoint_sectors, projection.coef_gradient)


@pytest.mark.parametrize("tile", [16, 32])
def test_copies_and_gradient_in_place(tile):
    """Copy segments and long segment lists (a four-subsystem superblock), against the
    adjoint and the gradient of its bilinear form; then gpsi written over psi itself."""
    import paper_1309_5571_amd as dm

    p = gen.hubbard_l11r_synthetic(128, seed=6)
    plan = dm.Plan(p, tiles=((1 << 30,), (tile,)))

    one = np.eye(len(p.coef))
    gradient = lambda p, psi, g: np.array([g @ l11r.project_sectors(p, psi, coef=c) for c in one])
    _check(dm, p, plan, 9, lambda p, g: projection.project_adjoint_sectors(l11r.to_lr(p), g), gradient)
    rng = np.random.default_rng(10)
    psi, g = (torch.from_numpy(rng.standard_normal(plan.n)).cuda() for _ in range(2))
    gpsi, gcoef = plan.backward_raw(psi, g)
    over, coef = psi.clone(), torch.empty_like(gcoef)
    ptr = lambda t: t.data_ptr()
    dm.N.check(dm.N.lib().dmrg_project_backward(plan._h, ptr(plan.coef), ptr(over), ptr(g), ptr(over), ptr(coef),
                                                torch.cuda.current_stream().cuda_stream))
    assert torch.equal(over, gpsi) and torch.equal(coef, gcoef)
