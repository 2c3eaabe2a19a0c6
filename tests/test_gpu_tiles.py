"""The FP64 tile kernels (32 x 32 tiles with the contraction split, 64 x 64 tiles
through LDS) at the edges of their tiles and contraction windows: block orders
around 1, 16, 32 and 64, odd and even, every operand layout (forward and
adjoint), one superblock and enough of them for the 64 x 64 tiles.

Tolerance: every output is a sum of products in FP64; with at most a few
hundred terms of comparable size the normwise error of either order of
summation is below K u ~ 1e-13, so 1e-12 as for every FP64 projection.
"""
import numpy as np
import pytest

import gen
from gen.workloads import Operator, Problem, Space
from oracle import projection

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = [(1, 2, 15), (16, 17, 31), (32, 33, 47), (48, 63, 64), (65, 96, 129), (1, 64, 127), (95, 16, 1), (191, 3, 70)]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()


def _problem(ldims, rdims, seed):
    """Three sectors a side, target 0: dense operators that keep and shift the
    label, diagonal factors on either side of a dense one, and identities."""
    rng = np.random.default_rng(seed)
    L, R = Space([[-1], [0], [1]], ldims), Space([[-1], [0], [1]], rdims)

    def ops(sp):
        def dense(shift):
            pairs = [(s, s + shift) for s in range(3) if 0 <= s + shift < 3]
            return Operator("dense", src=[a for a, _ in pairs], dst=[b for _, b in pairs],
                            blocks=[rng.standard_normal((sp.dims[b], sp.dims[a])) for a, b in pairs])
        return [Operator("identity"), dense(0), dense(1), dense(-1), Operator("diag", diag=rng.standard_normal(sp.m))]

    terms = [(1, 0), (0, 1), (2, 3), (3, 2), (1, 4), (4, 1), (4, 4), (1, 1)]
    return Problem(L, R, [0], ops(L), ops(R), terms, rng.standard_normal(len(terms)))


def _tiles64(probs):
    up = lambda d: (int(d) + 63) // 64
    return sum(up(p.left.dims[a]) * up(p.right.dims[b]) for p in probs for a in range(p.left.nsec)
               for b in range(p.right.nsec) if p.left.labels[a, 0] + p.right.labels[b, 0] == 0)


def _check(plan, probs, psi, g):
    y = plan.project_raw(_dev(psi)).cpu().numpy()
    gpsi, gcoef = (t.cpu().numpy() for t in plan.backward_raw(_dev(psi), _dev(g)))
    only_psi, _ = plan.backward_raw(_dev(psi), _dev(g), want_coef=False)
    _, only_coef = plan.backward_raw(_dev(psi), _dev(g), want_psi=False)
    assert np.array_equal(only_psi.cpu().numpy(), gpsi) and np.array_equal(only_coef.cpu().numpy(), gcoef)
    mo, t = plan.member_off, 0
    for i, p in enumerate(probs):
        s = slice(mo[i], mo[i + 1])
        ref = projection.project_sectors(p, psi[s])
        assert np.linalg.norm(y[s] - ref) <= 1e-12 * np.linalg.norm(ref), i
        ref = projection.project_adjoint_sectors(p, g[s])
        assert np.linalg.norm(gpsi[s] - ref) <= 1e-12 * np.linalg.norm(ref), i
        ref = projection.coef_gradient(p, psi[s], g[s])
        assert np.max(np.abs(gcoef[t:t + len(ref)] - ref)) <= 1e-12 * np.abs(ref).max(), i
        t += len(ref)


@pytest.mark.parametrize("e", range(len(EDGES)))
def test_tiles32_edges(e):
    import paper_1309_5571_amd as dm

    p = _problem(EDGES[e], EDGES[-1 - e], 10 + e)
    plan = dm.Plan(p, tiles=((1 << 30,), (32,)))
    rng = np.random.default_rng(e)
    _check(plan, [p], rng.standard_normal(plan.n), rng.standard_normal(plan.n))


@pytest.mark.parametrize("dfold", [False, True])
def test_tiles64_edges(dfold):
    """All edge shapes in one plan of more than 320 tiles of 64 x 64; inside
    Davidson the kernel takes the folded diagonal and leaves Rayleigh rows
    (checked through the converged energies)."""
    import paper_1309_5571_amd as dm
    from oracle import davidson as odav

    if not dfold:
        probs = [_problem(a, b, 100 + 10 * i + j) for i, a in enumerate(EDGES) for j, b in enumerate(EDGES)]
        assert _tiles64(probs) >= 320
        plan = dm.Plan(probs, tiles=None)
        rng = np.random.default_rng(1)
        _check(plan, probs, rng.standard_normal(plan.n), rng.standard_normal(plan.n))
        return
    probs = [gen.heisenberg_synthetic(m, seed=50 + m) for m in range(300, 480, 6)]
    assert _tiles64(probs) >= 320
    plan = dm.Plan(probs, tiles=None)
    x0 = np.random.default_rng(2).standard_normal(plan.n)
    _, E, info, st = plan.davidson(_dev(x0), tol=1e-10)
    assert st == 0
    mo = plan.member_off
    for i in (0, 7, 19):
        ref = odav.ground_state_davidson(probs[i], x0[mo[i]:mo[i + 1]], tol=1e-10)
        assert abs(E[i] - ref.energy) <= 1e-10, i


def test_many_segments_and_copies():
    """Tiles whose descriptor list is longer than the staged window, and copy
    segments (the site factors of a four-subsystem superblock)."""
    import paper_1309_5571_amd as dm
    from oracle import l11r

    p = gen.hubbard_l11r_synthetic(128, seed=5)
    plan = dm.Plan(p, tiles=((1 << 30,), (32,)))
    psi = np.random.default_rng(3).standard_normal(plan.n)
    y = plan.project_raw(_dev(psi)).cpu().numpy()
    ref = l11r.project_sectors(p, psi)
    assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("e", range(len(EDGES)))
def test_fused_edges(e, prec):
    """16 x 16 tiles: contractions and intermediates around 16, 36 and 64 (one
    piece, several pieces, two stages), with packed descriptors and tiles
    without a segment.  FP32 against the accumulation envelope K 2^-24 + 6 u
    of the exact product magnitudes."""
    import paper_1309_5571_amd as dm
    from oracle import precision

    p = _problem(EDGES[e], EDGES[-1 - e], 30 + e)
    if e == 0:  # only diagonal terms reach some of the tiles
        p.terms, p.coef = p.terms[[2, 6]], p.coef[[2, 6]]
    plan = dm.Plan(p, prec=prec, tiles=((1 << 30,), (16,)))
    psi = np.random.default_rng(e).standard_normal(plan.n)
    y = plan.project_raw(_dev(psi), prec=prec).cpu().numpy()
    ref = projection.project_sectors(p, psi)
    if prec == "f64":
        assert np.linalg.norm(y - ref) <= 1e-12 * np.linalg.norm(ref)
    else:
        env = (precision.max_contraction(p) + 6) * 2.0 ** -24 * np.linalg.norm(precision.project_magnitude(p, psi))
        assert np.linalg.norm(y - ref) <= env
