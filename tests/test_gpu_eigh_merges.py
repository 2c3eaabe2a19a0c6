"""The reduction at the edges of its rows (60, 120 and 180 by four, eight and
twelve rows a wavefront) and the merges of the divide and conquer at those of
their teams and tiles
(16 roots a panel, 96 or 64 rows a group; two panels a wavefront above order
256), for spectra that deflate in different ways.  Tolerances as in the tests of
the eigen-decomposition: 16 d u |A|_F."""
import numpy as np
import pytest
import torch

from test_gpu_eigh import _check, _run, _sym

pytestmark = pytest.mark.gpu


def _blocks(d, rng):
    q = np.linalg.qr(rng.standard_normal((d, d)))[0]
    clustered = (q * rng.integers(0, 3, d)) @ q.T  # three eigenvalues: chains of rotations
    decaying = (q * np.exp(-0.7 * np.arange(d))) @ q.T  # most weights negligible
    t = np.diag(rng.standard_normal(d)) + np.diag(np.where(rng.random(d - 1) < 0.3, 0.0, rng.standard_normal(d - 1)), 1)
    split = t + np.triu(t, 1).T  # tears without coupling
    glued = np.kron(np.eye((d + 8) // 9), _sym(rng, 9))[:d, :d]  # equal halves: pairs of equal poles
    return [_sym(rng, d), (clustered + clustered.T) / 2, (decaying + decaying.T) / 2, split, (glued + glued.T) / 2]


@pytest.mark.parametrize("d", [9, 15, 16, 17, 31, 33, 60, 61, 63, 65, 95, 97, 120, 121, 127, 179, 180, 181, 191,
                               193, 255, 256, 257, 289, 511])
def test_merge_edges(d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"merges of order {d}", flush=True)
    blocks = _blocks(d, np.random.default_rng(d))
    res, info = _run(blocks)
    assert np.all(info >= 1)
    _check(blocks, res)
