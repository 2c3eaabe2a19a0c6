"""Many blocks in one call: those of order up to 8 share workgroups (by a wavefront
each, in groups that depend on the number of blocks, 256 the last one without), and the
output's grid has fewer panels than a block's columns need.  Orders mixed so
that a group holds some, one or none of them.  Tolerances as in the tests of the
eigen-decomposition: 16 d u |A|_F."""
import numpy as np
import pytest
import torch

from test_gpu_eigh import _check, _run, _sym

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5, 256, 257, 770, 3400])
@pytest.mark.parametrize("kind", ["small", "mixed"])
def test_many_blocks(n, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"{n} {kind} blocks", flush=True)
    rng = np.random.default_rng(n)
    if kind == "small":
        orders = rng.integers(1, 9, n)
    else:  # runs of larger blocks among small ones, and one of several panels
        orders = np.where(np.arange(n) // 6 % 3 == 1, rng.integers(9, 13, n), rng.integers(1, 10, n))
        orders[n // 2] = 150
    blocks = [_sym(rng, int(d)) for d in orders]
    res, info = _run(blocks)
    assert np.all(info >= 0)
    _check(blocks, res)
