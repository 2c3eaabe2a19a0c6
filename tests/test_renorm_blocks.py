"""The packed block descriptors of renormalize against one ctypes structure each."""
import numpy as np
import pytest

import paper_1309_5571_amd as dm
from paper_1309_5571_amd import _native as N


@pytest.mark.parametrize("blocks", [
    [],
    [(1, 2, 3, 4, 5, 6, 7, 8, 1)],
    [tuple(np.int64(v) for v in (2 ** 40, 0, 1, -1, 5, 6, 7, 8, 0)), [9, 8, 7, 6, 5, 4, 3, 2, 1]],
    [(1.9, 2, 3, 4, 5, 6, 7, 8, True)],  # truncated as int() does
    [(1, 2, 3, 4, 5, 6, 7, 8)],  # diag left out: 0
    [(1, 2, 3, 4, 2 ** 32 + 5, 6, 7, 8, 0), (2 ** 63, 2, 3, 4, 5, 6, 7, 8, 0)],  # wrapped as ctypes does
], ids=["none", "one", "numpy", "float", "short", "wide"])
def test_packed_blocks(blocks):
    ref = (N.RenormBlock * max(len(blocks), 1))()
    for i, b in enumerate(blocks):
        ref[i] = N.RenormBlock(*[int(v) for v in b])
    assert bytes(dm._renorm_blocks(blocks)) == bytes(ref)


@pytest.mark.parametrize("block", [(1, 2, 3, 4, 5, 6, 7, 8, 1), (1, 2, 3, 4, 5, 6, 7, 8),
                                   (1, 2, 3, 4, 2 ** 32 + 5, 6, 7, 8, 0)], ids=["whole", "short", "wide"])
def test_fields_from_an_iterator(block):
    """A block's fields may come from an iterator, read once whichever way it is packed."""
    ref = (N.RenormBlock * 1)(N.RenormBlock(*block))
    assert bytes(dm._renorm_blocks([iter(block)])) == bytes(ref)


def test_generator_of_blocks_is_refused():
    with pytest.raises(TypeError):
        dm.renormalize(None, None, (b for b in [(1, 2, 3, 4, 5, 6, 7, 8, 1)]), 1)
