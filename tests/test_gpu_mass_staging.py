"""The mass before and after a labelling (which leaves the handle pinned memory
that the masses then come back through), and of a batch with more boxes than
that memory holds: the same bits, and the sum of the field."""
import numpy as np
import pytest
import torch

from paper_2105_01865_amd import ch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbox", [1, 3, 1025, 1026])
def test_masses_are_the_same_after_a_labelling(nbox):
    rng = np.random.default_rng(nbox)
    C = rng.random((nbox, 8, 8, 9))
    b = ch.Batch([(8, 8, 9)] * nbox, [0.125] * nbox, [0.1] * nbox, [5.0] * nbox,
                 stream=torch.cuda.Stream())
    b.set_field(b.pack(list(C), "c"))
    before = b.mass()
    root, cells = b.drops(nbox - 1)
    assert cells.sum() == (C[-1] >= 0.5).sum()
    after = b.mass()
    b.close()
    assert before == after
    # 576 values in double: sums of either order agree to 576 eps
    want = C.reshape(nbox, -1).sum(1) * 0.125 ** 3
    assert np.abs(np.array(after) - want).max() <= 576 * 2.3e-16 * want.max()
