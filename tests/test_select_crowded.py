"""top_a with so many kept entries that the threshold's bin is taken apart by a histogram of its own
(more than 1,024 entries), or, where most of them are equal, digit by digit."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding as B
from paper_1907_09356_amd import synth
from tests.parity_util import Pair


@pytest.mark.gpu
@pytest.mark.timeout(200)
@pytest.mark.parametrize("d,k,grid,order", [
    (2_300_001, 700_000, 0, B.ORDER_COMPRESS_THEN_MIX),       # 2,000 to 4,000 entries in the bin
    (2_300_001, 700_000, 0, B.ORDER_MIX_THEN_COMPRESS),
    (2_300_001, 2_299_999, 0, B.ORDER_COMPRESS_THEN_MIX),     # the list is the row
    (600_000, 300_000, 5000, B.ORDER_COMPRESS_THEN_MIX),      # a few hundred equal magnitudes in a sub-bin
    (2_300_001, 700_000, 200, B.ORDER_COMPRESS_THEN_MIX),     # thousands of them
])
def test_crowded_threshold_bin(d, k, grid, order):
    X0 = synth.normal_state(3, d, seed=k)
    if grid:
        X0 = np.round(X0 * grid) / np.float32(grid)
    pair = Pair(X0, synth.ring_csr(3), 0.1, compressor=B.Q_TOPK, k=k, order=order)
    grads = synth.GradientStream(3, d, seed=2)
    try:
        for t in range(3):
            det = pair.step(grads.next(), 0.0 if grid else 0.05)
            pair.check(det, tag="step %d" % t)
    finally:
        pair.close()
