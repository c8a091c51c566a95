"""top_a with so many kept entries that the threshold's bin is taken apart by a histogram of its own
(more than 1,024 entries), or, where most of them are equal, digit by digit."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding as B
from paper_1907_09356_amd import synth
from tests.parity_util import Pair


def test_room_for_the_bin():
    """... is kept for as many entries as the bin is likely to hold, and for rows and layers that take it apart only."""
    def workspace(n, d, k, **kw):
        cfg, keep = B.make_config(n, d, *synth.ring_csr(n), 0.1, B.Q_TOPK, k=k, **kw)
        return B.workspace_bytes(cfg)

    # from one block to several per row (k of some 6,550 on): a histogram per block and 1,024 entries
    assert workspace(1000, 20_000, 8000) - workspace(1000, 20_000, 6500) < 1000 * (16 * 2048 * 4 + 1024 * 8 + 1500 * 4 * 20)
    # thirty layers that share launches cost the same beside a layer that is taken apart as without it
    def layered(lengths, fraction):
        t = synth.layer_table(lengths, fraction=fraction)
        return workspace(64, synth.layers_dim(t), 1, layers=t)
    alone, both = layered([300_000], 0.05), layered([300_000] + [11_000] * 30, 0.05)
    lists = 64 * 31 * 32 * (2 * 4 * 15_000 // 32 + 1) * 8     # (every set's candidate lists are as long as the longest)
    assert both - alone < lists + 64 * 30 * 11_000 * 6


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
