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

    # from one block to several per row (k of some 6,550 on): a histogram per block and the row, where all of it may be listed
    assert workspace(1000, 20_000, 8000) - workspace(1000, 20_000, 6500) < 1000 * (16 * 2048 * 4 + 20_000 * 8 + 1500 * 4 * 20)
    assert workspace(1000, 40_000, 8000) - workspace(1000, 40_000, 6500) < 1000 * (16 * 2048 * 4 + 1024 * 8 + 1500 * 4 * 20)
    # thirty layers that share launches cost the same beside a layer that is taken apart as without it
    def layered(lengths, fraction):
        t = synth.layer_table(lengths, fraction=fraction)
        return workspace(64, synth.layers_dim(t), 1, layers=t)
    alone, both = layered([300_000], 0.05), layered([300_000] + [11_000] * 30, 0.05)
    lists = 64 * 31 * 32 * (2 * 4 * 15_000 // 32 + 1) * 8     # (every set's candidate lists are as long as the longest)
    assert both - alone < lists + 64 * 30 * 11_000 * 6


def occupancy(keys, T, shift):
    """(least, most) entries that a bin of 2^shift keys around the key T holds, wherever the bins start."""
    w = 1 << shift
    starts = T - np.unique(np.linspace(0, w - 1, 257).astype(np.int64))
    held = np.searchsorted(keys, starts + w) - np.searchsorted(keys, starts)
    return held.min(), held.max()


@pytest.mark.gpu
@pytest.mark.timeout(200)
@pytest.mark.parametrize("d,k,grid,order,reached", [
    (2_300_001, 700_000, 0, B.ORDER_COMPRESS_THEN_MIX, "histogram"),
    (2_300_001, 700_000, 0, B.ORDER_MIX_THEN_COMPRESS, None),
    (2_300_001, 2_299_999, 0, B.ORDER_COMPRESS_THEN_MIX, None),          # the list is the row
    (20_001, 8000, 0, B.ORDER_COMPRESS_THEN_MIX, None),                  # ... and the bins as wide as half an octave
    (600_000, 300_000, 5000, B.ORDER_COMPRESS_THEN_MIX, None),           # about 1,000 entries in the bin
    (2_300_001, 700_000, 5000, B.ORDER_COMPRESS_THEN_MIX, "histogram"),  # a few hundred equal magnitudes in a sub-bin
    (2_300_001, 700_000, 200, B.ORDER_COMPRESS_THEN_MIX, "sub-bin"),     # thousands of them
    (2_300_001, 700_000, 3, B.ORDER_COMPRESS_THEN_MIX, "bin"),           # more than the bin's list has room for
])
def test_crowded_threshold_bin(d, k, grid, order, reached):
    X0 = synth.normal_state(3, d, seed=k)
    if grid:
        X0 = np.round(X0 * grid) / np.float32(grid)
    if grid and d > 2_000_000:
        # the workers alike, so that the mix leaves the grid as it is: the second threshold is 0.5 of a normal
        # deviate, with 2 * 0.35 * 2.3 M / grid entries at it, and a mean bin holds 2,054 to 4,101
        X0[:] = X0[0]
    pair = Pair(X0, synth.ring_csr(3), 0.1, compressor=B.Q_TOPK, k=k, order=order)
    grads = synth.GradientStream(3, d, seed=2)
    want, room = k + k // 2, min(max((k + k // 2) // 32, 1024), 32768)
    before, seen = None, set()
    try:
        for t in range(3):
            G, lr = grads.next(), 0.0 if grid else 0.05
            v = (pair.ref.X - np.float32(lr) * np.float32(G)) - pair.ref.Xhat
            det = pair.step(G, lr)
            pair.check(det, tag="step %d" % t)
            if reached is None:
                continue
            scal = pair.gpu.last_scalars()
            keys = np.sort(v.view(np.uint32) & 0x7FFFFFFF, axis=1).astype(np.int64)
            for i in range(3):
                T, listed = int(scal[i, 0]), int(scal[i, 5])
                if before is not None and scal[i, 3] == 0:
                    # the bins are 256 to 511 between this step's guess and where its threshold was expected
                    kT, klisted, kkeys = before[i]
                    if klisted > k:
                        for G0 in (kkeys[d - klisted], kkeys[max(d - klisted - 1, 0)]):
                            delta = max(1, (kT - int(G0)) * want // (klisted - k))
                            least, most = occupancy(keys[i], T, max(0, delta.bit_length() - 9))
                            ties = np.count_nonzero(keys[i] == T)
                            seen.add("bin" if ties > room else "sub-bin" if 1024 < ties and most <= room
                                     else "histogram" if 1024 < least and most <= room and ties <= 1024 else "other")
            before = [(int(scal[i, 0]), int(scal[i, 5]), keys[i]) for i in range(3)]
        assert reached is None or reached in seen, seen
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(200)
def test_crowded_threshold_bin_random_a():
    """random_a with bins of 2,246 of the uniform keys: 2.3 M entries, bins of 2^22 keys (750,000 entries are wanted
    beyond the kept ones, 0.33 of 2^32 keys, in 256 to 511 bins)."""
    d, k = 2_300_001, 1_500_000
    extra = k // 2
    width = 1 << ((extra << 32) // d).bit_length() - 9
    assert 1024 < d * width >> 32 <= extra // 32
    pair = Pair(synth.normal_state(3, d, seed=3), synth.ring_csr(3), 0.1, compressor=B.Q_RANDK, k=k, seed=11)
    grads = synth.GradientStream(3, d, seed=2)
    try:
        for t in range(4):
            pair.check(pair.step(grads.next(), 0.05), tag="step %d" % t)
        assert np.all(pair.gpu.last_scalars()[:, 3] == 0)
    finally:
        pair.close()
