"""GPU parity of the mix's tile shapes at the edges of their ranges: worker counts at which the
workgroup shape changes, columns around the end of a tile, rows of W beyond what a tile stages."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding as B
from paper_1907_09356_amd import synth
from tests.parity_util import Pair

pytestmark = pytest.mark.gpu


def walk(n, d, topo, comp, steps=3, momentum=False, ld_align=32, **kw):
    """A few fused iterations, the state compared bit for bit after each."""
    pair = Pair(synth.normal_state(n, d, seed=n + d), topo, 0.2, comp, seed=5, ld_align=ld_align, **kw)
    grads = synth.GradientStream(n, d, seed=n)
    for t in range(steps):
        g = grads.next()
        det = pair.step_momentum(g, 0.1, 0.9, 1e-3) if momentum else pair.step(g, 0.1)
        pair.check(det, tag="n=%d d=%d step %d" % (n, d, t))
    pair.close()


@pytest.mark.parametrize("n", [9, 12, 13, 16, 17, 20, 21, 24, 25, 32, 33, 40, 41, 48, 49, 64])
@pytest.mark.parametrize("comp", [B.Q_TOPK, B.Q_RANDK])
def test_narrow_tile_by_number_of_workers(n, comp):
    d = 64 * 9 + (n * 7) % 64           # the last tile is cut anywhere
    walk(n, d, synth.ring_csr(n), comp, k=max(1, d // 20), momentum=n % 2 == 0, randk_rescale=int(comp == B.Q_RANDK and n % 3 == 0))


@pytest.mark.parametrize("d", [1, 63, 64, 65, 127, 128, 129, 64 * 128 - 1, 64 * 128 + 1, 64 * 300 + 3])
@pytest.mark.parametrize("comp,order", [(B.Q_TOPK, B.ORDER_COMPRESS_THEN_MIX), (B.Q_RANDK, B.ORDER_COMPRESS_THEN_MIX),
                                        (B.Q_RANDK, B.ORDER_MIX_THEN_COMPRESS)])
def test_narrow_tile_by_columns(d, comp, order):
    """Around one tile, and around the 128 tiles that share out eight dies."""
    walk(16, d, synth.torus_csr(4, 4), comp, k=max(1, d // 30), order=order)


@pytest.mark.parametrize("n", [31, 33, 64])
def test_narrow_tile_with_more_neighbours_than_it_stages(n):
    """The complete graph: 961 entries of W (staged), 1,089 and 4,096 (read from memory)."""
    walk(n, 300, synth.complete_csr(n), B.Q_TOPK, k=10)


@pytest.mark.parametrize("n,d,align", [(64, 17_000, 32), (16, 66_000, 32), (12, 90_001, 4)])
def test_mix_of_a_state_that_is_streamed(n, d, align):
    """Past the caches (4 to 12 MB per array), on whole lines and off them (the wide tile)."""
    walk(n, d, synth.ring_csr(n), B.Q_TOPK, steps=2, k=d // 100, ld_align=align)


@pytest.mark.parametrize("n", [8, 9, 12, 13, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("comp", [B.Q_SIGN, B.Q_QSGD])
@pytest.mark.parametrize("layered", [False, True])
def test_dense_tiles_by_number_of_workers(n, comp, layered):
    lengths = [700, 3, 64, 129, 5000 + n]
    d = synth.layers_dim(synth.layer_table(lengths)) if layered else 64 * 9 + (n * 7) % 64
    walk(n, d, synth.ring_csr(n), comp, levels=8, momentum=n % 2 == 0,
         layers=synth.layer_table(lengths) if layered else None)


@pytest.mark.parametrize("n,d,align", [(8, 140_001, 32), (16, 66_003, 4), (64, 17_000, 32)])
@pytest.mark.parametrize("comp", [B.Q_SIGN, B.Q_QSGD])
@pytest.mark.parametrize("layered", [False, True])
def test_local_update_formed_twice(n, d, align, comp, layered):
    """States streamed past the caches (4 to 12 MB per array): the norm pass does not store x - lr g."""
    lengths = [d // 2, 37, d - d // 2 - 40 - 300, 255]
    layers = synth.layer_table(lengths) if layered else None
    walk(n, synth.layers_dim(layers) if layered else d, synth.ring_csr(n), comp, steps=2, levels=8, ld_align=align,
         layers=layers)


@pytest.mark.parametrize("n,d", [(1, (1 << 21) + 1), (12, (1 << 21) + 1), (13, (1 << 21) + 131)])
@pytest.mark.parametrize("polls", [None, "0"])
def test_topk_update_formed_for_the_keys_only(n, d, polls, monkeypatch):
    """Rows above 2^21 entries of a state that is streamed (below 12 MB or above 96 MB per array): the
    candidate pass stores no x, neither does the repair of a failed guess (the first step, and the one
    after the state has been scaled), nor the row scan that is left when the repair's bounded wait is
    over at once (polls = 0)."""
    if polls is not None:
        monkeypatch.setenv("CHOCO_FALLBACK_SPIN_LIMIT", polls)
    pair = Pair(synth.normal_state(n, d, seed=3), synth.ring_csr(n), 0.2, B.Q_TOPK, k=d // 1000, ld_align=32)
    pair.gpu.set_profiling(True)
    grads = synth.GradientStream(n, d, seed=4)
    modes = []
    for t in range(4):
        pair.check(pair.step(grads.next(), 0.1 if t != 2 else 50.0), tag="step %d" % t)
        modes.append(set(pair.gpu.last_scalars()[:, 3]))
    assert pair.gpu.profile_report()["k_sel_compact_redo"][0] == 4
    assert modes[0] == {2.0 if polls else 0.0}       # (rebuilt: the select then takes the list)
    assert np.all(pair.gpu.last_scalars()[:, 4] >= 2)   # steps whose guess failed
    pair.close()


@pytest.mark.parametrize("n,d", [(24, 256 * 256), (24, 256 * 256 + 1), (64, 250), (24, 256 * 512), (24, 256 * 512 + 1)])
def test_norm_finished_in_the_apply_pass_or_before_it(n, d):
    """sign with 17 to 32 workers, a state of 12 MB or more: up to 512 tiles of 256 columns the apply pass
    finishes the norms itself (in the test of the launches: which does)."""
    walk(n, d, synth.ring_csr(n), B.Q_SIGN, steps=2)


@pytest.mark.parametrize("n", [9, 13, 20, 24, 32, 40, 48, 64])
def test_random_a_with_x_streamed_and_xhat_cached(n):
    """12 to 96 MB per array, every shape of the narrow tile."""
    d = (13 << 18) // n + n % 5
    walk(n, d, synth.ring_csr(n), B.Q_RANDK, steps=2, k=d // 50, momentum=n % 2 == 0)


@pytest.mark.parametrize("n,d,align", [(20, 256 * 391, 32), (40, 256 * 200 - 3, 32), (40, 256 * 350, 32), (48, 52_001, 32),
                                       (64, 256 * 180, 32), (64, 2001, 4), (24, 256 * 300 + 1, 4)])
@pytest.mark.parametrize("comp", [B.Q_SIGN, B.Q_QSGD])
def test_norms_finished_in_the_apply_pass_of_more_than_sixteen_workers(n, d, align, comp):
    walk(n, d, synth.ring_csr(n), comp, steps=2, levels=16, ld_align=align, momentum=n == 48)


@pytest.mark.parametrize("n", [9, 12, 13, 16])
@pytest.mark.parametrize("d", [256 * 511 - 4, 256 * 511 + 1])
@pytest.mark.parametrize("comp,order", [(B.Q_SIGN, B.ORDER_COMPRESS_THEN_MIX), (B.Q_QSGD, B.ORDER_COMPRESS_THEN_MIX),
                                        (B.Q_TOPK, B.ORDER_COMPRESS_THEN_MIX), (B.Q_SIGN, B.ORDER_MIX_THEN_COMPRESS),
                                        (B.Q_QSGD, B.ORDER_MIX_THEN_COMPRESS), (B.Q_RANDK, B.ORDER_MIX_THEN_COMPRESS)])
def test_wide_tile_around_512_tiles(n, d, comp, order):
    """Four waves of four rows or a row per wave; rows off whole lines, where there is no narrow tile."""
    walk(n, d, synth.ring_csr(n), comp, steps=2, levels=16, k=500, order=order, ld_align=4)


@pytest.mark.parametrize("n", [9, 12, 13, 16])
@pytest.mark.parametrize("tiles", [511, 512])
@pytest.mark.parametrize("comp", [B.Q_SIGN, B.Q_QSGD])
def test_layers_around_512_tiles(n, tiles, comp):
    """The layers' norms come from the apply pass (sign, a row per wave) or from a launch of their own."""
    layers = synth.layer_table([60_000, 7, 256 * tiles - 60_000 - 12 - 30_001, 29_989])
    d = synth.layers_dim(layers)
    assert (d + 255) // 256 == tiles
    walk(n, d, synth.ring_csr(n), comp, steps=2, levels=16, ld_align=4, layers=layers, momentum=n == 12)
