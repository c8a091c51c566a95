"""top_a on rows that one workgroup (or wave) selects out of its registers."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding as B
from paper_1907_09356_amd import synth
from tests.launches import recorded
from tests.parity_util import Pair


def test_which_rows_are_selected_out_of_registers():
    out = recorded("""
out = {}
for d, k, kw in ((768, 7, {}), (769, 7, {}), (1024, 1024, {}), (1025, 1025, {}), (6144, 3072, {}), (6144, 3073, {}), (6145, 160, {}),
                 (6145, 161, {}), (8192, 160, {}), (8193, 128, {}), (8193, 129, {}), (10240, 128, {}), (10241, 10, {}),
                 (1000, 10, dict(order=1)), (1000, 10, dict(mix_form=B.MIX_INCREMENTAL_S))):
    c = Context(5, d, B.Q_TOPK, k=k, **kw)
    out["%d %d %s" % (d, k, sorted(kw))] = [x[0] for x in c.step()][:-1]
    c.close()
for n, k in ((32, 160), (33, 160), (33, 64), (33, 65)):
    c = Context(n, 8192, B.Q_TOPK, k=k)
    out["n = %d, k = %d" % (n, k)] = [x[0] for x in c.step()][:-1]
    c.close()
c = Context(65, 1000, B.Q_TOPK, k=10)     # no tile of all rows
out["n = 65"] = [x[0] for x in c.step()]
""")
    assert out["768 7 []"] == ["k_row_compress<64,false>"]
    words = {"1024 1024 []", "6144 3072 []", "6145 160 []", "8192 160 []", "8193 128 []", "10240 128 []", "n = 32, k = 160", "n = 33, k = 64"}
    assert out["769 7 []"] == ["k_row_compress<1024,false>"]
    assert {c for c, l in out.items() if l == ["k_row_compress<1024,true>"]} == words
    assert sum(any(x.startswith("k_row_compress") for x in l) for l in out.values()) == 2 + len(words)


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,grid,mode", [
    (3, 1, 1, 0, "step"), (4, 5, 2, 0, "halves"), (8, 767, 766, 0, "step"), (6, 768, 1, 0, "momentum"), (9, 769, 300, 0, "step"),
    (2, 4097, 41, 0, "momentum"), (64, 1030, 50, 0, "step"), (5, 6144, 3072, 0, "halves"), (12, 8189, 160, 0, "step"), (4, 10240, 128, 0, "step"),
    (5, 700, 200, 3, "step"), (5, 3001, 900, 3, "step"), (3, 1024, 1024, 3, "step"),
    (5, 9001, 100, 50, "step"), (9, 5001, 30, 50, "step"),   # a dozen ties among the listed, in three sweeps and in two
    (3, 6144, 1500, 2, "step"),                              # more ties than are listed
    (3, 1000, 800, 1, "step"), (4, 700, 600, 1, "halves"), (3, 6000, 2900, -1, "step"),   # k includes zeros
])
def test_rows_selected_out_of_registers(n, d, k, grid, mode):
    """Lengths around a wave's, a sweep's and the longest; ties (values on a grid); a scale that jumps, so that
    the bracket around the last threshold misses.  The figures of the select are those of what was sent."""
    X0 = synth.normal_state(n, d, seed=d)
    if grid < 0:
        X0[:, ::2] = X0[:, ::3] = 0.0                        # (two thirds)
    elif grid:
        X0 = np.round(X0 * grid) / np.float32(grid)
    pair = Pair(X0, synth.ring_csr(n) if n > 2 else synth.complete_csr(n), 0.2, compressor=B.Q_TOPK, k=k, ld_align=32 if n % 2 else 4)
    grads = synth.GradientStream(n, d, seed=2)
    missed = 0
    try:
        for t, lr in enumerate([0.0 if grid else 0.05, 0.0 if grid else 0.05, 500.0, 0.01, 0.01]):
            g = grads.next()
            if mode == "momentum":
                det = pair.step_momentum(g, lr, 0.9, 1e-3)
            elif mode == "halves":
                pair.sgd_step(g, lr)
                det = pair.gossip_step()
            else:
                det = pair.step(g, lr)
            pair.check(det, tag="step %d" % t)
            idx, val = (a.cpu().numpy() for a in pair.gpu.last_selection())
            key = val.view(np.uint32) & 0x7FFFFFFF
            scal = pair.gpu.last_scalars()
            for i in range(n):
                last = key[i].min()
                assert scal[i, 0] == last and scal[i, 1] == idx[i][key[i] == last].max()
            missed += int(np.all(scal[:, 3] == 2))
            assert set(scal[:, 3]) <= {0.0, 2.0} and np.all(scal[:, 4] >= missed)
        assert missed >= 1                               # (the first step has no threshold to go by)
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [3, 40])
def test_layers_that_keep_zeros(n):
    """More kept than there are values other than zero, in layers of a wave, of small and of large workgroups."""
    layers = synth.layer_table([600, 2000, 9000, 40, 5000], fraction=0.5)
    d = synth.layers_dim(layers)
    X0 = synth.normal_state(n, d, seed=1)
    X0[:, np.arange(d) % 3 != 0] = 0.0
    pair = Pair(X0, synth.ring_csr(n), 0.2, compressor=B.Q_TOPK, layers=layers)
    grads = synth.GradientStream(n, d, seed=2)
    try:
        for t, lr in enumerate([0.0, 0.0, 0.05]):
            pair.check(pair.step(grads.next(), lr), tag="step %d" % t)
            if t == 0:
                assert np.all(pair.gpu.layer_scalars()[:, :, 0] == 0.0)
    finally:
        pair.close()
