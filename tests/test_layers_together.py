"""top_a layer by layer with layers of every kind in two launches: which tables take them, and parity at the edges of the
kinds (768 / 769 entries a wave or a 256-thread workgroup, 3,072 / 3,073 that or 1024 threads, 10,240 / 10,241 registers or
the pass over the long layers)."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding, synth
from tests.launches import recorded
from tests.parity_util import Pair

EDGES = [1, 768, 3072, 3073, 10240, 10241, 769, 5, 12288, 12289, 9216, 2304, 16, 36864, 3]


@pytest.mark.timeout(300)
def test_which_tables_take_two_launches():
    """Long layers of up to 2^19 entries, some of 3,073 to 10,240 and some shorter ones; whatever the workers and the order."""
    out = recorded("""
out = {}
for name, lengths in (("all", [20000, 4000, 100]), ("no long", [4000, 100]), ("no middle", [20000, 100]), ("no short", [20000, 4000]),
                      ("longest", [1 << 19, 4000, 100]), ("longer", [(1 << 19) + 1, 4000, 100])):
    for n in (2, 16, 64, 65):
        for order in (0, 1):
            for op, comp in (("topk", B.Q_TOPK), ("randk", B.Q_RANDK)):
                if name.startswith("long") and n > 2:
                    continue
                t = synth.layer_table(lengths, fraction=0.01)
                c = Context(n, synth.layers_dim(t), comp, layers=t, order=order)
                out["%s %s %d %d" % (op, name, n, order)] = [x[0].split("<")[0] + " " + x[1] for x in c.step()]
                c.close()
""")
    for key, launches in out.items():
        together = [x for x in launches if x.startswith("k_layers")]
        assert [x.split()[0] for x in together] == (
            ["k_layers_pass", "k_layers_select"] if key.startswith("topk") and ("all" in key or "longest" in key) else []), key
        assert not together or not any(x.startswith(("k_sel", "k_layer_")) for x in launches), key
    assert out["topk all 64 0"][:2] == ["k_layers_pass %dx64x1" % (1 + (20000 // 4 + 255) // 256), "k_layers_select 2x64x1"]


@pytest.mark.gpu
@pytest.mark.parametrize("n,table,form", [
    (2, "aligned", "step"), (5, "generic", "step"), (12, "aligned", "step"), (12, "aligned", "momentum"),
    (33, "aligned", "step"), (33, "aligned", "printed"), (17, "generic", "printed"), (70, "aligned", "step")])
def test_parity_where_the_kinds_meet(n, table, form):
    start, length, k = synth.layer_table(EDGES, fraction=0.02)
    if table == "generic":      # layers that start anywhere, with gaps
        start = np.cumsum([3] + [int(a) + 1 + (j % 3) for j, a in enumerate(length)])[:-1]
    k[1], k[7] = 0, length[7]   # a silent layer, a layer sent whole
    layers = (np.asarray(start, dtype=np.int64), length, k)
    d = int(layers[0][-1] + length[-1])
    order = binding.ORDER_MIX_THEN_COMPRESS if form == "printed" else binding.ORDER_COMPRESS_THEN_MIX
    pair = Pair(synth.normal_state(n, d, seed=n), synth.ring_csr(n), 0.1, seed=3, compressor=binding.Q_TOPK, layers=layers, order=order)
    g = synth.GradientStream(n, d, seed=4)
    for t in range(4):
        det = pair.step_momentum(g.next(), 0.05, 0.9, 1e-4) if form == "momentum" else pair.step(g.next(), 0.05)
        pair.check(det, tag="%d workers, %s table, %s, step %d" % (n, table, form, t))
    pair.gpu.set_profiling(True)
    pair.step(g.next(), 0.05)
    names = pair.gpu.profile_report()
    assert any(x.startswith("k_layers_pass") for x in names) and any(x.startswith("k_layers_select") for x in names), names
    pair.close()
