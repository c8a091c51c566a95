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
    """Long layers of up to 2^19 entries and some of up to 3,072; whatever the workers and the order.  Layers of 3,073 to
    10,240 entries go through lists like the long ones where all lists are short, else through registers; in lists they
    take the same launches without any of up to 3,072."""
    out = recorded("""
out = {}
for name, lengths in (("all", [20000, 4000, 100]), ("no long", [4000, 100]), ("no middle", [20000, 100]), ("no short", [20000, 4000]),
                      ("longest", [1 << 19, 4000, 100]), ("longer", [(1 << 19) + 1, 4000, 100]), ("many kept", [100000, 4000, 100])):
    for n in (2, 16, 64, 65):
        for order in (0, 1):
            for op, comp in (("topk", B.Q_TOPK), ("randk", B.Q_RANDK)):
                if name.startswith("long") and n > 2:
                    continue
                t = synth.layer_table(lengths, fraction=0.01)
                c = Context(n, synth.layers_dim(t), comp, layers=t, order=order)
                c.step()
                out["%s %s %d %d" % (op, name, n, order)] = [x[0].split("<")[0] + " " + x[1] for x in c.step()]
                c.close()
""")
    for key, launches in out.items():
        first = [x.split()[0] for x in launches if x.startswith(("k_layer", "k_sel"))]
        op, name = key.rsplit(" ", 2)[0].split(" ", 1)
        if op == "randk":
            assert not any(x.startswith("k_layers") for x in first), key
        elif name in ("all", "no middle", "no short"):
            assert first == ["k_layers_pass", "k_sel_refine"], key
        elif name in ("longest", "many kept"):
            assert first == ["k_layers_pass", "k_layers_select"], key
        else:
            assert not any(x.startswith("k_layers") for x in first), key
            assert "k_layer_compress" in first, key
    assert out["topk all 64 0"][:2] == ["k_layers_pass %dx64x1" % (1 + (20000 // 4 + 255) // 256 + (4000 // 4 + 255) // 256),
                                        "k_sel_refine 64x2x1"]
    assert out["topk no short 64 0"][:2] == ["k_layers_pass %dx64x1" % ((20000 // 4 + 255) // 256 + (4000 // 4 + 255) // 256),
                                             "k_sel_refine 64x2x1"]
    assert out["topk many kept 64 0"][:2] == ["k_layers_pass %dx64x1" % (1 + (100000 // 4 + 255) // 256), "k_layers_select 2x64x1"]


def test_no_launch_covers_more_chunks_than_the_layers_have():
    """200 layers of 5,000 entries beside a long one, with and without a short one: the streaming pass launches their chunks
    of 1,024 entries and one workgroup for the short layer."""
    out = recorded("""
out = {}
for name, n, more in (("short", 8, [100]), ("none", 8, []), ("none", 64, [])):
    t = synth.layer_table([1 << 19] + [5000] * 200 + more, fraction=0.0015)
    c = Context(n, synth.layers_dim(t), B.Q_TOPK, layers=t)
    out["%s %d" % (name, n)] = [x[:3] for x in c.step() + c.step()]
    c.close()
""")
    for name, launches in out.items():
        assert not any(x[0].startswith(("k_sel_compact", "k_layer_compress")) for x in launches), name
        grid = "%dx%dx1" % (512 + 5 * 200 + name.startswith("short"), int(name.split()[1]))
        assert [x[1:] for x in launches if x[0].startswith("k_layers_pass")] == [[grid, "256x1x1"]] * 2, name


def test_threads_of_the_select():
    """1024 in a context's first step, whatever its step counter, and for up to 512 workgroups; 512 for up to 3,072, then 256."""
    out = recorded("""
out = {}
for name, n, mids, t0 in (("512", 64, 7, 0), ("513", 27, 18, 0), ("3072", 64, 47, 0), ("3073", 7, 438, 0), ("resumed", 64, 47, 1000)):
    t = synth.layer_table([300000] + [3100] * mids, fraction=0.0015)
    c = Context(n, synth.layers_dim(t), B.Q_TOPK, layers=t)
    c.set_step(t0)
    out[name] = [[x[1:3] for x in c.step() if x[0].startswith("k_sel_refine")] for _ in range(3)]
    c.close()
""")
    for name, threads, grid in (("512", 1024, "64x8x1"), ("513", 512, "27x19x1"), ("3072", 512, "64x48x1"), ("3073", 256, "7x439x1"),
                                ("resumed", 512, "64x48x1")):
        assert out[name] == [[[grid, "%dx1x1" % t]] for t in (1024, threads, threads)], (name, out[name])


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,spread", [(64, 2.0 ** -1), (64, 2.0 ** -5), (64, 0.0), (20, 2.0 ** -3)])
def test_failed_guesses_and_ties_with_few_threads(n, spread):
    """Selects of 256 threads (512 with 20 workers): values of few magnitudes, steps whose size jumps (layers scanned, lists
    beyond what the threads hold), and a run that is resumed at another step."""
    lengths = [20000, 12000] + [3073, 3100, 3074, 3200] * 11 + [10240, 5000, 4096, 9216, 100]
    layers = synth.layer_table(lengths, fraction=0.015)
    d, rng = synth.layers_dim(layers), np.random.default_rng(5)

    def values():
        v = rng.standard_normal((n, d)).astype(np.float32)
        return np.round(v / np.float32(spread)) * np.float32(spread) if spread else v

    pair = Pair(values(), synth.ring_csr(n), 0.25, seed=3, compressor=binding.Q_TOPK, layers=layers)
    pair.gpu.set_step(1000)
    pair.ref.t = 1000
    scanned = []
    for t, lr in enumerate((0.5, 0.5, 0.25, 2.0, 0.5, 64.0, 0.5, 0.0)):
        pair.check(pair.step(values(), lr), tag="%d workers, %g, step %d" % (n, spread, t))
        scanned.append(pair.gpu.layer_scalars()[:, :-1, 3] == 0)
    assert scanned[0].all() and scanned[5].mean() > 0.5 and any(0 < s.mean() < 0.5 for s in scanned[1:5])
    pair.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,lengths,start0", [(9, [20000, 3073, 4096, 10240, 9216, 100, 1 << 19], 0), (33, [12000, 4096, 5000, 3333], 0),
                                              (2, [1 << 21, 700000], 3), (2, [1 << 21, 5000], 0)])
def test_layers_of_one_magnitude(n, lengths, start0):
    """Constant layers that get no gradients: every step scans them, all entries in one bin of each digit, and the cut is by the
    index; long layers up to the 2^21 entries (and three before them) below which the index's first digit is known."""
    start, length, k = synth.layer_table(lengths, fraction=0.01)
    k = np.minimum(k, 700)
    layers = (np.asarray(start) + start0, length, k)
    d = int(layers[0][-1] + length[-1])
    rng = np.random.default_rng(n)
    X0 = np.ones((n, d), dtype=np.float32)
    X0[:, ::3] = -1.0
    X0[0, rng.integers(0, d, 7)] = 1.5
    pair = Pair(X0, synth.ring_csr(n), 0.05, seed=3, compressor=binding.Q_TOPK, layers=layers)
    g = np.zeros((n, d), dtype=np.float32)
    for t in range(5):
        if t == 3:
            g[:, rng.integers(0, d, 50)] = 2.0
        pair.check(pair.step(g, 0.25), tag="%d workers, %s, step %d" % (n, lengths, t))
    assert np.any(pair.gpu.layer_scalars()[:, :, 3] == 0)
    pair.close()


def workspace(n, lengths, fraction, silent=()):
    start, length, k = synth.layer_table(lengths, fraction=fraction)
    k[list(silent)] = 0
    d = int(start[-1] + length[-1])
    cfg, keep = binding.make_config(n, d, *synth.ring_csr(n), 0.1, binding.Q_TOPK, layers=(start, length, k))
    return binding.workspace_bytes(cfg), 4 * n * d


@pytest.mark.parametrize("n,lengths,fraction,listed", [
    (64, [20000] + [4000] * 40, 0.01, True), (64, [20000] + [3100] * 1000, 0.01, True), (8, [1 << 19] + [5000] * 200, 0.0015, True),
    (64, [16000] + [3100] * 1000, 0.05, True), (64, [10300] + [3100] * 5000, 0.079, False), (64, [11000] + [3100] * 1000, 0.19, False)])
def test_lists_take_no_more_than_two_arrays(n, lengths, fraction, listed):
    """What the layers of 3,073 to 10,240 entries add to the workspace: their sub-lists, as many as a layer has chunks, and the
    counters; a silent one takes the table to registers."""
    lists, state = workspace(n, lengths, fraction)
    registers, _ = workspace(n, lengths, fraction, silent=[1])
    assert (lists > registers + state // 20) == listed
    assert lists <= registers + 2 * state
    if listed:
        chunks = sum((m + 1023) // 1024 for m in lengths[1:])
        room = min(1024, max(64, int(2.5 * lengths[1] * fraction + 120) * 2))   # of a sub-list, generously
        assert lists <= registers + n * (8 * room * chunks + 4 * 32 * 32 * len(lengths[1:])) + 4096 * len(lengths)


def test_a_workspace_that_was_enough_is_accepted():
    """Bytes that were asked for before layers of 3,073 to 10,240 entries went through lists: enough for the register form, and
    for a table without such layers."""
    out = recorded("""
out = {}
for name, n, lengths, fraction, ws in (("41", 64, [20000] + [4000] * 40, 0.01, 65611264), ("201", 8, [1 << 19] + [5000] * 200, 0.0015, 52669952),
                                       ("image", 64, list(synth.resnet20_like_lengths()), 0.01, 175791360),
                                       ("long", 8, [12000] * 40, 0.01, 101414400)):
    t = synth.layer_table(lengths, fraction=fraction)
    out[name] = []
    for given in (ws, None):
        c = Context(n, synth.layers_dim(t), B.Q_TOPK, layers=t, ws=given)
        assert c.rc == B.OK, (name, given, c.asked)
        c.step()
        out[name].append([x[0].split("<")[0] for x in c.step()])
        c.close()
    assert name == "long" or Context(n, synth.layers_dim(t), B.Q_TOPK, layers=t, ws=ws // 2).rc == B.E_NOMEM
""")
    for name, (before, asked) in out.items():
        if name == "long":
            assert before == asked, name
        else:
            assert any(x in ("k_layers_select", "k_layer_compress") for x in before), name
            assert asked[:2] == ["k_layers_pass", "k_sel_refine"], name


@pytest.mark.gpu
def test_parity_in_a_workspace_without_the_lists(monkeypatch):
    lengths, n = [20000, 4000, 100, 9216, 3073, 10240], 9
    layers = synth.layer_table(lengths, fraction=0.01)
    d = synth.layers_dim(layers)
    least = workspace(n, lengths, 0.01, silent=[1])[0] + (1 << 16)    # registers, what the silent layer keeps, longer rows
    assert least < workspace(n, lengths, 0.01)[0]
    monkeypatch.setattr(binding, "workspace_bytes", lambda cfg: least)
    pair = Pair(synth.normal_state(n, d, seed=8), synth.ring_csr(n), 0.05, seed=3, compressor=binding.Q_TOPK, layers=layers)
    g = synth.GradientStream(n, d, seed=9)
    for t in range(4):
        pair.check(pair.step(g.next(), 0.05), tag="registers, step %d" % t)
    pair.gpu.set_profiling(True)
    pair.step(g.next(), 0.05)
    assert any(x.startswith("k_layers_select") for x in pair.gpu.profile_report())
    pair.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,table,form,fraction", [
    (2, "aligned", "step", 0.02), (5, "generic", "step", 0.02), (12, "aligned", "step", 0.02), (12, "aligned", "momentum", 0.02),
    (33, "aligned", "step", 0.02), (33, "aligned", "printed", 0.02), (17, "generic", "printed", 0.02), (70, "aligned", "step", 0.02),
    (5, "generic", "step", 0.06), (33, "aligned", "momentum", 0.06), (12, "aligned", "printed", 0.06), (64, "many", "step", 0.01),
    (64, "many", "printed", 0.002), (5, "no short", "step", 0.02), (33, "no short", "momentum", 0.01), (64, "no short", "printed", 0.02)])
def test_parity_where_the_kinds_meet(n, table, form, fraction):
    """Lists through selects of 1024 threads (512 with more than 512 of them), at 6 % registers."""
    edges = EDGES if table != "many" else EDGES + [3073, 3074, 3500, 4000, 4096, 4097, 5000, 6144, 7000, 8191]
    if table == "no short":
        edges = [x for x in EDGES if x > 3072] + [3073, 3074, 4096, 4097, 7168]
    start, length, k = synth.layer_table(edges, fraction=fraction)
    if table == "generic":      # layers that start anywhere, with gaps
        start = np.cumsum([3] + [int(a) + 1 + (j % 3) for j, a in enumerate(length)])[:-1]
    if table != "no short":
        k[1], k[7] = 0, length[7]   # a silent layer, a layer sent whole
        k[2], k[5] = 1, max(k[5], 1)
    layers = (np.asarray(start, dtype=np.int64), length, k)
    d = int(layers[0][-1] + length[-1])
    order = binding.ORDER_MIX_THEN_COMPRESS if form == "printed" else binding.ORDER_COMPRESS_THEN_MIX
    pair = Pair(synth.normal_state(n, d, seed=n), synth.ring_csr(n), 0.1, seed=3, compressor=binding.Q_TOPK, layers=layers, order=order)
    g = synth.GradientStream(n, d, seed=4)
    for t in range(4):
        det = pair.step_momentum(g.next(), 0.05, 0.9, 1e-4) if form == "momentum" else pair.step(g.next(), 0.05)
        pair.check(det, tag="%d workers, %s table, %s, %g, step %d" % (n, table, form, fraction, t))
    pair.gpu.set_profiling(True)
    pair.step(g.next(), 0.05)
    names = pair.gpu.profile_report()
    assert any(x.startswith("k_layers_pass") for x in names), names
    assert any(x.startswith("k_layers_select") for x in names) == (fraction == 0.06), names
    pair.close()


@pytest.mark.gpu
@pytest.mark.parametrize("spread", [2.0 ** -3, 2.0 ** -12])
def test_layer_scalars_are_those_of_the_register_form(spread):
    """Layers of 3,073 to 10,240 entries, many entries of one magnitude: x, and where ties are cut threshold key, entries kept
    of those that hold it and how many these are, by lists (a long layer behind them) and by registers (none)."""
    import torch
    lengths, n = [3073, 5000, 10240, 100, 9216], 6
    common = synth.layers_dim(synth.layer_table(lengths))
    got = []
    for more in ([], [20000]):
        layers = synth.layer_table(lengths + more, fraction=0.01)
        d = synth.layers_dim(layers)
        ld = (d + 63) // 64 * 64
        x = torch.from_numpy(synth.normal_state(n, 1 << 16, seed=5))[:, :ld].div(spread).round().mul(spread).contiguous().cuda()
        ctx = binding.Choco(x, d, *synth.ring_csr(n), 0.25, binding.Q_TOPK, seed=3, layers=layers)
        g = torch.from_numpy(synth.normal_state(n, 1 << 16, seed=6)).div(spread).round().mul(spread).cuda()
        scal, sel = [], []
        for t in range(6):
            ctx.step(g[:, 64 * t:64 * t + ld].contiguous(), 0.5 if t != 4 else 20.0)
            scal.append(ctx.layer_scalars()[:, :len(lengths), :3])
            sel.append(x[:, :common].cpu().numpy())
        got.append((np.array(scal), np.array(sel)))
        ctx.close()
    np.testing.assert_array_equal(got[0][1], got[1][1])
    registers, lists = (a[:, :, [0, 1, 2, 4]] for a in (got[0][0], got[1][0]))
    tied = registers[:, :, :, 2] > registers[:, :, :, 1]
    np.testing.assert_array_equal(registers[tied], lists[tied])
    # all that hold the threshold key are kept: the search of the register form may end below the last kept key
    np.testing.assert_array_equal(lists[~tied][:, 1], lists[~tied][:, 2])
    assert np.all(lists[~tied][:, 1] >= 1) and np.all(lists[~tied][:, 0] >= registers[~tied][:, 0])
    if spread == 2.0 ** -3:
        assert np.any(tied)


@pytest.mark.gpu
@pytest.mark.parametrize("fraction", [0.001, 0.01, 0.03])
def test_large_entries_that_lie_together_stay_in_the_lists(fraction):
    """All of a layer's large entries in one chunk of 1,024: its sub-list holds them."""
    lengths, n = [20000, 9216, 5000, 100, 10240], 5
    start, length, k = layers = synth.layer_table(lengths, fraction=fraction)
    d = int(start[-1] + length[-1])
    where = np.zeros(d, dtype=np.float32)
    for a, m in zip(start, length):
        where[a + min(1024, m // 2):a + min(2048, m)] = 1.0

    def clustered(v):
        return (np.asarray(v) * (0.001 + where)).astype(np.float32)

    pair = Pair(clustered(synth.normal_state(n, d, seed=8)), synth.ring_csr(n), 0.05, seed=3, compressor=binding.Q_TOPK, layers=layers)
    g = synth.GradientStream(n, d, seed=9)
    for t in range(8):
        det = pair.step(clustered(g.next()), 0.5)
        pair.check(det, tag="clustered, %g, step %d" % (fraction, t))
        if t > 2:
            assert np.all(pair.gpu.layer_scalars()[:, [1, 2, 4], 3] == 1), t
    pair.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,table", [(5, "aligned"), (5, "generic"), (64, "aligned")])
def test_layers_with_fewer_values_than_are_kept(n, table):
    """Layers without gradients whose values have all been sent, and such of which few entries get one: the zeros that are
    kept with the others are the first, and once the layer has come to that its lists say so (no scan)."""
    lengths = [20000, 4000, 3500, 9216, 100, 10240, 5000, 3073, 2500, 12000, 7000, 3100, 6000, 8000, 3300, 9999, 4097, 30000]
    start, length, k = synth.layer_table(lengths, fraction=0.01)
    if table == "generic":
        start = np.cumsum([3] + [int(a) + 1 + (j % 3) for j, a in enumerate(length)])[:-1]
    k[2], k[9], k[13] = 819, 700, 1
    layers = (np.asarray(start, dtype=np.int64), length, k)
    d = int(layers[0][-1] + length[-1])
    rng = np.random.default_rng(n)
    # values left to be sent (the same of all workers, so that the mix adds none), entries that get a gradient
    left = [3.5, 0.5, 0.3, 0, 1.5, 2.2, 9, 0.9, 1.7, 0.6, 0, 2, 1, 1, 0.2, 0, 1.1, 0.4]
    moving = [0, 0, 0.7, 0, 0, 0.5, 3, 0, 0, 0.9, 0.4, 0.97, 0, 0, 1, 0, 0, 0.3]
    X0, at = np.zeros((n, d), dtype=np.float32), []
    for l, (a, m, kk) in enumerate(zip(layers[0], length, k)):
        places = a + rng.permutation(m if l % 2 else min(m, 2 * kk))[:int(np.ceil(left[l] * kk))]
        X0[:, places] = rng.standard_normal(len(places)).astype(np.float32)
        # among the first entries, about the k-th, anywhere
        near = [min(m, 2 * kk), min(m, kk + 40), m][l % 3]
        at.append(a + rng.permutation(near)[:min(near, int(moving[l] * kk))])
    at = np.concatenate(at)
    pair = Pair(X0, synth.ring_csr(n), 0.02, seed=3, compressor=binding.Q_TOPK, layers=layers)
    before = np.zeros((n, len(lengths)), dtype=bool)
    seen = 0
    for t in range(14):
        g = np.zeros((n, d), dtype=np.float32)
        g[:, at] = rng.standard_normal((1 if t < 11 else n, len(at))).astype(np.float32)
        v = (pair.ref.X - np.float32(0.25) * g) - pair.ref.Xhat
        pair.check(pair.step(g, 0.25), tag="%d workers, %s, step %d" % (n, table, t))
        scal = pair.gpu.layer_scalars()
        for l, (a, m, kk) in enumerate(zip(layers[0], length, k)):
            some = np.count_nonzero(v[:, a:a + m], axis=1)
            now = some < kk
            if m <= 10240:
                np.testing.assert_array_equal(scal[now, l, :3], np.stack([0 * some, kk - some, m - some], axis=1)[now])
            else:
                assert np.all(scal[now, l, 0] == 0)
            assert np.all(scal[now & before[:, l], l, 3] == 1), (t, l)
            seen += int((now & before[:, l]).sum())
            before[:, l] = now
    assert seen > 50 * n
    pair.close()
