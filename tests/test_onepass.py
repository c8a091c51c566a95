"""top_a and gsgd in one pass over the state: every bit as the oracle has it, also where the pass went by a wrong
threshold, left tiles unmixed, could not take its mix back without the records, or has to be undone."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding as B
from paper_1907_09356_amd import synth
from tests.launches import recorded
from tests.parity_util import Pair


def test_where_top_a_takes_one_pass():
    """Two to eight workers, whole vectors in the default order, more than 96 MiB per array, few marked columns."""
    out = recorded("""
out = {}
D = 3_200_000
for name, n, d, kw in (
        ("n8", 8, D, {}), ("n8 momentum", 8, D, {}), ("n2", 2, 4 * D, {}), ("n9", 9, D, {}), ("n1", 1, 8 * D, {}),
        ("96 MiB", 8, 96 * 2**20 // 32, {}), ("printed", 8, D, dict(order=1)), ("sums", 8, D, dict(mix_form=B.MIX_INCREMENTAL_S)),
        ("many kept", 8, D, dict(k=D // 500)), ("many kept, large", 8, 2 * D, dict(k=2 * D // 500)),
        ("more kept, large", 8, 2 * D, dict(k=2 * D // 300)), ("rescale", 8, D, dict(randk_rescale=1)), ("odd", 8, D + 1, {})):
    c = Context(n, d, B.Q_TOPK, **{"k": d // 1000, **kw})
    first = c.step()
    l = c.step_momentum() if "momentum" in name else c.step()
    out[name] = [[x[0].split("<")[0] for x in y] for y in (first, l)] + [l[0][1:3]]
    c.close()
""")
    # (also the first step, which has no threshold to go by: it may be captured, and replayed as a later one)
    launches = ["k_onepass_mix", "k_onepass_list", "k_onepass_restore", "k_sel_fallback", "k_sel_refine", "k_onepass_finish"]
    one = {"n8", "n8 momentum", "n2", "many kept, large", "odd"}
    for name, (a, b, shape) in out.items():
        if name in one:
            drop = {"k_sel_hist_parts", "k_sel_emit_parts"}
            norm = lambda l: ["k_sel_refine" if x == "k_sel_finish" else x for x in l if x not in drop]  # noqa: E731
            assert norm(a) == norm(b) == launches, name
        else:
            assert not any(x.startswith("k_onepass") for x in a + b), name
    assert out["odd"][2] == ["12501x1x1", "512x1x1"] and out["n2"][2][1] == "128x1x1"


def test_where_gsgd_takes_one_pass():
    """Two to eight workers, whole vectors in the default order, more than 96 MiB per array, few levels above zero."""
    out = recorded("""
out = {}
D = 3_200_000
for name, n, d, kw in (
        ("n8", 8, D, {}), ("n8 momentum", 8, D, {}), ("n2", 2, 4 * D + 1, dict(levels=64)), ("n9", 9, D, {}), ("n1", 1, 8 * D, {}),
        ("96 MiB", 8, 96 * 2**20 // 32, {}), ("printed", 8, D, dict(order=1)), ("levels", 8, D, dict(levels=16)),
        ("layers", 8, D, dict(layers=synth.layer_table([D // 2, D // 2])))):
    c = Context(n, d, B.Q_QSGD, **{"levels": 8, **kw})
    first = c.step()
    l = c.step_momentum() if "momentum" in name else c.step()
    out[name] = [[x[0].split("<")[0] for x in y] for y in (first, l)]
    c.close()
""")
    for name, (first, later) in out.items():
        assert not any(x.startswith("k_onepass") for x in first), name     # no norm to go by yet
        if name in ("n8", "n8 momentum", "n2"):
            assert first == ["k_dense_stat", "k_dense_finalise", "k_dense_apply_mix"], name
            assert later == ["k_onepass_mix", "k_group_reduce", "k_dense_finalise", "k_onepass_encode"], name
        else:
            assert later == first, name


def test_a_workspace_for_two_passes_is_accepted():
    """What choco_workspace_bytes asks for has room for one pass; without it the steps take two."""
    out = recorded("""
out = {}
for name, comp, kw in (("topk", B.Q_TOPK, dict(k=4000)), ("qsgd", B.Q_QSGD, dict(levels=8))):
    n, d = 8, 3_200_000
    full = Context(n, d, comp, **kw)
    lo, hi = 0, full.asked            # a size that is refused and one that is taken
    while hi - lo > 256:
        mid = (lo + hi) // 2
        c = Context(n, d, comp, ws=mid, **kw)
        if c.rc == B.OK:
            hi = mid
            c.close()
        else:
            assert c.rc == B.E_NOMEM, c.rc
            lo = mid
    steps = []
    for ws in (hi, full.asked - 1, full.asked):
        c = Context(n, d, comp, ws=ws, **kw)
        c.step()
        steps.append([x[0].split("<")[0] for x in c.step()])
        c.close()
    out[name] = [hi / (4 * n * d), full.asked / (4 * n * d), steps]
    full.close()
""")
    two = {"topk": ["k_sel_compact", "k_sel_fallback", "k_sel_refine", "k_tile_mix"],
           "qsgd": ["k_dense_stat", "k_dense_finalise", "k_dense_apply_mix"]}
    for name, (least, asked, steps) in out.items():
        assert least < 1.17 and 1.5 < asked < 1.75, name
        assert steps[0] == steps[1] == two[name] and steps[2][0] == "k_onepass_mix", name


def test_no_one_pass_where_the_state_fills_the_card():
    """Above 48 GiB per array the workspace stays that of two passes."""
    for comp, kw in ((B.Q_TOPK, dict(k=100_000)), (B.Q_QSGD, dict(levels=16))):
        arrays = []
        for d in (1_600_000_000, 1_620_000_000):
            cfg, keep = B.make_config(8, d, *synth.ring_csr(8), 0.1, comp, **kw)
            arrays.append(B.workspace_bytes(cfg) / (32 * d))
        assert arrays[0] > 1.5 and arrays[1] < 1.17


def graph(name, n):
    if name == "irregular":                         # unequal degrees and weights
        return synth.metropolis_csr(synth.irregular_graph(n, n - 2, seed=n))
    return synth.complete_csr(n) if name == "complete" else synth.ring_csr(n)


def same_message(pair, det, tag):
    """gsgd: the bit planes that the last step left decode to the oracle's levels times the step, every one."""
    if pair.codes is None:
        return
    q = pair.gpu.unpack_messages(pair.gpu.pack_messages())[:, :pair.d].cpu().numpy()
    step = np.float32(pair.gpu.last_scalars()[:, 3:4])
    assert np.array_equal(q, det["codes"].astype(np.float32) * step), tag + ": messages differ"


def steps(pair, grads, lr, mode, count, tag):
    for t in range(count):
        g = grads.next()
        if mode == "momentum":
            det = pair.step_momentum(g, lr, 0.9, 1e-3)
        elif mode == "halves":
            pair.sgd_step(g, lr)
            det = pair.gossip_step()
        else:
            det = pair.step(g, lr)
        pair.check(det, tag="%s step %d" % (tag, t))
        same_message(pair, det, "%s step %d" % (tag, t))
    return det


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,d,k,topo,mode,align", [
    (8, 3_150_001, 2000, "ring", "step", 4),        # a last tile of one column, rows off whole lines
    (7, 3_600_255, 900, "complete", "momentum", 4),
    (3, 8_400_300, 12_000, "ring", "halves", 64),   # (multi-block select)
    (2, 12_600_000, 1, "ring", "step", 4),
    (5, 5_100_001, 3000, "irregular", "step", 64),
    (6, 4_300_002, 2000, "irregular", "halves", 4),
])
def test_one_pass_steps(n, d, k, topo, mode, align):
    X0 = synth.normal_state(n, d, seed=n)
    X0[:, 5000:5400] *= 30.0                        # tiles with more candidates than there are slots
    pair = Pair(X0, graph(topo, n) if n > 2 else synth.complete_csr(2), 0.3, compressor=B.Q_TOPK, k=k, ld_align=align)
    try:
        steps(pair, synth.GradientStream(n, d, seed=2), 0.05, mode, 4, mode)
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
def test_one_pass_captured_first_step():
    """A first step that was captured: its replays go by the thresholds of those before, like eager steps."""
    import torch
    n, d, k = 8, 3_150_336, 2000
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        pair = Pair(synth.normal_state(n, d, seed=1), synth.ring_csr(n), 0.3, compressor=B.Q_TOPK, k=k)
        grads = synth.GradientStream(n, d, seed=2)
        try:
            G = grads.next()
            Gd = torch.zeros_like(pair.X)
            Gd[:, :d] = torch.from_numpy(np.ascontiguousarray(G, dtype=np.float32)).to(pair.X.device)
            pair.gpu.sync()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                pair.gpu.step(Gd, 0.05)
            side.synchronize()
            for t in range(6):
                if t == 3:                                   # the program's own work between the replays
                    steps(pair, grads, 0.05, "step", 1, "eager")
                graph.replay()
                side.synchronize()
                pair.ref.sgd_step(G, 0.05)
                pair.check(pair.ref.gossip_step(want_details=True), tag="replay %d" % t)
            scal = pair.gpu.last_scalars()
            assert np.all(scal[:, 3] == 0) and np.all(scal[:, 4] == 1), "only the first step has no threshold"
        finally:
            pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
def test_one_pass_taken_back():
    """Thresholds that fall by a factor between two steps (no list holds its k largest entries), with columns
    and whole tiles whose mix has no exact inverse (entries put right by units in the last place, or recorded), and
    ties at the threshold."""
    n, d, k = 8, 3_150_336, 1500
    rng = np.random.default_rng(5)
    X0 = synth.normal_state(n, d, seed=3)
    pair = Pair(X0, synth.ring_csr(n), 0.7, compressor=B.Q_TOPK, k=k)
    grads = synth.GradientStream(n, d, seed=4)
    try:
        steps(pair, grads, 0.05, "step", 2, "start")
        # xhat of its own at three columns of every tile, and everywhere in the tiles from column 100,000 to
        # 120,000: where the workers' xhat differ by as much as x, x' cannot be found again from the mixed x
        for where in (slice(7, d, 256), slice(100, d, 256), slice(255, d, 256), slice(100_000, 120_000)):
            pair.ref.Xhat[:, where] = pair.ref.X[:, where] + 1e-3 * rng.standard_normal(pair.ref.X[:, where].shape).astype(np.float32)
        pair.force_state()
        steps(pair, grads, 0.05, "step", 2, "lost")
        # a thousandth of the distance: every guess is too high
        pair.ref.X[:] = pair.ref.Xhat + (pair.ref.X - pair.ref.Xhat) * np.float32(1e-3)
        pair.force_state()
        steps(pair, grads, 1e-6, "step", 3, "fallen")
        assert np.all(pair.gpu.last_scalars()[:, 4] >= 2), "the thresholds were to be missed"
        # one worker's threshold only
        pair.ref.X[3] = pair.ref.Xhat[3] + (pair.ref.X[3] - pair.ref.Xhat[3]) * np.float32(0.01)
        pair.force_state()
        steps(pair, grads, 1e-6, "step", 2, "one row")
        # values on a grid: thousands of equal magnitudes around the threshold, lists that overflow
        pair.ref.X[:] = pair.ref.Xhat + np.round(X0 * 4) / np.float32(4)
        pair.force_state()
        steps(pair, grads, 0.0, "step", 2, "ties")
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,d,levels,topo,mode,align,outlier", [
    (8, 3_200_001, 8, "ring", "step", 4, False),
    (7, 3_700_255, 4, "complete", "momentum", 64, False),
    (3, 8_500_003, 16, "ring", "halves", 4, False),
    (2, 12_800_000, 64, "ring", "step", 4, False),
    (4, 6_400_003, 16, "irregular", "step", 64, False),
    (6, 4_300_001, 12, "irregular", "halves", 4, False),
    (8, 3_200_000, 8, "ring", "step", 4, True),      # one entry carries a row's norm: the level s itself
])
def test_one_pass_gsgd(n, d, levels, topo, mode, align, outlier):
    X0 = synth.normal_state(n, d, seed=n)
    X0[:, 70_000:70_400] *= 100.0                    # tiles with more columns to record than there are slots
    if outlier:
        X0[2, 12_345], X0[0, d - 1] = 3e6, -5e5
    pair = Pair(X0, graph(topo, n) if n > 2 else synth.complete_csr(2), 0.3, compressor=B.Q_QSGD, levels=levels, seed=9,
                ld_align=align)
    try:
        det = steps(pair, synth.GradientStream(n, d, seed=2), 0.05, mode, 4, mode)
        # (400 columns 100 times as large, |z| up to 4.5: s |v| / ||v|| = 100 s |z| / sqrt(d + 4e6) up to 1.3 with eight levels
        # of 3.2 M, 2.2 with sixteen of 6.4 M, 0.65 with four)
        assert np.abs(det["codes"]).max() >= (levels if outlier else 2 if levels >= 8 else 1)
        pair.gpu.set_step((1 << 33) + 2)             # a counter that is moved, back too: the dither follows it
        pair.ref.t = (1 << 33) + 2
        steps(pair, synth.GradientStream(n, d, seed=3), 0.05, "step", 1, "counter up")
        pair.gpu.set_step(2)
        pair.ref.t = 2
        steps(pair, synth.GradientStream(n, d, seed=4), 0.05, "step", 1, "counter back")
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
def test_one_pass_gsgd_taken_back():
    """Norms that shrink between two steps, of all workers or of one, beyond the bound that the pass went by; xhat of
    its own in some columns of every tile (no exact inverse of the mix) and an xhat of minus zero."""
    n, d = 8, 3_200_100
    rng = np.random.default_rng(5)
    pair = Pair(synth.normal_state(n, d, seed=3), synth.ring_csr(n), 0.7, compressor=B.Q_QSGD, levels=4, seed=2)
    grads = synth.GradientStream(n, d, seed=4)
    try:
        steps(pair, grads, 0.05, "step", 2, "start")
        for where in (slice(7, d, 256), slice(100, d, 256), slice(100_000, 120_000)):
            pair.ref.Xhat[:, where] = pair.ref.X[:, where] + 1e-3 * rng.standard_normal(pair.ref.X[:, where].shape).astype(np.float32)
        pair.ref.Xhat[:, 200_000:200_010] = -0.0
        pair.force_state()
        steps(pair, grads, 0.05, "step", 2, "lost")
        pair.ref.X[:] = pair.ref.Xhat + (pair.ref.X - pair.ref.Xhat) * np.float32(0.1)
        pair.force_state()
        steps(pair, grads, 1e-6, "step", 2, "shrunk")
        pair.ref.X[3] = pair.ref.Xhat[3] + (pair.ref.X[3] - pair.ref.Xhat[3]) * np.float32(0.5)
        pair.force_state()
        steps(pair, grads, 1e-6, "step", 2, "one row")
        pair.ref.X[:] = pair.ref.Xhat                # nothing to send: a norm of zero, and one again after it
        pair.force_state()
        steps(pair, grads, 0.0, "step", 1, "zero")
        steps(pair, grads, 0.05, "step", 2, "again")
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
def test_one_pass_gsgd_sends_what_xhat_cannot_show():
    """Levels whose value is below half a unit in the last place of xhat: they are sent though xhat stays as it is."""
    n, d, levels = 8, 3_200_000, 8
    rng = np.random.default_rng(1)
    X0 = np.tile(np.float32(1000.0) + rng.standard_normal(d).astype(np.float32), (n, 1))
    pair = Pair(X0, synth.ring_csr(n), 0.3, compressor=B.Q_QSGD, levels=levels, seed=5)
    zero = synth.GradientStream(n, d, seed=4)
    try:
        pair.ref.Xhat[:] = X0
        for i in range(n):                                   # four entries per tile and row, one unit apart
            pair.ref.X[i, i::64] = np.nextafter(X0[i, i::64], np.float32(0.0))
        pair.force_state()
        for t in range(3):
            det = steps(pair, zero, 0.0, "step", 1, "unit %d" % t)
            assert np.all(np.abs(det["codes"]).sum(axis=1) > 500) and np.array_equal(pair.ref.Xhat, X0)
    finally:
        pair.close()


def bounds_missed(r):
    """gsgd, from s / ||v|| of each row step by step (the first is the two-pass step): which later steps fail."""
    r = np.float32(r)
    missed = []
    for t in range(2, len(r) + 1):
        before = r[t - 3] if t > 2 else np.zeros_like(r[0])
        change = np.where(before > 0, np.minimum(np.abs(r[t - 2] / np.where(before > 0, before, 1) - 1), 1), 0)
        missed.append(bool(t <= len(r) and np.any(r[t - 1] > r[t - 2] * (1.02 + 2 * change))))
    return missed


def held_back(missed):
    """Two for a failure, one back for a step that went well; held from six on, down to two."""
    count, held, out = 0, False, []
    for m in missed:
        out.append(held)
        count = min(count + 2, 12) if m else max(count - 1, 0)
        held = count >= 6 or (held and count > 2)
    return out


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("op", ["topk", "qsgd"])
def test_one_pass_held_back(op):
    """Failures in a row, after which the pass leaves all tiles unmixed (also through a further failure), and steps that
    go well until it mixes again; gsgd then has norms that grow, with a bound too wide for the slots."""
    n, d = 8, 3_200_100
    kw = dict(compressor=B.Q_TOPK, k=1500) if op == "topk" else dict(compressor=B.Q_QSGD, levels=12)
    X0 = synth.normal_state(n, d, seed=3)
    pair = Pair(X0, synth.ring_csr(n), 0.2, seed=2, **kw)
    grads = synth.GradientStream(n, d, seed=4)
    figures = []

    def go(lr, count, tag):
        for _ in range(count):
            steps(pair, grads, lr, "step", 1, "%s, step %d" % (tag, len(figures)))
            figures.append(pair.gpu.last_scalars()[:, 4 if op == "topk" else 2].copy())

    try:
        go(1e-4, 2, "start")
        for shrink in range(1, 5):
            pair.ref.X[:] = X0 * np.float32(1e-3 ** shrink)
            pair.ref.Xhat[:] = 0
            pair.force_state()
            go(0.0, 1, "failing")
        go(0.0, 12, "well again")
        if op == "topk":
            missed = [bool(np.any(b > a)) for a, b in zip(figures, figures[1:])]
        else:
            missed = bounds_missed(figures)
        held = held_back(missed)
        assert missed[1:5] == [True] * 4 and held[4] and not held[-1], (missed, held)
        if op == "qsgd":
            pair.ref.X[:] = pair.ref.Xhat + (pair.ref.X - pair.ref.Xhat) * np.float32(5)
            pair.force_state()
            go(0.0, 3, "grown")
    finally:
        pair.close()


@pytest.mark.gpu
@pytest.mark.timeout(300)
@pytest.mark.parametrize("op", ["topk", "qsgd"])
def test_one_pass_extreme_values(op):
    """Entries that carry a row by themselves (1e30), entries and a whole row below the normal range, zeros of both signs."""
    n, d = 8, 3_200_000
    X0 = synth.normal_state(n, d, seed=3)
    X0[1] *= np.float32(1e-39)
    X0[2, 5::1_000_000] = 1e30
    X0[:, 100_000:100_040] = 1e-42
    X0[:, 200_000:200_040] = -0.0
    X0[3, 300_000:1_300_000] = 0.0
    kw = dict(compressor=B.Q_TOPK, k=1500) if op == "topk" else dict(compressor=B.Q_QSGD, levels=8)
    pair = Pair(X0, synth.ring_csr(n), 0.3, seed=2, **kw)
    try:
        steps(pair, synth.GradientStream(n, d, seed=4), 0.0, "step", 3, "no gradient")
        steps(pair, synth.GradientStream(n, d, seed=4), 0.05, "step", 2, "gradient")
    finally:
        pair.close()
