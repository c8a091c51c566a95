"""Which kernels a configuration runs, and in what shape: the rules of the dispatch, on the CPU."""
import pytest

from tests.launches import recorded

pytestmark = pytest.mark.timeout(300)


def names(launches):
    return [l[0].split("<")[0] for l in launches]


def test_metrics_in_one_launch_only_where_one_workgroup_is_enough():
    out = recorded("""
out = {}
for n, d in ((1000, 1024), (64, 1025), (64, 2048), (65, 2048), (8, 2049), (8, 4096), (1000, 4096)):
    c = Context(n, d, B.Q_SIGN)
    out["%d %d" % (n, d)] = c.metrics()
    c.close()
""")
    one = {k for k, v in out.items() if len(v) == 1}
    assert one == {"1000 1024", "64 1025", "64 2048"}
    assert out["1000 1024"][0][:3] == ["k_metrics_small<256>", "1x1x1", "256x1x1"]
    assert out["64 2048"][0][:3] == ["k_metrics_small<512>", "1x1x1", "512x1x1"]
    for k, blocks in (("8 4096", 4), ("1000 4096", 4), ("65 2048", 2), ("8 2049", 3)):
        assert names(out[k]) == ["k_metrics_partial", "k_metrics_final"]
        assert out[k][0][1:3] == ["%dx1x1" % blocks, "256x1x1"]


def test_a_context_needs_no_pinned_memory():
    """... not even for its metrics: they are copied then (a kernel that does not run leaves zeros)."""
    out = recorded("""
stub.stub_fail_pinned(1)
c = Context(8, 5000, B.Q_SIGN)
out = [c.rc, len(c.step()), len(c.metrics()), c.figures]
stub.stub_fail_pinned(0)
d = Context(8, 5000, B.Q_SIGN)
out += [d.rc, len(d.metrics()), len(c.metrics()), c.figures]
""")
    assert out == [0, 2, 2, [0.0, 0.0, 0.0], 0, 2, 2, [0.0, 0.0, 0.0]]


def test_sixty_four_contexts_share_a_page_of_pinned_memory():
    out = recorded("""
cs = [Context(3, 64, B.Q_SIGN) for _ in range(64)]
out = [stub.stub_pinned_calls()]
more = [Context(3, 64, B.Q_SIGN) for _ in range(2)]       # no slot left: an allocation each
out += [stub.stub_pinned_calls(), [m.rc for m in more], [len(m.metrics()) for m in more]]
more[0].close(); cs[5].close(); cs[63].close()
again = [Context(3, 64, B.Q_SIGN) for _ in range(3)]      # the two slots given back, then one allocation
out += [stub.stub_pinned_calls(), [len(c.metrics()) for c in again]]
""")
    assert out == [1, 3, [0, 0], [1, 1], 4, [1, 1, 1]]


def test_what_the_narrow_tile_streams():
    """<.., x past the caches, update of xhat, xhat past the caches>"""
    out = recorded("""
out = {}
for n, d in ((64, 40_000), (64, 65_000), (64, 270_000), (64, 400_000)):
    for op, comp in (("topk", B.Q_TOPK), ("randk", B.Q_RANDK)):
        for order in (0, 1):
            c = Context(n, d, comp, k=d // 100, align=64, order=order)
            tiles = [l[0] for l in c.step() if l[0].startswith("k_tile_mix")]
            out["%s %d %d" % (op, d, order)] = tiles[0].split("<")[1].split(",", 2)[2][:-1] if tiles else ""
            c.close()
""")
    streamed, cached, hat = "true,true,true", "false,true,false", "true,true,false"
    assert [out["topk %d 0" % d] for d in (40_000, 65_000, 270_000, 400_000)] == [streamed, cached, streamed, streamed]
    assert [out["randk %d 0" % d] for d in (40_000, 65_000, 270_000, 400_000)] == [streamed, hat, hat, streamed]
    assert [out["randk %d 1" % d] for d in (40_000, 65_000, 270_000, 400_000)] == [
        "true,false,true", "false,false,false", "true,false,false", "true,false,true"]


def test_where_the_apply_pass_finishes_the_norms():
    """A launch of k_dense_finalise or none; above 16 workers the latter is for few tiles."""
    out = recorded("""
out = {}
for op, comp in (("sign", B.Q_SIGN), ("gsgd", B.Q_QSGD)):
    for n, tiles, align in ((8, 4096, 64), (16, 4096, 64), (20, 391, 64), (20, 586, 64), (20, 700, 64), (24, 300, 64),
                            (24, 300, 4), (24, 700, 4), (24, 1030, 4), (32, 513, 64), (40, 200, 64), (40, 500, 64), (40, 513, 64), (48, 200, 64), (48, 285, 64),
                            (24, 512, 64), (24, 513, 64), (64, 100, 64), (64, 180, 64), (64, 220, 64), (64, 100, 4), (64, 260, 4)):
        d = 256 * tiles - 64
        c = Context(n, d - (align == 4) * 5, comp, levels=16, align=align)
        l = c.step()
        assert len(l) == (3 if "k_dense_finalise" in names(l) else 2)
        out["%s %d %d %d" % (op, n, tiles, align)] = "k_dense_finalise" not in names(l)
        c.close()
""".replace("out = {}", "names = lambda l: [x[0].split('<')[0] for x in l]\nout = {}"))
    folded = {k for k, v in out.items() if v}
    assert folded == {
        "sign 8 4096 64", "sign 16 4096 64", "sign 20 391 64", "sign 20 586 64", "sign 24 300 64", "sign 24 300 4", "sign 24 700 4", "sign 24 512 64",
        "sign 40 200 64", "sign 40 500 64", "sign 48 200 64", "sign 64 180 64", "sign 64 100 4",
        "gsgd 8 4096 64", "gsgd 16 4096 64", "gsgd 24 300 4", "gsgd 40 200 64", "gsgd 64 100 4"}


def test_waves_and_rows_of_the_wide_tile():
    """Four waves of four rows for 9 to 12 workers, in the printed order's mix for 9 to 16, from 512 tiles on."""
    out = recorded("""
out = {}
for n in (8, 9, 12, 13, 16, 17):
    for tiles in (511, 512):
        for order in (0, 1):
            c = Context(n, 256 * tiles - 5, B.Q_SIGN, order=order)
            l = [x for x in c.step() if x[0].startswith("k_tile_mix" if order else "k_dense_apply_mix")]
            assert len(l) == 1
            rows, waves = map(int, l[0][0].split("<")[1].split(",")[1:3])
            assert l[0][2] == "%dx1x1" % (64 * waves) and rows * waves >= n
            out["%d %d %d" % (n, tiles, order)] = [rows, waves]
            c.close()
""")
    one = {8: [1, 8], 9: [1, 12], 12: [1, 12], 13: [1, 16], 16: [1, 16], 17: [2, 16]}
    for n in one:
        for order in (0, 1):
            assert out["%d 511 %d" % (n, order)] == one[n]
            assert out["%d 512 %d" % (n, order)] == ([4, 4] if 9 <= n <= (16 if order else 12) else one[n])


def test_layer_scales_are_made_exactly_once():
    """Either by a launch of k_layer_finalise or by the form of the apply kernel that makes them (its
    last parameter 2), whatever the tile; never by the apply pass where it takes several rows at a time."""
    out = recorded("""
out = {}
for n in (2, 8, 9, 12, 13, 16, 17, 32, 33, 64):
    for lengths in ([700, 65536, 3], [65537, 700], [256 * 511 // 2 - 40] * 2, [256 * 512 // 2 - 4] * 2, [60000] * 3):
        for align in (4, 32):
            t = synth.layer_table(lengths)
            for op, comp in (("sign", B.Q_SIGN), ("gsgd", B.Q_QSGD)):
                c = Context(n, synth.layers_dim(t), comp, layers=t, align=align, levels=16)
                l = [x[0] for x in c.step()]
                apply = [x for x in l if x.startswith("k_dense_apply_mix")]
                assert len(apply) == 1, l
                out["%s %d %s %d" % (op, n, lengths[:2], align)] = [
                    sum(x.startswith("k_layer_finalise") for x in l), int(apply[0].rstrip(">").split(",")[-1]), apply[0]]
                c.close()
""")
    assert len(out) == 200
    for key, (launches, layered, kernel) in out.items():
        assert (launches, layered) in ((1, 1), (0, 2)), key
        args = kernel.split("<")[1].split(",")
        if layered == 2:
            assert key.startswith("sign") and "65537" not in key and args[1] == "1", (key, kernel)
    assert sum(v[1] == 2 for v in out.values()) > 40


def test_narrow_tile_on_whole_lines_whatever_the_size():
    """Above 8 workers, rows and X on 128 bytes; otherwise the tile of 256 columns."""
    out = recorded("""
out = {}
for op, comp in (("topk", B.Q_TOPK), ("randk", B.Q_RANDK)):
    for n, d, align, off in ((16, 1000, 32, 0), (16, 400_000, 32, 0), (16, 540_000, 32, 0), (16, 1_000_000, 32, 0), (64, 120_000, 32, 0),
                             (64, 1000, 4, 0), (64, 1000, 32, 64), (8, 1000, 32, 0), (65, 1000, 32, 0)):
        c = Context(n, d, comp, k=10, align=align, x_off=off)
        l = [x[0].split("<")[0] for x in c.step()]
        out["%s %d %d %d %d" % (op, n, d, align, off)] = [x for x in l if "mix" in x]
        c.close()
""")
    for key, tile in out.items():
        n, d, align, off = map(int, key.split()[1:])
        want = "k_mix_incremental" if n > 64 else "k_tile_mix_narrow" if n > 8 and align == 32 and not off else "k_tile_mix"
        assert tile == [want], key


def test_where_the_update_is_formed_twice():
    """Streamed states (4 to 12 MB per array, above 96 MB), plain SGD; top_a on rows above 2^21 entries."""
    out = recorded("""
redo = lambda l: [x[0].rstrip(">").split(",")[-1] == "true" for x in l if x[0].startswith("k_sel_compact")]
out = {}
for n, d in ((1, 1 << 21), (1, (1 << 21) + 1), (2, (1 << 21) + 1), (9, (1 << 21) + 130), (12, (1 << 21) + 1)):
    c = Context(n, d, B.Q_TOPK, k=100, align=32)
    out["%d %d" % (n, d)] = redo(c.step()) + redo(c.step_momentum())
    c.close()
""")
    assert out == {"1 2097152": [False, False], "1 2097153": [True, False], "2 2097153": [False, False],
                   "9 2097282": [False, False], "12 2097153": [True, False]}


def test_metrics_blocks_fill_the_scratch_of_the_call_without_allocations():
    """1,024 blocks write all of it, five a small part (what the test of two calls in a row relies on)."""
    out = recorded("""
out = []
for n, d in ((2, 1_050_001), (5, 4100)):
    c = Context(n, d, B.Q_SIGN)
    out.append(c.metrics_noalloc())
    c.close()
""")
    assert [l[0][:2] for l in out] == [["k_metrics_partial", "1024x1x1"], ["k_metrics_partial", "5x1x1"]]


def test_many_neighbours_keep_the_narrow_tile():
    """Above 32 workers, or 256 tiles, the norms get a launch of their own on dense graphs."""
    out = recorded("""
out = {}
for n, d in ((24, 60_000), (24, 100_000), (33, 20_000), (48, 20_000)):
    for topo in ("ring", "complete"):
        c = Context(n, d, B.Q_SIGN, topo=synth.ring_csr(n) if topo == "ring" else synth.complete_csr(n), align=64)
        out["%d %d %s" % (n, d, topo)] = [x[0].split("<")[0] for x in c.step()]
        c.close()
""")
    folded = {k for k, v in out.items() if len(v) == 2}
    assert folded == {"24 60000 ring", "24 100000 ring", "33 20000 ring", "48 20000 ring", "24 60000 complete"}
    assert all(v[-1] == ("k_dense_apply_mix" if k in folded else "k_dense_apply_mix_narrow") for k, v in out.items())


def test_room_that_random_a_leaves_the_step():
    """The draw beside a step: workgroups that stay, one to a compute unit, two where a few would be left over."""
    out = recorded("""
out = {}
for n, d in ((2, 3_000_000), (8, 3_000_000), (9, 2_200_000), (12, 2_200_000), (13, 2_200_000), (64, 2_200_000), (8, 2_000_000), (9, 8_400_000)):
    c = Context(n, d, B.Q_RANDK, k=d // 100)
    out["%d %d" % (n, d)] = [l[1:] for l in c.step() if l[0] == "k_sel_draw"]
    c.close()
""")
    assert out == {"2 3000000": [["128x2x1", "256x1x1", "73728"]], "8 3000000": [["32x8x1", "256x1x1", "73728"]],
                   "9 2200000": [["32x9x1", "256x1x1", "49152"]], "12 2200000": [["32x12x1", "256x1x1", "49152"]],
                   "13 2200000": [["32x13x1", "256x1x1", "73728"]], "64 2200000": [["32x64x1", "256x1x1", "73728"]],
                   "8 2000000": [], "9 8400000": [["32x9x1", "256x1x1", "73728"]]}
