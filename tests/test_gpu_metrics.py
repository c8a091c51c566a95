"""choco_metrics and choco_metrics_noalloc against the same sums in extended precision (64-bit
mantissa on x86), at the edges of their launches and on states that are hard to sum."""
import numpy as np
import pytest

from paper_1907_09356_amd import binding as B
from paper_1907_09356_amd import synth

pytestmark = pytest.mark.gpu


def state(n, d, kind, seed):
    rng = np.random.default_rng(seed)
    X = (0.05 + 1e-3 * rng.standard_normal((n, d))).astype(np.float32)
    if kind == "outlier":      # worker 0 far from the others, who agree
        X[0] = 7.0 + rng.random(d).astype(np.float32)
    elif kind == "late":       # ... the same with a worker of the second group of eight
        X[min(n - 1, 8)] = 7.0 + rng.random(d).astype(np.float32)
    elif kind == "offset":     # a common offset a million times the spread
        X += np.float32(1000.0)
    return X, X + (1e-2 * rng.standard_normal((n, d))).astype(np.float32)


def exact(X, H):
    X, H = X.astype(np.longdouble), H.astype(np.longdouble)
    xbar = X.mean(0)
    dev = ((X - xbar) ** 2).sum()
    return dict(consensus=dev / len(X), mean_norm=np.sqrt((xbar ** 2).sum()), psi=dev + ((X - H) ** 2).sum())


def open_ctx(X, H):
    import torch
    n, d = X.shape
    ld = (d + 3) // 4 * 4
    Xd = torch.full((n, ld), float("nan"), dtype=torch.float32, device="cuda:0")   # pad columns do not count
    Xd[:, :d] = torch.from_numpy(X).cuda()
    ctx = B.Choco(Xd, d, *synth.ring_csr(n), 0.3, B.Q_SIGN)
    ctx.xhat()[:, :d] = torch.from_numpy(H).cuda()
    return ctx


def check(ctx, X, H):
    import torch
    n = len(X)
    out = torch.empty(3, dtype=torch.float64, device="cuda:0")
    ctx.metrics_noalloc(out)
    got, want = ctx.metrics(), exact(X, H)
    assert list(out.cpu().numpy()) == [got["consensus"], got["mean_norm"], got["psi"]]
    # batches of eight rows, each with a few roundings that none of the later ones amplifies (a factor of
    # two at most), then a tree over the columns; the other two sums go row by row
    for key, terms in (("consensus", n / 4 + 40), ("mean_norm", n + 40), ("psi", n + 40)):
        err = abs(np.longdouble(got[key]) - want[key]) / want[key]
        assert err <= terms * 2.0 ** -53, (key, float(err), terms * 2.0 ** -53)


@pytest.mark.parametrize("n", [2, 8, 9, 16, 17, 64, 65, 100])
@pytest.mark.parametrize("d", [1, 3, 1024, 1025, 2048, 2049, 4099])
def test_edges_of_the_launches(n, d):
    X, H = state(n, d, "outlier" if (n + d) % 2 else "plain", seed=n * 10_000 + d)
    ctx = open_ctx(X, H)
    check(ctx, X, H)
    ctx.close()


@pytest.mark.parametrize("n,d", [(9, 37), (64, 1500), (1000, 37), (1000, 3000), (20_000, 5)])
@pytest.mark.parametrize("kind", ["plain", "outlier", "late", "offset"])
def test_no_digits_are_lost(n, d, kind):
    X, H = state(n, d, kind, seed=n + d)
    ctx = open_ctx(X, H)
    check(ctx, X, H)
    ctx.close()


def test_more_contexts_at_once_than_share_the_pinned_page():
    states = [state(2, 50, "plain", seed=s) for s in range(70)]
    ctxs = [open_ctx(*s) for s in states]
    for ctx, s in zip(ctxs[::-1], states[::-1]):
        check(ctx, *s)
    for ctx in ctxs[::2]:
        ctx.close()
    again = [open_ctx(*s) for s in states[:10]]
    for ctx, s in list(zip(ctxs[1::2], states[1::2])) + list(zip(again, states)):
        check(ctx, *s)
    for ctx in ctxs + again:
        ctx.close()
