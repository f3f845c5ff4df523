"""The kNN build's Gram forms: what the proof of each shortlist rests on, and
the order in which the forms take over from each other."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hn():
    import paper_2505_17368_amd as m
    m.load_library()
    return m


def _layer0(hn, Xd, **kw):
    idx = hn.henn_build(Xd, max_layers=0, **kw)
    adj = idx.export_layer(0)[1]
    idx.free()
    return adj


@pytest.mark.parametrize("d,scale", [(4, 1e-19), (8, 1e-19), (8, 3e-19), (8, 1.0), (8, 1e15)])
def test_fp16_residuals_of_small_and_large_rows(hn, d, scale):
    """Two tight groups far from the layer's mean, so that rows are near each
    other against their norms.  At 1e-19 the squared FP16 residuals of the rows
    are below the smallest FP32 number although the squared distances are not:
    the proof has to hold all the same.  Checked against FP64: no neighbour
    that was left out is nearer than the farthest listed one by more than the
    canonical FP32 distance's own rounding (d <= 8 coordinates: each
    difference within 2^-24, each square and sum within 2^-24 relative or half
    a subnormal step, 2^-150), for both distances of the comparison."""
    n, R = 3000, 16
    g = np.random.default_rng(1)
    u = g.standard_normal(d)
    u /= np.linalg.norm(u)
    sign = g.integers(0, 2, n) * 2 - 1
    X = ((sign[:, None] * u + 0.05 / np.sqrt(d) * g.standard_normal((n, d))) * scale).astype(
        np.float32)
    adj = _layer0(hn, to_dev(X), degree=R)
    assert (adj >= 0).all()
    X64 = X.astype(np.float64)
    bad = []
    for r in range(n):
        D = ((X64 - X64[r]) ** 2).sum(1)
        D[r] = np.inf
        true = np.partition(D, R - 1)[R - 1]
        worst = D[adj[r]].max()
        tol = 2 * (worst * (2 + d) * 2.0 ** -23 + d * 2.0 ** -150)
        if worst > true + tol:
            bad.append((r, worst, true))
    assert not bad, f"{len(bad)} rows of {n} miss a nearer neighbour, first {bad[0]}"


def test_layers_of_several_launches(hn):
    """More rows than one launch takes (4,096 blocks): the lists are kept for a
    launch's rows only.  FP16 first and FP32 alone give the same graph."""
    g = np.random.default_rng(3)
    X = g.standard_normal((4096 * 128 + 5000, 8)).astype(np.float32)
    Xd = to_dev(X)
    assert np.array_equal(_layer0(hn, Xd, degree=17), _layer0(hn, Xd, degree=17, gram=1))


@pytest.mark.parametrize("n,d,metric,degree", [(26_000, 16, 0, 16), (33_003, 40, 1, 32),
                                               (33_001, 130, 0, 8), (66_001, 8, 0, 32),
                                               (65_700, 140, 1, 5)])
@pytest.mark.parametrize("kind", ["scales", "gauss", "mixed"])
def test_pilot_keeps_or_rejects_the_fp16_form(hn, n, d, metric, degree, kind):
    """Layers without a pilot, with a small one and with one of 256 blocks:
    rows of one scale, where the FP16 form goes on; rows of very different
    scales, where the next form takes the whole layer; and a pilot of one kind
    before a layer of the other.  The graph is that of FP32 tiles alone, with no tolerance."""
    g = np.random.default_rng(n + d)
    X = g.standard_normal((n, d)).astype(np.float32)
    scale = np.exp2(g.integers(-12, 13, size=(n, 1))).astype(np.float32)
    if kind == "scales":
        X *= scale
    elif kind == "mixed":
        X[n * 5 // 9:] *= scale[n * 5 // 9:]
    Xd = to_dev(X)
    kw = dict(degree=degree, metric=metric)
    assert np.array_equal(_layer0(hn, Xd, **kw), _layer0(hn, Xd, gram=1, **kw))
