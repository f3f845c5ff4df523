"""Searches of rows of more than 512 coordinates (more than 64 chunks: eight
chunks per lane) in every storage form, list form and launch form."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hn():
    import paper_2505_17368_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("metric", [0, 1])
@pytest.mark.parametrize("d", [513, 600, 768, 1024])
def test_wide_rows_of_exact_codes_search_the_same_in_every_storage(hn, d, metric):
    """Integers in [-7, 7] with a 7 in every row are exact in FP32, BF16 and
    (scaled by 2^-6) FP8, and with integer queries in [-20, 20] so is every
    distance: sums of squares stay below 1024 * 27^2 < 2^20, scaled products
    below 1024 * 64 * 7 * 20 < 2^24.  So the storages return the same bits, for
    one query and for batches, with the list in registers and in LDS, with
    per-query times asked for, and in the persistent form."""
    import torch
    rng = np.random.default_rng(78)
    n = 3000
    X = rng.integers(-7, 8, size=(n, d)).astype(np.float32)
    X[np.arange(n), rng.integers(0, d, size=n)] = 7.0
    Q = rng.integers(-20, 21, size=(1200, d)).astype(np.float32)
    kw = dict(degree=16, metric=metric, graph="knn_sym", max_degree=32)
    base = hn.henn_build(to_dev(X), **kw)
    ex = [base.export_layer(i) for i in range(base.num_layers)]
    base.free()
    ref = {}
    for storage in ("f32", "bf16", "fp8"):
        idx = hn.henn_import(to_dev(X), [e[0] for e in ex], [e[1] for e in ex], storage=storage,
                             **kw)
        for ef in (32, 200, 300):  # two blocks of registers, four, LDS
            for nq, form in ((1200, {}), (1, {}), (300, {}), (300, dict(with_times=True)),
                             (300, dict(persistent=True)), (65, dict(exact_visited=True))):
                print(storage, ef, nq, form, flush=True)
                out = hn.henn_search_batch(idx, to_dev(Q[:nq]), k=10, ef=ef, **form)
                torch.cuda.synchronize()
                got = out[0].cpu().numpy(), out[1].cpu().numpy().view(np.uint32)
                if "with_times" in form:
                    assert (out[2].cpu().numpy() > 0).all()
                # the first storage's largest batch is the reference
                want = ref.setdefault((ef, "exact_visited" in form), got)
                m = min(nq, want[0].shape[0])
                for a, b in zip(got, want):
                    assert np.array_equal(a[:m], b[:m]), (storage, ef, nq, form)
        idx.free()
