"""The launch shape a search takes by itself: what it may cost, and that it
never changes a result."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import to_dev

pytestmark = pytest.mark.gpu

LDS = 160 * 1024  # bytes of a CU


@pytest.fixture(scope="module")
def hn():
    import paper_2505_17368_amd as m
    m.load_library()
    return m


def _shape(index, nq, **kw):
    from paper_2505_17368_amd import henn
    return henn.search_shape(index, nq, **kw)


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _base_bits(ef):
    """Table size before any growth, for an index of one-byte tags."""
    return (10 if ef <= 64 else 11 if ef <= 256 else 12) + 1


@pytest.mark.parametrize("storage", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("d", [16, 24, 40, 100, 128])
def test_default_table_keeps_no_wave_out(hn, storage, d):
    """A visited table larger than the base size leaves LDS for every wave that
    the kernel's registers let a CU hold, or that the batch gives it."""
    idx = hn.henn_build(to_dev(wl.uniform(2000, d, 7)), degree=16, max_degree=32,
                        graph="knn_sym", storage=storage)
    grown = 0
    for ef in (16, 64, 84, 128, 140, 256, 300):
        for nq in (1, 300, 1000, 3000, 10_000, 30_000):
            s = _shape(idx, nq, k=10, ef=ef)
            waves = min(s.register_waves, -(-nq // _cus()))
            assert s.vis_bits >= _base_bits(ef)
            if s.vis_bits > _base_bits(ef):
                grown += 1
                assert s.lds_per_wave * waves <= LDS, (ef, nq, s.vis_bits, s.register_waves)
    assert grown > 0
    idx.free()


@pytest.mark.parametrize("storage", ["f32", "bf16", "fp8"])
def test_every_default_shape_gives_the_same_bits(hn, storage):
    """Batches on either side of each line of the default shape: all rows they
    have in common are equal, and the shapes do differ."""
    X = wl.gauss_mix(20_000, 100, 10, 0.3, 53)
    Qd = to_dev(wl.gauss_mix(8300, 100, 10, 0.3, 54))
    idx = hn.henn_build(to_dev(X), degree=32, max_degree=60, graph="knn_sym", storage=storage)
    for ef in (100, 200):
        sizes = (1, 257, 2048, 2049, 3072, 3073, 8192, 8193)
        shapes = [_shape(idx, nq, k=10, ef=ef) for nq in sizes]
        assert len({s.vis_bits for s in shapes}) > 1
        assert {s.list_blocks for s in shapes} == ({2} if ef == 100 else
                                                   {4} if storage == "f32" else {0, 4})
        if storage != "f32":
            assert len({s.lanes_per_vec for s in shapes}) > 1
        ref_i, ref_d = hn.henn_search_batch(idx, Qd[:8193], k=10, ef=ef)
        for nq in sizes:
            i, d = hn.henn_search_batch(idx, Qd[:nq], k=10, ef=ef)
            assert np.array_equal(i.cpu().numpy(), ref_i[:nq].cpu().numpy()), (ef, nq)
            assert np.array_equal(d.cpu().numpy().view(np.uint32),
                                  ref_d[:nq].cpu().numpy().view(np.uint32)), (ef, nq)
    idx.free()


@pytest.mark.parametrize("n,d,storage,nq,ef", [(20_000, 128, "f32", 2000, 250),
                                               (20_000, 40, "fp8", 64, 500),
                                               (5000, 32, "bf16", 500, 64)])
def test_tuned_index_keeps_the_best_tried_or_the_default(hn, n, d, storage, nq, ef):
    """What a tuned index runs is either the shape the tuner returns or, in its
    table or as a whole, the untuned shape; other beam widths stay untuned."""
    X = wl.uniform(n, d, 71)
    Qd = to_dev(wl.uniform(nq, d, 72))
    idx = hn.henn_build(to_dev(X), degree=24, max_degree=48, graph="knn_sym", storage=storage)

    def fields(s):
        return s.lanes_per_vec, s.waves_per_block, s.vis_bits, bool(s.persistent)

    plain = fields(_shape(idx, nq, k=10, ef=ef))
    other = fields(_shape(idx, nq, k=10, ef=8 * ef if ef <= 256 else 16))
    ref_i, ref_d = hn.henn_search_batch(idx, Qd, k=10, ef=ef)
    t = hn.henn_autotune(idx, Qd, k=10, ef=ef)
    tuned = t["lanes_per_vec"], t["waves_per_block"], t["vis_bits"], t["persistent"]
    assert 8 <= t["vis_bits"] <= 12
    own_table = fields(_shape(idx, nq, k=10, ef=ef, lanes_per_vec=t["lanes_per_vec"],
                              waves_per_block=t["waves_per_block"], persistent=t["persistent"]))
    now = fields(_shape(idx, nq, k=10, ef=ef))
    assert now in (plain, tuned, own_table)
    assert fields(_shape(idx, nq, k=10, ef=8 * ef if ef <= 256 else 16)) == other
    i, dd = hn.henn_search_batch(idx, Qd, k=10, ef=ef)
    assert np.array_equal(i.cpu().numpy(), ref_i.cpu().numpy())
    assert np.array_equal(dd.cpu().numpy().view(np.uint32), ref_d.cpu().numpy().view(np.uint32))
    idx.free()
