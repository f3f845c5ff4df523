"""Serving form: continuous batching with memory-based admission.  Each
request's result is the same alone, in a mix of concurrent requests with
other k / beam widths, and in a plain batched search with the same shape."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import paper_2505_17368_amd as hn
    X, Q = wl.make("uniform_10k_d32")
    idx = hn.henn_build(to_dev(X), degree=16, graph=1, max_degree=32, root_complete_max=1000,
                        storage=1)
    yield hn, X, Q, idx
    idx.free()


def _batch(hn, idx, Q, k, ef):
    import torch
    gi, gd = hn.henn_search_batch(idx, to_dev(Q), k=k, ef=ef, k_max=10, ef_max=64, vis_bits=10)
    torch.cuda.synchronize()
    return gi.cpu().numpy(), gd.cpu().numpy()


def _drain(srv, expected):
    got = {}
    for _ in range(100000):
        srv.tick()
        tags, ids, dist = srv.poll()
        for t, i, d in zip(tags, ids, dist):
            got[int(t)] = (i.copy(), d.copy())
        if len(got) == expected:
            return got
    raise AssertionError("server did not finish")


def test_alone_equals_batch(setup):
    hn, X, Q, idx = setup
    ref_i, ref_d = _batch(hn, idx, Q[:8], 10, 64)
    for j in range(8):
        srv = hn.Server(idx, max_slots=4, k_max=10, ef_max=64, steps_per_tick=5, vis_bits=10)
        srv.submit(Q[j], 10, 64, j)
        got = _drain(srv, 1)
        assert np.array_equal(got[j][0], ref_i[j])
        assert np.array_equal(got[j][1].view(np.uint32), ref_d[j].view(np.uint32))
        srv.close()


def test_mix_with_staggered_arrivals_and_memory_admission(setup):
    hn, X, Q, idx = setup
    n = 300
    rng = np.random.default_rng(7)
    ks = rng.choice([1, 5, 10], size=n)
    efs = rng.choice([16, 32, 64], size=n)
    refs = {}
    for kk in (1, 5, 10):
        for ee in (16, 32, 64):
            sel = np.where((ks == kk) & (efs == ee))[0]
            if len(sel):
                bi, bd = _batch(hn, idx, Q[sel], kk, ee)
                for r, qi in enumerate(sel):
                    refs[int(qi)] = (bi[r], bd[r])
    # a pool with room for ~20 requests of the largest state: admission waits on memory
    srv = hn.Server(idx, max_slots=64, pool_bytes=20 * (512 + 4096), k_max=10, ef_max=64,
                    steps_per_tick=7, vis_bits=10)
    got = {}
    submitted = 0
    for tick in range(100000):
        burst = int(rng.integers(0, 9))
        for _ in range(burst):
            if submitted < n:
                srv.submit(Q[submitted], int(ks[submitted]), int(efs[submitted]), submitted)
                submitted += 1
        srv.tick()
        st = srv.stats()
        assert st["active"] <= 64 and st["pool_bytes_used"] <= 20 * (512 + 4096)
        tags, ids, dist = srv.poll()
        for t, i, d in zip(tags, ids, dist):
            got[int(t)] = (i.copy(), d.copy())
        if len(got) == n:
            break
    assert len(got) == n
    st = srv.stats()
    assert st["max_active"] > 1          # requests overlapped on the device
    # memory bounded the batch: the smallest request state (list of 16 keys +
    # 1,024-entry visited table of 16-bit tags on this index, 256-aligned)
    smallest = -(-(16 * 8 + 1024 * 2) // 256) * 256
    assert st["max_active"] <= 20 * 4608 // smallest < 64
    for qi, (ids, dist) in got.items():
        ri, rd = refs[qi]
        assert np.array_equal(ids, ri), qi
        assert np.array_equal(dist.view(np.uint32), rd.view(np.uint32)), qi
    srv.close()


def test_waves_separated_by_idle_ticks(setup):
    """A wave that finishes within one step, then ticks with nothing active,
    then a second wave into the same slots: every request gets its own
    result (the completion counter a step counts into starts from zero
    whatever the ticks in between did)."""
    hn, X, Q, idx = setup
    ref_i, ref_d = _batch(hn, idx, Q[:32], 10, 64)
    srv = hn.Server(idx, max_slots=16, k_max=10, ef_max=64, steps_per_tick=100000, vis_bits=10)
    got = {}
    for wave in range(2):
        for j in range(16 * wave, 16 * wave + 16):
            srv.submit(Q[j], 10, 64, j)
        for _ in range(4):  # the step, its retirement, then idle ticks
            srv.tick()
            tags, ids, dist = srv.poll()
            for t, i, d in zip(tags, ids, dist):
                got[int(t)] = (i.copy(), d.copy())
        assert len(got) == 16 * (wave + 1)
        assert srv.stats()["active"] == 0
    srv.close()
    for j in range(32):
        assert np.array_equal(got[j][0], ref_i[j]), j
        assert np.array_equal(got[j][1].view(np.uint32), ref_d[j].view(np.uint32)), j


def test_cancel_waiting_and_admitted_requests(setup):
    """Cancelled requests return nothing; every other request still equals
    the batch search, and the freed slots and bytes are reused."""
    hn, X, Q, idx = setup
    n = 96
    ref_i, ref_d = _batch(hn, idx, Q[:n], 10, 64)
    srv = hn.Server(idx, max_slots=16, k_max=10, ef_max=64, steps_per_tick=4, vis_bits=10)
    for j in range(n):
        srv.submit(Q[j], 10, 64, j)
    waiting = [40, 41, 95]
    assert [srv.cancel(t) for t in waiting] == [1, 1, 1]
    srv.tick()  # admits 0..15, launches their first step
    admitted = [3, 7]
    assert [srv.cancel(t) for t in admitted] == [2, 2]
    assert srv.cancel(1000) == 0
    got = {}
    for _ in range(100000):
        srv.tick()
        tags, ids, dist = srv.poll()
        for t, i, d in zip(tags, ids, dist):
            got[int(t)] = (i.copy(), d.copy())
        if srv.stats()["pending"] == 0 and srv.stats()["active"] == 0 and \
                len(got) == n - len(waiting) - len(admitted):
            break
    st = srv.stats()
    srv.close()
    assert st["cancelled"] == 5 and st["pool_bytes_used"] == 0
    assert set(got) == set(range(n)) - set(waiting) - set(admitted)
    for j in got:
        assert np.array_equal(got[j][0], ref_i[j]), j
        assert np.array_equal(got[j][1].view(np.uint32), ref_d[j].view(np.uint32)), j


@pytest.mark.parametrize("storage", [0, 2])
def test_serving_and_captured_graph_after_updates(storage):
    """After Delete(x) and Insert(x) on an NSW index, the serving form and a
    captured search graph (both created afterwards) return the batched
    search's ids, which are point ids, not layer positions."""
    import torch

    import paper_2505_17368_amd as hn
    X = wl.uniform(6000, 16, 81)
    Xn = wl.uniform(1000, 16, 82)
    Q = wl.uniform(64, 16, 83)
    idx = hn.henn_build(to_dev(X), degree=8, max_degree=16, graph=4, storage=storage,
                        root_complete_max=400)
    gone = np.arange(0, 6000, 4, dtype=np.int32)
    # a server and a graph made before the updates refuse to run after them
    # (the check is on the host: nothing is launched)
    old_srv = hn.Server(idx, max_slots=16, k_max=10, ef_max=64, steps_per_tick=8)
    old_g = hn.SearchGraph(idx, to_dev(Q), k=10, ef=64, k_max=10, ef_max=64)
    hn.henn_delete(idx, gone)
    hn.henn_insert(idx, to_dev(Xn))
    with pytest.raises(hn.HennError):
        old_srv.tick()
    with pytest.raises(hn.HennError):
        old_g.launch()
    old_srv.close()
    old_g.free()
    ref_i, ref_d = _batch(hn, idx, Q, 10, 64)
    assert not np.isin(ref_i, gone).any() and (ref_i >= 6000).any()
    srv = hn.Server(idx, max_slots=16, k_max=10, ef_max=64, steps_per_tick=8, vis_bits=10)
    for j in range(len(Q)):
        srv.submit(Q[j], 10, 64, j)
    got = _drain(srv, len(Q))
    srv.close()
    for j in range(len(Q)):
        assert np.array_equal(got[j][0], ref_i[j]), j
        assert np.array_equal(got[j][1].view(np.uint32), ref_d[j].view(np.uint32)), j
    g = hn.SearchGraph(idx, to_dev(Q), k=10, ef=64, k_max=10, ef_max=64)
    for _ in range(3):
        g.launch()
        torch.cuda.synchronize()
        assert np.array_equal(g.ids.cpu().numpy(), ref_i)
    g.free()
    idx.free()


def test_upper_layer_beam_wider_than_the_request_list():
    """A server whose beam above layer 0 (ef_upper = 16) is wider than a
    request's own list (k = 1, ef = 8): each request's state holds the wider
    list, and the result alone, in a mix and in the batched search agree."""
    import torch

    import paper_2505_17368_amd as hn
    X, Q = wl.make("uniform_10k_d32")
    idx = hn.henn_build(to_dev(X), degree=16, graph=1, max_degree=32)
    assert idx.num_layers >= 3             # greedy layers above layer 0
    Qs = Q[:48]
    ref_i, ref_d = hn.henn_search_batch(idx, to_dev(Qs), k=1, ef=8, k_max=10, ef_max=64,
                                        ef_upper=16, vis_bits=10)
    torch.cuda.synchronize()
    ref_i, ref_d = ref_i.cpu().numpy(), ref_d.cpu().numpy()
    kw = dict(k_max=10, ef_max=64, ef_upper=16, steps_per_tick=3, vis_bits=10)
    for j in (0, 5):
        srv = hn.Server(idx, max_slots=4, **kw)
        srv.submit(Qs[j], 1, 8, j)
        got = _drain(srv, 1)
        srv.close()
        assert np.array_equal(got[j][0], ref_i[j]), j
        assert np.array_equal(got[j][1].view(np.uint32), ref_d[j].view(np.uint32)), j
    srv = hn.Server(idx, max_slots=32, **kw)
    efs = [8, 64, 8, 32]
    ks = [1, 10, 1, 5]
    for j in range(len(Qs)):
        srv.submit(Qs[j], ks[j % 4], efs[j % 4], j)
    got = _drain(srv, len(Qs))
    srv.close()
    for j in range(len(Qs)):
        if ks[j % 4] != 1 or efs[j % 4] != 8:
            continue
        assert np.array_equal(got[j][0], ref_i[j]), j
        assert np.array_equal(got[j][1].view(np.uint32), ref_d[j].view(np.uint32)), j
    idx.free()


def test_list_changes_its_place_while_requests_are_in_flight(setup):
    """Beams of 129 to 256: a tick of many requests (over eight a CU) keeps the
    lists in LDS, one of few in registers.  Requests that are saved under one
    form and go on under the other return what a plain search returns."""
    hn, X, Q, idx = setup
    import torch
    line = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    n = line + 700
    Qm = wl.uniform(n, 32, 61)
    rng = np.random.default_rng(9)
    ks = rng.choice([1, 10], size=n).astype(np.int32)
    efs = rng.choice([16, 60, 130, 200], size=n).astype(np.int32)
    srv = hn.Server(idx, max_slots=n, pool_bytes=64 << 20, k_max=10, ef_max=200,
                    steps_per_tick=7)
    srv.submit_batch(Qm, ks, efs, np.arange(n, dtype=np.int64))
    got, active = {}, []
    while len(got) < n:
        active.append(srv.tick())
        for t, i, d in zip(*srv.poll()):
            got[int(t)] = (i.copy(), d.copy())
        assert len(active) < 100000
    assert max(active) > line and any(0 < a <= line for a in active)
    gi, gd = hn.henn_search_batch(idx, to_dev(Qm), k_arr=to_dev(ks), ef_arr=to_dev(efs), k_max=10,
                                  ef_max=200)
    gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    for j in range(n):
        assert np.array_equal(got[j][0], gi[j]), j
        assert np.array_equal(got[j][1].view(np.uint32), gd[j].view(np.uint32)), j
    srv.close()
