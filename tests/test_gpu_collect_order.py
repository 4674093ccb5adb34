"""wpm_collect at the sizes where its path changes: results below and above the
key-range split (4096 of an instance), lists that are prefixes of others (cycle
unions), more than 128 facets, against the oracle and Python's own sort."""
import itertools

import numpy as np
import pytest

import oracle as O
import wpm_inputs as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_00806_amd import engine
    return engine


@pytest.mark.parametrize("v", [4, 7, 8])
def test_cycle_unions(E, v):
    # K_v: unions of disjoint cycles, so that one list can be a prefix of another
    F = [(1 << a) | (1 << b) for a, b in itertools.combinations(range(v), 2)]
    p = E.prepare(2, v, facets=F, max_facets=0)
    _, sets = E.sweep([p])
    assert sets[0] == O.enumerate_wpm(2, F, 0)
    prefixes = sum(a == b[:len(a)] for a, b in zip(sets[0], sets[0][1:]))
    assert (prefixes > 0) == (v >= 6)


def test_many_results_in_mixed_batch(E):
    # one instance with tens of thousands of results among small ones, and one
    # with more than 128 facets
    insts = [i for i in W.batch(E.kdim, count=64) if i.meta["k"] <= 14][:6] + [W.single(E.kdim)]
    insts += [i for i in W.batch(E.kdim, count=256) if i.meta["k"] == 20 and i.n == 7][:1]
    preps = E.prepare_many(insts)
    assert len(preps[-1].facets) > 128
    res, sets = E.sweep(preps, cbits=10)
    assert max(res.counts) > 8192 and min(res.counts) < 4096
    for p, got, n in zip(preps, sets, res.counts):
        assert len(got) == n and got == O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets)


def test_sizes_only_and_short_output(E):
    import ctypes
    from paper_2301_00806_amd import _lib as L
    p = E.prepare(3, 7, lam=W.fano().lam)
    batch = E.DeviceBatch([p])
    sw = E.Sweeper(batch, cap=4096)
    sw.set_items(E.build_queue(batch.k, 7, 64))
    sw.launch(L.SCHED_DYNAMIC, wg_size=64)
    counts, words, offs = sw.collect_raw()
    hosts, _ = batch.host_views()
    h = np.zeros(1, np.uint64)
    need, o2, out = ctypes.c_int64(0), np.zeros(2, np.int64), np.zeros(len(words), np.uint32)
    call = lambda buf, cap: L.lib().wpm_collect(
        hosts, 1, sw.surv.data_ptr(), sw.cap, sw.counts.data_ptr(), sw.total.data_ptr(), E._ptr(h, L.c_u64p),
        buf, cap, ctypes.byref(need), E._ptr(o2, L.c_i64p), None)
    assert call(None, 0) == L.WPM_ECAP and need.value == len(words) and list(o2) == list(offs)
    assert call(E._ptr(out), len(words) - 1) == L.WPM_ECAP and not out.any()
    assert call(E._ptr(out), len(words)) == L.WPM_OK and np.array_equal(out, words) and h[0] == counts[0]
