"""Tables without a level section on the GPU: the walk of every vector, alone
and in one launch with descended tables, against the oracle.

The packer gives nearly every table a level section, so these tests take the
bit that announces it out of the header (the rest of the table does not
depend on it) and check which kernel a batch gets."""
import copy
import ctypes

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


def walked(p):
    """The instance with a table that is walked."""
    q = copy.copy(p)
    q.table = p.table.copy()
    q.table[11] &= ~np.uint32(2)
    return q


def oracle_sets(preps):
    return [O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets) for p in preps]


def sorted_records(surv, total):
    rec = surv[:int(total[1])].cpu().numpy()
    rec = rec[rec[:, 1] != -1]
    return rec[np.lexsort((rec[:, 0], rec[:, 1]))]


# ------------------------------------------------- both kinds in one launch

def mixed(E):
    insts = [i for i in W.batch(E.kdim, count=64) if 12 <= i.meta["k"] <= 14][:6]
    preps = E.prepare_many(insts)
    assert all(E.descended(p) for p in preps)
    preps = [walked(p) if j % 3 == 1 else p for j, p in enumerate(preps)]
    assert [E.descended(p) for p in preps] == [True, False, True] * 2
    return preps


@pytest.mark.parametrize("mode,grid", [(0, 0), (1, 7), (1, 0), (2, 1), (2, 3), (2, 17), (2, 0), (3, 5)])
@pytest.mark.parametrize("cbits", [7, 10])
def test_mixed_launch(E, mode, grid, cbits):
    from paper_2301_00806_amd import _lib as L
    preps = mixed(E)
    batch = E.DeviceBatch(preps)
    assert batch.c_batch.flags == 0
    one = E.build_queue(batch.k, cbits, 64)
    # each kind's malformed items: chunk bits below 7, a lane window across an
    # aligned group, chunks beyond 2^k; and instances that are not there
    bad = np.zeros(8, dtype=E.ITEM_DTYPE)
    for j, i in enumerate((0, 1)):
        bad[3 * j:3 * j + 3] = [(i, 5, 64, 0), (i, 7, 64, 480), (i, 7, 64, 1 << (preps[i].k - 7))]
    bad[6:] = [(len(preps), 7, 64, 0), (1 << 31, 7, 64, 0)]
    rep = 40 if cbits == 7 else 3
    if mode == 0:
        items = np.concatenate([one, bad[:6]])  # (plain mode refuses unknown instances)
        items = items[np.argsort(items["instance"], kind="stable")]
        rep = 1
    else:
        items = np.concatenate([np.concatenate([one] * rep), bad])
        items = items[np.random.default_rng(3).permutation(len(items))]
    nbad = len(items) - rep * len(one)
    bins = np.linspace(0, len(items), grid + 1).astype(np.int64) if mode == 3 else None
    d_bins = None if bins is None else torch.from_numpy(bins).to("cuda")
    d_items = torch.from_numpy(items.view(np.int64).reshape(-1).copy()).to("cuda")
    counts = torch.full((len(preps),), 7, dtype=torch.int64, device="cuda")
    total = torch.full((L.TOTAL_WORDS,), 7, dtype=torch.int64, device="cuda")
    surv = torch.empty((1 << 20, 2), dtype=torch.int64, device="cuda")
    scratch = torch.full((L.QUEUE_SCRATCH_WORDS // 2,), 5, dtype=torch.int64, device="cuda")
    want = oracle_sets(preps)
    for words in (0, L.QUEUE_SCRATCH_WORDS):
        s = L.Sched(mode=mode, wg_size=64, grid=grid, flags=0, d_items=d_items.data_ptr(),
                    h_items=items.ctypes.data, num_items=len(items), d_scratch=scratch.data_ptr(),
                    scratch_words=words, d_bin_offsets=None if bins is None else d_bins.data_ptr())
        print(f"[gpu] mixed launch mode {mode} grid {grid} items {len(items)}", flush=True)
        L.check("enumerate", L.lib().wpm_enumerate(
            ctypes.byref(batch.c_batch), ctypes.byref(s), surv.data_ptr(), 1 << 20, counts.data_ptr(),
            total.data_ptr(), None, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        torch.cuda.synchronize()
        tot = total.cpu().tolist()
        assert tot[2] == nbad
        assert counts.cpu().tolist() == [rep * len(w) for w in want] and tot[0] == rep * sum(map(len, want))
        rec = sorted_records(surv, total)
        assert len(rec) == tot[0]
        uniq, times = np.unique(rec, axis=0, return_counts=True)
        assert (times == rep).all() and len(uniq) == sum(map(len, want))


# ------------------------------------------ descended tables under the walk

@pytest.mark.parametrize("mode", [1, 2, 3])
def test_walk_flag_gives_the_same_sweep(E, mode):
    # tables of both kinds, walked in one launch
    from paper_2301_00806_amd import _lib as L
    preps = mixed(E)
    batch = E.DeviceBatch(preps)
    items = E.build_queue(batch.k, 9, 128)
    bins = torch.from_numpy(np.linspace(0, len(items), 6).astype(np.int64)).to("cuda")
    sw = E.Sweeper(batch, cap=1 << 20)
    sw.set_items(items, split_classes=False)
    for flags in (0, L.FLAG_WALK):
        s = L.Sched(mode=mode, wg_size=128, grid=5, flags=flags, d_items=sw._items_dev.data_ptr(),
                    num_items=len(items), d_scratch=sw.scratch.data_ptr(), d_bin_offsets=bins.data_ptr())
        L.check("enumerate", L.lib().wpm_enumerate(
            ctypes.byref(batch.c_batch), ctypes.byref(s), sw.surv.data_ptr(), sw.cap, sw.counts.data_ptr(),
            sw.total.data_ptr(), sw.stats.data_ptr(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
        res = sw.result()
        assert (res.stats[5:8] == 0).all() == (flags == L.FLAG_WALK)
        assert sw.collect() == oracle_sets(preps)


@pytest.mark.parametrize("mode", [1, 3])
def test_short_items_are_walked_in_static_and_packed_launches(E, mode):
    from paper_2301_00806_amd import scheduler as S
    insts = [i for i in W.batch(E.kdim, count=160) if 16 < i.meta["k"] <= 24]
    preps = E.prepare_many(insts, prune=True, min_free=7)
    preps = [p for p in preps if E.descended(p)]
    batch = E.DeviceBatch(preps)
    sw = E.Sweeper(batch, cap=1 << 22)
    plan = S.make_plan(batch, {1: "static", 3: "packed"}[mode], cbits=7, wg=256)
    assert plan.mode == mode
    assert [E.walks_short_items(plan.items[s.start:s.end], 256, len(preps)) for s in plan.segments] == [True]
    want = [O.count_wpm(p.n, [int(f) for f in p.facets], p.max_facets) for p in preps]
    sw.set_items(plan.items, segments=plan.segments)
    for _ in range(2):
        sw.launch(mode, wg_size=256)
        res = sw.result()
        assert [int(c) for c in res.counts] == want and (res.stats[5:8] == 0).all()
    sw.launch_fetch(mode, wg_size=256)
    assert [int(c) for c in sw.result().counts] == want
