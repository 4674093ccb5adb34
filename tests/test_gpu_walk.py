"""Tables without a level section on the GPU: the walk of every vector, alone
and in one launch with descended tables, against the oracle.

The packer gives every table a level section, so these tests take the bit that
announces it out of the header (the rest of the table does not depend on it)
and check which kernel a batch gets."""
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
    assert all(E.descended(p) for p in preps)
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


# ----------------------------------------------------------- the walk alone

def walk_batch(E, preps):
    from paper_2301_00806_amd import _lib as L
    preps = [walked(p) for p in preps]
    batch = E.DeviceBatch(preps)
    assert batch.c_batch.flags == L.BATCH_WALK
    assert all(b.flags == L.BATCH_WALK for b in batch.class_batches.values())
    return preps, batch


def sweep(E, preps, mode=2, cbits=10, wg=256, waves=0, cap=1 << 22, split=True, **kw):
    """Sets and result of a sweep of the instances, all of them walked."""
    preps, batch = walk_batch(E, preps)
    sw = E.Sweeper(batch, cap=cap)
    sw.set_items(E.build_queue(batch.k, cbits, wg, blocks=batch.blocks, **kw), split_classes=split)
    print(f"[gpu] walk of {len(preps)} instances, mode {mode} cbits {cbits} wg {wg} waves {waves}", flush=True)
    sw.launch(mode, wg_size=wg, waves=waves)
    res = sw.result()
    assert (res.stats[5:8] == 0).all()  # (the descent opens sub-cubes)
    return sw.collect(), res


def graphs(E, sizes=(5, 6, 7, 8), **kw):
    import itertools
    return [E.prepare(2, v, facets=[(1 << a) | (1 << b) for a, b in itertools.combinations(range(v), 2)],
                      max_facets=0, **kw) for v in sizes]


@pytest.mark.parametrize("waves", [7, 8])
@pytest.mark.parametrize("cbits,wg", [(13, 128), (10, 512), (7, 64), (12, 256)])
def test_walk_matches_oracle_under_both_register_budgets(E, waves, cbits, wg):
    insts = [i for i in W.batch(E.kdim, count=96) if i.meta["k"] <= 20][:16]
    preps = E.prepare_many(insts)
    sets, res = sweep(E, preps, cbits=cbits, wg=wg, waves=waves)
    want = oracle_sets(preps)
    assert sets == want and list(res.counts) == [len(w) for w in want]


@pytest.mark.parametrize("waves", [7, 8])
def test_walk_across_segments_and_full_lists(E, waves):
    # chunks of 2^14 steps cross the 4096-step segments; complete graphs fill the
    # candidate lists, so that overflow steps are rechecked (stats[4])
    inst = W.single(E.kdim)
    p = E.prepare(inst.n, inst.m, lam=inst.lam)
    sets, _ = sweep(E, [p], cbits=14, wg=64, waves=waves)
    assert sets == oracle_sets([p])
    preps = graphs(E)
    sets, res = sweep(E, preps, cbits=12, waves=waves)
    assert sets == oracle_sets(preps) and int(res.stats[4]) > 0


@pytest.mark.parametrize("waves", [7, 8])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("kind", ["walked", "descended"])
def test_sweep_without_critical_ridges(E, waves, mode, kind):
    # six disjoint K_4 have no critical ridge: every vector is a complex
    from paper_2301_00806_amd import _lib as L
    import itertools
    F = [(1 << (4 * g + a)) | (1 << (4 * g + b)) for g in range(6) for a, b in itertools.combinations(range(4), 2)]
    p = E.prepare(2, 24, facets=F, max_facets=0)
    assert p.k == 18 and p.info.n_crit == 0
    batch = E.DeviceBatch([walked(p) if kind == "walked" else p])
    assert batch.c_batch.flags == (L.BATCH_WALK if kind == "walked" else L.BATCH_TREE)
    sw = E.Sweeper(batch, cap=1 << 19)
    sw.set_items(E.build_queue(batch.k, 8, 128))
    sw.launch(mode, wg_size=128, waves=waves)
    res = sw.result()
    assert res.total == 8 ** 6 - 1 == int(res.counts[0])  # every union of the seven cycles of each
    counts, words, offs = sw.collect_raw()
    assert list(offs) == [0, len(words)] and int(counts[0]) == 8 ** 6 - 1
    one = [[]] + [c for c in oracle_sets(graphs(E, (4,)))[0]]
    assert len(one) == 8 and len(words) == 8 ** 6 - 1 + 6 * 8 ** 5 * sum(map(len, one))


def test_walk_of_cosets_and_properties(E):
    from test_conditions import _conditions_for, oracle_filtered
    insts = [W.fano()] + [i for i in W.batch(E.kdim, count=64) if i.meta["k"] <= 18][:11]
    preps, wants = [], []
    for j, inst in enumerate(insts):
        F = E.candidates(inst.n, inst.m, inst.lam)
        mf = E.default_max_facets(inst.n, inst.m)
        I, J, props = _conditions_for(inst.n, F, mf, j)
        kw = [dict(forced_in=I, forced_out=J), dict(properties=props),
              dict(forced_in=I, forced_out=J, properties=props)][j % 3]
        preps.append(E.prepare(inst.n, inst.m, lam=inst.lam, **kw))
        wants.append(oracle_filtered(inst.n, F, mf, kw.get("forced_in") or (), kw.get("forced_out") or (),
                                     kw.get("properties") or ()))
    assert any(p.offset is not None for p in preps)
    for cbits, wg, mode, waves in ((7, 64, 2, 7), (9, 256, 1, 8), (12, 256, 0, 7)):
        sets, res = sweep(E, preps, mode=mode, cbits=cbits, wg=wg, waves=waves)
        assert sets == wants and list(res.counts) == [len(w) for w in wants]


def test_walk_of_mixed_strides_and_deferred_ridges(E):
    insts = [i for i in W.batch(E.kdim, count=48) if 14 <= i.meta["k"] <= 20][:8]
    preps = [E.prepare(i.n, i.m, lam=i.lam, max_groups=1 + j % 2) for j, i in enumerate(insts)]
    preps += graphs(E, (7, 8)) + graphs(E, (7, 8), max_groups=1)
    assert {p.info.slots for p in preps} == {4, 8} and sum(p.info.n_deferred for p in preps) > 0
    want = oracle_sets(preps)
    for mode, cbits, waves in ((2, 9, 7), (0, 7, 8), (1, 10, 8)):
        sets, res = sweep(E, preps, mode=mode, cbits=cbits, waves=waves, split=False)
        assert sets == want and list(res.counts) == [len(w) for w in want]


@pytest.mark.parametrize("policy", ["plain", "static", "dynamic", "packed"])
def test_walk_schedules(E, policy):
    from paper_2301_00806_amd import scheduler as S
    insts = [i for i in W.batch(E.kdim, count=96) if i.meta["k"] <= 20][:24]
    preps, batch = walk_batch(E, E.prepare_many(insts))
    want = oracle_sets(preps)
    sw = E.Sweeper(batch, cap=1 << 22)
    plan = S.make_plan(batch, policy, cbits=9, wg=256, plain_min_items=3)
    sw.set_items(plan.items, segments=plan.segments)
    sw.launch(plan.mode, wg_size=256)
    sw.result()
    assert sw.collect() == want
    rec = np.asarray(sw.launch_fetch(plan.mode, wg_size=256, parts=3))
    assert (rec[:, 1] != -1).sum() == sum(len(w) for w in want)


def test_walk_of_a_pruned_batch(E):
    insts = [i for i in W.batch(E.kdim, count=96) if i.meta["k"] <= 20][:24]
    preps = E.prepare_many(insts, prune=True, min_free=10)
    assert sum(p.visited for p in preps) < sum(p.vectors for p in preps)
    sets, _ = sweep(E, preps, cbits=9, order=1, cost=np.arange(1, len(preps) + 1, dtype=np.float32))
    assert sets == oracle_sets(preps)


@pytest.mark.parametrize("mode", [1, 2])
def test_walk_skips_and_counts_malformed_items(E, mode):
    from paper_2301_00806_amd import _lib as L
    insts = [i for i in W.batch(E.kdim, count=32) if i.meta["k"] <= 16][:3]
    preps = E.prepare_many(insts)
    want = oracle_sets(preps)
    alone, batch = walk_batch(E, preps[:2])
    both = E.DeviceBatch(alone + preps[2:])
    good = E.build_queue(batch.k, 7, 64)
    bad = np.zeros(5, dtype=E.ITEM_DTYPE)
    bad[0] = (0, 5, 64, 0)                                   # cbits < 7
    bad[1] = (0, 7, 64, 480)                                 # 480 + 64 > 512
    bad[2] = (1, 7, 64, (1 << (max(preps[1].k, 7) - 7)))     # beyond 2^k
    bad[3] = (1 << 20, 7, 64, 0)                             # unknown instance
    bad[4] = (2, 7, 64, 0)                                   # a table of the other kind
    batch = both
    batch.c_batch.flags = L.BATCH_WALK
    sw = E.Sweeper(batch, cap=1 << 20)
    sw.set_items(np.concatenate([good, bad]), split_classes=False)
    print("[gpu] malformed items under the walk", flush=True)
    sw.launch(mode, wg_size=64, grid=2)
    torch.cuda.synchronize()
    assert int(sw.total.cpu()[2]) == 5
    assert [int(c) for c in sw.counts.cpu()] == [len(want[0]), len(want[1]), 0]
    with pytest.raises(L.WpmError):
        sw.collect()


def test_walk_counts_are_exact_after_record_overflow(E):
    from paper_2301_00806_amd import _lib as L
    preps, batch = walk_batch(E, graphs(E, (7, 8), max_groups=1))
    want = [O.count_wpm(p.n, [int(f) for f in p.facets], p.max_facets) for p in preps]
    sw = E.Sweeper(batch, cap=64)
    sw.set_items(E.build_queue(batch.k, 8, 64))
    sw.launch(2, wg_size=64)
    res = sw.result()
    assert res.slots > 64 and [int(c) for c in res.counts] == want
    with pytest.raises(L.WpmError) as ei:
        sw.collect()
    assert ei.value.status == L.WPM_ECAP
