"""Launch classes of a batch: each holds tables of one kind, so that no launch
looks at the items of the other kernel (host logic, no GPU)."""
import itertools

import numpy as np
import pytest

import wpm_inputs as W
from paper_2301_00806_amd import _lib as L
from paper_2301_00806_amd import engine as E


@pytest.fixture(scope="module")
def preps():
    insts = [i for i in W.batch(E.kdim, count=96) if i.meta["k"] <= 22][:48]
    out = E.prepare_many(insts, prune=True, min_free=7)
    for p in out[::3]:
        p.table[11] &= ~np.uint32(2)  # without the bit that announces the level section
    assert {E.descended(p) for p in out} == {True, False}
    return out


def test_every_packed_table_has_a_level_section():
    # also where its tests reject nothing: disjoint K_4 have no critical ridge
    for groups in (1, 5, 6, 8):
        F = [(1 << (4 * g + a)) | (1 << (4 * g + b)) for g in range(groups)
             for a, b in itertools.combinations(range(4), 2)]
        p = E.prepare(2, 4 * groups, facets=F, max_facets=0)
        assert p.k == 3 * groups and p.info.n_crit == 0 and E.descended(p)
    insts = [i for i in W.batch(E.kdim, count=128) if i.meta["k"] <= 20]
    for mf in (7, 10):
        assert all(E.descended(p) for p in E.prepare_many(insts, prune=True, min_free=mf))


def test_classes_hold_one_kind(preps):
    batch = E.DeviceBatch(preps, device="cpu")
    assert batch.c_batch.flags == 0
    for c, b in batch.class_batches.items():
        kinds = {E.descended(p) for p, q in zip(preps, batch.cls) if q == c}
        assert len(kinds) == 1
        assert b.flags == (L.BATCH_TREE if kinds == {True} else L.BATCH_WALK)
        assert E.class_row_words(c) in E.LDS_CLASSES
        assert b.max_row_words <= E.class_row_words(c)
    assert len(batch.class_batches) >= 2


def test_items_are_split_by_kind(preps):
    batch = E.DeviceBatch(preps, device="cpu")
    items = E.build_queue(batch.k, 9, 64, blocks=batch.blocks)
    out, segs = E.split_by_class(batch, items)
    assert sorted(map(tuple, out.tolist())) == sorted(map(tuple, items.tolist()))
    assert len(segs) == len(batch.class_batches)
    for s in segs:
        part = out[s.start:s.end]["instance"]
        assert {E.descended(preps[i]) for i in part} == {batch.class_batches[s.cls].flags == L.BATCH_TREE}


def test_one_kind_keeps_the_width_classes():
    insts = [i for i in W.batch(E.kdim, count=32) if i.meta["k"] <= 22]
    plain = E.prepare_many(insts)
    batch = E.DeviceBatch(plain, device="cpu")
    assert all(E.descended(p) for p in plain)
    assert np.array_equal(batch.cls, [E.lds_class(p.info) for p in plain])
    assert batch.c_batch.flags == L.BATCH_TREE


@pytest.mark.parametrize("wg", [64, 256, 512])
def test_walked_short_items(wg):
    # fewer than 64 vectors per lane of the workgroup on average, 2^15 items and
    # more, 64 of an instance and more
    def walked(n, per_instance, lanes, cbits):
        items = np.zeros(n, dtype=E.ITEM_DTYPE)
        items["lanes"], items["cbits"] = lanes, cbits
        return E.walks_short_items(items, wg, -(-n // per_instance))
    n = 1 << 15
    assert walked(n, 64, wg - 1, 6) and walked(n + 77, 1 << 20, 1, 6)
    assert not walked(n, 64, wg, 6) and not walked(n, 64, 1, 63)
    assert not walked(n - 1, 64, wg - 1, 6) and not walked(0, 64, 1, 7) and not walked(1, 64, 1, 7)
    assert not walked(n, 63, wg - 1, 6)


def test_tuner_times_register_budgets_of_walked_tables_alone(preps):
    from paper_2301_00806_amd import tune as T
    mixed = E.DeviceBatch(preps, device="cpu")
    descended = E.DeviceBatch([p for p in preps if E.descended(p)], device="cpu")
    walked = E.DeviceBatch([p for p in preps if not E.descended(p)], device="cpu")
    assert T.wave_choices(descended, T.WAVES) == T.WAVES[:1]
    assert T.wave_choices(walked, T.WAVES) == T.wave_choices(mixed, T.WAVES) == T.WAVES
