"""Fewer items than workgroups: items handed out in parts, with short items
among long ones, at grids where each number of parts is chosen, without a host
copy of the items, against the oracle's sets."""
import ctypes

import numpy as np
import pytest

import oracle as O
import wpm_inputs as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("grid", [4, 8, 17, 40, 64, 150, 512, 0])
def test_parts_of_short_and_long_items(mode, grid):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_00806_amd import _lib as L, engine as E
    insts = W.batch(E.kdim, count=512)
    insts = [next(i for i in insts if i.meta["k"] == k) for k in (12, 16, 18, 20)]
    preps = E.prepare_many(insts)
    assert all(int(p.table[11]) & 2 for p in preps)
    batch = E.DeviceBatch(preps)
    items = np.concatenate([E.build_queue(np.where(np.arange(4) == j, batch.k, 0).astype(np.int32), c, 256)
                            for j, c in enumerate((7, 8, 9, 12))])
    assert len(items) <= 8
    sw = E.Sweeper(batch, cap=1 << 20)
    sw.set_items(items, split_classes=False)
    sw._items_ptr = 0  # (no host copy)
    sw.launch(mode, wg_size=256, grid=grid)
    sw.result()
    assert sw.collect() == [O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets) for p in preps]
