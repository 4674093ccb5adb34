"""The dynamic queue with one head and with eight: the same sweep, at item
numbers around the blocks that go round the heads (64), the grid and one item
more or fewer, with whole items and a small grid, against the oracle's counts."""
import numpy as np
import pytest

import oracle as O
import wpm_inputs as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid", [1, 3, 8, 61, 0])
@pytest.mark.parametrize("num_items", [1, 7, 65, 256, 257, 319, 321, 575, 1037])
def test_heads_take_every_item_once(grid, num_items):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import ctypes
    from paper_2301_00806_amd import _lib as L, engine as E
    insts = [i for i in W.batch(E.kdim, count=64) if 12 <= i.meta["k"] <= 14][:3]
    preps = E.prepare_many(insts)
    want = [len(O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets)) for p in preps]
    batch = E.DeviceBatch(preps)
    one = E.build_queue(batch.k, 7, 64)
    # whole sweeps of the three instances in turn, cut after num_items items
    rep = -(-num_items // len(one))
    items = np.concatenate([one] * rep)[:num_items].copy()
    per_item = None
    for words in (0, L.QUEUE_SCRATCH_WORDS):
        counts = torch.full((len(preps),), 7, dtype=torch.int64, device="cuda")
        total = torch.full((L.TOTAL_WORDS,), 7, dtype=torch.int64, device="cuda")
        surv = torch.empty((1 << 20, 2), dtype=torch.int64, device="cuda")
        scratch = torch.full((L.QUEUE_SCRATCH_WORDS // 2,), 5, dtype=torch.int64, device="cuda")
        d_items = torch.from_numpy(items.view(np.int64).reshape(-1).copy()).to("cuda")
        s = L.Sched(mode=L.SCHED_DYNAMIC, wg_size=64, grid=grid, flags=0, d_items=d_items.data_ptr(),
                    h_items=items.ctypes.data, num_items=len(items), d_scratch=scratch.data_ptr(),
                    scratch_words=words)
        st = L.lib().wpm_enumerate(ctypes.byref(batch.c_batch), ctypes.byref(s), surv.data_ptr(), 1 << 20,
                                   counts.data_ptr(), total.data_ptr(), None,
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        L.check("enumerate", st)
        torch.cuda.synchronize()
        got = counts.cpu().tolist()
        if num_items % len(one) == 0:
            assert got == [w * (num_items // len(one)) for w in want]
        rec = surv[:int(total[1])].cpu().numpy()
        rec = rec[rec[:, 1] != -1]
        rec = rec[np.lexsort((rec[:, 0], rec[:, 1]))].tobytes()
        if per_item is None:
            per_item = (got, rec)
        assert (got, rec) == per_item
