"""Record slots past the caller's buffer: a sweep that adds to the totals of
earlier ones (more results than 36 and than 43 bits count) writes none of its
records, wherever the slot counter stands, and its counts stay exact."""
import ctypes

import numpy as np
import pytest

import oracle as O
import wpm_inputs as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CAP = 1 << 16


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("at", [CAP - 100, CAP, (1 << 36) - 192, 1 << 36, (1 << 43) - 192, 3 << 43])
def test_nothing_is_written_past_the_buffer(mode, at):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_00806_amd import _lib as L, engine as E
    insts = [i for i in W.batch(E.kdim, count=64) if 12 <= i.meta["k"] <= 14][:3]
    preps = E.prepare_many(insts)
    want = [len(O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets)) for p in preps]
    assert 512 < sum(want) < CAP - 8192
    batch = E.DeviceBatch(preps)
    items = E.build_queue(batch.k, 9, 64)
    d_items = torch.from_numpy(items.view(np.int64).reshape(-1).copy()).to("cuda")
    counts = torch.zeros(len(preps), dtype=torch.int64, device="cuda")
    total = torch.tensor([0, at, 0, 0], dtype=torch.int64, device="cuda")
    surv = torch.full((CAP, 2), 7, dtype=torch.int64, device="cuda")
    scratch = torch.zeros(L.QUEUE_SCRATCH_WORDS // 2, dtype=torch.int64, device="cuda")
    s = L.Sched(mode=mode, wg_size=64, grid=3, flags=L.FLAG_ACCUMULATE, d_items=d_items.data_ptr(),
                h_items=items.ctypes.data, num_items=len(items), d_scratch=scratch.data_ptr(),
                scratch_words=L.QUEUE_SCRATCH_WORDS)
    L.check("enumerate", L.lib().wpm_enumerate(
        ctypes.byref(batch.c_batch), ctypes.byref(s), surv.data_ptr(), CAP, counts.data_ptr(), total.data_ptr(),
        None, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    assert counts.cpu().tolist() == want
    tot = total.cpu().tolist()
    assert tot[0] == sum(want) and tot[1] >= at + sum(want) and tot[2] == 0
    rec = surv.cpu().numpy()
    first = min(at, CAP)
    assert (rec[:first] == 7).all()
    assert (rec[first:, 1] != 7).all()
