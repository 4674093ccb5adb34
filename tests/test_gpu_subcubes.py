"""The sub-cubes that the descent says it opened (d_stats[5..7]) are those that
the level rows of the tables leave, each counted once, however many waves
share it."""
import numpy as np
import pytest

import wpm_inputs as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def opened(p):
    """(2^18, 2^12, 2^6) sub-cubes opened in a sweep of all 2^k vectors."""
    import tablesim as TS
    from test_tree_levels import EIGHTEEN, LEVEL_WORDS, SIX, SIX2, TWELVE, fails, level_rows
    R = level_rows(p.table)
    kp = max(p.k, 7)
    off = R[kp] if p.offset is not None else np.zeros(LEVEL_WORDS, np.uint64)
    R = R[:kp]
    assert TS.header(p.table)["kp"] == kp
    alive = np.zeros(1, np.uint64)  # sub-cubes of 2^kp, split level by level
    at, out = max(kp, 18), []
    for bits, bases in ((18, (EIGHTEEN,)), (12, (TWELVE,)), (6, (SIX, SIX2))):
        n = max(0, min(at, kp) - bits)
        sub = ((alive[:, None] << np.uint64(n)) | np.arange(1 << n, dtype=np.uint64)[None]).reshape(-1)
        i = sub << np.uint64(bits)
        x = (i ^ (i >> np.uint64(1)))
        bad = np.zeros(len(sub), bool)
        for b in bases:
            bad |= fails(R, off, x, b)
        alive, at = sub[~bad], bits
        out.append(len(alive))
    return out


@pytest.mark.parametrize("wg", [64, 128, 256, 512])
@pytest.mark.parametrize("mode", [1, 2, 3])
def test_opened_subcubes(wg, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_00806_amd import engine as E
    from test_tree_levels import level_rows
    insts = W.batch(E.kdim, count=256)
    insts = [next(i for i in insts if i.meta["k"] == k) for k in (12, 14, 18, 20, 21)]
    preps = E.prepare_many(insts)
    F = [int(f) for f in E.candidates(insts[2].n, insts[2].m, insts[2].lam)]
    preps.append(E.prepare(insts[2].n, insts[2].m, lam=insts[2].lam, forced_in=F[:1]))
    assert preps[-1].offset is not None and all(level_rows(p.table) is not None for p in preps)
    want = np.array([opened(p) for p in preps]).sum(0)
    batch = E.DeviceBatch(preps)
    # whole groups of 2^18, or whole instances
    items = np.concatenate([E.build_queue(np.where(np.arange(len(preps)) == j, batch.k, 0).astype(np.int32),
                                          12 if p.k >= 18 else max(p.k - 6, 7), 64) for j, p in enumerate(preps)])
    grid = 3
    bins = np.linspace(0, len(items), grid + 1).astype(np.int64)
    sw = E.Sweeper(batch, cap=1 << 20)
    sw.set_items(items, bin_offsets=bins)
    sw.launch(mode, wg_size=wg, grid=grid)
    assert (np.array(sw.result().stats[5:8]) == want).all(), want
