"""The level section of packed tables (host logic, no GPU): the sub-cube
tests of the tree descent are constant over their sub-cubes and never reject
a weak pseudo-manifold, for plain, pruned and coset instances."""
import numpy as np
import pytest

import oracle as O
import tablesim as TS
import wpm_inputs as W
from paper_2301_00806_amd import engine as E

LEVEL_WORDS = 20
LEAF, SIX, SIX2, TWELVE, EIGHTEEN = 0, 4, 8, 12, 16


def level_rows(tab):
    """[kp (+ offset row)][16] of the level section, or None."""
    h = TS.header(tab)
    if not int(tab[11]) & 2:
        return None
    nrows = h["kp"] + (1 if h["offset"] else 0)
    at = TS.HDR + nrows * h["RS"]
    return tab[at:at + nrows * LEVEL_WORDS].reshape(nrows, LEVEL_WORDS).astype(np.uint64)


def fails(R, off, xs, base):
    """Whether the 4-word group at `base` rejects each x."""
    v = np.repeat(off[None, base:base + 4], len(xs), 0)
    for t in range(R.shape[0]):
        v = v ^ (R[t, base:base + 4][None] * ((xs >> np.uint64(t)) & np.uint64(1))[:, None])
    a, u, c, w = v.T
    return TS.at_least3([a, a ^ u, c, c ^ w]) != 0


def test_no_level_rejects_a_member():
    seen = 0
    insts = W.batch(E.kdim, count=96)
    preps = [E.prepare(i.n, i.m, lam=i.lam) for i in insts if i.meta["k"] <= 13][:16]
    for i in insts:
        if i.meta["k"] in (14, 15) and len(preps) < 24:
            F = [int(f) for f in E.candidates(i.n, i.m, i.lam)]
            p = E.prepare(i.n, i.m, lam=i.lam, forced_in=F[:1])
            if p.feasible and 12 <= p.k <= 13:
                preps.append(p)
    for p in preps:
        R = level_rows(p.table)
        if R is None:
            continue
        off = R[p.k] if p.offset is not None else np.zeros(LEVEL_WORDS, np.uint64)
        R = R[:p.k]
        # constant over the sub-cube: the free coordinates' rows are zero
        assert not R[:6, SIX:].any() and not R[:12, TWELVE:].any() and not R[:18, EIGHTEEN:].any()
        xs = np.array(TS.survivors_direct(p.table), dtype=np.uint64)
        for base in (LEAF, SIX, SIX2, TWELVE, EIGHTEEN):
            assert not len(xs) or not fails(R, off, xs, base).any(), (p.k, base)
        seen += 1
        if p.offset is not None:
            seen += 1000
    assert seen > 1000, seen


@pytest.mark.parametrize("k_lo,k_hi,prune", [(22, 28, False), (22, 28, True), (30, 32, False)])
def test_levels_keep_every_oracle_member(k_lo, k_hi, prune):
    """Larger instances: the oracle's complexes, expressed in the kernel
    basis, pass every level."""
    inst = next(i for i in W.batch(E.kdim, count=512) if k_lo <= i.meta["k"] <= k_hi)
    p = E.prepare(inst.n, inst.m, lam=inst.lam, prune=prune, min_free=16)
    R = level_rows(p.table)
    assert R is not None
    sets = O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets, node_limit=0)
    # coordinates of each complex: solve against the basis by elimination
    pos = {int(f): j for j, f in enumerate(p.facets)}
    rows = [(sum(int(p.basis[t, w]) << (32 * w) for w in range(p.W)), 1 << t) for t in range(p.k)]
    piv = []
    for v, x in rows:
        for b, pv, px in piv:
            if v >> b & 1:
                v, x = v ^ pv, x ^ px
        b = v.bit_length() - 1
        piv = [(bb, pv ^ v, px ^ x) if pv >> b & 1 else (bb, pv, px) for bb, pv, px in piv] + [(b, v, x)]
    xs = []
    for K in sets[:20000]:
        v, x = sum(1 << pos[f] for f in K), 0
        for b, pv, px in piv:
            if v >> b & 1:
                v, x = v ^ pv, x ^ px
        assert v == 0
        xs.append(x)
    xs = np.array(xs, dtype=np.uint64)
    off = np.zeros(LEVEL_WORDS, np.uint64)
    for base in (LEAF, SIX, SIX2, TWELVE, EIGHTEEN):
        assert not fails(R, off, xs, base).any(), base
    # and they do reject: a random vector rarely passes all of them
    rng = np.random.default_rng(1)
    rx = rng.integers(0, 1 << p.k, 4096, dtype=np.uint64)
    left = ~(fails(R, off, rx, SIX) | fails(R, off, rx, SIX2) | fails(R, off, rx, TWELVE))
    assert left.mean() < 0.5
