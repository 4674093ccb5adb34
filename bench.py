"""Benchmark: kernel vectors checked per second on one MI355X.

Workload: 16384 seeded characteristic matrices lambda = [I_n | 4 uniform
columns], n = 5 + (i mod 4), m = n + 4, kept when the kernel dimension k of
their candidate set is at most 36 (the learned-scheduler workload).  A step is
one pass of the hot path over the whole batch with the packed tables already
resident in HBM: cost prediction, queue packing, the persistent sweep of all
sum_i 2^k_i kernel vectors into exact per-instance counts (read back) and
survivor records (left in HBM by default; the end-to-end figure copies them
to the host and expands them).  The plain schedule (one launch per instance) is
timed on the same batch for comparison, and so is the pruned sweep over a
convenient kernel basis (Section 2.1: same results, fewer vectors visited),
reported beside the headline figure.

Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

import numpy as np


def log(msg: str) -> None:
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


# Integer VALU peak: 256 CUs x 128 32-bit lane-ops per clock (a wave64 VALU op
# every 2 clocks on each of 4 SIMDs, the same issue rate as fp32 FMA behind the
# 157.3 TFLOP/s figure) x 2.4 GHz.  wpm_valu_probe measures it on the device.
INT32_PEAK = 256 * 128 * 2.4e9
# Fast filter per kernel vector: 4 XORs and 2 threshold ops, plus a 3-input
# minimum, a minimum and a compare shared by the four chains of a step.
ALG_OPS_PER_VECTOR = 4 + 2 + 3 / 4
# Tree descent, int32 ops for each of the 64 parts of an opened sub-cube: of
# 2^18 vectors (4 XORs, 2 threshold ops), of 2^12 (two ridge groups: 8 XORs, 4
# threshold ops, 1 OR), of 2^6 (4 XORs, 2 threshold ops, a compare and an add
# that collects its bit).  The checks of candidates are not counted.
DESCENT_OPS = (6, 13, 8)


def walked(p) -> bool:
    """Is this instance's table without a level section (swept vector by
    vector)?"""
    return not int(p.table[11]) & 2


def sweep_ops(preps, stats) -> float:
    """int32 ops of the tests a sweep of `preps` made: the descent's by the
    sub-cubes it opened, the walk's by vectors."""
    ops = 64.0 * sum(c * float(n) for c, n in zip(DESCENT_OPS, stats[5:8]))
    return ops + ALG_OPS_PER_VECTOR * float(sum(int(p.visited) for p in preps if p.k > 0 and walked(p)))


def kernel_sources_sha256() -> str:
    import hashlib
    h = hashlib.sha256()
    for f in ("sweep_kernel.h", "tree_kernel.h"):
        with open(os.path.join(ROOT, "paper_2301_00806_amd", "csrc", f), "rb") as src:
            h.update(src.read())
    return h.hexdigest()


def ops_alg_plain(p) -> int:
    """Work per kernel vector of the plain per-ridge check (the paper's
    kernel in bit-mask form): W XORs for the Gray step, for every ridge with
    at least 4 parents an AND and a popcount per facet word holding one of
    its parents plus one compare, and W popcounts plus a compare for the
    facet bound."""
    facets = [int(f) for f in p.facets]
    words, parents = {}, {}
    for j, f in enumerate(facets):
        v = f
        while v:
            r = f & ~(v & -v)
            words.setdefault(r, set()).add(j >> 5)
            parents[r] = parents.get(r, 0) + 1
            v &= v - 1
    W = (len(facets) + 31) // 32
    return W + sum(2 * len(words[r]) + 1 for r in words if parents[r] >= 4) + W + 1


WORKLOADS = {
    "learned": "learned-scheduler batch: {count} lambda = [I_n | 4 uniform], n = 5..8, m = n + 4, k <= 36",
    "batch": "batch: {count} lambda = [I_n | 4 uniform], n = 4..7, m = n + 4, 12 <= k <= 32",
    "stress": "stress: {count} random 0.75-dense subsets of the 7-subsets of [11], 32 <= k <= 40",
}


def build_workload(count: int, workload: str = "learned", seed_start: int = 0):
    import wpm_inputs as W
    from paper_2301_00806_amd import engine as E
    t = time.time()
    if workload == "learned":
        insts = W.learned(E.kdim, count=count, start=seed_start)
    elif workload == "batch":
        insts = W.batch(E.kdim, count=count, start=seed_start)
    else:
        insts = W.stress(E.kdim, count=count, start=seed_start)
    log(f"selected {len(insts)} instances in {time.time() - t:.1f}s")
    t = time.time()
    preps = E.prepare_many(insts)
    log(f"prepared (candidates, basis, packing) in {time.time() - t:.1f}s")
    return insts, preps


def oracle_counts_match(counts, workload, n_inst):
    """Per-instance counts against the oracle's, stored for each workload at
    its full size by tests/golden/make_counts.py (None for other sizes)."""
    path = os.path.join(ROOT, "tests", "golden", f"{workload}{n_inst}_counts.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        gold = np.array(json.load(f)["counts"], dtype=np.uint64)
    return bool(np.array_equal(np.asarray(counts, dtype=np.uint64), gold))


def cpu_baseline(preps, budget_s: float):
    """The oracle (plain CPU backtracking) on a bounded sample of the same
    instances, one instance per host thread; reported in kernel vectors
    covered per second (sum of 2^k of the instances it finished)."""
    import oracle as O
    from concurrent.futures import ThreadPoolExecutor, as_completed
    cores = min(16, os.cpu_count() or 1)
    order = sorted(range(len(preps)), key=lambda i: preps[i].k)
    rng = np.random.default_rng(7)
    # a sample spanning the k range: every stride-th instance by k
    sample = order[::max(1, len(order) // 512)]
    rng.shuffle(sample)
    done_vec, done_n, t0 = 0.0, 0, time.time()
    with ThreadPoolExecutor(max_workers=cores) as ex:
        futs = {}
        it = iter(sample)
        def submit():
            try:
                i = next(it)
            except StopIteration:
                return False
            p = preps[i]
            futs[ex.submit(O.enumerate_wpm, p.n, [int(f) for f in p.facets], p.max_facets)] = i
            return True
        for _ in range(cores):
            submit()
        while futs:
            for f in as_completed(list(futs)):
                i = futs.pop(f)
                f.result()
                done_vec += float(1 << preps[i].k)
                done_n += 1
                if time.time() - t0 < budget_s:
                    submit()
                break
    el = time.time() - t0
    # the same oracle on one thread: instances of the sample in k order, about 5 s
    one_vec, one_n, t1 = 0.0, 0, time.time()
    for i in sorted(sample, key=lambda i: preps[i].k)[::max(1, len(sample) // 64)]:
        if time.time() - t1 > 5.0:
            break
        p = preps[i]
        O.enumerate_wpm(p.n, [int(f) for f in p.facets], p.max_facets)
        one_vec += float(1 << p.k)
        one_n += 1
    el1 = time.time() - t1
    return {"value": done_vec / el, "unit": "kernel vectors/s", "cores": cores, "kind": "oracle",
            "sample": f"{done_n} of the {len(preps)} instances (spread over the k range), "
                      f"{el:.1f}s wall, one instance per thread; vectors = sum of 2^k",
            "single_thread_value": one_vec / el1 if el1 > 0 else None,
            "single_thread_sample": f"{one_n} instances of that sample in k order, {el1:.1f}s, one thread"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="learned", choices=sorted(WORKLOADS),
                    help="learned (the headline), batch or stress")
    ap.add_argument("--instances", type=int, default=0, help="0 = the workload's own size")
    ap.add_argument("--cbits", type=int, default=0, help="lane chunk bits (0 = autotuned)")
    ap.add_argument("--wg", type=int, default=0, help="workgroup size (0 = autotuned)")
    ap.add_argument("--waves", type=int, default=0, help="kernel register budget: 7 or 8 waves per SIMD (0 = autotuned)")
    ap.add_argument("--max-items", type=int, default=0)
    ap.add_argument("--no-plain", action="store_true")
    ap.add_argument("--no-static", action="store_true")
    ap.add_argument("--cap", type=int, default=1 << 26, help="survivor records in HBM")
    ap.add_argument("--plain-min-items", type=int, default=512,
                    help="plain schedule: split each instance over at least this many workgroups")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--train-instances", type=int, default=4096)
    ap.add_argument("--epochs", type=int, default=200)
    ap.add_argument("--learned-policy", default="dynamic", choices=["packed", "dynamic"])
    ap.add_argument("--only-learned", action="store_true",
                    help="time only the learned schedule (profiling runs)")
    ap.add_argument("--no-split", action="store_true",
                    help="one launch under the largest kernel template instead of one per class")
    ap.add_argument("--cpu-budget", type=float, default=15.0)
    ap.add_argument("--no-e2e", action="store_true",
                    help="skip the end-to-end run (table upload, step, collect to facet lists)")
    ap.add_argument("--no-pruned", action="store_true",
                    help="skip the convenient-basis (pruned) sweep of the same batch")
    ap.add_argument("--min-free", type=int, default=0,
                    help="free coordinates a pruned instance keeps (0 = engine default)")
    ap.add_argument("--records", default="hbm", choices=["hbm", "host", "copy"],
                    help="survivor records left in HBM (the step's output), written by the sweep into "
                         "pinned host memory, or written to HBM and copied back in parts that overlap the sweep")
    ap.add_argument("--parts", type=int, default=4,
                    help="--records copy: sub-launches of the largest class, so that record copies overlap the sweep")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 256 MiB device copy (for counter calibration)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU: the engine runs on a single device "
              "(--gpus must be 1)", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2301_00806_amd import _lib as L
    from paper_2301_00806_amd import engine as E
    torch.cuda.set_device(0)
    cus, clk_khz, lds = E.device_query()
    log(f"device: {cus} CUs, wallclock {clk_khz} kHz, LDS/block {lds}")

    if args.instances == 0:
        args.instances = {"learned": 16384, "batch": 4096, "stress": 64}[args.workload]
    insts, preps = build_workload(args.instances, args.workload)
    batch = E.DeviceBatch(preps)
    vectors = batch.vectors
    log(f"sum 2^k = {vectors:.4e}; tables {batch.table_bytes / 1e6:.1f} MB in HBM")
    stream = torch.cuda.current_stream()
    tuned = None
    if args.cbits == 0 or args.wg == 0 or args.waves == 0:
        from paper_2301_00806_amd import tune as T
        tuned = T.tune(preps, log=log)
        log(f"autotuner ({'cached' if tuned['cached'] else 'measured'}, {tuned['key']}): "
            f"cbits={tuned['cbits']} wg={tuned['wg']}")
        args.cbits = args.cbits or tuned["cbits"]
        args.wg = args.wg or tuned["wg"]
        args.waves = args.waves or tuned.get("waves", 0)
    sw = E.Sweeper(batch, cap=args.cap, records_on_host=args.records == "host")

    # ---- learned part: labels from timed sweeps of the batch workload, MLP
    # trained on the GPU by the engine's own forward/backward/Adam kernels
    from paper_2301_00806_amd import costmodel as CM
    from paper_2301_00806_amd import scheduler as S
    t = time.time()
    import wpm_inputs as W
    train_insts = W.batch(E.kdim, count=args.train_instances)
    train_preps = E.prepare_many(train_insts)
    Xtr, Ttr, _ = S.measure_labels(train_preps, cbits=12, wg=args.wg)
    model = CM.CostModel(seed=0)
    model.fit(Xtr, Ttr, epochs=args.epochs, lr=3e-3, batch=512)
    okt = np.isfinite(Ttr).all(1)
    train_loss = model.loss(Xtr[okt], Ttr[okt])
    log(f"cost model trained on {len(Xtr)} instances in {time.time() - t:.1f}s, loss {train_loss:.4f}")

    feats = CM.features_of(preps)

    # a side stream for the cost model's inference, so that the next step's
    # plan can be made while the current step's sweep runs
    side = torch.cuda.Stream()

    def plan_learned(st=None):
        cost = S.per_vector_cost(model, feats, stream=st)   # MLP inference on the GPU
        return S.make_plan(batch, args.learned_policy, cost=cost, cbits=args.cbits, wg=args.wg,
                           split=not args.no_split)

    def timed_plan(make, steps, warmup, label, sw=sw, n_inst=len(preps), vec=vectors):
        plan = make()
        for _ in range(warmup):
            sw.set_items(plan.items, segments=plan.segments)
            if args.records == "hbm":
                sw.launch(plan.mode, wg_size=args.wg, stream=stream, waves=args.waves)
            else:
                sw.launch_fetch(plan.mode, wg_size=args.wg, stream=stream, parts=args.parts, waves=args.waves)
            # the timed steps make the next plan on the side stream: its first
            # use there carries a one-time cost (several ms), paid here
            make(side)
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        kern_ms, seg_ms, walls = [], {}, []
        t0 = time.perf_counter()
        # Scheduling is part of every step: the first step's plan is made in
        # the timed region, and each later one while the step before it
        # sweeps (host queue building and the model's inference on a side
        # stream overlap the GPU), as a pipeline over successive batches would.
        plan = make()
        for step in range(steps):
            ts = time.perf_counter()
            sw.set_items(plan.items, segments=plan.segments)
            nxt = {}

            def plan_next():
                if step + 1 < steps:
                    nxt["plan"] = make(side)
            e0.record(stream)
            if args.records == "hbm":
                # the sweep; its survivor records stay in HBM
                sw.launch(plan.mode, wg_size=args.wg, stream=stream, seg_events=True, waves=args.waves)
                e1 = torch.cuda.Event(enable_timing=True)
                e1.record(stream)
                plan_next()
                rec = None
            else:
                # records in pinned host memory: written there by the sweep,
                # or copied there while the later sub-launches still run
                rec = sw.launch_fetch(plan.mode, wg_size=args.wg, stream=stream, parts=args.parts,
                                      seg_events=True, waves=args.waves, while_running=plan_next)
                e1 = sw.launch_end
            plan = nxt.get("plan", plan)
            counts = sw.counts[:n_inst].cpu()          # synchronises the stream
            tot, slots = (int(v) for v in sw.total.cpu()[:2])
            if slots > sw.cap:
                raise SystemExit(f"survivor buffer too small: {slots} > {sw.cap}")
            assert rec is None or len(rec) == slots
            kern_ms.append(e0.elapsed_time(e1))
            for cls, a0, a1 in sw.seg_events:
                seg_ms.setdefault(cls, []).append(a0.elapsed_time(a1))
            walls.append(time.perf_counter() - ts)
        torch.cuda.synchronize()
        wall = (time.perf_counter() - t0) / steps
        timed_plan.medians = (float(np.median(walls)) * 1e3, float(np.median(kern_ms)))
        res = sw.result()
        log(f"{label}: kernel {np.mean(kern_ms):.2f} ms, step {wall * 1e3:.2f} ms, "
            f"{vec / wall:.3e} vectors/s, total WPMs {res.total}, stats {res.stats[:3]}")
        timed_plan.seg_ms = {c: float(np.mean(v)) for c, v in seg_ms.items()}
        return wall, float(np.mean(kern_ms)), res

    t_b, k_b, res_b = timed_plan(plan_learned, args.steps, args.warmup, f"learned-{args.learned_policy}")
    step_med, kern_med = timed_plan.medians

    # ---- roofline launch: the learned plan once more, every class as a
    # single dispatch with HIP events around each (with --records copy the
    # timed steps split the largest class into parts); its events time the
    # dominant kernel
    plan = plan_learned()
    sw.set_items(plan.items, segments=plan.segments)
    sw.launch(plan.mode, wg_size=args.wg, stream=stream, seg_events=True, waves=args.waves)
    torch.cuda.synchronize()
    seg_ms = {(None if cls is None else int(cls)): a0.elapsed_time(a1) for cls, a0, a1 in sw.seg_events}
    assert np.array_equal(sw.counts[:len(preps)].cpu().numpy().astype(np.uint64), res_b.counts)

    # ---- end to end once: packed tables host -> HBM, one step, records back
    # and expanded into canonical facet lists by wpm_collect
    e2e = None
    if not args.no_e2e:
        sw.reserve_host_staging()   # set-up: pinned memory the records are copied into
        host_tab = batch.tables.cpu().pin_memory()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        batch.tables.copy_(host_tab)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        plan = plan_learned()
        sw.set_items(plan.items, segments=plan.segments)
        sw.launch(plan.mode, wg_size=args.wg, stream=stream, waves=args.waves)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        d2h_ms = None
        if not sw.records_on_host:
            # the survivor records over PCIe into pinned host memory
            slots = min(int(sw.total[1].item()), sw.cap)
            torch.cuda.synchronize()
            ta = time.perf_counter()
            sw._staging[:slots].copy_(sw.surv[:slots], non_blocking=True)
            torch.cuda.synchronize()
            d2h_ms = (time.perf_counter() - ta) * 1e3
        t2b = time.perf_counter()
        cnt_e, words_e, _ = sw.collect_raw()
        t3 = time.perf_counter()
        assert np.array_equal(cnt_e, res_b.counts)
        step_s, collect_s = t2 - t1, t3 - t2b
        e2e = {"h2d_ms": (t1 - t0) * 1e3, "step_ms": step_s * 1e3,
               "records_d2h_ms": d2h_ms, "collect_ms": collect_s * 1e3,
               "total_ms": (t1 - t0 + step_s + collect_s) * 1e3,
               "vectors_per_s": vectors / (t1 - t0 + step_s + collect_s),
               "pcie_inclusive_step_vectors_per_s": None if d2h_ms is None else
               vectors / (step_s + d2h_ms * 1e-3),
               "table_bytes": batch.table_bytes, "facet_words": int(len(words_e)),
               "note": "collect = records to host + expansion to sorted facet lists, 16 host threads; "
                       "pcie_inclusive_step = step + survivor records to pinned host memory"}
        log(f"end to end: {e2e}")
        del words_e
    # the dominant launch: the launch class holding most of the vectors
    cls_vec = {}
    for p, c in zip(preps, batch.cls):
        if p.k > 0:
            cls_vec[int(c)] = cls_vec.get(int(c), 0) + (1 << p.k)
    dom = max(cls_vec, key=cls_vec.get)
    dom_ms = seg_ms[dom]
    waves_used = args.waves if args.waves in (7, 8) else 8
    dom_preps = [p for p, c in zip(preps, batch.cls) if int(c) == dom and p.k > 0]
    kinds = {"sweep_kernel<%d>" % waves_used if walked(p) else "tree_kernel<7>" for p in dom_preps}
    # its statistics: the class alone, once more
    seg = next(s for s in plan.segments if s.cls is None or int(s.cls) == dom)
    sw.set_items(plan.items[seg.start:seg.end], segments=[E.Segment(seg.cls, 0, seg.end - seg.start, seg.bins)])
    sw.launch(plan.mode, wg_size=args.wg, stream=stream, waves=args.waves)
    torch.cuda.synchronize()
    roof_stats = sw.stats.cpu().numpy().astype(np.uint64)
    dom_name = "%s (rows of at most %d words)" % (" + ".join(sorted(kinds)), E.class_row_words(dom))
    log(f"dominant launch {dom_name}: {cls_vec[dom]:.4e} vectors in {dom_ms:.2f} ms "
        f"({cls_vec[dom] / dom_ms * 1e3:.3e} vectors/s); per-class ms {seg_ms}")
    out = {}
    sp = not args.no_split
    others = [("static", lambda st=None: S.make_plan(batch, "static", cbits=args.cbits, wg=args.wg, split=sp)),
              ("dynamic_pow2", lambda st=None: S.make_plan(batch, "dynamic", cbits=args.cbits, wg=args.wg, split=sp)),
              ("packed_pow2", lambda st=None: S.make_plan(batch, "packed", cbits=args.cbits, wg=args.wg, split=sp))]
    if not args.no_plain:
        others.append(("plain", lambda st=None: S.make_plan(batch, "plain", cbits=args.cbits, wg=args.wg,
                                                    plain_min_items=args.plain_min_items, split=sp)))
    other_pol = "packed" if args.learned_policy == "dynamic" else "dynamic"
    others.append((f"{other_pol}_model", lambda st=None: S.make_plan(
        batch, other_pol, cost=S.per_vector_cost(model, feats, stream=st), cbits=args.cbits, wg=args.wg,
        split=sp)))
    for name, mk in ([] if args.only_learned else others):
        if args.no_static and name == "static":
            continue
        st = max(1, args.steps // 2) if name != "plain" else 1
        t_o, k_o, res_o = timed_plan(mk, st, 1, name)
        assert np.array_equal(res_o.counts, res_b.counts), f"{name} counts differ"
        out[name] = {"value": vectors / t_o, "ms_per_step": t_o * 1e3, "kernel_ms": k_o}

    # ---- convenient-basis block pruning: the same batch, the same results,
    # fewer vectors visited
    pruned = None
    if not args.no_pruned:
        t = time.time()
        cb_p = args.cbits
        if args.min_free:
            mf = args.min_free
            preps_p = E.prepare_many(insts, prune=True, min_free=mf)
            tuned_p = None
        else:
            # free coordinates and chunk bits from the pruned autotuner
            from paper_2301_00806_amd import tune as T
            tuned_p, preps_p = T.tune_pruned(insts, wg=args.wg, waves=args.waves or 8, log=log)
            mf, cb_p = int(tuned_p["min_free"]), int(tuned_p["cbits"])
            log(f"pruned autotuner ({'cached' if tuned_p['cached'] else 'measured'}, {tuned_p['key']}): "
                f"min_free={mf} cbits={cb_p}")
        prep_s = time.time() - t
        batch_p = E.DeviceBatch(preps_p)
        visited = batch_p.visited
        log(f"pruned: prepared in {prep_s:.1f}s, visits {visited:.4e} of {vectors:.4e} vectors "
            f"({visited / vectors:.3f})")
        sw_p = E.Sweeper(batch_p, cap=args.cap, records_on_host=args.records == "host")
        feats_p = CM.features_of(preps_p)

        def plan_pruned(st=None):
            cost = S.per_vector_cost(model, feats_p, stream=st)
            return S.make_plan(batch_p, "dynamic", cost=cost, cbits=cb_p, wg=args.wg,
                               split=not args.no_split)
        t_p, k_p, res_p = timed_plan(plan_pruned, args.steps, args.warmup, "pruned-dynamic",
                                     sw=sw_p, n_inst=len(preps_p), vec=vectors)
        assert np.array_equal(res_p.counts, res_b.counts), "pruned counts differ"
        pruned = {"min_free": mf, "cbits": cb_p, "tuned": None if tuned_p is None else
                  {"cached": tuned_p["cached"], "results": tuned_p["results"]},
                  "visited_vectors": visited, "covered_vectors": vectors,
                  "ms_per_step": t_p * 1e3, "kernel_ms": k_p,
                  "covered_per_s": vectors / t_p, "visited_per_s": visited / t_p,
                  "speedup_vs_learned_step": t_b / t_p, "prep_s": prep_s,
                  # the tests' ops over the kernel time
                  "frac_of_peak": sweep_ops(preps_p, res_p.stats) / (k_p * 1e-3) / INT32_PEAK,
                  "counts_equal_to_full_sweep": True}
        del sw_p, batch_p

    # model error on the fresh instances: measured per-instance time vs
    # prediction (skipped with --only-learned, which measures no labels)
    model_err = None
    if not args.only_learned:
        _, Tte, _ = S.measure_labels(preps, cbits=args.cbits, wg=args.wg, repeats=1)
        pred = model.predict(feats)
        ok = np.isfinite(Tte[:, 0])
        err = pred[ok, 0] - Tte[ok, 0]
        base = np.median(Ttr[okt, 0]) - Tte[ok, 0]     # "cost proportional to 2^k": constant ns/vector
        # the large instances: those holding 90% of the vectors
        vec_ok = np.array([float(1 << p.k) for p in preps])[ok]
        big = np.argsort(-vec_ok)
        big = big[:int(np.searchsorted(np.cumsum(vec_ok[big]) / vec_ok.sum(), 0.9)) + 1]
        model_err = {"log_rmse": float(np.sqrt(np.mean(err ** 2))),
                     "mape": float(np.mean(np.abs(np.expm1(err)))),
                     "log_rmse_pow2_heuristic": float(np.sqrt(np.mean(base ** 2))),
                     "mape_pow2_heuristic": float(np.mean(np.abs(np.expm1(base)))),
                     "large_instances": int(len(big)),
                     "log_rmse_large": float(np.sqrt(np.mean(err[big] ** 2))),
                     "log_rmse_pow2_heuristic_large": float(np.sqrt(np.mean(base[big] ** 2))),
                     "train_instances": len(Xtr), "train_loss": train_loss}
        log(f"model error on fresh instances: {model_err}")

    if args.copy_calibration:
        a = torch.empty(1 << 26, dtype=torch.int32, device="cuda")
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()

    dom_ops = sweep_ops(dom_preps, roof_stats)
    achieved = dom_ops / (dom_ms * 1e-3) / 1e12
    # the same launch priced at the plain per-ridge check's work per vector
    # (AND + popcount per parent word of every critical ridge), weighted by 2^k
    plain_ops = sum(float(1 << p.k) * ops_alg_plain(p) for p, c in zip(preps, batch.cls)
                    if int(c) == dom and p.k > 0)
    plain_per_vec = plain_ops / cls_vec[dom]
    effective = plain_ops / (dom_ms * 1e-3) / 1e12
    probe = E.valu_probe(0, 4)
    # the walk's fast step: its instruction-mix ceiling: per vector 4.5 two-source ops
    # (4 XORs, a quarter of a minimum and of a compare) and 2.25 three-source
    # ops (2 logic ops, a quarter of a 3-input minimum) at the probe's rates
    # (nothing to compare a descent with)
    mix_ceiling = None
    if any(walked(p) for p in dom_preps):
        probe3 = E.valu_probe(1, 8)
        probe2 = E.valu_probe(0, 8)
        mix_ceiling = ALG_OPS_PER_VECTOR / (4.5 / probe2 + 2.25 / probe3)
    def profiled(name):
        path = os.path.join(ROOT, "profiles", name)
        if not os.path.exists(path):
            return None
        with open(path) as f:
            j = json.load(f)
        same = (j.get("kernel_source_sha256") == kernel_sources_sha256() and j.get("kernel") == dom_name
                and j.get("vectors") == float(cls_vec[dom]))
        return j if same else None
    counters = profiled("sweep_counters.json")
    traffic = (profiled("sweep_traffic.json") or {}).get("bytes_per_launch")
    line = {
        "metric": "kernel vectors checked/sec + WPM count (bit-exact); batched+learned vs plain",
        "value": vectors / t_b,
        "unit": "kernel vectors/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": t_b * 1e3,
        "ms_per_step_median": step_med,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "u32",
        "data": "synthetic (seeded SplitMix64 inputs)",
        "config": {"workload": WORKLOADS[args.workload].format(count=len(preps)),
                   "instances": len(preps), "sum_2k": vectors, "cbits": args.cbits,
                   "wg_size": args.wg, "waves_per_simd": waves_used, "records": args.records,
                   "record_copy_parts": args.parts if args.records == "copy" else None,
                   "schedule": f"learned: {args.learned_policy}, LPT on MLP-predicted cost"},
        "wpm_total": int(res_b.total),
        "wpm_counts_sha256": __import__("hashlib").sha256(res_b.counts.tobytes()).hexdigest(),
        "wpm_counts_match_oracle": oracle_counts_match(res_b.counts, args.workload, len(preps)),
        "kernel_ms": k_b,
        "kernel_ms_median": kern_med,
        "end_to_end": e2e,
        "schedules": out,
        "pruned": pruned,
        "cost_model": model_err,
        "autotune": None if tuned is None else {"key": tuned["key"], "cbits": tuned["cbits"],
                                                "wg": tuned["wg"], "waves": tuned.get("waves"),
                                                "cached": tuned["cached"]},
        "roofline": {"bound": "alu", "achieved": achieved, "peak": INT32_PEAK / 1e12,
                     "unit": "Tops/s (int32 VALU lane-ops)", "frac": achieved / (INT32_PEAK / 1e12),
                     "traffic": traffic, "kernel": dom_name, "kernel_ms": dom_ms,
                     "vectors_per_launch": cls_vec[dom], "ops_per_vector": dom_ops / cls_vec[dom],
                     "subcubes_opened": {b: int(n) for b, n in zip(("2^18", "2^12", "2^6"), roof_stats[5:8])},
                     "candidates": int(roof_stats[0]),
                     "ops_alg_plain_per_vector": plain_per_vec,
                     "effective_plain": effective, "effective_plain_frac": effective / (INT32_PEAK / 1e12),
                     "note": "every kernel vector is decided: by a ridge that fails for its whole sub-cube, or "
                             "down to the vector itself (every count equals the oracle's). frac counts the int32 ops "
                             "of the tests made; effective_plain prices all vectors at the plain per-ridge "
                             "AND+popcount check",
                     "measured_int32_xor_peak": probe / 1e12,
                     "mix_ceiling": None if mix_ceiling is None else mix_ceiling / 1e12,
                     "mix_ceiling_frac": None if mix_ceiling is None else mix_ceiling / INT32_PEAK,
                     "executed_frac": None if counters is None else
                     counters["executed_lane_ops_per_s"] / INT32_PEAK,
                     "valu_busy": None if counters is None else counters["valu_busy"]},
    }
    if not args.no_cpu:
        line["cpu_baseline"] = cpu_baseline(preps, args.cpu_budget)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
