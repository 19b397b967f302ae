#!/usr/bin/env python3
"""Throughput of node2vec second-order walks on one MI355X.

A step is one pass of the whole hot path over one batch: every walk of the
workload (r walks from every vertex, L moves each) generated by the persistent
walk kernel from a resident graph into a resident output matrix.  The graph is
built on the device (R-MAT generator and CSR build) before timing.

Prints one JSON line: transitions per second (moves actually taken), the
dominant kernel's achieved algorithmic bandwidth against the HBM peak, the
plain one-launch-per-move form measured on the same GPU, and the CPU oracle
timed on a bounded sample of the same workload.  Other workloads: c1, c2 and
c5 (visit counts), c4 (serving, p50/p99 latency), the paper's graph families
(skew<S>, wec<K>, er<K>; --approx T for FN-Approx) and their whole studies
(paper-skew, paper-wec, paper-er: one JSON line per cell).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "2nd-order walk steps/sec + % HBM roofline, 1 MI355X; p50/p99 request latency"
HBM_PEAK_GBS = 8000.0
KERNEL = "k_persistent"
KERNEL_SRC = os.path.join(ROOT, "paper_1805_00280_amd", "csrc", "walk.hip")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def finite(x):
    """x with every non-finite float replaced by None (the output line is strict JSON)."""
    if isinstance(x, float) and not np.isfinite(x):
        log(f"[bench] non-finite value {x} reported as null")
        return None
    if isinstance(x, dict):
        return {k: finite(v) for k, v in x.items()}
    if isinstance(x, (list, tuple)):
        return [finite(v) for v in x]
    return x


def emit_line(line):
    print(json.dumps(finite(line), allow_nan=False), flush=True)


def kernel_sha():
    return hashlib.sha256(open(KERNEL_SRC, "rb").read()).hexdigest()[:16]


def load_traffic(workload):
    """The committed rocprofv3 counter summary of the workload (HBM bytes per
    launch, L2 hit rate), when it was taken on the current kernel source."""
    path = os.path.join(ROOT, "profiles", f"traffic_{workload}.json")
    if not os.path.exists(path):
        return None
    try:
        t = json.load(open(path))
    except ValueError:
        return None
    # also sources whose k_persistent device assembly was compared equal to
    # the profiled build's (listed in the summary with how that was checked)
    if kernel_sha() not in [t.get("kernel_sha")] + list(t.get("same_code_shas", [])):
        return None
    return t


def available_cores():
    """Cores this process may use on the host: its affinity set, capped by a cgroup CPU quota."""
    n = len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else (os.cpu_count() or 1)
    try:
        quota, period = open("/sys/fs/cgroup/cpu.max").read().split()[:2]
        if quota != "max":
            n = min(n, max(1, -(-int(quota) // int(period))))
    except (OSError, ValueError):
        pass
    return max(1, n)


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def cpu_baseline(w, target_s, max_threads=0, approx_t=0):
    """The oracle timed on seeded samples of the workload's walks, on every core
    available to this process and on one thread, plus the oracle's isolated
    algorithmic-bytes model over a sample of the same walks, split by class."""
    import oracle as O
    threads = available_cores() if not max_threads else max(1, min(max_threads, available_cores()))
    t0 = time.perf_counter()
    og = O.rmat_csr(*w.rmat_args(), weighted=w.weighted, nthreads=threads)
    log(f"[cpu] oracle CSR scale {w.scale}: {time.perf_counter() - t0:.1f}s, m={og.m}")

    def timed_sample(nth, target, seed):
        # grow the sample until one timed run takes at least 0.7 of target
        count = 64
        while True:
            ids = w.sample_walk_ids(count, seed=seed)
            t1 = time.perf_counter()
            r = O.walk(og, (ids % w.n).astype(np.uint32), w.L, w.p, w.q, w.seed, wids=ids, want_out=False,
                       nthreads=nth, approx_t=approx_t)
            dt = time.perf_counter() - t1
            if dt >= 0.7 * target or count >= w.walks:
                return count, r["transitions"], dt
            count = int(min(w.walks, count * min(64.0, max(2.0, 1.2 * target / max(dt, 1e-3)))))

    count, moves, dt = timed_sample(threads, target_s, 12)
    log(f"[cpu] oracle {count} walks, {moves} moves in {dt:.1f}s on {threads} threads")
    count1, moves1, dt1 = timed_sample(1, target_s * 0.6, 14)
    log(f"[cpu] oracle {count1} walks, {moves1} moves in {dt1:.1f}s on 1 thread")
    cost_ids = w.sample_walk_ids(min(count, 2048), seed=13)
    t0 = time.perf_counter()
    cls = O.walk_cost_classes(og, (cost_ids % w.n).astype(np.uint32), cost_ids, w.L, w.p, w.q, w.seed,
                              nthreads=threads, approx_t=approx_t)
    hub_b, hub_m, oth_b, oth_m = cls
    log(f"[cpu] cost model {len(cost_ids)} walks: {(hub_b + oth_b) / max(hub_m + oth_m, 1):.1f} B/move isolated, "
        f"other moves {oth_b / max(oth_m, 1):.1f} B/move ({time.perf_counter() - t0:.1f}s)")
    base = {"value": moves / dt, "unit": "steps/s", "cores": threads, "kind": "oracle",
            "value_1thread": moves1 / dt1, "host_cpus": os.cpu_count(), "cpu_model": cpu_model(),
            "sample": f"{count} seeded-random walks of the {w.name} workload ({moves} moves) on {threads} threads, "
                      f"{count1} walks ({moves1} moves) on 1 thread; walk phase only, graph prebuilt"
                      + (f", FN-Approx 1/{approx_t}" if approx_t else "")}
    model = {"isolated_bytes_per_move": (hub_b + oth_b) / max(hub_m + oth_m, 1),
             "other_bytes_per_move": oth_b / max(oth_m, 1), "hub_share": hub_m / max(hub_m + oth_m, 1),
             "sample_walks": len(cost_ids)}
    return base, model


MEMO_MAX_DEG = 4161536


def pass_bytes(off, out, L, d_rule, memo_min, weighted):
    """Memo-aware algorithmic bytes of one pass, read off its walk matrix (the
    model the oracle defines in or_memo_pass_bytes, evaluated with torch on the
    matrix's device, one column at a time).  A second-order move at a vertex
    above d_rule pays v's offset lines, its output, and the cheaper of a cold
    evaluation (merge N(v) with N(t), or search N(t)'s members in N(v)) and,
    where v keeps pair summaries, a warm one (v's summary row, 6 bytes per
    segment, 22 on weighted graphs, the half segment of N(v) holding the draw
    and N(t)'s share of it); each distinct
    pair whose moves read a summary pays its intersection once.  Returns the
    hub-move bytes with summaries (memo) and without (cold), and the counts."""
    import torch
    dev = out.device
    off = off.to(dev).long()
    deg = off[1:] - off[:-1]
    mask32 = 0xFFFFFFFF

    def lines(elem, lo, hi):
        return torch.where(hi > lo, ((hi * elem - 1) >> 6) - ((lo * elem) >> 6) + 1, torch.zeros_like(lo))

    def levels(d):
        k = torch.ones_like(d)
        for j in range(1, 40):
            k += ((16 << j) < d).long()
        return k

    memo_b = torch.zeros((), dtype=torch.int64, device=dev)
    cold_b = torch.zeros((), dtype=torch.int64, device=dev)
    warm_b = torch.zeros((), dtype=torch.int64, device=dev)  # moves that read a summary
    hub_m = other_m = warm_m = 0
    keys = []
    summaries = memo_min is not None
    for s in range(L):
        valid = out[:, s + 1] != -1
        if s == 0:
            other_m += int(valid.sum().item())
            continue
        v = out[valid, s].long() & mask32
        t = out[valid, s - 1].long() & mask32
        dv = deg[v]
        hub = dv > d_rule
        other_m += int((~hub).sum().item())
        v, t, dv = v[hub], t[hub], dv[hub]
        if v.numel() == 0:
            continue
        hub_m += v.numel()
        dt = deg[t]
        ov, ot = off[v], off[t]
        rt = lines(4, ot, ot + dt)
        wl = lines(2, ov, ov + dv) if weighted else torch.zeros_like(dv)
        cold = torch.minimum(lines(4, ov, ov + dv) + rt + wl, rt + dt * levels(dv) + wl)
        offl = lines(8, v, v + 2)
        cold_b += ((offl + cold) * 64 + 4).sum()
        if not summaries:
            memo_b += ((offl + cold) * 64 + 4).sum()
            continue
        keep = (dv >= memo_min) & (dv <= MEMO_MAX_DEG)
        tiles = (dv + 511) // 512
        per = (tiles + 63) // 64
        seglen = per * 512
        h = torch.minimum(seglen // 2, dv)
        ht = (dt * h + dv - 1) // dv
        segs = (((tiles + per - 1) // per) + 1) & ~1  # the row's segments, rounded up to even
        if weighted:  # the row's weight sums, the half segment's weights
            warm = (22 * segs + 63) // 64 + (4 * h + 63) // 64 + (2 * h + 63) // 64 + (4 * ht + 63) // 64
        else:
            warm = (6 * segs + 63) // 64 + (4 * h + 63) // 64 + (4 * ht + 63) // 64
        usew = keep & (warm < cold)
        warm_m += int(usew.sum().item())
        memo_b += ((offl + torch.where(usew, warm, cold)) * 64 + 4).sum()
        warm_b += (((offl + warm) * 64 + 4) * usew).sum()
        tk = (dt >= memo_min) & (dt <= MEMO_MAX_DEG) & (not weighted)
        a = torch.where(tk, torch.minimum(t, v), v)
        b = torch.where(tk, torch.maximum(t, v), t)
        k = ((a << 32) | b)[usew]
        if k.numel():
            keys.append(torch.unique(k))
    inter = 0
    inter_b = torch.zeros((), dtype=torch.int64, device=dev)
    if keys:
        k = torch.unique(torch.cat(keys))
        keys.clear()
        inter = k.numel()
        a, b = k >> 32, k & mask32
        da, db = deg[a], deg[b]
        if weighted:  # keys (v, t): the directed cold evaluation, weights of N(v) included
            rt = lines(4, off[b], off[b] + db)
            wl = lines(2, off[a], off[a] + da)
            pair = torch.minimum(lines(4, off[a], off[a] + da) + rt + wl, rt + db * levels(da) + wl)
        else:
            dense = lines(4, off[a], off[a] + da) + lines(4, off[b], off[b] + db)
            first = da <= db
            sh = torch.where(first, a, b)
            dsh = torch.where(first, da, db)
            dlo = torch.where(first, db, da)
            search = lines(4, off[sh], off[sh] + dsh) + dsh * levels(dlo)
            pair = torch.minimum(dense, search)
        inter_b = (pair * 64).sum()
        memo_b += inter_b
    return {"hub_bytes": int(memo_b.item()), "hub_bytes_cold": int(cold_b.item()), "hub_moves": hub_m,
            "other_moves": other_m, "warm_moves": warm_m, "intersections": inter,
            "warm_bytes": int(warm_b.item()), "intersection_bytes": int(inter_b.item())}


def copy_calibration():
    """Three copies of 4 GiB: a kernel of known traffic (4 GiB read and 4 GiB
    written per copy) against which FETCH_SIZE and WRITE_SIZE are scaled."""
    import torch
    n = 1 << 30
    a = torch.empty(n, dtype=torch.int32, device="cuda")
    b = torch.empty(n, dtype=torch.int32, device="cuda")
    a.fill_(1)
    torch.cuda.synchronize()
    for _ in range(3):
        t0 = time.perf_counter()
        b.copy_(a)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        log(f"[copy] 4 GiB in {dt * 1e3:.1f} ms: {2 * n * 4 / dt / 1e9:.0f} GB/s")


def counts(args, w):
    """Counts form (by default R-MAT scale 27, about 4.2G directed entries, u64
    offsets): every vertex starts one walk of 80 moves; walks run in chunks of
    --chunk walks (walk_base keeps each walk's random stream; by default one
    chunk) and reduce on the device to per-vertex visit counts plus a 64-bit
    checksum."""
    import torch
    import paper_1805_00280_amd as P

    dev = "cuda:0"
    t0 = time.perf_counter()
    g = P.Graph.from_rmat(*w.rmat_args(), weighted=False, device=dev)
    torch.cuda.synchronize()
    log(f"[counts] graph scale {w.scale} built in {time.perf_counter() - t0:.1f}s: m={g.m}")
    # sketches for the hub rows that fit in free device memory (highest degrees first)
    memo = 0
    if not args.no_memo:
        # one contiguous allocation: hand the allocator's cached blocks back first
        torch.cuda.empty_cache()
        free, _ = torch.cuda.mem_get_info()
        memo = g.attach_memo(budget=max(0, free - (8 << 30)))
        log(f"[counts] {free / 2**30:.1f} GiB free: pair sketches {memo / 2**30:.1f} GiB for rows of degree >= "
            f"{g.memo_min_degree}")
    cnt = torch.zeros(w.n, dtype=torch.int32, device=dev)
    cs = torch.zeros(1, dtype=torch.int64, device=dev)
    stream = torch.cuda.current_stream()
    opts = P.exec_opts(g)

    def one_pass(tag):
        cnt.zero_()
        cs.zero_()
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        ev0 = torch.cuda.Event(enable_timing=True)
        ev1 = torch.cuda.Event(enable_timing=True)
        ev0.record(stream)
        g.memo_clear(stream)
        for lo in range(0, w.walks, args.chunk):
            hi = min(lo + args.chunk, w.walks)
            st = torch.arange(lo, hi, dtype=torch.int64, device=dev).remainder_(w.n).to(torch.int32)
            g.walk_counts(st, w.L, w.p, w.q, w.seed, cnt, cs, walk_base=lo, opts=opts, stream=stream,
                          approx_t=args.approx)
            torch.cuda.synchronize()
            log(f"[counts] {tag}: walks [{lo}, {hi}) done at {time.perf_counter() - t1:.1f}s")
        ev1.record(stream)
        torch.cuda.synchronize()
        return time.perf_counter() - t1, ev0.elapsed_time(ev1)

    for i in range(args.warmup):
        one_pass(f"warmup {i}")
    walls, kms = [], []
    for i in range(args.steps):
        wall, km = one_pass(f"step {i}")
        walls.append(wall)
        kms.append(km)
    g.check_starts()
    visits = int(cnt.to(torch.int64).sum().item())
    moves = visits - w.walks
    # mean visits per equi-width degree bucket (the paper's frequency-versus-degree figure)
    dmax = int((g.off[1:] - g.off[:-1]).max().item())
    width = max(1, -(-dmax // 64))
    pv, pc = g.visit_profile(cnt, width, 66)
    pv, pc = pv.cpu().numpy(), pc.cpu().numpy()
    profile = {"width": width, "buckets": [[int(k) * width, int(pv[k]), float(pc[k] / pv[k])]
                                           for k in range(66) if pv[k]]}
    checksum = int(cs.cpu().numpy().view(np.uint64)[0])
    ms = float(np.mean(walls)) * 1000.0
    log(f"[counts] {moves} moves, {ms:.0f} ms/pass, {moves / ms * 1e3 / 1e6:.1f} M moves/s, checksum {checksum:#x}")
    line = {"metric": METRIC, "value": moves / (ms / 1000.0), "unit": "steps/s", "n_gpus": 1, "steps": args.steps,
            "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "u32", "data": "synthetic",
            "config": {"workload": w.name, "scale": w.scale, "edge_factor": w.edge_factor, "abc": [w.a, w.b, w.c],
                       "p": w.p, "q": w.q, "walks": w.walks, "walk_length": w.L, "entries": g.m,
                       "chunk_walks": args.chunk, "outputs": "visit counts + checksum", "pair_sketch_bytes": memo,
                       "approx_t": args.approx,
                       "pair_sketch_min_degree": g.memo_min_degree if memo else None,
                       "checksum": f"{checksum:#018x}", "visits": visits, "event_ms": float(np.mean(kms))},
            "visit_profile": profile}
    paper = paper_context(w)
    if paper:
        line["paper"] = paper
    emit_line(line)


def serving(loads, warm, measured, check=3, sat_requests=240, window=32, log_tag="serve"):
    """Serving workload: the R-MAT scale-22 graph resident with pair sketches, a
    server with a 24 GiB pool (65536-walk chunks, 64 chunks and 2^19 walks per
    tick) and the Philox-drawn request stream (sizes floor(2^(20U)) in
    [1, 2^20], L in {20, 40, 80}, p and q over {1/4, 1/2, 1, 2, 4}).
    Saturation is measured in a closed loop that keeps `window` requests
    outstanding; then, for each offered load rho, `warm` warm-up and `measured`
    timed requests arrive as a Poisson stream at rho x saturation.  Latency is
    completion minus submission (the server's own stamps).  A seeded subset of
    each load's requests is checked against the same request walked alone and
    against the oracle on sampled rows."""
    import threading

    import torch
    import oracle as O
    import paper_1805_00280_amd as P
    from paper_1805_00280_amd import workloads as WL

    w = WL.C4
    dev = "cuda:0"
    g = P.Graph.from_rmat(*w.rmat_args(), weighted=False, device=dev)
    memo = g.attach_memo()
    torch.cuda.synchronize()
    log(f"[{log_tag}] graph scale {w.scale}: m={g.m}, pair sketches {memo / 2**30:.1f} GiB")
    og = O.rmat_csr(*w.rmat_args(), weighted=False, nthreads=available_cores())
    srv = P.Server(g, pool_bytes=24 << 30, chunk_walks=65536, max_inflight=64, tick_walks=1 << 19)
    next_j = [0]

    def draw(k):
        reqs = WL.serving_requests(k, w.n, first=next_j[0])
        next_j[0] += k
        return reqs

    def work(r):
        return len(r["starts"]) * r["L"]

    def closed_loop(reqs):
        """Keeps `window` requests outstanding; returns moves/s between the
        completion of the first sixth and of the last request."""
        pending, times, moves, i = {}, [], [], 0
        while i < len(reqs) or pending:
            while i < len(reqs) and len(pending) < window:
                r = reqs[i]
                pending[srv.submit(r["starts"], r["L"], r["p"], r["q"], r["seed"])] = work(r)
                i += 1
            for t in list(pending):
                res = srv.poll(t)
                if res is not None:
                    times.append(res.done_ns / 1e9)
                    moves.append(pending.pop(t))
                    srv.release(t)
            time.sleep(0.0002)
        k0 = len(times) // 6
        order = np.argsort(times)
        tt = np.array(times)[order]
        mv = np.array(moves)[order]
        return float(mv[k0 + 1:].sum() / (tt[-1] - tt[k0]))

    def open_loop(reqs, rate, check_idx):
        arrive = WL.arrival_times(reqs, rate)
        tickets = [None] * len(reqs)

        def client():
            t0 = time.perf_counter()
            for i, r in enumerate(reqs):
                d = t0 + arrive[i] - time.perf_counter()
                if d > 0:
                    time.sleep(d)
                tickets[i] = srv.submit(r["starts"], r["L"], r["p"], r["q"], r["seed"])

        th = threading.Thread(target=client)
        t0 = time.perf_counter()
        th.start()
        lat = [None] * len(reqs)
        left, checked = set(range(len(reqs))), {}
        depth = []
        while left:
            for i in list(left):
                if tickets[i] is None:
                    continue
                res = srv.poll(tickets[i])
                if res is None:
                    continue
                lat[i] = (res.done_ns - res.submit_ns) / 1e6
                if i in check_idx:
                    checked[i] = srv.result_tensor(res)
                srv.release(tickets[i])
                left.discard(i)
            depth.append(srv.stats()[0] + srv.stats()[1])
            time.sleep(0.0002)
        th.join()
        return np.array(lat), time.perf_counter() - t0, checked, float(np.mean(depth))

    sat = closed_loop(draw(sat_requests))
    log(f"[{log_tag}] saturation {sat / 1e6:.1f} M moves/s (closed loop, {sat_requests} requests, "
        f"{window} outstanding)")
    rng = np.random.default_rng(11)
    out = {"saturation_steps_per_s": sat, "loads": []}
    for rho in loads:
        wreqs, mreqs = draw(warm), draw(measured)
        mean_work = np.mean([work(r) for r in mreqs])
        rate = rho * sat / mean_work
        open_loop(wreqs, rate, set())
        check_idx = set(rng.choice(len(mreqs), size=min(check, len(mreqs)), replace=False).tolist())
        lat, dt, checked, depth = open_loop(mreqs, rate, check_idx)
        mism_alone = mism_oracle = 0
        for i, got in checked.items():
            r = mreqs[i]
            st = torch.from_numpy(r["starts"].view(np.int32)).to(dev)
            alone = g.walk(st, r["L"], r["p"], r["q"], r["seed"]).cpu().numpy().view(np.uint32)
            mism_alone += int(not np.array_equal(got, alone))
            n = len(r["starts"])
            idx = np.arange(n) if n <= 512 else np.sort(rng.choice(n, size=512, replace=False))
            want = O.walk(og, r["starts"][idx], r["L"], r["p"], r["q"], r["seed"], wids=idx.astype(np.uint64),
                          nthreads=available_cores())["out"]
            mism_oracle += int(not np.array_equal(got[idx], want))
        moves = sum(work(r) for r in mreqs)
        rec = {"offered_load": rho, "arrival_rate_per_s": rate, "requests": len(mreqs), "warmup_requests": len(wreqs),
               "p50_ms": float(np.percentile(lat, 50)), "p99_ms": float(np.percentile(lat, 99)),
               "mean_ms": float(lat.mean()), "max_ms": float(lat.max()), "steps_per_s": moves / dt,
               "mean_queue_depth": depth, "checked_requests": len(checked),
               "mismatch_vs_alone": mism_alone, "mismatch_vs_oracle": mism_oracle}
        log(f"[{log_tag}] rho {rho}: {len(mreqs)} requests at {rate:.1f}/s: p50 {rec['p50_ms']:.1f} ms, "
            f"p99 {rec['p99_ms']:.1f} ms, {moves / dt / 1e6:.1f} M moves/s, depth {depth:.1f}, "
            f"mismatches alone {mism_alone} oracle {mism_oracle}")
        out["loads"].append(rec)
    srv.close()
    g.detach_memo()
    del g
    torch.cuda.empty_cache()
    return out


def serve(args):
    """The serving workload on its own line: p50/p99 latency per offered load."""
    loads = [float(x) for x in args.loads.split(",")]
    res = serving(loads, args.warm_requests, args.requests, check=args.check_requests)
    main = res["loads"][min(range(len(loads)), key=lambda i: abs(loads[i] - 0.8))]
    line = {"metric": METRIC, "value": main["steps_per_s"], "unit": "steps/s", "n_gpus": 1,
            "steps": main["requests"], "warmup": main["warmup_requests"],
            "ms_per_step": main["mean_ms"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "u32", "data": "synthetic",
            "config": {"workload": "rmat22-serving", "scale": 22, "pool_bytes": 24 << 30, "chunk_walks": 65536,
                       "tick_walks": 1 << 19, "requests_per_load": args.requests, "loads": loads},
            "latency_ms": {"p50": main["p50_ms"], "p99": main["p99_ms"]}, "serving": res}
    emit_line(line)


def skipgram_leg(steps=16, warmup=2, batch=1 << 16, window=10, negatives=64, log_tag="sgns"):
    """Skip-gram with negative sampling over node2vec walks: walks of the scale-20
    weighted workload (p = 1, q = 1/2, one 80-move walk per vertex) generated on
    the device, then `steps` timed SGD steps of `batch` walks each (dimension
    128, window 10, 64 shared negatives per walk, noise weights degree^0.75).
    Roofline: the useful dot products (3 x 2 x 128 flops per center-target
    pair) against the bf16 MFMA peak, and the bytes a step must move (the rows
    it gathers, their fp32 gradient read-modify-writes and the update pass over
    both tables) against the HBM peak."""
    import torch
    import paper_1805_00280_amd as P
    from paper_1805_00280_amd import workloads as WL

    dev = "cuda:0"
    w = WL.C2
    g = P.Graph.from_rmat(*w.rmat_args(), weighted=True, device=dev)
    n = w.n
    starts = torch.arange(n, dtype=torch.int32, device=dev)
    walks = g.walk(starts, w.L, w.p, w.q, w.seed)
    deg = (g.off[1:] - g.off[:-1]).double()
    cum = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    cum[1:] = torch.cumsum(torch.floor(deg.pow(0.75) * 1024.0).long(), 0)
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    win = ((torch.rand((n, 128), generator=gen, device=dev) - 0.5) / 128.0).float()
    wout = ((torch.rand((n, 128), generator=gen, device=dev) - 0.5) / 128.0).float()
    sg = P.SkipGram(n, win, wout, cum, window=window, negatives=negatives, lr=0.025, seed=11, max_walks=batch)
    stream = torch.cuda.current_stream()
    nb = walks.shape[0] // batch
    lens = (walks != -1).sum(1).long()  # rows end at their first sentinel
    m = lens.double()
    # (center, context) pairs of a walk of m positions: sum_i min(i, w) + min(m - 1 - i, w)
    i = torch.arange(walks.shape[1], device=dev).double()
    pairs = ((torch.minimum(i, torch.tensor(float(window), device=dev)).unsqueeze(0)
              + torch.minimum((m.unsqueeze(1) - 1 - i).clamp(min=0), torch.tensor(float(window), device=dev)))
             * (i.unsqueeze(0) < m.unsqueeze(1))).sum(1)
    flops_walk = 3 * 2 * 128 * (pairs + m * negatives)
    rows_walk = m + m + negatives * (m > 0).double()
    bytes_walk = rows_walk * 512 * 3  # gather, then the gradient row read and written
    apply_bytes = 2 * n * 128 * 4 * 4  # both tables: read w and g, write w and g
    for k in range(warmup):
        sg.step(walks[(k % nb) * batch:(k % nb + 1) * batch], walk_base=(k % nb) * batch, stream=stream)
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    a.record(stream)
    flops = byts = 0.0
    for k in range(steps):
        lo = (k % nb) * batch
        sg.step(walks[lo:lo + batch], walk_base=lo, stream=stream)
    b.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms = a.elapsed_time(b)
    for k in range(steps):
        lo = (k % nb) * batch
        flops += float(flops_walk[lo:lo + batch].sum().item())
        byts += float(bytes_walk[lo:lo + batch].sum().item()) + apply_bytes
    loss = float(sg.loss.item())
    tfs = flops / (ms / 1000.0) / 1e12
    gbs = byts / (ms / 1000.0) / 1e9
    res = {"walks_per_s": steps * batch / (ms / 1000.0), "ms_per_step": ms / steps, "wall_ms_per_step": wall * 1000 / steps,
           "steps": steps, "batch_walks": batch, "dim": 128, "window": window, "negatives": negatives,
           "graph": w.name, "loss_per_step": loss / (steps + warmup),
           "roofline": {"mfma": {"achieved": tfs, "peak": 2500.0, "unit": "TFLOP/s", "frac": tfs / 2500.0},
                        "hbm": {"achieved": gbs, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": gbs / HBM_PEAK_GBS},
                        "flops_per_step": flops / steps, "bytes_per_step": byts / steps}}
    res["roofline"]["bound"] = "hbm" if gbs / HBM_PEAK_GBS >= tfs / 2500.0 else "mfma"
    log(f"[{log_tag}] {steps} steps of {batch} walks: {ms / steps:.2f} ms/step, {res['walks_per_s'] / 1e6:.2f} M walks/s, "
        f"{tfs:.1f} TFLOP/s ({tfs / 2500.0:.4f} of bf16 peak), {gbs:.0f} GB/s ({gbs / HBM_PEAK_GBS:.3f} of HBM)")
    del sg, walks, g
    torch.cuda.empty_cache()
    return res


def count_moves(out, rows=1 << 22):
    """Entries past column 0 that hold a vertex, counted a block of rows at a
    time (the matrix can be most of the device's memory)."""
    total = 0
    for lo in range(0, out.shape[0], rows):
        total += int((out[lo:lo + rows, 1:] != -1).sum().item())
    return total


def paper_context(w):
    """The paper's own figure for the same graph family and (p, q), when it
    prints one (its 12-machine cluster: context, not a target)."""
    from paper_1805_00280_amd import workloads as WL
    fam = w.name.split("-")[0]
    out = {}
    if fam.startswith(("skew", "wec", "er")):
        t1 = WL.PAPER_TABLE1.get(fam)
        if t1:
            out["table1_entries"], out["table1_max_degree"] = t1
    if (w.p, w.q) == (0.5, 2.0) and fam in WL.PAPER_FN_BASE_SECONDS:
        out["fn_base_seconds"] = WL.PAPER_FN_BASE_SECONDS[fam]
        out["fn_base_hardware"] = "12 machines, 2 Xeon CPUs each, GraphLite (Section 4)"
    sp = WL.PAPER_FN_APPROX_SPEEDUP.get((fam, w.p, w.q))
    if sp:
        out["fn_approx_speedup_over_fn_base"] = sp
    return out


def paper_table(args):
    """The paper's graph-family studies, one 80-move walk from every vertex at
    (p, q) = (0.5, 2) and (2, 0.5), exact and FN-Approx, one JSON line per cell
    (graph built once per member, one untimed pass, one timed):
    paper-skew: Skew-S for S in 1.78, 2, 3, 4, 5 (Section 4.6);
    paper-wec: WeC-K for K in 20, 22, 24, 26 (Section 4.5);
    paper-er: ER-K for K in 20, 22, 24, 26, 28 (Section 4.4)."""
    import torch
    import paper_1805_00280_amd as P
    from paper_1805_00280_amd import workloads as WL

    dev = "cuda:0"
    torch.cuda.set_device(0)
    stream = torch.cuda.current_stream()
    members = {"paper-skew": [(WL.skew, S) for S in (1.78, 2.0, 3.0, 4.0, 5.0)],
               "paper-wec": [(WL.wec, K) for K in (20, 22, 24, 26)],
               "paper-er": [(WL.er, K) for K in (20, 22, 24, 26, 28)]}[args.workload]
    for make, S in members:
        w0 = make(S)
        t0 = time.perf_counter()
        g = P.Graph.from_rmat(*w0.rmat_args(), weighted=False, device=dev)
        memo = 0 if args.no_memo else g.attach_memo()
        deg = g.off[1:] - g.off[:-1]
        dmax = int(deg.max().item())
        torch.cuda.synchronize()
        log(f"[table] {w0.name.split('-')[0]}: m={g.m} max degree {dmax} built in {time.perf_counter() - t0:.1f}s, "
            f"sketches {memo / 2**30:.1f} GiB")
        starts = torch.arange(w0.walks, dtype=torch.int32, device=dev)
        out = torch.empty((w0.walks, w0.L + 1), dtype=torch.int32, device=dev)
        opts = P.exec_opts(g)
        for p, q in WL.PAPER_PQ:
            w = make(S, p, q)

            def timed(approx_t):
                g.memo_clear(stream)
                g.walk(starts, w.L, w.p, w.q, w.seed, out=out, opts=opts, stream=stream, approx_t=approx_t)
                torch.cuda.synchronize()
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                t1 = time.perf_counter()
                a.record(stream)
                g.memo_clear(stream)
                g.walk(starts, w.L, w.p, w.q, w.seed, out=out, opts=opts, stream=stream, approx_t=approx_t)
                b.record(stream)
                torch.cuda.synchronize()
                wall = time.perf_counter() - t1
                g.check_starts()
                return wall, a.elapsed_time(b), count_moves(out)

            wall, kms, moves = timed(0)
            awall, akms, amoves = timed(args.approx or 1000)
            line = {"metric": METRIC, "value": moves / wall, "unit": "steps/s", "n_gpus": 1, "steps": 1, "warmup": 1,
                    "ms_per_step": wall * 1000.0, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
                    "dtype": "u32", "data": "synthetic",
                    "config": {"workload": w.name, "scale": w.scale, "edge_factor": w.edge_factor,
                               "abc": [w.a, w.b, w.c], "p": p, "q": q, "walks": w.walks, "walk_length": w.L,
                               "entries": g.m, "max_degree": dmax, "pair_sketch_bytes": memo, "kernel_ms": kms},
                    "fn_approx": {"approx_t": args.approx or 1000, "ms_per_step": awall * 1000.0,
                                  "kernel_ms": akms, "moves": amoves, "speedup_vs_exact": wall / awall},
                    "paper": paper_context(w)}
            log(f"[table] {w.name}: exact {wall * 1e3:.1f} ms ({moves / wall / 1e6:.1f} M moves/s), "
                f"FN-Approx {awall * 1e3:.1f} ms ({wall / awall:.2f}x)")
            emit_line(line)
        del g, out, starts
        torch.cuda.empty_cache()


def resolve_workload(args):
    from paper_1805_00280_amd import workloads as WL
    if args.workload in ("c1", "c2", "c3", "c5"):
        return {"c1": WL.C1, "c2": WL.C2, "c3": WL.C3, "c5": WL.C5}[args.workload]
    p, q = (float(x) for x in args.pq.split(","))
    return WL.paper_family(args.workload, p, q)


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None, help="timed passes (default: 1 for c3, 3 otherwise)")
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="c3",
                    help="c1, c2, c3 (default), c4 (serving), c5 (counts); the paper's families skew<S>, wec<K>, "
                         "er<K>; paper-skew, paper-wec, paper-er for a whole family table")
    ap.add_argument("--pq", default="0.5,2", help="paper families: p,q (the paper uses 0.5,2 and 2,0.5)")
    ap.add_argument("--approx", type=int, default=0,
                    help="FN-Approx threshold 1/APPROX at hub moves (the paper's 1e-3 is 1000; 0: exact)")
    ap.add_argument("--outputs", choices=["walks", "counts"], default="walks",
                    help="paper families: full walk matrix, or visit counts + checksum (graphs too big for the matrix)")
    ap.add_argument("--chunk", type=int, default=1 << 27,
                    help="c5: walks per launch (default: all 2^27 in one launch, so pair sketches serve the whole pass)")
    ap.add_argument("--requests", type=int, default=2000, help="c4: measured requests per offered load")
    ap.add_argument("--warm-requests", type=int, default=200, help="c4: warm-up requests per offered load")
    ap.add_argument("--check-requests", type=int, default=5, help="c4: requests per load checked for parity")
    ap.add_argument("--loads", default="0.5,0.8,0.95", help="c4: offered loads as fractions of saturation")
    ap.add_argument("--no-skipgram", action="store_true", help="headline run: skip the Skip-gram leg")
    ap.add_argument("--no-serving", action="store_true",
                    help="headline run: skip the short serving leg (p50/p99 at 0.8 of saturation)")
    ap.add_argument("--no-plain", action="store_true", help="skip the plain one-launch-per-move form")
    ap.add_argument("--no-sketch-leg", action="store_true", help="skip the pass without pair sketches")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--cpu-threads", type=int, default=0, help="oracle threads (0: every core available)")
    ap.add_argument("--autotune", action="store_true", help="tune execution options before timing")
    ap.add_argument("--no-memo", action="store_true", help="do not attach pair-sketch memory")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run three 4 GiB device-to-device copies (scale reference for HBM byte counters)")
    args = ap.parse_args()
    if args.copy_calibration:
        copy_calibration()
        return
    if args.steps is None:
        args.steps = 1 if args.workload == "c3" else (16 if args.workload == "sgns" else 3)

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(f"bench.py: measures one GPU only (asked for {max(args.gpus, world)}); "
              f"the walk path would shard by walk ids with no exchange between GPUs", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_1805_00280_amd as P
    from paper_1805_00280_amd import workloads as WL

    if args.workload == "c4":
        serve(args)
        return
    if args.workload == "sgns":
        res = skipgram_leg(steps=args.steps or 16, warmup=args.warmup)
        line = {"metric": "Skip-gram walks/sec over node2vec walks, 1 MI355X", "value": res["walks_per_s"],
                "unit": "walks/s", "n_gpus": 1, "steps": res["steps"], "warmup": args.warmup,
                "ms_per_step": res["ms_per_step"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
                "dtype": "bf16", "data": "synthetic",
                "config": {"workload": "sgns-" + res["graph"], "batch_walks": res["batch_walks"], "dim": 128,
                           "window": res["window"], "negatives": res["negatives"]},
                "roofline": res["roofline"], "loss_per_step": res["loss_per_step"]}
        emit_line(line)
        return
    if args.workload in ("paper-skew", "paper-wec", "paper-er"):
        paper_table(args)
        return
    try:
        w = resolve_workload(args)
    except ValueError as e:
        print(f"bench.py: {e}", file=sys.stderr)
        sys.exit(2)
    if args.workload == "c5" or args.outputs == "counts":
        counts(args, w)
        return
    dev = "cuda:0"
    torch.cuda.set_device(0)
    log(f"[bench] workload {w.name}: n={w.n} walks={w.walks} L={w.L}")
    t0 = time.perf_counter()
    g = P.Graph.from_rmat(*w.rmat_args(), weighted=w.weighted, device=dev)
    torch.cuda.synchronize()
    log(f"[bench] graph built on device in {time.perf_counter() - t0:.2f}s: m={g.m}")
    memo_bytes = 0 if args.no_memo else g.attach_memo()
    log(f"[bench] pair-sketch memory: {memo_bytes / 2**30:.1f} GiB")
    starts = torch.arange(w.walks, dtype=torch.int64, device=dev).remainder_(w.n).to(torch.int32)
    out = torch.empty((w.walks, w.L + 1), dtype=torch.int32, device=dev)
    opts = P.exec_opts(g)
    if args.autotune:
        best, ms = g.autotune(1 << 16, w.L, w.p, w.q)
        opts = best
        log(f"[bench] autotuned {best.as_dict()} ({ms:.2f} ms on the tuning sample)")
    stream = torch.cuda.current_stream()

    def step():
        # a cold pass: sketches persist across calls, so the pass starts from cleared ones
        g.memo_clear(stream)
        g.walk(starts, w.L, w.p, w.q, w.seed, out=out, opts=opts, stream=stream, approx_t=args.approx)

    for i in range(args.warmup):
        t1 = time.perf_counter()
        step()
        torch.cuda.synchronize()
        log(f"[bench] warmup {i}: {time.perf_counter() - t1:.3f}s")
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i, (a, b) in enumerate(evs):
        a.record(stream)
        step()
        b.record(stream)
        if i + 1 < args.steps:  # progress line; the last step is closed by the synchronize below
            b.synchronize()
            log(f"[bench] step {i}: {a.elapsed_time(b):.1f} ms")
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    kernel_ms = float(np.mean([a.elapsed_time(b) for a, b in evs]))
    g.check_starts()
    moves = count_moves(out)
    ms_per_step = wall * 1000.0 / args.steps
    value = moves / (ms_per_step / 1000.0)
    log(f"[bench] persistent: {ms_per_step:.1f} ms/step wall, {kernel_ms:.1f} ms kernel, {moves} moves, "
        f"{value / 1e9:.3f} G steps/s")

    # algorithmic bytes of this launch, read off its own walk matrix (every form
    # below produces the same matrix)
    model = None
    if not args.approx:
        t1 = time.perf_counter()
        model = pass_bytes(g.off, out, w.L, g.d_rule, g.memo_min_degree if memo_bytes else None, w.weighted)
        log(f"[bench] bytes model ({time.perf_counter() - t1:.1f}s): {model}")

    nosk = None
    if memo_bytes and not args.no_sketch_leg:
        # the same pass without pair sketches (every hub move evaluated from scratch)
        nopts = P.exec_opts(g, memo=0)
        out2 = torch.empty_like(out)
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        g.walk(starts, w.L, w.p, w.q, w.seed, out=out2, opts=nopts, stream=stream, approx_t=args.approx)
        b.record(stream)
        torch.cuda.synchronize()
        nms = a.elapsed_time(b)
        same = bool(torch.equal(out, out2))
        nosk = {"ms_per_step": nms, "value": moves / (nms / 1000.0), "unit": "steps/s", "identical_to_persistent": same}
        log(f"[bench] no sketches: {nms:.1f} ms/step, {moves / nms / 1e6:.3f} G steps/s, identical={same}")
        del out2

    plain = None
    if not args.no_plain:
        popts = P.exec_opts(g, mode=P.MODE_PLAIN)
        pws = P._alloc(g.walk_workspace(w.walks, w.L, popts), dev)
        out2 = torch.empty_like(out)

        def plain_call():
            torch.cuda.synchronize()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            g.memo_clear(stream)
            g.walk(starts, w.L, w.p, w.q, w.seed, out=out2, opts=popts, ws=pws, stream=stream, approx_t=args.approx)
            b.record(stream)
            torch.cuda.synchronize()
            return a.elapsed_time(b)

        # the first call launches its L+2 or 2L+2 kernels directly; a repeat of the
        # same call is captured into a graph and replayed from then on, so
        # short passes are timed again on a replay
        direct = plain_call()
        pms, replayed = direct, None
        if direct < 1000.0:
            plain_call()
            replayed = plain_call()
            pms = replayed
        same = bool(torch.equal(out, out2))
        plain = {"ms_per_step": pms, "value": moves / (pms / 1000.0), "unit": "steps/s",
                 "most_launches_per_step": 1 + 2 * w.L, "direct_ms": direct, "replayed_ms": replayed,
                 "persistent_speedup": pms / kernel_ms, "identical_to_persistent": same}
        log(f"[bench] plain: {pms:.1f} ms/step (direct {direct:.2f} ms, replayed {replayed} ms), "
            f"{moves / pms / 1e6:.3f} G steps/s, identical={same}")
        del out2, pws

    cpu, cost = None, None
    if not args.no_cpu_baseline:
        cpu, cost = cpu_baseline(w, args.cpu_seconds, args.cpu_threads, args.approx)

    serv = None
    if args.workload == "c3" and not args.no_serving and not args.approx:
        # request latency beside the throughput: a short run of the serving workload
        # (its full protocol is --workload c4)
        g_memo = memo_bytes
        g.detach_memo()
        del out, starts
        torch.cuda.empty_cache()
        serv = serving([0.8], warm=50, measured=300, check=2, sat_requests=160, log_tag="serving")
        memo_bytes = g_memo
    sgns = None
    if args.workload == "c3" and not args.no_skipgram and not args.approx:
        # the stage the walks feed: Skip-gram steps over walks of the scale-20 workload
        try:
            del out
        except NameError:
            pass
        sgns = skipgram_leg(steps=8, warmup=2, log_tag="skipgram")

    counters = None if args.approx else load_traffic(w.name)
    traffic = counters.get("bytes_per_launch") if counters else None
    roof = {"bound": "hbm", "achieved": None, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": None,
            "traffic": traffic, "kernel": KERNEL, "kernel_ms": kernel_ms, "moves_per_launch": moves,
            "bytes_model": "memo-aware (oracle or_memo_pass_bytes; other moves at the oracle's sampled mean)"}
    if model is not None and cost is not None:
        other = model["other_moves"] * cost["other_bytes_per_move"]
        alg = other + model["hub_bytes"]
        achieved = alg / (kernel_ms / 1000.0) / 1e9
        roof.update({"achieved": achieved, "frac": achieved / HBM_PEAK_GBS, "bytes_per_launch": alg,
                     "bytes_by_class": {"intersections": model["intersection_bytes"], "warm_moves": model["warm_bytes"],
                                        "cold_moves": model["hub_bytes"] - model["intersection_bytes"]
                                        - model["warm_bytes"], "other_moves": other},
                     "bytes_per_move": alg / max(moves, 1), "hub_moves": model["hub_moves"],
                     "warm_hub_moves": model["warm_moves"], "intersections": model["intersections"],
                     "other_moves": model["other_moves"], "other_bytes_per_move": cost["other_bytes_per_move"],
                     "isolated_bytes_per_move": cost["isolated_bytes_per_move"],
                     "isolated_equiv_GBs": cost["isolated_bytes_per_move"] * moves / (kernel_ms / 1000.0) / 1e9})
        if roof["frac"] > 1.0:
            log(f"[bench] the bytes model gives {roof['frac']:.2f} of the HBM peak: not a roofline fraction, "
                f"frac withheld")
            roof["frac_withheld"] = roof["frac"]
            roof["frac"] = None
        if nosk is not None:
            nalg = other + model["hub_bytes_cold"]
            nosk["bytes_per_launch"] = nalg
            nosk["achieved_GBs"] = nalg / (nosk["ms_per_step"] / 1000.0) / 1e9
            nosk["frac"] = nosk["achieved_GBs"] / HBM_PEAK_GBS
    if traffic is not None:
        # measured HBM bytes of the same launch (counter run on this kernel source)
        roof["measured_GBs"] = traffic / (kernel_ms / 1000.0) / 1e9
        roof["measured_frac"] = roof["measured_GBs"] / HBM_PEAK_GBS
        roof["traffic_per_move"] = traffic / max(moves, 1)
        if counters.get("l2_hit_rate") is not None:
            roof["l2_hit_rate"] = counters["l2_hit_rate"]
    line = {
        "metric": METRIC, "value": value, "unit": "steps/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "u32", "data": "synthetic",
        "config": {"workload": w.name, "scale": w.scale, "edge_factor": w.edge_factor, "abc": [w.a, w.b, w.c],
                   "weighted": w.weighted, "p": w.p, "q": w.q, "walks_per_vertex": w.r, "walk_length": w.L,
                   "walks": w.walks, "vertices": w.n, "entries": g.m, "form": "persistent",
                   "pair_sketch_bytes": memo_bytes, "approx_t": args.approx,
                   "exec_opts": opts.as_dict()},
        "roofline": roof, "no_sketches": nosk, "plain": plain, "cpu_baseline": cpu,
    }
    if sgns is not None:
        line["skipgram"] = sgns
    if serv is not None:
        ld = serv["loads"][0]
        line["latency_ms"] = {"p50": ld["p50_ms"], "p99": ld["p99_ms"], "workload": "rmat22-serving",
                              "offered_load": ld["offered_load"], "requests": ld["requests"]}
        line["serving"] = serv
    paper = paper_context(w)
    if paper:
        line["paper"] = paper
    emit_line(line)


if __name__ == "__main__":
    main()
