#!/usr/bin/env python3
"""Benchmark of the SpecEE speculative early-exit predictor on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--only NAME] [--no-cpu]

One *step* is the full per-token hot path at the Llama2-7B shape with K=4 (the
"32-layer exit sweep for one token" workload): 32 dependent specee_predict calls,
one per decoder layer with that layer's predictor, each consuming the local
probabilities the previous call produced.  The calls are captured once into a HIP
graph per input set and the timed region replays graphs, rotating over input sets
(different hidden states and speculative ids) so that the LM-head rows of a step
are not in cache from the step before.  All inputs are resident in HBM before the
timed region; nothing is copied from or to the host inside it.

The single JSON line also carries, under "extra", the latency of the other
workloads (single step, token trees, full-vocabulary head and the speed-up over
it) and a throughput mode (many independent problems per launch) with its own
fraction of the HBM roofline; "cpu_baseline" times the CPU oracle on the same
workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0   # MI355X HBM3E, published
H = 512

# HBM bytes per launch of the dominant kernels, from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE
# runs scaled by the same counters on specee_calib_copy (see profiles/); None = not measured.
MEASURED_TRAFFIC = {}
_traffic_file = os.path.join(ROOT, "profiles", "hbm_traffic.json.txt")
if os.path.exists(_traffic_file):
    try:
        MEASURED_TRAFFIC = {k: v["fetch_bytes"] + v["write_bytes"] for k, v in
                            json.loads(open(_traffic_file).read().split("---JSON---")[1]).items()}
    except Exception:  # noqa: BLE001 - a malformed summary must not break the benchmark
        MEASURED_TRAFFIC = {}


def predict_bytes(d, K, B=1, Hh=H, distinct_rows=None):
    """Algorithmic bytes of one predictor launch: hidden states + RMSNorm weight + distinct
    LM-head rows + predictor weights + ids/prev/outputs."""
    rows = B * K if distinct_rows is None else distinct_rows
    return B * d * 2 + d * 2 + rows * d * 2 + (3 * K * Hh + Hh) * 2 + B * (K * 4 + K * 4 + 2 * K * 4 + 8)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=2000)
    ap.add_argument("--warmup", type=int, default=200)
    ap.add_argument("--sets", type=int, default=64, help="rotating input sets")
    ap.add_argument("--only", default="", help="comma-separated sections: sweep,single,batch,tree,lmhead,q4,loop,c4,c5,copy")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--no-extra", action="store_true", help="only the headline step")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build measures one GPU only (--gpus 1); the predictor shards by token with no "
              "communication", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2504_08850_amd import specee as sp
    from paper_2504_08850_amd import synth

    sp.lib()
    assert torch.cuda.is_available(), "bench.py needs the GPU"
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)

    def up(a):
        return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(dev)

    last_spread = {}

    def ev_time(fn, iters, warm):
        """Milliseconds per call of fn (median over up to ten consecutive samples of the timed calls), from HIP
        events on the stream the kernels run on.  The spread of the samples is kept for spread()."""
        for _ in range(warm):
            fn()
        torch.cuda.synchronize()
        nsamp = min(10, iters)
        per = max(1, iters // nsamp)
        evs = [torch.cuda.Event(enable_timing=True) for _ in range(nsamp + 1)]
        evs[0].record()
        for i in range(nsamp):
            for _ in range(per):
                fn()
            evs[i + 1].record()
        torch.cuda.synchronize()
        ms = np.array([evs[i].elapsed_time(evs[i + 1]) / per for i in range(nsamp)])
        last_spread.update(p10=float(np.percentile(ms, 10)), median=float(np.median(ms)),
                           p90=float(np.percentile(ms, 90)), samples=nsamp, calls_per_sample=per)
        return float(np.median(ms))

    def spread(div=1.0):
        """p10 / p90 of the last ev_time() in microseconds per unit (div units per call of fn)."""
        return {"us_p10": last_spread["p10"] * 1e3 / div, "us_p90": last_spread["p90"] * 1e3 / div,
                "timing_samples": last_spread["samples"]}

    def capture(fn):
        """Capture fn's launches into a HIP graph; returns the graph."""
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            fn()
        torch.cuda.current_stream().wait_stream(s)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            fn()
        torch.cuda.synchronize()
        return g

    only = set(x for x in args.only.split(",") if x)

    def want(*names):
        return not only or bool(only & set(names))
    extra = {}
    c2 = synth.CONFIGS["C2"]
    d, V, K, L = c2.d, c2.V, c2.K, c2.L
    t_setup = time.time()
    lm_h = synth.lm_head(V, d, synth.lm_seed(c2))
    lm = up(lm_h)
    base = synth.make("C2", lm=lm_h)
    gamma = up(base["gamma"])
    W1, w2 = up(base["W1"]), up(base["w2"])           # one predictor per layer, shared by all tokens

    # ------------------------------------------------------------------ headline: C2 sweep, 32 dependent calls
    R = args.sets
    result = None
    if want("sweep"):
        sets = []
        for r in range(R):
            hid = up(synth.hidden_drift(L, 1, d, 50_000 + r))
            ids = up(synth.ids_uniform_distinct(1, K, V, 60_000 + r))
            out = dict(logits=torch.empty((L, 1, K), device=dev), probs=torch.empty((L, 1, K), device=dev),
                       scores=torch.empty((L, 1), device=dev), exit=torch.empty((L, 1), dtype=torch.int32, device=dev))
            zero = torch.zeros((1, K), device=dev)
            sets.append((hid, ids, out, zero))

        def sweep_calls(r):
            hid, ids, out, zero = sets[r]
            for l in range(L):
                o = dict(logits=out["logits"][l], probs=out["probs"][l], scores=out["scores"][l], exit=out["exit"][l])
                sp.predict(hid[l], gamma, lm, ids, zero if l == 0 else out["probs"][l - 1], W1[l], w2[l], out=o)

        graphs = [capture(lambda r=r: sweep_calls(r)) for r in range(R)]
        for w in range(args.warmup):
            graphs[w % R].replay()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        # marks inside the timed region (an event record costs the stream nothing measurable): twenty slices of it
        nsl = max(1, min(20, args.steps))
        cuts = sorted(set(int(round(i * args.steps / nsl)) for i in range(1, nsl)))
        marks = {c: torch.cuda.Event(enable_timing=True) for c in cuts}
        t0 = time.perf_counter()
        e0.record()
        for k in range(args.steps):
            if k in marks:
                marks[k].record()
            graphs[k % R].replay()
        e1.record()
        torch.cuda.synchronize()
        wall_ms = (time.perf_counter() - t0) * 1e3
        ms_per_step = e0.elapsed_time(e1) / args.steps
        us_per_call = ms_per_step * 1e3 / L
        edges = [(0, e0)] + [(c, marks[c]) for c in cuts] + [(args.steps, e1)]
        slice_us = np.array([a[1].elapsed_time(b[1]) * 1e3 / ((b[0] - a[0]) * L) for a, b in zip(edges, edges[1:])])
        alg = predict_bytes(d, K)
        achieved = alg / (us_per_call * 1e-6) / 1e9
        result = {
            "metric": "predictor evals/s (Llama2-7B shape, K=4; per-layer speculative early-exit predictor)",
            "value": L / (ms_per_step * 1e-3),
            "unit": "evals/s",
            "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
            "ms_per_step": ms_per_step,
            "us_per_call": us_per_call,
            "us_per_call_p10_median_p90": [float(np.percentile(slice_us, 10)), float(np.median(slice_us)),
                                           float(np.percentile(slice_us, 90))],
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "f32", "dtype_note": "fp16 inputs widened exactly, fp32 products and sums", "data": "synthetic",
            "config": {"workload": "C2: 32-layer exit sweep for one token, d=4096 V=32000 K=4, MLP 12->512->1, "
                                   "32 dependent specee_predict launches per step (HIP graph replay), "
                                   f"{R} rotating input sets", "batch": 1, "layers": L},
            "roofline": {"bound": "hbm", "kernel": "predict_kernel<4,2,false,true,256,2>", "achieved": achieved,
                         "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                         "algorithmic_bytes_per_launch": alg,
                         "traffic": MEASURED_TRAFFIC.get("predict_c2"),
                         "note": "one call moves 62 KB, far below the ~8 MB bandwidth-delay product of HBM: this "
                                 "mode is bound by two dependent memory round trips plus launch, not by bandwidth; "
                                 "see extra.throughput for the bandwidth-bound mode"},
            "wall_ms_timed_region": wall_ms,
        }
        # the same sweep as ONE launch of specee_predict_sweep (all layers' hidden states known up front)
        if not args.no_extra:
            hid0, ids0, _, _ = sets[0]
            so = sp.predict_sweep(hid0, gamma, lm, ids0, W1, w2)
            gs = [capture(lambda r=r: sp.predict_sweep(sets[r][0], gamma, lm, sets[r][1], W1, w2, out=so))
                  for r in range(min(R, 16))]
            it = [0]

            def rot():
                gs[it[0] % len(gs)].replay()
                it[0] += 1
            ms = ev_time(rot, 400, 40)
            extra["c2_one_launch_sweep"] = {"us_per_sweep": ms * 1e3, "evals_per_s": L / (ms * 1e-3), **spread(),
                                            "note": "one graph launch per sweep: includes the host's launch of the graph"}
            # the same sweeps back to back inside one graph (no host launch between them)
            nb = min(R, 16)
            gb = capture(lambda: [sp.predict_sweep(sets[r][0], gamma, lm, sets[r][1], W1, w2, out=so) for r in range(nb)])
            msb = ev_time(gb.replay, 50, 5) / nb
            extra["c2_one_launch_sweep"]["us_per_sweep_back_to_back"] = msb * 1e3
            extra["c2_one_launch_sweep"]["back_to_back_spread"] = spread(nb)

    # ------------------------------------------------------------------ C1: isolated single call, cold vs warm
    if want("single") and not args.no_extra:
        t1 = synth.make("C1", lm=lm_h)
        R1 = 256
        hid = up(synth.hidden(R1, d, 123))
        ids = up(synth.ids_uniform_distinct(R1, K, V, 124))
        prev = up(synth.prob_rows(R1, K, 125))
        w1_1, w2_1 = up(t1["W1"]), up(t1["w2"])
        outs = sp.predict(hid[:1], gamma, lm, ids[:1], prev[:1], w1_1, w2_1)

        def cold_calls():
            for r in range(R1):
                sp.predict(hid[r:r + 1], gamma, lm, ids[r:r + 1], prev[r:r + 1], w1_1, w2_1, out=outs)

        def warm_calls():
            for r in range(R1):
                sp.predict(hid[:1], gamma, lm, ids[:1], prev[:1], w1_1, w2_1, out=outs)
        gc, gw = capture(cold_calls), capture(warm_calls)
        us_cold = ev_time(gc.replay, 20, 3) * 1e3 / R1
        sp_cold = spread(R1)
        us_warm = ev_time(gw.replay, 20, 3) * 1e3 / R1
        # the 256 rotating inputs above fit the 256 MB last-level cache; 7680 tokens whose rows cover the whole
        # head (and 63 MB of hidden states) do not, so these calls find their rows in HBM
        R2 = 7680
        rng = np.random.default_rng(77)
        hid2 = up(rng.standard_normal((R2, d), dtype=np.float32).astype(np.float16))
        ids2 = up(rng.permutation(V)[:R2 * K].reshape(R2, K).astype(np.int32))
        prev2 = up(synth.prob_rows(R2, K, 126))

        def hbm_calls():
            for r in range(R2):
                sp.predict(hid2[r:r + 1], gamma, lm, ids2[r:r + 1], prev2[r:r + 1], w1_1, w2_1, out=outs)
        gh = capture(hbm_calls)
        us_hbm = ev_time(gh.replay, 3, 1) * 1e3 / R2
        del gh
        extra["c1_single_call"] = {"us_per_call_rotated_ids": us_cold, "us_per_call_same_inputs": us_warm,
                                   "us_per_call_rows_from_hbm": us_hbm, "rotated_ids": sp_cold,
                                   "algorithmic_bytes": predict_bytes(d, K)}

    # ------------------------------------------------------------------ full-vocabulary head, N=1 (what the predictor replaces)
    lm_us = None
    if want("lmhead") and not args.no_extra:
        hid = up(synth.hidden(8, d, 321))
        out_full = torch.empty((1, V), device=dev)
        it = [0]

        def full():
            sp.lm_head_gemv(hid[it[0] % 8:it[0] % 8 + 1], gamma, lm, out=out_full)
            it[0] += 1
        g = capture(lambda: [full() for _ in range(8)])
        lm_us = ev_time(g.replay, 30, 5) * 1e3 / 8
        sp_lm = spread(8)
        byts = V * d * 2 + d * 4 + V * 4
        extra["lm_head_gemv_32000x4096"] = {
            "us_per_call": lm_us, **sp_lm, "achieved_GBps": byts / lm_us / 1e3, "frac_of_8TBps": byts / lm_us / 1e3 / HBM_PEAK_GBS,
            "algorithmic_bytes": byts, "traffic": MEASURED_TRAFFIC.get("lm_head_gemv_7b"),
            "note": "262 MB head is re-read every call; the 256 MB Infinity Cache can hold part of it"}
        vids = up(synth.ids_uniform_distinct(1, K, V, 5))
        vout = sp.verify(hid[:1], gamma, lm, vids)
        vws = torch.empty(sp.workspace_bytes(sp.OP_VERIFY, sp.Dims(d, V, K, 1, 1e-5, 0.5), 1), dtype=torch.uint8,
                          device=dev)
        gv = capture(lambda: [sp.verify(hid[i:i + 1], gamma, lm, vids, out=vout, workspace=vws) for i in range(8)])
        v_us = ev_time(gv.replay, 30, 5) * 1e3 / 8
        extra["specee_verify_32000x4096"] = {"us_per_call": v_us, **spread(8), "achieved_GBps": V * d * 2 / v_us / 1e3}
        if result is not None:
            extra["speedup_vs_full_vocab_head"] = {
                "predictor_us": result["us_per_call"], "lm_head_gemv_us": lm_us,
                "ratio": lm_us / result["us_per_call"]}

    # ------------------------------------------------------------------ throughput mode: many independent tokens per launch
    if want("batch") and not args.no_extra:
        tp = {}
        t1 = synth.make("C1", lm=lm_h)
        w1_1, w2_1 = up(t1["W1"]), up(t1["w2"])
        for B in (16, 256, 2048, 8000, 16384):
            rng = np.random.default_rng(B)
            hid = up(rng.standard_normal((B, d), dtype=np.float32).astype(np.float16))
            # distinct ids across the whole batch while the vocabulary allows it (then the kernel's
            # traffic equals the algorithmic bytes); beyond that rows repeat and are re-fetched
            if B * K <= V:
                ids_h = rng.permutation(V)[:B * K].reshape(B, K).astype(np.int32)
            else:
                ids_h = rng.integers(0, V, size=(B, K)).astype(np.int32)
            ids = up(ids_h)
            prev = up(synth.prob_rows(B, K, 9))
            o = sp.predict(hid, gamma, lm, ids, prev, w1_1, w2_1)
            reps = 8
            g = capture(lambda: [sp.predict(hid, gamma, lm, ids, prev, w1_1, w2_1, out=o) for _ in range(reps)])
            us = ev_time(g.replay, 20, 3) * 1e3 / reps
            byts = predict_bytes(d, K, B, distinct_rows=len(np.unique(ids_h)))
            tp[f"B={B}"] = {"us_per_launch": us, **spread(reps), "evals_per_s": B / us * 1e6, "algorithmic_bytes": byts,
                            "achieved_GBps": byts / us / 1e3, "frac_of_8TBps": byts / us / 1e3 / HBM_PEAK_GBS}
        # ids as a draft model would give them: Zipf(1.1) ranks over the vocabulary (the 16-sequence workload's
        # recipe).  Hot rows repeat across tokens and stay in L2, so the launch moves little more than the
        # hidden states; no de-duplication pass is needed for that.
        B = 16384
        rng = np.random.default_rng(3)
        hid = up(rng.standard_normal((B, d), dtype=np.float32).astype(np.float16))
        ids_h = synth.ids_zipf_vocab(B, K, V, 4242)
        ids, prev = up(ids_h), up(synth.prob_rows(B, K, 9))
        o = sp.predict(hid, gamma, lm, ids, prev, w1_1, w2_1)
        g = capture(lambda: [sp.predict(hid, gamma, lm, ids, prev, w1_1, w2_1, out=o) for _ in range(8)])
        us = ev_time(g.replay, 20, 3) * 1e3 / 8
        byts = predict_bytes(d, K, B, distinct_rows=len(np.unique(ids_h)))
        tp["B=16384_zipf_ids"] = {"us_per_launch": us, **spread(8), "evals_per_s": B / us * 1e6,
                                  "distinct_rows": int(len(np.unique(ids_h))), "algorithmic_bytes": byts,
                                  "achieved_GBps": byts / us / 1e3, "frac_of_8TBps": byts / us / 1e3 / HBM_PEAK_GBS,
                                  "traffic": MEASURED_TRAFFIC.get("predict_B16384_zipf"),
                                  "path": "specee_predict, one workgroup per token; repeated rows served by L2"}
        # the same batch through the merged mapping: groups of Ng tokens scored as one "tree" each against the
        # union of their ids (specee_predict_tree without parents), so that a row shared inside a group is read once
        merged_alt = {}
        for Ng, cap in ((32, 128), (64, 256)):
            Gg = B // Ng
            Mg = [len(np.unique(ids_h[i * Ng:(i + 1) * Ng])) for i in range(Gg)]
            if max(Mg) > cap:
                merged_alt[f"groups_of_{Ng}"] = {"skipped": f"a group's union ({max(Mg)}) exceeds {cap} rows"}
                continue
            ot = sp.predict_tree(hid.view(Gg, Ng, d), gamma, lm, ids.view(Gg, Ng, K), prev.view(Gg, Ng, K), w1_1, w2_1,
                                 Mcap=cap)
            wst = ot.pop("_workspace")
            g = capture(lambda: [sp.predict_tree(hid.view(Gg, Ng, d), gamma, lm, ids.view(Gg, Ng, K),
                                                 prev.view(Gg, Ng, K), w1_1, w2_1, Mcap=cap, out=ot, workspace=wst)
                                 for _ in range(4)])
            usm = ev_time(g.replay, 10, 2) * 1e3 / 4
            torch.cuda.synchronize()
            same = bool(torch.allclose(ot["scores"].flatten(), o["scores"], rtol=2e-3, atol=2e-6))
            merged_alt[f"groups_of_{Ng}"] = {"us_per_launch": usm, **spread(4), "mean_union": float(np.mean(Mg)),
                                             "rows_read": int(np.sum(Mg)), "scores_agree_with_direct_path": same}
        tp["B=16384_zipf_ids"]["merged_mapping_alternative"] = merged_alt
        # B=8000 touches every row of the 262 MB head, most of which the 256 MB last-level cache can keep from
        # one launch to the next; alternating between two different heads takes that help away
        lm_b = up(synth.lm_head(V, d, synth.lm_seed(c2) + 1))
        B = 8000
        rng = np.random.default_rng(B)
        hid = up(rng.standard_normal((B, d), dtype=np.float32).astype(np.float16))
        ids_h = rng.permutation(V)[:B * K].reshape(B, K).astype(np.int32)
        ids, prev = up(ids_h), up(synth.prob_rows(B, K, 9))
        o = sp.predict(hid, gamma, lm, ids, prev, w1_1, w2_1)
        g = capture(lambda: [sp.predict(hid, gamma, lm if r % 2 == 0 else lm_b, ids, prev, w1_1, w2_1, out=o)
                             for r in range(8)])
        us = ev_time(g.replay, 20, 3) * 1e3 / 8
        byts = predict_bytes(d, K, B, distinct_rows=B * K)
        tp["B=8000_two_heads_alternating"] = {"us_per_launch": us, **spread(8), "evals_per_s": B / us * 1e6,
                                              "algorithmic_bytes": byts, "achieved_GBps": byts / us / 1e3,
                                              "frac_of_8TBps": byts / us / 1e3 / HBM_PEAK_GBS}
        del lm_b
        tp["traffic_B8000"] = MEASURED_TRAFFIC.get("predict_B8000")
        extra["throughput_predict_7b"] = tp

    # ------------------------------------------------------------------ C3 tree (latency) and batches of trees (throughput)
    if want("tree") and not args.no_extra:
        c3 = synth.CONFIGS["C3"]
        trees = [synth.make("C3", seed=s, lm=lm_h) for s in range(32)]
        tw1, tw2 = up(trees[0]["W1"]), up(trees[0]["w2"])
        dev_trees = [(up(t["hidden"]), up(t["ids"]), up(t["prev_probs"]), up(t["parent"])) for t in trees]
        Ms = [len(np.unique(t["ids"])) for t in trees]
        o = sp.predict_tree(dev_trees[0][0], gamma, lm, dev_trees[0][1], dev_trees[0][2], tw1, tw2,
                            parent=dev_trees[0][3], Mcap=c3.Mcap)
        ws = o["_workspace"]
        # preallocate outputs once so the graph holds no allocations
        outs = [sp.predict_tree(hh, gamma, lm, ii, pp, tw1, tw2, parent=par, Mcap=c3.Mcap, workspace=ws)
                for (hh, ii, pp, par) in dev_trees]

        def tree_calls_prealloc():
            for (hh, ii, pp, par), oo in zip(dev_trees, outs):
                oo2 = {k: (v[None] if v is not None else None) for k, v in oo.items() if k != "_workspace"}
                sp.predict_tree(hh[None], gamma, lm, ii[None], pp[None], tw1, tw2, parent=par[None], Mcap=c3.Mcap,
                                out=oo2, workspace=ws)
        g = capture(tree_calls_prealloc)
        us = ev_time(g.replay, 20, 3) * 1e3 / len(dev_trees)
        byts = int(np.mean([c3.N * d * 2 + m * d * 2 for m in Ms])) + d * 2 + (3 * K * H + H) * 2
        extra["c3_tree_N60"] = {"us_per_call": us, **spread(len(dev_trees)), "mean_M": float(np.mean(Ms)), "algorithmic_bytes": byts,
                                "achieved_GBps": byts / us / 1e3, "node_evals_per_s": c3.N / us * 1e6}
        # throughput: G different trees per launch (own hidden states, own id pools)
        for G in (64, 256):
            tg = [synth.make("C3", seed=1000 + i, lm=lm_h) for i in range(G)]
            hh = up(np.stack([t["hidden"] for t in tg]))
            ii_h = np.stack([t["ids"] for t in tg])
            ii, pp = up(ii_h), up(np.stack([t["prev_probs"] for t in tg]))
            par = up(np.stack([t["parent"] for t in tg]))
            og = sp.predict_tree(hh, gamma, lm, ii, pp, tw1, tw2, parent=par, Mcap=c3.Mcap)
            wsg = og.pop("_workspace")
            # several launches per graph (so that the graph's own launch cost is not in the figure), rotating
            # over enough different batches -- other hidden states, ids shifted to other rows -- that the
            # 256 MB last-level cache cannot serve one launch from the previous ones
            per_set = G * c3.N * d * 2 + sum(len(np.unique(x)) for x in ii_h) * d * 2
            nsets = int(min(12, max(2, -(-700_000_000 // per_set))))
            hsets = [hh] + [torch.randn(hh.shape, device=dev, dtype=torch.float16) for _ in range(nsets - 1)]
            isets = [ii] + [((ii + 7919 * r) % V).to(torch.int32) for r in range(1, nsets)]
            reps = nsets * max(1, 8 // nsets)
            g = capture(lambda: [sp.predict_tree(hsets[r % nsets], gamma, lm, isets[r % nsets], pp, tw1, tw2,
                                                 parent=par, Mcap=c3.Mcap, out=og, workspace=wsg)
                                 for r in range(reps)])
            us = ev_time(g.replay, 20, 3) * 1e3 / reps
            # hidden states of every tree + every LM-head row the batch touches, once
            bytsG = G * c3.N * d * 2 + len(np.unique(ii_h)) * d * 2 + d * 2 + (3 * K * H + H) * 2
            # what the launch really requests: every tree reads its own merged rows (rows shared between
            # trees are served by the caches the second time, but they do cross the memory path)
            bytsT = G * c3.N * d * 2 + sum(len(np.unique(x)) for x in ii_h) * d * 2 + d * 2 + (3 * K * H + H) * 2
            extra[f"c3_tree_batch_G{G}"] = {"us_per_launch": us, **spread(reps), "node_evals_per_s": G * c3.N / us * 1e6,
                                            "distinct_rows_in_batch": int(len(np.unique(ii_h))),
                                            "algorithmic_bytes": bytsG, "achieved_GBps": bytsG / us / 1e3,
                                            "frac_of_8TBps": bytsG / us / 1e3 / HBM_PEAK_GBS,
                                            "bytes_with_rows_counted_per_tree": bytsT,
                                            "frac_of_8TBps_rows_per_tree": bytsT / us / 1e3 / HBM_PEAK_GBS,
                                            "rotating_batches": nsets,
                                            "traffic": MEASURED_TRAFFIC.get(f"tree_c3_batch_G{G}")}

    # ------------------------------------------------------------------ 4-bit group-quantised LM-head rows
    if want("q4") and not args.no_extra:
        group = 128
        qh, sh, zh = synth.quantize_q4(lm_h, group)
        qd, sd, zd = up(qh.view(np.int32)), up(sh), up(zh)
        t1 = synth.make("C1", lm=lm_h)
        w1_1, w2_1 = up(t1["W1"]), up(t1["w2"])
        row_bytes = d // 2 + 2 * (d // group) * 2

        def q4_bytes(B, rows):
            return B * d * 2 + d * 2 + rows * row_bytes + (3 * K * H + H) * 2 + B * (K * 4 + K * 4 + 2 * K * 4 + 8)
        R1 = 256
        hid = up(synth.hidden(R1, d, 223))
        ids = up(synth.ids_uniform_distinct(R1, K, V, 224))
        prev = up(synth.prob_rows(R1, K, 225))
        o1 = sp.predict_q4(hid[:1], gamma, qd, sd, zd, group, ids[:1], prev[:1], w1_1, w2_1)
        g = capture(lambda: [sp.predict_q4(hid[r:r + 1], gamma, qd, sd, zd, group, ids[r:r + 1], prev[r:r + 1], w1_1,
                                           w2_1, out=o1) for r in range(R1)])
        res = {"group": group, "row_bytes": row_bytes, "fp16_row_bytes": 2 * d,
               "us_per_call_rotated_ids": ev_time(g.replay, 20, 3) * 1e3 / R1,
               "algorithmic_bytes_one_token": q4_bytes(1, K)}
        for B in (8000, 16384):
            rng = np.random.default_rng(B)
            hb = up(rng.standard_normal((B, d), dtype=np.float32).astype(np.float16))
            ids_h = (rng.permutation(V)[:B * K].reshape(B, K) if B * K <= V
                     else rng.integers(0, V, size=(B, K))).astype(np.int32)
            ib, pb = up(ids_h), up(synth.prob_rows(B, K, 9))
            o = sp.predict_q4(hb, gamma, qd, sd, zd, group, ib, pb, w1_1, w2_1)
            reps = 8
            g = capture(lambda: [sp.predict_q4(hb, gamma, qd, sd, zd, group, ib, pb, w1_1, w2_1, out=o)
                                 for _ in range(reps)])
            us = ev_time(g.replay, 20, 3) * 1e3 / reps
            byts = q4_bytes(B, len(np.unique(ids_h)))
            res[f"B={B}"] = {"us_per_launch": us, **spread(reps), "evals_per_s": B / us * 1e6, "algorithmic_bytes": byts,
                             "achieved_GBps": byts / us / 1e3, "frac_of_8TBps": byts / us / 1e3 / HBM_PEAK_GBS}
        extra["q4_predict_7b"] = res
        # the full head and the verification step on the same quantised head (70 MB instead of 262 MB)
        hid8 = up(synth.hidden(8, d, 321))
        out_q = torch.empty((1, V), device=dev)
        g = capture(lambda: [sp.lm_head_gemv_q4(hid8[i:i + 1], gamma, qd, sd, zd, group, out=out_q) for i in range(8)])
        us = ev_time(g.replay, 30, 5) * 1e3 / 8
        head_bytes = V * (row_bytes) + d * 4 + V * 4
        extra["lm_head_gemv_q4_32000x4096"] = {"us_per_call": us, **spread(8), "algorithmic_bytes": head_bytes,
                                               "achieved_GBps": head_bytes / us / 1e3,
                                               "frac_of_8TBps": head_bytes / us / 1e3 / HBM_PEAK_GBS,
                                               "traffic": MEASURED_TRAFFIC.get("lm_head_gemv_q4_7b")}
        vids = up(synth.ids_uniform_distinct(1, K, V, 5))
        vo_q = sp.verify_q4(hid8[:1], gamma, qd, sd, zd, group, vids)
        vws_q = torch.empty(sp.workspace_bytes(sp.OP_VERIFY_Q4, sp.Dims(d, V, K, 1, 1e-5, 0.5), 1), dtype=torch.uint8,
                            device=dev)
        g = capture(lambda: [sp.verify_q4(hid8[i:i + 1], gamma, qd, sd, zd, group, vids, out=vo_q, workspace=vws_q)
                             for i in range(8)])
        us = ev_time(g.replay, 30, 5) * 1e3 / 8
        extra["specee_verify_q4_32000x4096"] = {"us_per_call": us, **spread(8),
                                                "achieved_GBps": V * row_bytes / us / 1e3,
                                                "frac_of_8TBps": V * row_bytes / us / 1e3 / HBM_PEAK_GBS,
                                                "traffic": MEASURED_TRAFFIC.get("verify_q4_7b")}
        # token trees on the quantised head: 256 trees of the 60-node shape per launch, one workgroup per tree
        c3 = synth.CONFIGS["C3"]
        Gq = 256
        tq = [synth.make("C3", seed=3000 + i, lm=np.zeros((1, 1), np.float16)) for i in range(Gq)]
        ids_hq = np.stack([t["ids"] for t in tq])
        tw1q, tw2q = up(tq[0]["W1"]), up(tq[0]["w2"])
        prevq, parq = up(np.stack([t["prev_probs"] for t in tq])), up(np.stack([t["parent"] for t in tq]))
        hq = [torch.randn((Gq, c3.N, d), device=dev, dtype=torch.float16) for _ in range(4)]
        iq = [((up(ids_hq) + 7919 * r) % V).to(torch.int32) for r in range(4)]
        oq = sp.predict_tree_q4(hq[0], gamma, qd, sd, zd, group, iq[0], prevq, tw1q, tw2q, parent=parq, Mcap=c3.Mcap)
        g = capture(lambda: [sp.predict_tree_q4(hq[r], gamma, qd, sd, zd, group, iq[r], prevq, tw1q, tw2q, parent=parq,
                                                Mcap=c3.Mcap, out=oq) for r in range(4)])
        us = ev_time(g.replay, 20, 3) * 1e3 / 4
        bq = Gq * c3.N * d * 2 + sum(len(np.unique(x)) for x in ids_hq) * row_bytes + d * 2 + (3 * K * H + H) * 2
        extra["q4_tree_batch_G256"] = {"us_per_launch": us, **spread(4), "node_evals_per_s": Gq * c3.N / us * 1e6,
                                       "bytes_with_rows_counted_per_tree": bq,
                                       "frac_of_8TBps_rows_per_tree": bq / us / 1e3 / HBM_PEAK_GBS,
                                       "traffic": MEASURED_TRAFFIC.get("tree_q4_batch_G256")}
        del hq, iq
        del qd, sd, zd

    # ------------------------------------------------------------------ layer loop with device-side control (one token)
    if want("loop") and not args.no_extra:
        t2 = synth.make("C2", lm=lm_h)
        hid_l = up(t2["hidden"])                       # [L][1][d]
        ids_l = up(t2["ids"]).clone()
        done = torch.zeros(1, dtype=torch.int32, device=dev)
        zero = torch.zeros((1, K), device=dev)
        po = [dict(logits=torch.empty((1, K), device=dev), probs=torch.empty((1, K), device=dev),
                   scores=torch.empty(1, device=dev), exit=torch.empty(1, dtype=torch.int32, device=dev))
              for _ in range(L)]
        vo = [dict(token=torch.empty(1, dtype=torch.int32, device=dev), max_logit=torch.empty(1, device=dev),
                   hit=torch.empty(1, dtype=torch.int32, device=dev)) for _ in range(L)]
        vws = torch.empty(sp.workspace_bytes(sp.OP_VERIFY, sp.Dims(d, V, K, H, 1e-5, 0.5), 1), dtype=torch.uint8,
                          device=dev)

        def loop(threshold):
            done.zero_()
            prev = zero
            for l in range(L):
                sp.predict(hid_l[l], gamma, lm, ids_l, prev, W1[l], w2[l], threshold=threshold, out=po[l], done=done)
                sp.verify(hid_l[l], gamma, lm, ids_l, gate=po[l]["exit"], done=done, out=vo[l], workspace=vws)
                prev = po[l]["probs"]
        res = {}
        # never fires: every layer pays the predictor and two empty verification launches
        g = capture(lambda: loop(2.0))
        res["never_fires_us_per_token"] = ev_time(g.replay, 50, 5) * 1e3
        res["never_fires_spread"] = spread()
        # always fires, never hits: every layer pays a full-vocabulary verification
        g = capture(lambda: loop(-1.0))
        res["always_fires_never_hits_us_per_token"] = ev_time(g.replay, 20, 3) * 1e3
        # fires everywhere and is accepted on the way: the arg-max token of layer 10 is among the ids
        full10 = sp.lm_head_gemv(hid_l[10], gamma, lm)
        ids_l[0, 0] = int(full10.argmax())
        g = capture(lambda: loop(-1.0))
        res["fires_everywhere_accepted_us_per_token"] = ev_time(g.replay, 20, 3) * 1e3
        torch.cuda.synchronize()
        # layer 10's arg-max token usually leads at earlier layers too (the hidden state drifts slowly)
        res["fires_everywhere_accepted_exit_layer"] = int(torch.stack([v["hit"] for v in vo]).flatten().nonzero()[0])
        res["launches_per_layer"] = 3
        extra["layer_loop_device_control_7b"] = res
        # the same loop as one call (specee_layer_loop): no launch per layer, the exit decided on the device
        ids_rand = up(t2["ids"]).clone()
        lo = sp.layer_loop(hid_l, gamma, lm, ids_rand, W1, w2, threshold=2.0)
        lws = lo.pop("_workspace")

        def one_launch(threshold, ids_):
            return capture(lambda: sp.layer_loop(hid_l, gamma, lm, ids_, W1, w2, threshold=threshold, out=lo,
                                                 workspace=lws))
        r1 = {}
        g = one_launch(2.0, ids_rand)
        us = ev_time(g.replay, 200, 20) * 1e3
        r1["never_fires_us_per_token"] = us
        r1["never_fires_spread"] = spread()
        r1["never_fires_us_per_layer"] = us / L
        # four tokens' loops back to back inside one graph: the device time without the host's launch of a graph
        g4 = capture(lambda: [sp.layer_loop(hid_l, gamma, lm, ids_rand, W1, w2, threshold=2.0, out=lo, workspace=lws)
                              for _ in range(4)])
        us4 = ev_time(g4.replay, 50, 5) * 1e3 / 4
        r1["never_fires_back_to_back_us_per_token"] = us4
        r1["never_fires_back_to_back_us_per_layer"] = us4 / L
        g = one_launch(-1.0, ids_rand)
        us = ev_time(g.replay, 20, 3) * 1e3
        torch.cuda.synchronize()
        r1["always_fires_never_hits_us_per_token"] = us
        r1["always_fires_never_hits_verifications"] = int(lo["exit"].sum())
        g = one_launch(-1.0, ids_l)                    # ids_l holds layer 10's arg-max token
        us = ev_time(g.replay, 50, 5) * 1e3
        torch.cuda.synchronize()
        r1["fires_everywhere_accepted_us_per_token"] = us
        r1["fires_everywhere_accepted_exit_layer"] = int(lo["exit_layer"][0])
        r1["status"] = int(lo["status"][0])
        r1["launches_per_token"] = 2
        # sixteen tokens walk the stack in the same launch (a group of 16 workgroups each)
        B16 = 16
        hid16 = up(np.concatenate([synth.make("C2", seed=100 + i, lm=np.zeros((1, 1), np.float16))["hidden"]
                                   for i in range(B16)], axis=1))       # [L][16][d]
        ids16 = up(synth.ids_uniform_distinct(B16, K, V, 321))
        l16 = sp.layer_loop(hid16, gamma, lm, ids16, W1, w2, threshold=2.0)
        w16 = l16.pop("_workspace")
        g16 = capture(lambda: [sp.layer_loop(hid16, gamma, lm, ids16, W1, w2, threshold=2.0, out=l16, workspace=w16)
                               for _ in range(4)])
        us16 = ev_time(g16.replay, 50, 5) * 1e3 / 4
        r1["sixteen_tokens_never_fires_back_to_back_us"] = us16
        r1["sixteen_tokens_never_fires_us_per_token_layer"] = us16 / (B16 * L)
        # the scheduler's active set (Sec. 5.3): the last five tokens left the model at layers 19..24, two layers either
        # side of each stay active, plus an offline subset of every eighth layer
        sched = sp.Scheduler(L, Q=5, radius=2, offline_mask=[1 if l % 8 == 0 else 0 for l in range(L)])
        for e in (22, 19, 24, 21, 22):
            sched.push(e)
        act_h = sched.active()
        act_d = up(np.asarray(act_h, np.int32))
        ga = capture(lambda: [sp.layer_loop(hid_l, gamma, lm, ids_rand, W1, w2, active=act_d, threshold=2.0, out=lo,
                                            workspace=lws) for _ in range(4)])
        usa = ev_time(ga.replay, 50, 5) * 1e3 / 4
        r1["scheduled_active_layers"] = int(sum(act_h))
        r1["scheduled_never_fires_back_to_back_us_per_token"] = usa
        extra["layer_loop_one_launch_7b"] = r1
        # the same loop on the 4-bit group-quantised head (specee_layer_loop_q4)
        qh_l, sh_l, zh_l = synth.quantize_q4(lm_h, 128)
        qd_l, sd_l, zd_l = up(qh_l.view(np.int32)), up(sh_l), up(zh_l)
        ids_q = up(t2["ids"]).clone()
        lq = sp.layer_loop_q4(hid_l, gamma, qd_l, sd_l, zd_l, 128, ids_q, W1, w2, threshold=2.0)
        lqws = lq.pop("_workspace")

        def one_launch_q4(threshold, ids_, reps=1):
            return capture(lambda: [sp.layer_loop_q4(hid_l, gamma, qd_l, sd_l, zd_l, 128, ids_, W1, w2,
                                                     threshold=threshold, out=lq, workspace=lqws) for _ in range(reps)])
        rq = {}
        rq["never_fires_back_to_back_us_per_token"] = ev_time(one_launch_q4(2.0, ids_q, 4).replay, 50, 5) * 1e3 / 4
        rq["never_fires_back_to_back_us_per_layer"] = rq["never_fires_back_to_back_us_per_token"] / L
        rq["never_fires_spread"] = spread(4)
        rq["always_fires_never_hits_us_per_token"] = ev_time(one_launch_q4(-1.0, ids_q).replay, 20, 3) * 1e3
        torch.cuda.synchronize()
        rq["always_fires_never_hits_verifications"] = int(lq["exit"].sum())
        full10q = sp.lm_head_gemv_q4(hid_l[10], gamma, qd_l, sd_l, zd_l, 128)
        ids_q[0, 0] = int(full10q.argmax())
        rq["fires_everywhere_accepted_us_per_token"] = ev_time(one_launch_q4(-1.0, ids_q).replay, 50, 5) * 1e3
        torch.cuda.synchronize()
        rq["fires_everywhere_accepted_exit_layer"] = int(lq["exit_layer"][0])
        rq["status"] = int(lq["status"][0])
        extra["layer_loop_one_launch_q4_7b"] = rq
        del qd_l, sd_l, zd_l

    # ------------------------------------------------------------------ C4: 13B shape, 16 sequences x 40 layers
    if want("c4") and not args.no_extra:
        del lm
        torch.cuda.empty_cache()
        c4 = synth.CONFIGS["C4"]
        lm4_h = synth.lm_head(c4.V, c4.d, synth.lm_seed(c4))
        lm4 = up(lm4_h)
        t4 = synth.make("C4", lm=lm4_h)
        T4 = {k: up(v) for k, v in t4.items() if k not in ("cfg", "lm_head")}
        # per-layer batched call (decode-time use): 40 dependent launches of B=16
        o4 = dict(logits=torch.empty((c4.L, c4.B, c4.K), device=dev), probs=torch.empty((c4.L, c4.B, c4.K), device=dev),
                  scores=torch.empty((c4.L, c4.B), device=dev),
                  exit=torch.empty((c4.L, c4.B), dtype=torch.int32, device=dev))
        zero = torch.zeros((c4.B, c4.K), device=dev)

        def c4_calls():
            for l in range(c4.L):
                o = {k: v[l] for k, v in o4.items()}
                sp.predict(T4["hidden"][l], T4["gamma"], lm4, T4["ids"], zero if l == 0 else o4["probs"][l - 1],
                           T4["W1"][l], T4["w2"][l], out=o)
        g = capture(c4_calls)
        ms = ev_time(g.replay, 50, 5)
        nrows = len(np.unique(t4["ids"]))
        byts_layer = predict_bytes(c4.d, c4.K, c4.B, distinct_rows=nrows)
        extra["c4_13b_16seq_per_layer_calls"] = {
            "us_per_layer_call": ms * 1e3 / c4.L, **spread(c4.L), "ms_all_40_layers": ms, "evals_per_s": c4.L * c4.B / (ms * 1e-3),
            "algorithmic_bytes_per_layer": byts_layer, "achieved_GBps": byts_layer / (ms * 1e3 / c4.L) / 1e3}
        so = sp.predict_sweep(T4["hidden"], T4["gamma"], lm4, T4["ids"], T4["W1"], T4["w2"])
        g = capture(lambda: sp.predict_sweep(T4["hidden"], T4["gamma"], lm4, T4["ids"], T4["W1"], T4["w2"], out=so))
        us = ev_time(g.replay, 100, 10) * 1e3
        sweep_spread = spread()
        g8 = capture(lambda: [sp.predict_sweep(T4["hidden"], T4["gamma"], lm4, T4["ids"], T4["W1"], T4["w2"], out=so)
                              for _ in range(8)])
        us_b2b = ev_time(g8.replay, 50, 5) * 1e3 / 8
        byts = c4.L * c4.B * c4.d * 2 + nrows * c4.d * 2 + c4.d * 2 + c4.L * (3 * c4.K * H + H) * 2
        extra["c4_13b_one_launch_sweep"] = {"us_per_launch": us, **sweep_spread, "evals_per_s": c4.L * c4.B / us * 1e6,
                                            "algorithmic_bytes": byts, "achieved_GBps": byts / us / 1e3,
                                            "frac_of_8TBps": byts / us / 1e3 / HBM_PEAK_GBS,
                                            "us_per_launch_back_to_back": us_b2b,
                                            "frac_of_8TBps_back_to_back": byts / us_b2b / 1e3 / HBM_PEAK_GBS,
                                            "note": "us_per_launch is one graph launch per sweep and includes the host's "
                                                    "launch of the graph; back_to_back is eight sweeps inside one graph",
                                            "distinct_rows": int(nrows), "row_reads": int(c4.L * c4.B * c4.K),
                                            "path": "specee_predict_sweep, one workgroup per (layer, token); the "
                                                    "distinct rows cross the fabric once and their repeats over "
                                                    "layers and tokens are served by L2 (no de-duplication pass)"}
        extra["c4_13b_16seq_per_layer_calls"]["path"] = ("specee_predict per layer, one workgroup per token; rows "
                                                         "repeated within a layer served by L2")
        del lm4, T4
        torch.cuda.empty_cache()
        lm = None

    # ------------------------------------------------------------------ C5: d=8192, V=128256, K=8, 64-node tree + full head
    if want("c5") and not args.no_extra:
        lm = None
        torch.cuda.empty_cache()
        c5 = synth.CONFIGS["C5"]
        lm5_h = synth.lm_head(c5.V, c5.d, synth.lm_seed(c5))
        lm5 = up(lm5_h)
        ts = [synth.make("C5", seed=s, lm=lm5_h) for s in range(8)]
        g5 = up(ts[0]["gamma"])
        tw1, tw2 = up(ts[0]["W1"]), up(ts[0]["w2"])
        dts = [(up(t["hidden"]), up(t["ids"]), up(t["prev_probs"]), up(t["parent"])) for t in ts]
        Ms = [len(np.unique(t["ids"])) for t in ts]
        outs = [sp.predict_tree(hh, g5, lm5, ii, pp, tw1, tw2, parent=par, Mcap=c5.Mcap) for (hh, ii, pp, par) in dts]
        ws = outs[0]["_workspace"]

        def c5_calls():
            for (hh, ii, pp, par), oo in zip(dts, outs):
                oo2 = {k: (v[None] if v is not None else None) for k, v in oo.items() if k != "_workspace"}
                sp.predict_tree(hh[None], g5, lm5, ii[None], pp[None], tw1, tw2, parent=par[None], Mcap=c5.Mcap,
                                out=oo2, workspace=ws)
        g = capture(c5_calls)
        us_tree = ev_time(g.replay, 20, 3) * 1e3 / len(dts)
        byts = int(np.mean([c5.N * c5.d * 2 + m * c5.d * 2 for m in Ms])) + c5.d * 2 + (3 * c5.K * H + H) * 2
        extra["c5_tree_N64_V128256"] = {"us_per_call": us_tree, **spread(len(dts)), "mean_M": float(np.mean(Ms)),
                                        "algorithmic_bytes": byts, "achieved_GBps": byts / us_tree / 1e3}
        full = torch.empty((c5.N, c5.V), device=dev)
        g = capture(lambda: sp.lm_head_gemv(dts[0][0], g5, lm5, out=full))
        # (the first few dozen passes over a 2 GB head run 10-20 % slower than the sustained rate -- successive
        # repetitions in one process on the same buffers read 501, 447, 438, 420 us -- so this one warms up longer)
        us64 = ev_time(g.replay, 30, 40) * 1e3
        b64 = c5.V * c5.d * 2 + c5.N * c5.d * 2 + c5.N * c5.V * 4
        extra["lm_head_gemv_128256x8192_N64"] = {"us_per_call": us64, **spread(), "algorithmic_bytes": b64,
                                                 "achieved_GBps": b64 / us64 / 1e3,
                                                 "frac_of_8TBps": b64 / us64 / 1e3 / HBM_PEAK_GBS,
                                                 "mfma_TFLOPs": 2 * 2.0 * c5.N * c5.V * c5.d / us64 / 1e6,
                                                 "traffic": MEASURED_TRAFFIC.get("lm_head_gemm_c5")}
        one = torch.empty((1, c5.V), device=dev)
        g = capture(lambda: sp.lm_head_gemv(dts[0][0][:1], g5, lm5, out=one))
        us1 = ev_time(g.replay, 30, 5) * 1e3
        b1 = c5.V * c5.d * 2 + c5.d * 4 + c5.V * 4
        extra["lm_head_gemv_128256x8192_N1"] = {"us_per_call": us1, **spread(), "algorithmic_bytes": b1,
                                                "achieved_GBps": b1 / us1 / 1e3,
                                                "frac_of_8TBps": b1 / us1 / 1e3 / HBM_PEAK_GBS}
        extra["c5_tree_N64_V128256"]["speedup_vs_full_head_N64"] = us64 / us_tree
        # throughput mode for this shape: G trees per launch (merged sets of ~140 rows: sixteen row tiles per
        # workgroup; 64 trees are scored node by node), two batches in rotation
        for G in (64, 256):
            batches, bytes_tree = [], 0
            for b in range(2):
                gen = torch.Generator(device=dev)
                gen.manual_seed(9000 + 10 * G + b)
                hid = torch.randn((G, c5.N, c5.d), device=dev, dtype=torch.float16, generator=gen)
                ids_h = np.stack([synth.make("C5", seed=500 + b * G + i, lm=np.zeros((1, 1), np.float16))["ids"]
                                  for i in range(G)])
                prev = up(synth.prob_rows(G * c5.N, c5.K, 77 + b).reshape(G, c5.N, c5.K))
                par = up(np.tile(ts[0]["parent"], (G, 1)))
                ids_d = up(ids_h)
                if b == 0:
                    bytes_tree = G * c5.N * c5.d * 2 + sum(len(np.unique(x)) for x in ids_h) * c5.d * 2
                o = sp.predict_tree(hid, g5, lm5, ids_d, prev, tw1, tw2, parent=par, Mcap=c5.Mcap)
                wsb = o.pop("_workspace")
                batches.append((hid, ids_d, prev, par, o, wsb))

            def c5_batch():
                for _ in range(2):
                    for (hid, ids_d, prev, par, o, wsb) in batches:
                        sp.predict_tree(hid, g5, lm5, ids_d, prev, tw1, tw2, parent=par, Mcap=c5.Mcap, out=o,
                                        workspace=wsb)
            g = capture(c5_batch)
            us = ev_time(g.replay, 10, 2) * 1e3 / 4
            extra[f"c5_tree_batch_G{G}"] = {"us_per_launch": us, **spread(4), "node_evals_per_s": G * c5.N / us * 1e6,
                                            "bytes_with_rows_counted_per_tree": bytes_tree,
                                            "frac_of_8TBps_rows_per_tree": bytes_tree / us / 1e3 / HBM_PEAK_GBS}
            del batches
        del lm5
        torch.cuda.empty_cache()

    # ------------------------------------------------------------------ counter calibration: plain copy of known size
    if want("copy"):
        src = torch.empty(256 << 20, dtype=torch.uint8, device=dev)
        dst = torch.empty_like(src)
        for _ in range(5):
            sp.calib_copy(dst, src)
        torch.cuda.synchronize()
        ms = ev_time(lambda: sp.calib_copy(dst, src), 20, 2)
        extra["calib_copy_256MiB"] = {"ms": ms, "GBps_read_plus_write": 2 * src.numel() / ms / 1e6}
        del src, dst

    # ------------------------------------------------------------------ CPU oracle on the same workload
    cpu = None
    if not args.no_cpu and want("sweep"):
        from oracle import specee_oracle as orc
        orc.build()
        orc.set_threads(1)
        hid = synth.hidden_drift(L, 1, d, 50_000)
        ids = synth.ids_uniform_distinct(1, K, V, 60_000)
        t0 = time.perf_counter()
        orc.predict_sweep(hid, base["gamma"], lm_h, ids, base["W1"], base["w2"])
        one = time.perf_counter() - t0
        reps = int(max(3, min(20000, 12.0 / max(one, 1e-6))))
        t0 = time.perf_counter()
        for _ in range(reps):
            orc.predict_sweep(hid, base["gamma"], lm_h, ids, base["W1"], base["w2"])
        dt = time.perf_counter() - t0
        cpu = {"value": reps * L / dt, "unit": "evals/s", "cores": orc.get_threads(), "kind": "oracle",
               "sample": f"{reps} repetitions of the same 32-layer sweep (one token) in {dt:.1f} s, "
                         "plain C float64 oracle, single thread",
               "us_per_call": dt / (reps * L) * 1e6}
        # context: the oracle's full-vocabulary head on a sample of rows
        rows = np.arange(0, V, 8, dtype=np.int32)
        t0 = time.perf_counter()
        orc.lm_head_rows(hid[0], base["gamma"], lm_h, rows)
        dt = time.perf_counter() - t0
        cpu["lm_head_gemv_us_extrapolated_from_4000_rows"] = dt * 8 * 1e6
        # context: the same oracle over independent tokens on all host cores it may use (its outer loop is
        # an OpenMP loop over tokens); a sample of the batched workload
        ncores = max(1, min(len(os.sched_getaffinity(0)), int(os.environ.get("OMP_NUM_THREADS", "16"))))
        orc.set_threads(ncores)
        Bc = 4096
        hid_b = synth.hidden(Bc, d, 70_000)
        ids_b = synth.ids_uniform_distinct(Bc, K, V, 70_001)
        prev_b = synth.prob_rows(Bc, K, 70_002)
        t0 = time.perf_counter()
        orc.predict(hid_b, base["gamma"], lm_h, ids_b, prev_b, base["W1"][0], base["w2"][0])
        dt = time.perf_counter() - t0
        cpu["batched_all_cores"] = {"value": Bc / dt, "unit": "evals/s", "cores": orc.get_threads(),
                                    "sample": f"{Bc} independent tokens (distinct ids), one layer, in {dt:.2f} s"}
        orc.set_threads(1)

    if result is None:
        result = {"metric": "section run", "value": None, "unit": "", "n_gpus": 1, "steps": args.steps,
                  "warmup": args.warmup, "config": {"workload": ",".join(sorted(only))}}
    # the same kernel where bandwidth, not latency, is the bound: thousands of tokens per launch
    tp_all = extra.get("throughput_predict_7b", {})
    tp8 = tp_all.get("B=8000_two_heads_alternating") or tp_all.get("B=8000")
    # a plain device-to-device copy (read + write) on this machine, as a second yardstick beside the 8 TB/s peak
    copy_gbps = extra.get("calib_copy_256MiB", {}).get("GBps_read_plus_write")
    if tp8 and "roofline" in result:
        result["roofline_throughput"] = {
            "bound": "hbm", "kernel": "predict_kernel<4,2,false,true,256,2>, 8000 tokens per launch (distinct ids), launches "
                                     "alternating between two LM heads so that the last-level cache cannot keep one",
            "achieved": tp8["achieved_GBps"], "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": tp8["frac_of_8TBps"],
            "algorithmic_bytes_per_launch": tp8["algorithmic_bytes"], "us_per_launch": tp8["us_per_launch"],
            "traffic": MEASURED_TRAFFIC.get("predict_B8000"),
            "copy_kernel_GBps": copy_gbps,
            "frac_of_copy_kernel": (tp8["achieved_GBps"] / copy_gbps) if copy_gbps else None,
            "note": "random gathers of 8 KB rows with no dependent trip reach 86 % of 8 TB/s on this chip "
                    "(streaming probe); the predictor makes two dependent trips per token; with one head "
                    "re-used by every launch the same kernel reads " +
                    (f"{tp_all['B=8000']['frac_of_8TBps'] * 100:.0f} %" if "B=8000" in tp_all else "more") +
                    " because most of the 262 MB head stays in the 256 MB last-level cache"}
    result["extra"] = extra
    result["cpu_baseline"] = cpu
    result["setup_s"] = time.time() - t_setup
    print(json.dumps(result))


if __name__ == "__main__":
    main()
