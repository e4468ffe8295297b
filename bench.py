#!/usr/bin/env python3
"""Benchmark of the embed-and-aggregate path on one MI355X.

A step is one pass of the whole path over one synthetic workload whose inputs
already sit in HBM: CSR construction from the raw pair list, plan creation,
then every round (dense transform + neighbourhood aggregation) and the final
classifier transform (or head mean).  The headline value is the edge*feature
arithmetic of all aggregations in the pass (2 flop per CSR entry and feature
column) divided by the wall time of the whole step.

With no --config the headline workload is the Reddit-shaped one (index 3) and the
ogbn-products-shaped one (index 4, the workload whose gathers really are HBM reads)
runs in the same process and is reported under "also".

Prints one JSON line.  Extra objects:
  roofline      the dominant kernel (the widest aggregation) against the 8 TB/s HBM peak;
                frac is measured-traffic bytes / time / peak and cannot exceed 1, the
                gather-model and compulsory figures stand beside it
  transforms    every dense transform timed alone: its rate, what it issues on the bf16 matrix cores, and HBM
  cpu_baseline  the CPU oracle timed on the same workload
"""
from __future__ import annotations

import argparse
import gc
import hashlib
import json
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
MFMA_BF16_PEAK_TFLOPS = 2500.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--config", type=int, default=None,
                    help="workload index (0-4; 3 = Reddit-shaped, 4 = ogbn-products-shaped); "
                         "default: 3 as the headline and 4 under 'also'")
    ap.add_argument("--no-cpu", action="store_true", help="skip the cpu_baseline leg")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the rows beyond the hot path (training step, backward, 16-bit table, partition)")
    ap.add_argument("--cpu-rows", type=int, default=0, help="rows in the oracle sample (0 = per-workload default)")
    ap.add_argument("--option", action="append", default=[], metavar="NAME=VALUE",
                    help="set a tuning knob of the library (retexo_set_option) before running, for experiments")
    ap.add_argument("--probe", action="store_true",
                    help="for rocprofv3 --pmc runs: one pass, then one 1 GiB device copy (the known-size "
                         "reference for the byte counters) and one launch of the dominant aggregation; no JSON")
    ap.add_argument("--probe-transforms", action="store_true",
                    help="for rocprofv3 --pmc runs: one pass, then every dense transform of the workload launched "
                         "once more on its own (the last transform dispatches of the run); no JSON")
    return ap.parse_args()


def library_source_hash():
    """sha256 over the library's sources: ties a stored counter summary to the kernels it was taken from."""
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2302_13053_amd", "csrc")
    for path in sorted(os.path.join(csrc, f) for f in os.listdir(csrc)) + [os.path.join(ROOT, "include", "retexo.h")]:
        with open(path, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def profiled_traffic(workload_name):
    """HBM-side bytes per launch of the dominant aggregation from the committed rocprofv3 summary
    (FETCH_SIZE + WRITE_SIZE runs): (bytes, source description, matches the current sources?)."""
    path = os.path.join(ROOT, "profiles", "bench_%s.md" % workload_name)
    if not os.path.exists(path):
        return None, "no profiles/bench_%s.md" % workload_name, False
    text = open(path).read()
    m = re.search(r"total per aggregation:.*?=\s*(\d+) bytes", text)
    if not m:
        return None, "profiles/bench_%s.md has no traffic total" % workload_name, False
    hm = re.search(r"library sources sha256:\s*([0-9a-f]+)", text)
    same = bool(hm) and hm.group(1) == library_source_hash()
    src = "profiles/bench_%s.md (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE of `bench.py --probe`, not this run; " \
          "taken from library sources %s, %s)" % (workload_name, hm.group(1) if hm else "unknown",
                                                  "same as now" if same else "CHANGED since: re-profile")
    return int(m.group(1)), src, same


def algorithmic_bytes(n, nnz, F, concat, gat_heads=0):
    """Bytes one aggregation must move in the gather model: one F-float row per
    CSR entry, the index arrays, the output, and the self copy if concatenated."""
    b = 4 * nnz * F + 4 * nnz + 8 * (n + 1) + 4 * n * F
    if concat:
        b += 2 * 4 * n * F           # read z_v, write it into the self half
    if gat_heads:
        b += 4 * nnz * gat_heads + 8 * n * gat_heads
    return b


def compulsory_bytes(n, nnz, F, concat):
    """Bytes with a perfect cache: every feature row read once, the indices once, the output written once."""
    return 4 * n * F + 4 * nnz + 8 * (n + 1) + 4 * n * (2 * F if concat else F)


def cpu_baseline(w, src, dst, feats, params, n_rows):
    """Oracle cost per unit on a bounded sample, scaled to one whole pass."""
    import oracle
    from paper_2302_13053_amd import workloads as wl
    n = w.n_nodes
    t0 = time.perf_counter()
    m = min(src.size, 4_000_000)
    oracle.csr_from_coo(src[:m], dst[:m], n, w.self_loops)
    t_csr = (time.perf_counter() - t0) * (src.size / max(m, 1))
    rp, ci = oracle.csr_from_coo(src, dst, n, w.self_loops)     # needed to run the sample; not timed
    rng = np.random.Generator(np.random.Philox(key=12345))
    rows = np.sort(rng.choice(n, size=min(n_rows, n), replace=False)).astype(np.int64)
    nnz = int(rp[-1])
    sample_edges = int((rp[rows + 1] - rp[rows]).sum())
    total = t_csr
    spent = 0.0
    for i, st in enumerate(w.stages):
        p = params[i]
        if i == 0:
            H = feats
        else:
            H = wl.random_matrix(n, st.d_in, 100 + i, ld=wl.pad_ld(st.d_in))
        if st.kind == "head_mean":
            t0 = time.perf_counter()
            oracle.head_mean(H[rows], st.heads, st.d_out)
            dt = time.perf_counter() - t0
            spent += dt
            total += dt * n / rows.size
            continue
        if st.w:
            t0 = time.perf_counter()
            oracle.transform(H, st.d_in, p.W, p.b, st.relu, rows=rows)
            dt = time.perf_counter() - t0
            spent += dt
            total += dt * n / rows.size
        if st.kind == "round":
            Z = H if not st.w else wl.random_matrix(n, st.d_out, 200 + i, ld=wl.pad_ld(st.d_out))
            t0 = time.perf_counter()
            oracle.aggregate(st.mode, rp, ci, Z, st.d_out, heads=st.heads, a_src=p.a_src, a_dst=p.a_dst,
                             self_concat=st.concat, rows=rows)
            dt = time.perf_counter() - t0
            spent += dt
            total += dt * nnz / max(sample_edges, 1)
    flops = sum(2.0 * nnz * st.d_out for st in w.stages if st.kind == "round")
    return {
        "value": flops / total / 1e9,
        "unit": "GFLOP/s (edge*feature, whole pass)",
        "cores": oracle.threads(),
        "kind": "oracle",
        "sample": "%d random rows of every stage (%d CSR entries) plus CSR build of the first %d pairs, "
                  "%.1f s of oracle time, scaled per row / per entry / per pair to one whole pass"
                  % (rows.size, sample_edges, m, spent),
        "estimated_pass_seconds": total,
    }


class Timer:
    """HIP events on the stream the library launches on (torch's current stream)."""

    def __init__(self, torch):
        self.torch = torch
        self.e0 = torch.cuda.Event(enable_timing=True)
        self.e1 = torch.cuda.Event(enable_timing=True)

    def ms(self, fn, reps):
        fn()
        self.torch.cuda.synchronize()
        self.e0.record()
        for _ in range(reps):
            fn()
        self.e1.record()
        self.torch.cuda.synchronize()
        return self.e0.elapsed_time(self.e1) / reps


def run_probe(w, pipe, torch, Hn, wl):
    pipe.run()
    torch.cuda.synchronize()
    ref_src = torch.empty(1 << 28, dtype=torch.float32, device="cuda").normal_()
    ref_dst = torch.empty_like(ref_src)
    torch.cuda.synchronize()
    ref_dst.copy_(ref_src)                       # 1 GiB read + 1 GiB written
    torch.cuda.synchronize()
    di = max((i for i, st in enumerate(w.stages) if st.kind == "round"), key=lambda i: w.stages[i].d_out)
    st = w.stages[di]
    Zin = pipe.H0 if not st.w else torch.empty((w.n_nodes, wl.pad_ld(st.d_out)), dtype=torch.float32,
                                               device="cuda").normal_()
    _, _, a_s, a_d = pipe.params[di]
    Hn.aggregate(pipe.graph, st.mode, Zin, st.d_out, heads=st.heads, a_src=a_s, a_dst=a_d, concat=st.concat)
    torch.cuda.synchronize()
    print("probe done: copy of %d bytes each way, then stage %d aggregation (F=%d)"
          % (ref_src.numel() * 4, di, st.d_out))


def bench_workload(index, args):
    import torch
    from paper_2302_13053_amd import binding as B
    from paper_2302_13053_amd import harness as Hn
    from paper_2302_13053_amd import workloads as wl

    w = wl.workload(index)
    t0 = time.perf_counter()
    src, dst = wl.make_graph(w)
    feats = wl.make_features(w, ld=wl.pad_ld(w.feat_dim))
    params = wl.make_params(w)
    t_gen = time.perf_counter() - t0

    pipe = Hn.Pipeline(w, src, dst, feats, params)
    if args.probe:
        run_probe(w, pipe, torch, Hn, wl)
        pipe.close()
        return None
    if args.probe_transforms:
        pipe.run()
        torch.cuda.synchronize()
        for i, st in enumerate(w.stages):
            if st.w:
                Hin = pipe.H0 if i == 0 else pipe.outs[i - 1]
                Hn.transform(Hin, st.d_in, pipe.params[i][0], pipe.params[i][1], st.relu)
                torch.cuda.synchronize()
                print("probe: transform %d x %d -> %d" % (w.n_nodes, st.d_in, st.d_out))
        pipe.close()
        return None
    for _ in range(args.warmup):
        pipe.run()
    torch.cuda.synchronize()

    events = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        pipe.run(events=events)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms_per_step = wall * 1e3 / args.steps

    n, nnz = w.n_nodes, pipe.graph.nnz
    timer = Timer(torch)
    reps = max(3, args.steps)
    # per-step-kind mean over the timed steps, from events on the launch stream
    per = {}
    for label, a, b in events:
        per.setdefault(label, []).append(a.elapsed_time(b))
    stages = []
    flops = 0.0
    dominant = None
    for i, st in enumerate(w.stages):
        label = "%s%d" % (st.kind, i)
        ms = float(np.mean(per[label]))
        rec = {"stage": label, "ms": ms, "d_in": st.d_in, "d_out": st.d_out}
        if st.kind == "round":
            ef = float(nnz) * st.d_out
            flops += 2.0 * ef
            rec["mode"] = st.mode
            rec["edge_features"] = ef
            rec["identity_transform"] = not st.w
            if not st.w:
                gb = algorithmic_bytes(n, nnz, st.d_out, st.concat, st.heads if st.mode == "gat_softmax" else 0)
                rec["agg_effective_GBs"] = gb / ms / 1e6
            if dominant is None or ef > dominant[1]:
                dominant = (i, ef)
        if st.w:
            rec["transform_gflop"] = 2.0 * n * st.d_in * st.d_out / 1e9
        stages.append(rec)

    # ---- roofline of the dominant aggregation: the aggregate call alone, on the launch stream
    di = dominant[0]
    dst_stage = w.stages[di]
    gat = dst_stage.mode == "gat_softmax"
    F = dst_stage.d_out
    if dst_stage.w:
        # the aggregation's input is the transform's output; a resident random matrix of that shape stands in
        Zin = torch.empty((n, wl.pad_ld(F)), dtype=torch.float32, device="cuda").normal_()
    else:
        Zin = pipe.H0 if di == 0 else pipe.outs[di - 1]
    W_, b_, a_s, a_d = pipe.params[di]
    agg_out = torch.empty((n, wl.pad_ld(dst_stage.out_width)), dtype=torch.float32, device="cuda")
    ws = Hn.ws_tensor(B.retexo_workspace_bytes(pipe.graph.plan, F, B.MODES[dst_stage.mode], dst_stage.heads,
                                               B.F_SELF_CONCAT if dst_stage.concat else 0))
    agg_ms = timer.ms(lambda: Hn.aggregate(pipe.graph, dst_stage.mode, Zin, F, heads=dst_stage.heads, a_src=a_s,
                                           a_dst=a_d, concat=dst_stage.concat, out=agg_out, workspace=ws), reps)
    g_bytes = algorithmic_bytes(n, nnz, F, dst_stage.concat, dst_stage.heads if gat else 0)
    c_bytes = compulsory_bytes(n, nnz, F, dst_stage.concat)
    traffic, traffic_src, traffic_current = profiled_traffic(w.name)

    def rate(nbytes):
        return None if nbytes is None else nbytes / agg_ms / 1e6          # GB/s

    def frac(nbytes):
        return None if nbytes is None else nbytes / agg_ms / 1e6 / HBM_PEAK_GBS
    roofline = {
        "bound": "hbm",
        "kernel": ("agg_gat_rows_kernel (slab of one head after the other, four rows per wave) or agg_gat_flash_kernel "
                   "(wave per row), scores formed from the gathered rows; other head widths: gat_scores_kernel + "
                   "agg_gat_fast_kernel with a score table"
                   if gat else
                   "aggregation call = agg_rowgroup_kernel + agg_grouped_kernel per source range (narrow slabs) "
                   "or agg_linear_kernel (whole rows), chosen by the plan"),
        "stage": "round%d aggregation, F=%d" % (di, F),
        # achieved / frac: bytes that crossed the L2 <-> fabric boundary (rocprofv3 counters of the same launch,
        # an upper bound on HBM bytes) per second of this run's launch time; cannot exceed the peak
        "achieved": rate(traffic),
        "peak": HBM_PEAK_GBS,
        "unit": "GB/s",
        "frac": frac(traffic),
        "traffic": traffic,
        "traffic_source": traffic_src,
        "traffic_matches_current_kernels": traffic_current,
        "ms_per_launch": agg_ms,
        # the three figures: gather model (every entry reads one row: what the kernel delivers to its lanes;
        # above 1 when most gathers are served by L2), measured traffic, and the perfect-cache bound
        "effective_gather": {"bytes": g_bytes, "GB/s": rate(g_bytes), "frac": frac(g_bytes)},
        "hbm_measured": {"bytes": traffic, "GB/s": rate(traffic), "frac": frac(traffic)},
        "compulsory": {"bytes": c_bytes, "GB/s": rate(c_bytes), "frac": frac(c_bytes)},
        "edge_features_per_s": float(nnz) * F / (agg_ms * 1e-3),
    }

    # ---- every dense transform alone, against the bf16 matrix cores that carry it and against HBM
    transforms = []
    for i, st in enumerate(w.stages):
        if not st.w:
            continue
        Hin = pipe.H0 if i == 0 else pipe.outs[i - 1]
        Wd, bd = pipe.params[i][0], pipe.params[i][1]
        Zt = torch.empty((n, wl.pad_ld(st.d_out)), dtype=torch.float32, device="cuda")
        tms = timer.ms(lambda: Hn.transform(Hin, st.d_in, Wd, bd, st.relu, out=Zt), reps)
        fl = 2.0 * n * st.d_in * st.d_out
        by = 4.0 * (n * st.d_in + n * st.d_out + st.d_in * st.d_out)
        ai = fl / by
        # what the matrix cores are issued by the block kernel: six bf16 products per float32 product, whole tiles of
        # columns (41 run as 64) and of sixteen k
        cols = next((t for t in (32, 64, 128, 192, 256) if st.d_out <= t), 256 * -(-st.d_out // 256))
        fl_issued = 6 * 2.0 * n * (-(-st.d_in // 16) * 16) * cols
        balance = MFMA_BF16_PEAK_TFLOPS * 1e3 / HBM_PEAK_GBS         # issued flop per byte where the two bounds meet
        transforms.append({"stage": "%s%d" % (st.kind, i), "shape": "%d x %d -> %d" % (n, st.d_in, st.d_out),
                           "ms_alone": tms, "TFLOP/s": fl / tms / 1e9, "issued_bf16_TFLOP/s": fl_issued / tms / 1e9,
                           "frac_bf16_mfma_issued": fl_issued / tms / 1e9 / MFMA_BF16_PEAK_TFLOPS,
                           "GB/s": by / tms / 1e6, "frac_hbm": by / tms / 1e6 / HBM_PEAK_GBS,
                           "flop_per_byte": ai, "flop_per_byte_issued": fl_issued / by,
                           "bound": "mfma" if fl_issued / by >= balance else "hbm"})
        del Zt

    out = {
        "ms_per_step": ms_per_step,
        "value": flops / (ms_per_step * 1e-3) / 1e9,
        "data": "synthetic (seeded %s graph, %s)" % (w.graph, w.stands_in_for),
        "config": {"workload": w.name, "config_index": w.index, "family": w.family, "nodes": n,
                   "raw_pairs": int(src.size), "csr_entries": int(nnz),
                   "max_degree": B.retexo_plan_max_degree(pipe.graph.plan), "feat_dim": w.feat_dim,
                   "stages": [st.kind + ":" + (st.mode if st.kind == "round" else "dense" if st.kind == "transform"
                                               else "heads") + ":%d->%d" % (st.d_in, st.d_out) for st in w.stages]},
        "csr_plan_ms": float(np.mean(per["csr+plan"])),
        "stages": stages,
        "input_generation_s": t_gen,
        "roofline": roofline,
        "transforms": transforms,
    }
    if not args.no_extras:
        extras(out, w, pipe, args, timer, reps, di, Zin, agg_out, ws, agg_ms)
    pipe.close()
    del pipe, Zin, agg_out, ws
    gc.collect()
    torch.cuda.empty_cache()
    if not args.no_cpu:
        default_rows = w.n_nodes      # the oracle is fast enough to run every row of every stage in 10-30 s
        out["cpu_baseline"] = cpu_baseline(w, src, dst, feats, params, args.cpu_rows or default_rows)
    return out


def extras(out, w, pipe, args, timer, reps, di, Zin, agg_out, ws, agg_ms):
    """Rows beyond the hot path, on the tensors that are already resident."""
    import torch
    from paper_2302_13053_amd import binding as B
    from paper_2302_13053_amd import harness as Hn
    from paper_2302_13053_amd import workloads as wl
    n, nnz = w.n_nodes, pipe.graph.nnz
    dst_stage = w.stages[di]
    gat = dst_stage.mode == "gat_softmax"
    F = dst_stage.d_out
    # one local training step (loss + gradients + SGD update) of the first trained layer with its
    # temporary classifier, on the aggregated features
    hidden = next((i for i, st in enumerate(w.stages) if st.kind == "round" and st.w and st.mode != "gat_softmax"),
                  None)
    if hidden is not None:
        st = w.stages[hidden]
        n_cls = w.stages[-1].d_out
        X = pipe.outs[hidden - 1] if hidden > 0 else pipe.H0
        g = torch.Generator(device="cuda").manual_seed(1234)
        labels = torch.randint(0, n_cls, (n,), generator=g, device="cuda", dtype=torch.int32)
        labels[torch.rand(n, generator=g, device="cuda") > 0.66] = -1       # two thirds are training nodes
        W1, b1 = pipe.params[hidden][0].clone(), pipe.params[hidden][1].clone()
        Wc = torch.empty((st.d_out, n_cls), dtype=torch.float32, device="cuda").uniform_(-0.1, 0.1, generator=g)
        bc = torch.zeros(n_cls, dtype=torch.float32, device="cuda")
        tws = Hn.ws_tensor(B.retexo_train_workspace_bytes(n, st.d_in, st.d_out, n_cls))
        losses = []

        def train_once(dropout=None):
            loss, *grads = Hn.layer_grad(X, st.d_in, labels, W1, b1, Wc, bc, workspace=tws, dropout=dropout)
            for p_, g_ in zip((W1, b1, Wc, bc), grads):
                B.check(B.retexo_sgd_update(p_.numel(), p_.data_ptr(), g_.data_ptr(), 0.01, Hn._stream_ptr()),
                        "retexo_sgd_update")
            losses.append(loss)
        tms = timer.ms(train_once, reps)
        tfl = (4.0 * n * st.d_in * st.d_out + 6.0 * n * st.d_out * n_cls) / tms / 1e9
        out["train_step"] = {"layer": "%d->%d (ReLU) + classifier %d->%d" % (st.d_in, st.d_out, st.d_out, n_cls),
                             "ms": tms, "TFLOP/s": tfl,
                             "loss_first": float(losses[0].cpu()[0]), "loss_last": float(losses[-1].cpu()[0]),
                             "sgd_steps": reps + 1}
        draw = [0]

        def train_dropout_once():       # the same step with dropout 0.5 on the hidden units (a fresh mask per step)
            draw[0] += 1
            train_once(dropout=(0.5, 20230213, draw[0]))
        out["train_step"]["ms_with_dropout"] = timer.ms(train_dropout_once, reps)
    # a layer whose aggregation has trainable parameters (edge softmax) trains with the aggregation in the
    # loop: its backward (dL/dZ and the attention-vector gradients) on the first such round's shape
    att = next((i for i, st in enumerate(w.stages) if st.kind == "round" and st.mode == "gat_softmax"
                and st.d_out <= 1024), None)
    if att is not None:
        st = w.stages[att]
        Fz, width = st.d_out, pipe.outs[att].shape[1]
        Zb = pipe.outs[att]                               # stands in for the round's transformed features
        Gb = torch.empty_like(Zb).normal_(generator=torch.Generator(device="cuda").manual_seed(4321))
        a_s, a_d = pipe.params[att][2], pipe.params[att][3]
        dZb = torch.empty_like(Zb)
        bws = Hn.ws_tensor(B.retexo_aggregate_backward_workspace_bytes(pipe.graph.plan, B.MODES[st.mode], Fz, st.heads))
        bms = timer.ms(lambda: Hn.aggregate_backward(pipe.graph, st.mode, Fz, Gb, Z=Zb, heads=st.heads, a_src=a_s,
                                                     a_dst=a_d, dZ=dZb, workspace=bws), reps)
        gbs = 2.0 * nnz * Fz * 4 / bms / 1e6              # two gather passes, one row of F floats per entry each
        out["aggregate_backward"] = {"shape": "%s F=%d heads=%d ld=%d" % (st.mode, Fz, st.heads, width), "ms": bms,
                                     "GB/s_algorithmic": gbs, "frac_hbm": gbs / HBM_PEAK_GBS}
        # in a training loop: the forward in save mode, then the backward that reuses what it kept (one gather pass)
        try:
            sws = Hn.ws_tensor(B.retexo_workspace_bytes(pipe.graph.plan, Fz, B.MODES[st.mode], st.heads, B.F_SAVE))
            fout = torch.empty_like(Zb)
            t_f = timer.ms(lambda: Hn.aggregate(pipe.graph, st.mode, Zb, Fz, heads=st.heads, a_src=a_s, a_dst=a_d,
                                                out=fout, workspace=sws, save=True), reps)
            t_b = timer.ms(lambda: Hn.aggregate_backward(pipe.graph, st.mode, Fz, Gb, Z=Zb, heads=st.heads, a_src=a_s,
                                                         a_dst=a_d, dZ=dZb, workspace=bws, saved=sws), reps)
            out["aggregate_backward"].update({"forward_save_mode_ms": t_f, "backward_after_save_ms": t_b,
                                              "GB/s_algorithmic_after_save": nnz * Fz * 4 / t_b / 1e6})
            del sws, fout
        except B.RetexoError:
            pass                                           # layout without save mode: the plain backward stands
        del Gb, dZb, bws
    # variant: the dominant aggregation over a table in 16-bit storage (half the gathered bytes; the stored value
    # is the float32 value rounded to nearest even, sums stay in float32)
    try:
        Z16 = Hn.store_rows(Zin, F, "bf16")               # the table the roofline figure above was measured on
        kw16 = dict(heads=dst_stage.heads, a_src=pipe.params[di][2], a_dst=pipe.params[di][3]) if gat else {}
        ms16 = timer.ms(lambda: Hn.aggregate_stored(pipe.graph, dst_stage.mode, Z16, F, "bf16", concat=dst_stage.concat,
                                                    out=agg_out, workspace=ws, **kw16), reps)
        out["stored_aggregation"] = {"storage": "bf16", "stage": out["roofline"]["stage"], "ms": ms16,
                                     "fp32_ms": agg_ms, "GB/s_algorithmic": nnz * F * 2 / ms16 / 1e6}
        del Z16
    except B.RetexoError:
        pass
    # The same aggregation call when every gathered row is an L2 hit: the graph keeps its rows, their lengths and
    # their split over the source ranges, but inside each of the plan's sixteen ranges the columns are squeezed
    # (monotonically) into a window of 1,024 sources, so that the 32-column slab of four ranges is 512 KB.  What
    # remains is the kernels' own request rate: how close the real call is to it says what the L2 misses cost.
    if w.index == 3 and not gat:
        group = (n + 15) // 16                            # sources per range of the plan's split
        col = pipe.col_idx[:nnz].to(torch.int64)
        base = (col // group) * group
        squeezed = (base + ((col - base) * 1024) // group).to(torch.int32)
        del col, base
        lg = Hn.DeviceGraph(n, int(nnz), pipe.row_ptr, squeezed)
        Hn.make_plan(lg, split_rows=True)
        l2_ms = timer.ms(lambda: Hn.aggregate(lg, dst_stage.mode, Zin, F, concat=dst_stage.concat, out=agg_out,
                                              workspace=ws), reps)
        out["roofline"]["same_call_all_gathers_in_l2"] = {
            "what": "same rows, row lengths and range split; the columns of each of the sixteen ranges squeezed into 1024 sources",
            "ms": l2_ms, "gather_model_TB/s": out["roofline"]["effective_gather"]["bytes"] / l2_ms / 1e9,
            "real_call_ms_over_this": agg_ms / l2_ms}
        lg.destroy()
        del squeezed
    # the partition-shaped run: worker 0's share of this graph (seeded random ownership over 4 workers for the
    # dense graph, 2 for the large sparse one, as the paper distributes them); the pack of what it owes its peers,
    # the unpack of what it receives, and the first round's aggregation on its local graph
    if w.index in (3, 4):
        n_workers = 4 if w.index == 3 else 2
        owner = torch.from_numpy(np.random.Generator(np.random.Philox(key=70 + w.index))
                                 .integers(0, n_workers, n).astype(np.int32)).cuda()
        share = Hn.partition_share(pipe.graph, owner, n_workers, 0)             # size query + real call
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            share = Hn.partition_share(pipe.graph, owner, n_workers, 0)
        torch.cuda.synchronize()
        share_ms = (time.perf_counter() - t0) / reps * 1e3
        st0 = w.stages[0]
        Fp = st0.d_out
        n_local = share.n_inner + share.n_halo
        gl = torch.Generator(device="cuda").manual_seed(99)
        table = torch.empty((n_local, wl.pad_ld(Fp)), dtype=torch.float32, device="cuda").normal_(generator=gl)
        n_send = int(share.send_ids.numel())
        sbuf = torch.empty((max(n_send, 1), wl.pad_ld(Fp)), dtype=torch.float32, device="cuda")
        rbuf = torch.empty((max(share.n_halo, 1), wl.pad_ld(Fp)), dtype=torch.float32, device="cuda").normal_(generator=gl)

        def exchange_compute_side():
            Hn.halo_pack(share.send_ids, table, Fp, buf=sbuf)        # owner side: inner rows its peers need
            Hn.halo_unpack(share.recv_ids, rbuf, table, Fp)          # receiver side: into the boundary rows
        pu_ms = timer.ms(exchange_compute_side, reps)
        local = Hn.make_plan(share.graph)
        lgat = st0.mode == "gat_softmax"
        lkw = dict(heads=st0.heads, a_src=pipe.params[0][2], a_dst=pipe.params[0][3]) if lgat else {}
        lout = torch.empty((n_local, wl.pad_ld(st0.out_width)), dtype=torch.float32, device="cuda")
        lws = Hn.ws_tensor(B.retexo_workspace_bytes(local.plan, Fp, B.MODES[st0.mode], st0.heads,
                                                    B.F_SELF_CONCAT if st0.concat else 0))
        l_ms = timer.ms(lambda: Hn.aggregate(local, st0.mode, table, Fp, concat=st0.concat, out=lout, workspace=lws,
                                             **lkw), reps)
        lg = algorithmic_bytes(n_local, share.graph.nnz, Fp, st0.concat, st0.heads if lgat else 0)
        g_ms = agg_ms if di == 0 else None
        out["partition"] = {"workers": n_workers, "inner": share.n_inner, "boundary": share.n_halo,
                            "local_entries": share.graph.nnz, "share_ms_incl_size_query_and_allocation": share_ms,
                            "send_rows": n_send, "recv_rows": share.n_halo, "width": Fp,
                            "pack_send_plus_unpack_recv_ms": pu_ms,
                            "GB/s_read_plus_write": 2.0 * (n_send + share.n_halo) * Fp * 4 / pu_ms / 1e6,
                            "local_round": {"what": "first round's aggregation (%s, F=%d) on worker 0's local graph: "
                                                    "%d rows over a table of %d rows" % (st0.mode, Fp, share.n_inner, n_local),
                                            "ms": l_ms, "algorithmic_bytes": lg,
                                            "effective_gather_GB/s": lg / l_ms / 1e6,
                                            "effective_gather_frac": lg / l_ms / 1e6 / HBM_PEAK_GBS,
                                            "hbm_measured_frac": None,
                                            "global_round_ms": g_ms,
                                            "global_round_ms_over_workers": None if g_ms is None else g_ms / n_workers,
                                            "share_of_global_round": None if g_ms is None else l_ms / g_ms}}
        local.destroy()
        del table, sbuf, rbuf, lout, lws


def main():
    args = parse()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on one GPU only (no collectives, no sharding); use --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2302_13053_amd import binding as B

    B.load()
    for item in args.option:
        name, _, value = item.partition("=")
        B.check(B.retexo_set_option(name, int(value)), "retexo_set_option(%s)" % item)
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)

    head_index = 3 if args.config is None else args.config
    head = bench_workload(head_index, args)
    if args.probe or args.probe_transforms:
        return
    out = {
        "metric": "aggregated edge*feature GFLOP/s per lazy-MP pass (whole path: CSR build, plan, all rounds)",
        "value": head.pop("value"),
        "unit": "GFLOP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head.pop("ms_per_step"),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "library_sources_sha256": library_source_hash(),
    }
    out.update(head)
    if args.config is None:
        # the workload whose gathers are real HBM reads, same process, same measurement
        also = bench_workload(4, args)
        also["unit"] = "GFLOP/s"
        out["also"] = also
    print(json.dumps(out))


if __name__ == "__main__":
    main()
