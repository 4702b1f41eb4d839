#!/usr/bin/env python3
"""Benchmark of the Wigner-6j convolution forward on one MI355X.

One step = the whole hot path over one synthetic input already resident in
HBM: the radius graph (CSR) followed by the Wigner-6j convolution forward
(device-side tile plan, solid harmonics, aggregation of the neighbours'
uncoupled products with their CG coupling, i-side 6j recoupling, per-irrep
fp32 channel mixing), on the 20,000-atom protein-scale workload (L = 4,
C = 128, 8 heads).

    python bench.py [--steps K] [--warmup W] [--workload NAME] [--no-cpu] [--no-configs]

Prints ONE JSON line.  Besides the step throughput it reports the forward
alone (atoms/s, edges/s), the per-edge tensor-product baseline on the same
inputs and GPU, the per-kernel times (HIP events on the launch stream,
recorded during the timed steps), the roofline of the dominant kernel and of
the whole forward, every workload's forward, baseline, speedup and sampled
parity (`configs`), the fp64 oracle timed on the host cores on a bounded row
sample, and the parity of the timed output on those rows.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "Wigner-6j conv fwd atoms/s + edges/s at Lmax=4, C=128; speedup vs edge-TP"
HBM_PEAK_GBS = 8000.0         # MI355X HBM3E
FP32_MFMA_PEAK_TFS = 157.3    # MI355X dense fp32 MFMA
BF16_MFMA_PEAK_TFS = 2500.0   # MI355X dense bf16 MFMA


def tri(a, b, c):
    return abs(a - b) <= c <= a + b


def layer_counts(L):
    """Index-structure counts of the factorised layer (per channel): rows of
    T, j-side matrix entries, i-side matrix entries, edge filter entries."""
    blocks = [(a, b, d) for a in range(L + 1) for b in range(L + 1) for d in range(abs(a - b), a + b + 1)
              if any(tri(a, b + u, o) and tri(u, d, o) for u in range(L - b + 1) for o in range(L + 1))]
    dimT = sum(2 * d + 1 for a, b, d in blocks)
    m_slots = sum((2 * d + 1) * (2 * a + 1) for a, b, d in blocks)
    q_slots = sum((2 * o + 1) * (2 * d + 1) for a, b, d in blocks for o in range(L + 1)
                  if any(tri(a, b + u, o) and tri(u, d, o) for u in range(L - b + 1)))
    return dict(dimT=dimT, m_slots=m_slots, q_slots=q_slots, k_slots=(L + 1) ** 4)


def coupling_entries(e2f, L):
    """Nonzero CG entries (row, alpha, beta) of the j-side coupling [h^(a) (x) R^(b)]^(d)
    over the blocks the layer uses (per channel)."""
    n = 0
    for a in range(L + 1):
        for b in range(L + 1):
            for d in range(abs(a - b), a + b + 1):
                if any(tri(a, b + u, o) and tri(u, d, o) for u in range(L - b + 1) for o in range(L + 1)):
                    n += int(np.count_nonzero(np.abs(e2f.e2f_real_cg(a, b, d)) > 1e-14))
    return n


def file_sha(path):
    with open(path, "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()


def central_crop(pos, side):
    """Atoms inside the central cube of the given side (re-indexed)."""
    lo, hi = pos.min(0), pos.max(0)
    c = (lo + hi) / 2
    keep = np.all(np.abs(pos - c) < side / 2, axis=1)
    return np.nonzero(keep)[0]


def alg_counts(e2f, L, C, H, n, E, fused=False):
    """Algorithmic work of the forward's kernels (per launch over the whole
    graph), counted from the real-basis tables: the aggregation as the
    factorised layer's a3 (dimT multiply-adds per edge and channel) plus the
    j-side coupling of every receiver (a2); the recouple (a4); the mixing
    (a5); and the compulsory bytes each kernel moves.  fused: the aggregation
    couples to the output itself (a2 + a3 + a4 in one kernel, y written
    instead of S)."""
    cnt = layer_counts(L)
    dimT, nk = cnt["dimT"], (L + 1) ** 2
    cpl = coupling_entries(e2f, L)
    mt = (nk + 15) // 16
    mp = 16 * mt  # components of R per MFMA tile column, padded to 16
    inputs = 4.0 * n * nk * C + 4.0 * E * nk + 4.0 * E * H + 4.0 * E + 8.0 * (n + 1)
    if fused:
        # issued: from L = 4 on the products as split bf16 (three
        # v_mfma_f32_16x16x32_bf16 of 16384 flops per 16 edges, 16 rows and 16
        # columns: six bf16 products per fp32 multiply-add), below as fp32;
        # then per receiver and 16 channels one fp32 16x16x4 MFMA per component
        # q and group of four rows (7 groups at L = 4, 12 and 13 at L = 5, 6)
        groups = {4: 7, 5: 12, 6: 13}.get(L, (nk + 3) // 4)
        cols = 16 * -(-C // 16)
        agg = dict(flops=2.0 * E * dimT * C + 2.0 * n * (cpl + cnt["q_slots"]) * C,
                   bytes=inputs + 4.0 * n * nk * C,
                   issued_flops=2.0 * n * cols * nk * groups * 64 + (0.0 if L >= 4 else 2.0 * E * mp * nk * cols))
        if L >= 4:
            agg["issued_bf16_flops"] = 12.0 * E * mp * nk * cols
    else:
        agg = dict(flops=2.0 * E * dimT * C + 2.0 * n * cpl * C, bytes=inputs + 4.0 * n * dimT * C,
                   issued_flops=2.0 * E * mp * nk * C + 2.0 * n * cpl * C)
    rec = dict(flops=2.0 * n * cnt["q_slots"] * C, bytes=4.0 * n * dimT * C + 4.0 * n * nk * C + 8.0 * n * nk)
    mix = dict(flops=2.0 * n * nk * C * C, bytes=8.0 * n * nk * C + 4.0 * (L + 1) * C * C)
    # the whole forward, fused: inputs and output once (h, positions, CSR,
    # attention weights, mixing weights, out), all the arithmetic above
    fwd = dict(flops=2.0 * E * dimT * C + 2.0 * n * (cpl + cnt["q_slots"]) * C + mix["flops"],
               bytes=4.0 * n * nk * C * 2 + 12.0 * n + 4.0 * E + 8.0 * (n + 1) + 4.0 * E * H + 4.0 * (L + 1) * C * C)
    return dict(aggregate=agg, recouple=rec, mix=mix, forward=fwd, dimT=dimT, coupling_entries=cpl,
                recouple_entries=cnt["q_slots"])


def morton_order(pos, cell=4.0):
    """Atom indices sorted by the Morton key of their 4 A cells."""
    q = np.floor((pos - pos.min(0)) / cell).astype(np.int64)
    key = np.zeros(len(pos), dtype=np.int64)
    for b in range(10):
        for a in range(3):
            key |= ((q[:, a] >> b) & 1) << (3 * b + a)
    return np.argsort(key, kind="stable").astype(np.int32)


def roof_of(bytes_, flops, t_ms, peak_tf):
    """Roofline position of one launch: the binding resource is the one
    whose lower-bound time is larger."""
    t_b, t_f = bytes_ / (HBM_PEAK_GBS * 1e9), flops / (peak_tf * 1e12)
    if t_b >= t_f:
        a = bytes_ / (t_ms * 1e-3) / 1e9
        return dict(bound="hbm", achieved=a, peak=HBM_PEAK_GBS, unit="GB/s", frac=a / HBM_PEAK_GBS)
    a = flops / (t_ms * 1e-3) / 1e12
    return dict(bound="mfma", achieved=a, peak=peak_tf, unit="TFLOP/s", frac=a / peak_tf)


def forward_floor(counts, t_ms):
    """T_roof / T_meas of the whole forward against the fused floor."""
    f = counts["forward"]
    t_roof = max(f["bytes"] / (HBM_PEAK_GBS * 1e9), f["flops"] / (FP32_MFMA_PEAK_TFS * 1e12)) * 1e3
    return dict(t_roof_ms=t_roof, t_meas_ms=t_ms, frac=t_roof / t_ms, flops=f["flops"], bytes=f["bytes"])


def time_gpu(fn, steps, warmup):
    """Mean wall time per call of `steps` calls after `warmup`, bracketed by
    device synchronisation."""
    import torch
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) * 1e3 / steps


def sweep_one(name, steps, warmup, crop=False, parity_rows=None, quiet=False):
    """One workload: the 6j forward and the edge-TP baseline (fp32 mixing),
    their speedup, and parity of both on sampled rows against the oracle.
    crop: the central 58.48 A sub-cube of the workload (the 200,000-atom
    system's baseline runs there).  Attention weights come from the seeded
    generator on the device for every edge; the sampled rows' weights are
    replaced by the host generator's, which the oracle reads, so both sides
    see the same inputs on those rows."""
    import torch
    import e2f_synth as syn
    import oracle
    import paper_2501_19216_amd as e2f

    wl = syn.WORKLOADS[name]
    if parity_rows is None:
        parity_rows = 256
    inp = syn.make_inputs(wl)
    dev = torch.device("cuda:0")
    pos_h, feat_h, gid_h, spc = inp.pos, inp.feat, inp.graph_id, inp.species
    if crop:
        keep = central_crop(inp.pos, syn._cube_side(20000))
        pos_h, feat_h, spc = np.ascontiguousarray(pos_h[keep]), np.ascontiguousarray(feat_h[keep]), spc[keep]
        gid_h = None if gid_h is None else gid_h[keep]
    if not quiet:
        print("[configs] %s%s: %d atoms generated" % (name, " crop" if crop else "", pos_h.shape[0]),
              file=sys.stderr, flush=True)
    ctx = e2f.e2f_create(wl.lmax, 0)
    pos = torch.from_numpy(pos_h).to(dev)
    feat = torch.from_numpy(feat_h).to(dev)
    gid = None if gid_h is None else torch.from_numpy(np.ascontiguousarray(gid_h)).to(dev)
    rp, ci = e2f.e2f_neighbor_list(ctx, pos, wl.cutoff, gid)
    rph, cih = rp.cpu().numpy(), ci.cpu().numpy()
    n, E = pos_h.shape[0], len(cih)
    al = syn.attention_weights_device(pos_h, spc, rph, cih, wl.heads, wl.cutoff, wl.species, wl.seed, dev)
    rows = np.arange(n, dtype=np.int32) if n <= parity_rows else \
        np.sort(np.random.default_rng(11).choice(n, parity_rows, replace=False)).astype(np.int32)
    # the sampled rows' weights from the host generator (each row's weights
    # depend on that row alone): a CSR of those rows, receiver k at node k,
    # sender j at node len(rows) + j
    sub_rp = np.concatenate([[0], np.cumsum(rph[rows + 1] - rph[rows])]).astype(np.int64)
    sub_e = np.concatenate([np.arange(rph[r], rph[r + 1]) for r in rows]).astype(np.int64)
    al_h = np.zeros((E, wl.heads), dtype=np.float32)
    if len(sub_e):
        rp_rows = np.concatenate([sub_rp, np.full(n, sub_rp[-1])]).astype(np.int64)
        al_rows = syn.attention_weights(np.concatenate([pos_h[rows], pos_h]), np.concatenate([spc[rows], spc]),
                                        rp_rows, (cih[sub_e] + len(rows)).astype(np.int32), wl.heads, wl.cutoff,
                                        wl.species, wl.seed)
        al_h[sub_e] = al_rows
        al[torch.from_numpy(sub_e).to(dev)] = torch.from_numpy(al_rows).to(dev)
    mix_w = torch.from_numpy(inp.mix_w).to(dev)
    out6 = torch.empty_like(feat)
    oute = torch.empty_like(feat)
    e2f.e2f_wigner6j_prepare(ctx, wl.lmax, wl.channels, wl.heads, wl.cutoff, mix_w=mix_w)
    k6 = max(2, steps // 4) if n > 50000 else steps
    f6 = lambda: e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, al, wl.lmax, wl.heads, wl.cutoff,
                                               mix_w=mix_w, graph_id=gid, out=out6)
    ms6 = time_gpu(f6, k6, warmup)
    res = {"workload": name + ("_crop" if crop else ""), "atoms": n, "edges": E, "lmax": wl.lmax,
           "channels": wl.channels, "heads": wl.heads, "cutoff": wl.cutoff, "fwd_ms": ms6,
           "atoms_per_s": n / ms6 * 1e3, "edges_per_s": E / ms6 * 1e3}
    run_edge = n <= 50000
    if run_edge:
        fe = lambda: e2f.e2f_edge_tp_conv_forward(ctx, pos, feat, rp, ci, al, wl.lmax, wl.heads, wl.cutoff,
                                                  mix_w=mix_w, out=oute)
        mse = time_gpu(fe, max(2, steps // 2) if wl.lmax >= 6 else steps, warmup)
        res.update(edge_tp_ms=mse, speedup_vs_edge_tp=mse / ms6)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ref = oracle.layer(wl.lmax, wl.heads, pos_h, feat_h, rph, cih, al_h, inp.path_w, inp.mix_w, rows=rows)
    res["parity"] = {"rows": int(len(rows)), "oracle_s": time.perf_counter() - t0,
                     "max_rel_err": oracle.max_rel_err(out6.cpu().numpy()[rows], ref, wl.lmax)}
    if run_edge:
        res["parity"]["edge_tp_max_rel_err"] = oracle.max_rel_err(oute.cpu().numpy()[rows], ref, wl.lmax)
    if n <= 50000:
        orp, oci = oracle.neighbor_list(pos_h, wl.cutoff, gid_h)
        res["parity"]["graph_bit_exact"] = bool(np.array_equal(orp, rph) and np.array_equal(oci, cih))
    ctx.close()
    return res


# The scaling study of the paper (Sec. 4.1, Fig. 2): (b.i) dense graphs
# (every atom attends to every other, k = 0 below) at L = 3 against N;
# k-nearest-neighbour graphs: (b.ii, b.iii) k = 32 at L = 2 and 3 against N,
# (c) N = 1000, k = 32 against L, (d) N = 1000, L = 3 against k.  Channels
# and heads are not stated there; 128 channels and 8 heads as in the
# protein-scale workload.
FIG2 = ([("b.i", 0, 3, n) for n in (250, 500, 1000, 2000, 4000)] +
        [("b.ii", 32, 2, n) for n in (1000, 2000, 5000, 10000, 20000, 50000)] +
        [("b.iii", 32, 3, n) for n in (1000, 2000, 5000, 10000, 20000, 50000)] +
        [("c", 32, L, 1000) for L in (1, 2, 3, 4, 5, 6)] +
        [("d", k, 3, 1000) for k in (64, 128, 256, 512)])


def fig2_point(panel, k, L, n, steps, warmup, C=128, H=8):
    """6j forward and edge-TP baseline on a kNN graph of n atoms (uniform at
    0.1 atoms/A^3, minimum distance 0.9 A), timed on the GPU."""
    import torch
    import e2f_synth as syn
    import paper_2501_19216_amd as e2f

    dev = torch.device("cuda:0")
    seed = 7000 + 10 * L + n + k
    pos_h = syn.positions_cube(n, syn._cube_side(n), 0.9, seed)
    rng = np.random.default_rng(seed)
    species = rng.integers(0, 10, size=n).astype(np.int32)
    feat = torch.from_numpy(rng.standard_normal((n, (L + 1) ** 2, C), dtype=np.float32)).to(dev)
    ctx = e2f.e2f_create(L, 0)
    pos = torch.from_numpy(pos_h).to(dev)
    ms_knn = None
    if k > 0:
        rp, ci = e2f.e2f_knn_graph(ctx, pos, k)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(3):
            e2f.e2f_knn_graph(ctx, pos, k)
        torch.cuda.synchronize()
        ms_knn = (time.perf_counter() - t0) * 1e3 / 3
        rph, cih = rp.cpu().numpy(), ci.cpu().numpy()
    else:  # the complete graph, for the per-edge baseline
        rph = np.arange(0, n * (n - 1) + 1, n - 1, dtype=np.int64)
        cih = np.delete(np.tile(np.arange(n, dtype=np.int32), n), np.arange(n) * (n + 1))
        rp, ci = torch.from_numpy(rph).to(dev), torch.from_numpy(cih).to(dev)
    d = np.linalg.norm(pos_h[np.repeat(np.arange(n), np.diff(rph))] - pos_h[cih], axis=1)
    reach = float(d.max()) * 1.001  # the graph's longest edge: envelope, default weights, tiles
    alpha = torch.from_numpy(syn.attention_weights(pos_h, species, rph, cih, H, reach, 10, seed)).to(dev)
    out = torch.empty_like(feat)

    def timed(fn):
        for _ in range(warmup):
            fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) * 1e3 / steps

    ms_split = ms_fused = None
    if k > 0:
        ms6 = timed(lambda: e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, reach, out=out))
        ms_split = timed(lambda: e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, reach, out=out,
                                                               form="split"))
        if L <= 4:
            ms_fused = timed(lambda: e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, reach,
                                                                   out=out, form="fused"))
    else:
        dense = torch.zeros(n, n, H, device=dev)
        dense[torch.from_numpy(np.repeat(np.arange(n), n - 1)).to(dev), ci.long()] = alpha
        ms6 = timed(lambda: e2f.e2f_wigner6j_conv_forward_dense(ctx, pos, feat, dense, L, H, reach, out=out))
        del dense
    mse = timed(lambda: e2f.e2f_edge_tp_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, reach, out=out))
    ctx.close()
    return {"panel": panel, "graph": "knn" if k > 0 else "dense", "k": k, "lmax": L, "atoms": n, "edges": int(len(cih)), "channels": C,
            "heads": H, "reach": reach, "knn_ms": ms_knn, "fwd_ms": ms6, "split_ms": ms_split, "fused_ms": ms_fused,
            "edge_tp_ms": mse, "speedup_vs_edge_tp": mse / ms6, "atoms_per_s": n / ms6 * 1e3}


def _cpu_model():
    """The host CPU's model name (first 'model name' line of /proc/cpuinfo), or None."""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


# Every workload of the benchmark, reported in the `configs` field: the five
# synthetic systems, and the central crop of the 200,000-atom one (where its
# per-edge baseline runs).
CONFIGS = [("cluster32_L2", False), ("molecules256x30_L3", False), ("water2000_L4", False),
           ("protein20k_L4", False), ("stress200k_L6", False), ("stress200k_L6", True)]


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="protein20k_L4")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle CPU baseline")
    ap.add_argument("--no-configs", action="store_true", help="skip the per-workload table")
    ap.add_argument("--cpu-rows", type=int, default=6144)
    ap.add_argument("--copy-calib", action="store_true",
                    help="also run a 1 GiB device copy and a 1 GiB device sum (counter calibration)")
    ap.add_argument("--sweep", action="store_true",
                    help="instead: one JSON line per workload (6j forward and edge-TP baseline times and speedup)")
    ap.add_argument("--sweep-workloads", default="", help="comma-separated subset of the sweep (default: all)")
    ap.add_argument("--paper-fig2", action="store_true",
                    help="instead: the scaling study on dense and kNN graphs (6j vs edge-TP), one JSON line per point")
    ap.add_argument("--fig2-panels", default="", help="comma-separated subset of the panels b.i,b.ii,b.iii,c,d")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py runs on one GPU only: the library has no multi-GPU path (no sharding, no collectives).",
              file=sys.stderr)
        sys.exit(2)

    import torch
    import e2f_synth as syn
    import paper_2501_19216_amd as e2f

    if args.paper_fig2:
        panels = [p for p in args.fig2_panels.split(",") if p]
        for panel, k, L, n in FIG2:
            if panels and panel not in panels:
                continue
            print(json.dumps(fig2_point(panel, k, L, n, args.steps, args.warmup)), flush=True)
        return

    if args.sweep:
        names = [w for w in args.sweep_workloads.split(",") if w]
        for name, crop in CONFIGS:
            if names and name not in names:
                continue
            print(json.dumps(sweep_one(name, args.steps, args.warmup, crop)), flush=True)
        return

    wl = syn.WORKLOADS[args.workload]
    inp = syn.make_inputs(wl)
    n, L, C, H = inp.pos.shape[0], wl.lmax, wl.channels, wl.heads
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    ctx = e2f.e2f_create(L, 0)
    pos = torch.from_numpy(inp.pos).to(dev)
    feat = torch.from_numpy(inp.feat).to(dev)
    mix_w = torch.from_numpy(inp.mix_w).to(dev)
    gid = None if inp.graph_id is None else torch.from_numpy(inp.graph_id).to(dev)

    # the graph once, to size buffers and draw the attention weights
    row_ptr, col = e2f.e2f_neighbor_list(ctx, pos, wl.cutoff, gid)
    E = col.numel()
    rp_h, ci_h = row_ptr.cpu().numpy(), col.cpu().numpy()
    alpha_h = syn.attention_weights(inp.pos, inp.species, rp_h, ci_h, H, wl.cutoff, wl.species, wl.seed)
    alpha = torch.from_numpy(alpha_h).to(dev)
    rp_buf = torch.empty(n + 1, dtype=torch.int64, device=dev)
    col_buf = torch.empty(E, dtype=torch.int32, device=dev)
    out = torch.empty_like(feat)
    # the caller-owned workspace of the one-pass forward, allocated once
    ws_bytes = e2f.e2f_wigner6j_workspace_size(ctx, n, E, L, C, H, wl.cutoff, mix_w=mix_w)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    e2f.e2f_wigner6j_prepare(ctx, L, C, H, wl.cutoff, mix_w=mix_w)

    def step():
        rp, ci = e2f.e2f_neighbor_list(ctx, pos, wl.cutoff, gid, rp_buf, col_buf)
        e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, rp, ci, alpha, L, H, wl.cutoff, mix_w=mix_w, graph_id=gid,
                                      out=out, workspace=ws)

    def fwd_only():
        e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, row_ptr, col, alpha, L, H, wl.cutoff, mix_w=mix_w,
                                      graph_id=gid, out=out, workspace=ws)

    out_e = torch.empty_like(feat)

    def edge_only():
        e2f.e2f_edge_tp_conv_forward(ctx, pos, feat, row_ptr, col, alpha, L, H, wl.cutoff, mix_w=mix_w, out=out_e)

    def nl_only():
        e2f.e2f_neighbor_list(ctx, pos, wl.cutoff, gid, rp_buf, col_buf)

    def timed(fn, k):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(k):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) * 1e3 / k

    for _ in range(args.warmup):
        step()
    # ---- the timed steps, with per-kernel event timing on the launch stream
    e2f.e2f_profile(ctx, True)
    ms_step = timed(step, args.steps)
    prof = e2f.e2f_profile_read(ctx)
    e2f.e2f_profile(ctx, False)
    print("[bench] %s: %d atoms, %d edges, step %.3f ms" % (wl.name, n, E, ms_step), file=sys.stderr, flush=True)
    out_step = out.cpu().numpy()
    # ---- the forward alone, the baseline, the graph alone
    for _ in range(2):
        fwd_only(), edge_only()
    ms_fwd = timed(fwd_only, args.steps)
    # the two-kernel form of the same layer (S written, then recoupled; the
    # context's own workspace, sized on the first call)
    out_s = torch.empty_like(feat)

    def fwd_split():
        e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, row_ptr, col, alpha, L, H, wl.cutoff, mix_w=mix_w,
                                      graph_id=gid, out=out_s, form="split")

    fwd_split()
    ms_fwd_split = timed(fwd_split, args.steps)
    ms_edge = timed(edge_only, args.steps)
    ms_nl = timed(nl_only, args.steps)
    # the attention weights of the same graph (q.k over 16 dims per head + 8 radial functions)
    g = torch.Generator(device=dev).manual_seed(5)
    q_att = torch.randn(n, H, 16, device=dev, generator=g)
    k_att = torch.randn(n, H, 16, device=dev, generator=g) / 4.0
    w_att = torch.randn(H, 8, device=dev, generator=g)
    a_out = torch.empty(E, H, device=dev)
    att_only = lambda: e2f.e2f_attention_weights(ctx, pos, row_ptr, col, wl.cutoff, q_att, k_att, w_att, out=a_out)
    att_only()
    ms_att = timed(att_only, args.steps)
    # uniform attention over all N^2 pairs (App. G): the global-moment form
    glob_out = torch.empty_like(feat)
    glob_only = lambda: e2f.e2f_wigner6j_conv_forward_global(ctx, pos, feat, L, H, wl.cutoff, mix_w=mix_w,
                                                             out=glob_out)
    glob_only()
    ms_glob = timed(glob_only, args.steps)
    # Alg. 1's per-degree weights alpha / D^f (the y_norm flag): both forms of
    # the factorised forward and the per-edge baseline
    yn_out = torch.empty_like(feat)
    yn = {}
    for form in ("fused", "split"):
        def fy(form=form):
            e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, row_ptr, col, alpha, L, H, wl.cutoff, mix_w=mix_w,
                                          graph_id=gid, out=yn_out, y_norm=True, form=form)
        fy()
        yn[form + "_ms"] = timed(fy, args.steps)

    def fy_edge():
        e2f.e2f_edge_tp_conv_forward(ctx, pos, feat, row_ptr, col, alpha, L, H, wl.cutoff, mix_w=mix_w,
                                     graph_id=gid, out=yn_out, y_norm=True)

    fy_edge()
    yn["edge_tp_ms"] = timed(fy_edge, args.steps)
    yn["speedup_vs_edge_tp"] = yn["edge_tp_ms"] / yn["fused_ms"]
    del yn_out
    # the backward of the timed forward (fp32 mixing): both products, then each alone
    g_out = torch.randn(out.shape, device=dev, generator=g)

    def bwd(wf, wa, wp=False):
        return lambda: e2f.e2f_wigner6j_conv_backward(ctx, pos, feat, g_out, row_ptr, col, alpha, L, H, wl.cutoff,
                                                      mix_w=mix_w, graph_id=gid, want_feat=wf, want_alpha=wa,
                                                      want_pos=wp)

    bwd(True, True, True)()
    ms_bwd = timed(bwd(True, True, True), args.steps)
    ms_bwd_pos = timed(bwd(False, False, True), args.steps)
    ms_bwd_feat = timed(bwd(True, False), args.steps)
    ms_bwd_alpha = timed(bwd(False, True), args.steps)
    print("[bench] fwd %.3f ms, edge-TP %.3f ms, graph %.3f ms" % (ms_fwd, ms_edge, ms_nl), file=sys.stderr,
          flush=True)

    # ---- the aggregation alone on stored node tensors T [n][H][dimT][C/H]
    # (random; the unfused form of the aggregation, for its HBM rate): kernel
    # time from HIP events, the call (with its checked plan and one read-back)
    # by the wall clock
    dimT = layer_counts(L)["dimT"]
    T_a3 = torch.randn(n, H, dimT, C // H, device=dev, generator=g)
    S_a3 = torch.empty_like(T_a3)
    order_a3 = torch.from_numpy(morton_order(inp.pos)).to(dev)  # blocks of close receivers
    a3_call = lambda: e2f.e2f_aggregate(ctx, T_a3, row_ptr, col, alpha, out=S_a3, order=order_a3)
    a3_call()
    e2f.e2f_profile(ctx, True)
    ms_a3_call = timed(a3_call, max(3, args.steps // 2))
    prof_a3 = e2f.e2f_profile_read(ctx)
    e2f.e2f_profile(ctx, False)
    t_a3 = prof_a3["a3_aggregate"][1] / prof_a3["a3_aggregate"][0]
    a3_bytes = 2.0 * 4 * n * dimT * C + E * (4.0 + 4.0 * H) + 8.0 * (n + 1)  # T once, S once, CSR, weights
    a3_flops = 2.0 * E * dimT * C
    a3 = {"kernel_ms": t_a3, "call_ms": ms_a3_call, "alg_bytes": a3_bytes, "alg_flops": a3_flops,
          "alg_GBps": a3_bytes / (t_a3 * 1e-3) / 1e9, "alg_frac_hbm": a3_bytes / (t_a3 * 1e-3) / 1e9 / HBM_PEAK_GBS,
          "alg_TFLOPs": a3_flops / (t_a3 * 1e-3) / 1e12, "traffic": None}
    a3_path = os.path.join(ROOT, "profiles", "traffic_a3_%s.json" % wl.name)
    if os.path.exists(a3_path):
        tr = json.load(open(a3_path))
        if tr.get("conv_sha256") == file_sha(os.path.join(ROOT, "paper_2501_19216_amd", "csrc", "conv.hip")):
            a3["traffic"] = tr["bytes_per_launch"]
            a3["traffic_GBps"] = tr["bytes_per_launch"] / (t_a3 * 1e-3) / 1e9
            a3["traffic_frac_hbm"] = a3["traffic_GBps"] / HBM_PEAK_GBS
    del T_a3, S_a3, order_a3
    print("[bench] aggregation alone %.3f ms (%.0f GB/s of compulsory bytes)" % (t_a3, a3["alg_GBps"]),
          file=sys.stderr, flush=True)

    kernels = {k: dict(launches=v[0] // args.steps, ms=v[1] / args.steps) for k, v in prof.items()}
    fused = "recouple" not in prof  # the aggregation coupled to the output itself
    counts = alg_counts(e2f, L, C, H, n, E, fused)
    peaks = {"aggregate": FP32_MFMA_PEAK_TFS, "recouple": FP32_MFMA_PEAK_TFS, "mix": FP32_MFMA_PEAK_TFS}
    for k, v in kernels.items():
        if k in peaks:
            tk = v["ms"] / max(1, v["launches"])
            v["alg_GBps"] = counts[k]["bytes"] / (tk * 1e-3) / 1e9
            v["alg_TFLOPs"] = counts[k]["flops"] / (tk * 1e-3) / 1e12
            r = roof_of(counts[k]["bytes"], counts[k]["flops"], tk, peaks[k])
            v["bound"], v["frac"] = r["bound"], r["frac"]
    dom = max((k for k in kernels if k in peaks), key=lambda k: kernels[k]["ms"])
    t_dom = kernels[dom]["ms"] / max(1, kernels[dom]["launches"])
    roof = roof_of(counts[dom]["bytes"], counts[dom]["flops"], t_dom, peaks[dom])
    roof["traffic"] = None
    roof["kernel"] = dom
    roof["launch_ms"] = t_dom
    roof["alg_flops"] = counts[dom]["flops"]
    roof["alg_bytes"] = counts[dom]["bytes"]
    if "issued_flops" in counts[dom]:
        roof["issued_flops"] = counts[dom]["issued_flops"]
        roof["issued_TFLOPs"] = counts[dom]["issued_flops"] / (t_dom * 1e-3) / 1e12
    if "issued_bf16_flops" in counts[dom]:
        # the fp32 products issued on the bf16 matrix cores (split operands);
        # issued_flops then counts the fp32 MFMAs alone
        roof["issued_bf16_flops"] = counts[dom]["issued_bf16_flops"]
        roof["issued_bf16_TFLOPs"] = counts[dom]["issued_bf16_flops"] / (t_dom * 1e-3) / 1e12
        roof["mfma_time_at_peak_ms"] = (counts[dom]["issued_flops"] / (FP32_MFMA_PEAK_TFS * 1e12)
                                        + counts[dom]["issued_bf16_flops"] / (BF16_MFMA_PEAK_TFS * 1e12)) * 1e3
    tr_path = os.path.join(ROOT, "profiles", "traffic_%s_%s.json" % (dom, wl.name))
    if os.path.exists(tr_path):
        tr = json.load(open(tr_path))
        src = "fused.hip" if dom == "aggregate" and fused else "conv.hip"
        if tr.get("source_sha256") == file_sha(os.path.join(ROOT, "paper_2501_19216_amd", "csrc", src)):
            roof["traffic"] = tr["bytes_per_launch"]
            # measured HBM rate: counter bytes over the same launch time
            roof["traffic_GBps"] = tr["bytes_per_launch"] / (t_dom * 1e-3) / 1e9
            roof["traffic_frac"] = roof["traffic_GBps"] / HBM_PEAK_GBS
    floor = forward_floor(counts, ms_fwd)

    # ---- the bf16 channel-mixing variant of the same forward
    mix_bf16 = mix_w.to(torch.bfloat16)

    def fwd_bf16():
        e2f.e2f_wigner6j_conv_forward(ctx, pos, feat, row_ptr, col, alpha, L, H, wl.cutoff, mix_w=mix_bf16,
                                      graph_id=gid, out=out, workspace=ws)

    for _ in range(2):
        fwd_bf16()
    e2f.e2f_profile(ctx, True)
    ms_fwd_bf16 = timed(fwd_bf16, args.steps)
    prof16 = e2f.e2f_profile_read(ctx)
    e2f.e2f_profile(ctx, False)
    mix16_ms = prof16["mix"][1] / prof16["mix"][0] if "mix" in prof16 else None
    bf16_res = {"ms": ms_fwd_bf16, "atoms_per_s": n / (ms_fwd_bf16 * 1e-3), "mix_ms": mix16_ms}
    if mix16_ms:
        mb = 8.0 * n * (L + 1) ** 2 * C + 2.0 * (L + 1) * C * C
        r = roof_of(mb, counts["mix"]["flops"], mix16_ms, BF16_MFMA_PEAK_TFS)
        bf16_res.update(mix_alg_GBps=mb / (mix16_ms * 1e-3) / 1e9,
                        mix_alg_TFLOPs=counts["mix"]["flops"] / (mix16_ms * 1e-3) / 1e12,
                        mix_bound=r["bound"], mix_frac=r["frac"])

    if args.copy_calib:
        x = torch.empty(1 << 28, dtype=torch.float32, device=dev)
        y = torch.empty_like(x)
        y.copy_(x)
        torch.cuda.synchronize()
        x.sum()
        torch.cuda.synchronize()

    # ---- oracle on the host cores, bounded row sample; parity of the timed output
    cpu = None
    parity = None
    if not args.no_cpu:
        import oracle
        orp, oci = oracle.neighbor_list(inp.pos, wl.cutoff, inp.graph_id)
        graph_equal = bool(np.array_equal(orp, rp_h) and np.array_equal(oci, ci_h))
        k = min(args.cpu_rows, n)
        rows = np.linspace(0, n - 1, k).astype(np.int32)
        cores = int(os.environ.get("OMP_NUM_THREADS") or len(os.sched_getaffinity(0)))
        t0 = time.perf_counter()
        ref = oracle.layer(L, H, inp.pos, inp.feat, orp, oci, alpha_h, inp.path_w, inp.mix_w, rows=rows)
        dt = time.perf_counter() - t0
        cpu = dict(value=k / dt, unit="atoms/s", cores=cores, kind="oracle",
                   sample="%d of %d receiver rows (evenly spaced), fp64 layer definition + mixing, %.1f s" % (k, n, dt),
                   cpu_model=_cpu_model())
        parity = dict(rows=k, max_rel_err=oracle.max_rel_err(out_step[rows], ref, L), graph_bit_exact=graph_equal)
    ctx.close()
    del ws

    # ---- every workload: forward, baseline, speedup, sampled parity
    configs = None
    if not args.no_configs:
        configs = []
        for name, crop in CONFIGS:
            if name == wl.name and not crop:
                configs.append({"workload": name, "atoms": n, "edges": E, "lmax": L, "channels": C, "heads": H,
                                "cutoff": wl.cutoff, "fwd_ms": ms_fwd, "atoms_per_s": n / ms_fwd * 1e3,
                                "edges_per_s": E / ms_fwd * 1e3, "edge_tp_ms": ms_edge,
                                "speedup_vs_edge_tp": ms_edge / ms_fwd, "parity": parity})
                continue
            r = sweep_one(name, max(3, args.steps // 4), 2, crop)
            print("[bench] %s: fwd %.3f ms%s, parity %.2e" % (
                r["workload"], r["fwd_ms"], (", edge-TP %.3f ms" % r["edge_tp_ms"]) if "edge_tp_ms" in r else "",
                r["parity"]["max_rel_err"]), file=sys.stderr, flush=True)
            configs.append(r)

    res = {
        "metric": METRIC,
        "value": n / (ms_step * 1e-3),
        "unit": "atoms/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "atoms": n, "edges": E, "lmax": L, "channels": C, "heads": H,
                   "cutoff": wl.cutoff, "mix": "fp32", "step": "radius graph + Wigner-6j conv forward"},
        "edges_per_s": E / (ms_step * 1e-3),
        "fwd": {"ms": ms_fwd, "atoms_per_s": n / (ms_fwd * 1e-3), "edges_per_s": E / (ms_fwd * 1e-3),
                "roofline": floor, "recouple_in_aggregation": fused, "two_kernel_ms": ms_fwd_split},
        "edge_tp": {"ms": ms_edge, "atoms_per_s": n / (ms_edge * 1e-3), "edges_per_s": E / (ms_edge * 1e-3)},
        "speedup_vs_edge_tp": ms_edge / ms_fwd,
        "fwd_bf16_mix": bf16_res,
        "neighbor_list_ms": ms_nl,
        "workspace_bytes": ws_bytes,
        "backward": {"ms": ms_bwd, "grad_feat_ms": ms_bwd_feat, "grad_alpha_ms": ms_bwd_alpha,
                     "grad_pos_ms": ms_bwd_pos},
        "global_moment": {"ms": ms_glob, "pairs": n * n, "atoms_per_s": n / (ms_glob * 1e-3)},
        "y_norm": yn,
        "attention": {"ms": ms_att, "dk": 16, "n_rbf": 8, "bytes_GBps": (E * (4 + 4 * H) + 12.0 * n) / (ms_att * 1e-3) / 1e9},
        "aggregate_alone": a3,
        "counts": {"dimT": counts["dimT"], "coupling_entries": counts["coupling_entries"],
                   "recouple_entries": counts["recouple_entries"]},
        "kernels": kernels,
        "roofline": roof,
        "cpu_baseline": cpu,
        "parity": parity,
        "configs": configs,
    }
    print(json.dumps(res))


if __name__ == "__main__":
    main()
