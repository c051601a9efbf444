#!/usr/bin/env python3
"""Benchmark of the per-partition GCN layer step on one MI355X.

A step = the whole hot path over the model of the chosen workload: for every layer the
forward step (cache test, message build, recovery, aggregation, dense transform) and the
backward step (dense gradients, transposed aggregation, cache test and message build on the
halo gradients). value = edges traversed per second = layers * nnz / step time, inputs
resident in HBM. The headline runs every layer in the generic order (aggregate first, then
transform); the same model with the per-layer choice of the order is timed beside it and
reported as `optimised_order`. One JSON line on stdout; progress on stderr.
"""
import argparse
import json
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
MFMA_PEAK_TFLOPS = {"f32": 157.3, "bf16": 2500.0}
AGG_KERNELS = ("spmm_walk_kernel", "spmm_transform_kernel")
SPLIT_AGG = "spmm_split_aggregation"   # all kernels of one aggregation of a matrix split by column class


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def spmm_bytes(rows_out, rows_in, nnz, dim, esz):
    """Bytes of one aggregation launch under two models: every needed input row read once
    (compulsory traffic), and one input row read per stored entry (no reuse at all: what the
    caches see). Both include the CSR arrays and the output rows."""
    csr = 8 * (rows_out + 1) + 8 * nnz
    out = rows_out * dim * esz
    return csr + out + rows_in * dim * esz, csr + out + nnz * dim * esz


def read_traffic(workload, order, kernels_sha):
    """profiles/traffic_<workload>.txt: per-launch FETCH_SIZE / WRITE_SIZE bytes of every kernel, from the
    two rocprofv3 --pmc runs of this same script. -> (dict kernel -> bytes, info) or (None, info)."""
    path = os.path.join(ROOT, "profiles", f"traffic_{workload}.txt")
    info = {"file": os.path.relpath(path, ROOT), "present": os.path.exists(path)}
    if not info["present"]:
        return None, info
    per = {}
    for line in open(path):
        line = line.strip()
        if line.startswith("#"):
            for key in ("kernels_sha", "order", "commit"):
                tag = key + "="
                if tag in line:
                    info[key] = line.split(tag)[1].split()[0]
            continue
        if "=" in line:
            name, rest = line.split("=")
            f_b, w_b = rest.split()[:2]
            per[name.strip()] = float(f_b) + float(w_b)
    info["stale"] = info.get("kernels_sha") != kernels_sha
    info["same_order"] = info.get("order") == order
    return per, info


def time_steps(model, first, steps):
    """`steps` steps bracketed by synchronisation: -> (wall seconds, [ms of every step from events
    recorded on the launch stream])."""
    import torch
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        ev[i].record()
        model.step(first + i)
    ev[steps].record()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    return elapsed, [ev[i].elapsed_time(ev[i + 1]) for i in range(steps)]


def cpu_baseline(model, budget_edges=12_000_000):
    """The oracle, as it stands, on a bounded sample of the same workload: every k-th local row of
    the partition (with all columns those rows touch), one stationary step of all layers."""
    import numpy as np
    import torch
    import oracle

    P, w = model.P, model.w
    oracle.build()
    cores = min(os.cpu_count() or 1, 16)
    oracle.set_threads(cores)
    stride = max(1, int(round(P.nnz / budget_edges)))
    rows = torch.arange(0, P.n_loc, stride, device=P.rowptr.device)
    lens = (P.rowptr[rows + 1] - P.rowptr[rows])
    ptr = torch.zeros(rows.numel() + 1, dtype=torch.int64, device=rows.device)
    torch.cumsum(lens, 0, out=ptr[1:])
    nnz_s = int(ptr[-1])
    seg = torch.repeat_interleave(torch.arange(rows.numel(), device=rows.device), lens)
    pos = torch.arange(nnz_s, device=rows.device) - ptr[seg] + P.rowptr[rows][seg]
    cols = P.colidx[pos].long()
    vals = P.vals[pos]
    # local ids: sampled rows first (they stay "local"), every other touched column is halo
    n_s = rows.numel()
    lid = torch.full((P.n_loc + P.n_halo,), -1, dtype=torch.int64, device=rows.device)
    lid[rows] = torch.arange(n_s, device=rows.device)
    other = torch.unique(cols[lid[cols] < 0])
    lid[other] = n_s + torch.arange(other.numel(), device=rows.device)
    h_s = other.numel()
    lc = lid[cols]
    order = torch.argsort(seg * (n_s + h_s) + lc)
    A = (ptr.cpu().numpy(), lc[order].to(torch.int32).cpu().numpy(), vals[order].cpu().numpy())
    order_t = torch.argsort(lc * n_s + seg)
    tptr = torch.zeros(n_s + h_s + 1, dtype=torch.int64, device=rows.device)
    torch.cumsum(torch.bincount(lc, minlength=n_s + h_s), 0, out=tptr[1:])
    At = (tptr.cpu().numpy(), seg[order_t].to(torch.int32).cpu().numpy(), vals[order_t].cpu().numpy())
    qs = {"minmax": oracle.Q_MINMAX, "symmetric": oracle.Q_SYMMETRIC, "none": oracle.Q_NONE}[w.qscheme]
    norm = {"linf": oracle.NORM_LINF, "l2": oracle.NORM_L2}[w.norm]

    def host(t):
        t = t.detach().cpu()
        if t.dtype == torch.bfloat16:
            return t.view(torch.int16).numpy().view(np.uint16).copy()
        return t.numpy().copy()

    # inputs of the sample: local rows from xfull, "halo" rows from the full xfull rows the sample
    # touches; their two alternating versions are the same matrix (local part) or the fresh versions
    state = []
    for li, L in enumerate(model.layers):
        I = model.inputs[li]
        if model.tf[li]:
            # transform-first layer: the exchanged rows are rows of T = X W. Columns of the sample
            # that are local rows of the partition get their T row from the oracle's own transform.
            is_h = other >= P.n_loc
            Wn = host(L.W)
            t_loc, _ = oracle.dense_fwd(host(L.x_local[other[~is_h]]), Wn, relu=False)
            fresh = []
            for v in range(2):
                fr = np.zeros((other.numel(), L.f_out), np.float32)
                fr[host(~is_h)] = t_loc
                fr[host(is_h)] = host(I.fresh[v][other[is_h] - P.n_loc])
                fresh.append(fr)
            state.append(dict(tf=True, x=host(L.x_local[rows]), t=np.zeros((n_s + h_s, L.f_out), np.float32),
                              fresh=fresh, sent=np.zeros_like(fresh[0]), gsent=np.zeros_like(fresh[0]), W=Wn,
                              dH=[host(I.dH[v][rows]) for v in range(2)]))
            continue
        full = [torch.cat([L.xfull[:P.n_loc], I.fresh[v]]) for v in range(2)]
        fresh = [host(f[other]) for f in full]
        x = np.concatenate([host(L.xfull[rows]), np.zeros_like(fresh[0])])
        state.append(dict(tf=False, x=x, fresh=fresh, sent=np.zeros_like(fresh[0]), gsent=np.zeros_like(fresh[0]),
                          W=host(L.W), dH=[host(I.dH[v][rows]) for v in range(2)]))
        del full
    nl = len(model.layers)

    def step(v):
        outs = []
        for li in range(nl):
            s = state[li]
            if s["tf"]:
                outs.append(oracle.layer_tf_fwd(A, n_s, h_s, s["x"], s["t"], s["fresh"][v], s["sent"], s["W"], w.eps,
                                                norm, w.bits, qs, oracle.COMMIT_CUR, li + 1 < nl, True))
                continue
            outs.append(oracle.layer_fwd(A, n_s, h_s, s["x"], s["fresh"][v], s["sent"], s["W"], w.eps, norm,
                                         w.bits, qs, oracle.COMMIT_CUR, li + 1 < nl, True))
        for li in reversed(range(nl)):
            s = state[li]
            if s["tf"]:
                oracle.layer_tf_bwd(At, n_s, h_s, s["x"], outs[li]["H"], s["dH"][v], s["W"], s["gsent"], w.eps, norm,
                                    w.bits, qs, oracle.COMMIT_CUR, li + 1 < nl, True, True)
                continue
            oracle.layer_bwd(At, n_s, h_s, outs[li]["M"], outs[li]["H"], s["dH"][v], s["W"], s["gsent"], w.eps,
                             norm, w.bits, qs, oracle.COMMIT_CUR, li + 1 < nl, True, True)

    step(0)                       # fills the caches (everything is sent once), not timed
    t0 = time.perf_counter()
    step(1)
    dt = time.perf_counter() - t0
    return {"value": nl * nnz_s / dt / 1e9, "unit": "GE/s", "cores": oracle.get_threads(), "kind": "oracle",
            "sample": f"every {stride}th local row of the partition: {n_s} rows, {h_s} other columns, "
                      f"{nnz_s} edges, all {nl} layers fwd+bwd, one stationary step in {dt:.2f} s"}


def kernel_report(cdf, model, w, steps):
    """Per-kernel durations from the events the library recorded inside the timed region, the
    aggregation launches by their position in a step, and every kernel against its own roof."""
    seq = cdf.cdf_profile_read_all()
    kernels = {}
    for name, ms in seq:
        kernels.setdefault(name, []).append(ms)
    esz = 2 if w.dtype == "bf16" else 4
    n, h, nnz = model.n_loc, model.n_halo, model.nnz
    widths = model.spmm_widths()
    # launch order of the aggregations within a step: forward layers 0..L-1 on A, then backward
    # layers L-1..0 on A^T (the library records which of its two aggregation kernels ran)
    per_step = [spmm_bytes(n, n + h, nnz, f, esz) for f in widths] + \
               [spmm_bytes(n + h, n, nnz, f, esz) for f in reversed(widths)]
    wid_of = list(widths) + list(reversed(widths))
    # a matrix split by column class is one aggregation too: its preparation, two walks and the sum of the partial rows
    # follow one another, and its time is that of them all
    agg, split = [], None
    for name, ms in seq:
        if name == "split_kernels" and split is None:
            split = 0.0
        if split is not None:
            split += ms
            if name == "split_combine_kernel":
                agg.append((SPLIT_AGG, split))
                split = None
        elif name in AGG_KERNELS:
            agg.append((name, ms))
    nl = len(per_step)
    positions = None
    if len(agg) == nl * steps:
        positions = []
        for i in range(nl):
            mine = agg[i::nl]
            assert len({name for name, _ in mine}) == 1
            positions.append({"kernel": mine[0][0], "width": wid_of[i], "matrix": "A" if i < nl // 2 else "A^T",
                              "avg_ms": sum(ms for _, ms in mine) / len(mine),
                              "no_reuse_bytes": per_step[i][1], "compulsory_bytes": per_step[i][0]})
    out = {name: {"launches": len(ms), "avg_ms": sum(ms) / len(ms), "ms_per_step": sum(ms) / steps}
           for name, ms in kernels.items()}
    return out, positions


def roofline(positions, traffic, tinfo):
    """The dominant kernel (the aggregation variant with the most time per step) against the HBM roof.
    achieved = bytes the hardware counters saw this kernel move per launch (FETCH_SIZE + WRITE_SIZE at the
    L2 <-> fabric interface, from the committed rocprofv3 runs of this script) / its average launch time
    measured here. The byte models are side figures: `l2_level` counts one feature row per stored entry
    (what the caches serve, can exceed the HBM peak), `compulsory` counts every input row once."""
    if not positions:
        return None
    by_kernel = {}
    for p in positions:
        by_kernel.setdefault(p["kernel"], []).append(p)
    name = max(by_kernel, key=lambda k: sum(p["avg_ms"] for p in by_kernel[k]))
    sel = by_kernel[name]
    avg_s = sum(p["avg_ms"] for p in sel) / len(sel) / 1e3
    bmax = sum(p["no_reuse_bytes"] for p in sel) / len(sel)
    bmin = sum(p["compulsory_bytes"] for p in sel) / len(sel)
    r = {"kernel": name, "bound": "hbm", "achieved": None, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": None,
         "traffic": None, "avg_launch_ms": avg_s * 1e3, "launches_per_step": len(sel),
         "l2_level_bytes_per_launch": bmax, "l2_level_GBps": bmax / avg_s / 1e9,
         "compulsory_bytes_per_launch": bmin, "compulsory_GBps": bmin / avg_s / 1e9,
         "compulsory_frac": bmin / avg_s / 1e9 / HBM_PEAK_GBS, "traffic_over_compulsory": None,
         "traffic_source": tinfo}
    usable = traffic is not None and name in traffic and tinfo.get("same_order")
    if usable:
        t = traffic[name]
        r["traffic"] = t
        r["achieved"] = t / avg_s / 1e9
        r["frac"] = r["achieved"] / HBM_PEAK_GBS
        r["traffic_over_compulsory"] = t / bmin
        if tinfo.get("stale"):
            log(f"[bench] WARNING: {tinfo['file']} was taken on other kernel sources "
                f"({tinfo.get('kernels_sha')}); roofline.traffic may be out of date")
    else:
        log(f"[bench] no usable counter summary for this workload / order ({tinfo}); roofline.frac is null")
    return r


def kernel_rooflines(model, w, kernels):
    """Every HBM-bound kernel against its own algorithmic bytes (streaming kernels: these are the bytes
    that must move), every dense kernel against the peak of the matrix instruction it executes."""
    esz = 2 if w.dtype == "bf16" else 4
    n, h = model.n_loc, model.n_halo
    widths = model.spmm_widths()

    def avg(xs):
        return sum(xs) / len(xs)
    lay = list(zip(widths, [g for _, g in w.layers()]))   # (width of the halo rows, f_out)
    sent_f = [int(L.n_sent.item()) for L in model.layers]
    sent_b = [int(L.gn_sent.item()) for L in model.layers]
    rb = [L.row_bytes for L in model.layers]
    alg = {
        "filter_kernel": avg([h * (2 * f * esz + 1) + 4 * sn[i] for sn in (sent_f, sent_b) for i, (f, _) in enumerate(lay)]),
        "quantize_kernel": avg([sn[i] * (3 * f * esz + rb[i] + 12) for sn in (sent_f, sent_b) for i, (f, _) in enumerate(lay)]),
        "dequantize_kernel": avg([sent_f[i] * (2 * f * esz + rb[i] + 12) for i, (f, _) in enumerate(lay)]),
        # one-pass test + message build: every row read once, sent rows committed and coded
        "test_encode_kernel": avg([h * (2 * f * esz + 1) + sn[i] * (f * esz + rb[i] + 8)
                                   for sn in (sent_f, sent_b) for i, (f, _) in enumerate(lay)]),
        "place_messages_kernel": avg([sn[i] * (2 * rb[i] + 16 + 4)
                                    for sn in (sent_f, sent_b) for i, (f, _) in enumerate(lay)]),
    }
    per_kernel = {}
    for name, b in alg.items():
        if name in kernels:
            gbs = b / (kernels[name]["avg_ms"] * 1e-3) / 1e9
            per_kernel[name] = {"bound": "hbm", "algorithmic_bytes_per_launch": b, "achieved_GBps": gbs,
                                "peak_GBps": HBM_PEAK_GBS, "frac": gbs / HBM_PEAK_GBS}
    flops = avg([2.0 * n * f * g for f, g in w.layers()])
    # everything runs on the bf16 matrix cores. bf16-stored activations: fp32 operands split into a high and
    # a low part (2, 2 and 3 products executed per useful one for the forward product, dW and dM); an fp32
    # workload: both operands split into three parts, six products
    executed = {"gemm_kernel<FWD>": 2, "gemm_kernel<DM>": 3, "gemm_kernel<DW>": 2} if w.dtype == "bf16" else \
        {"gemm_kernel<FWD>": 6, "gemm_kernel<DM>": 6, "gemm_kernel<DW>": 6}
    for name in ("gemm_kernel<FWD>", "gemm_kernel<DW>", "gemm_kernel<DM>"):
        if name in kernels:
            mult = executed.get(name, 1)
            peak = MFMA_PEAK_TFLOPS["bf16" if mult > 1 else "f32"]
            tf = flops / (kernels[name]["avg_ms"] * 1e-3) / 1e12
            per_kernel[name] = {"bound": "mfma", "instruction": "bf16" if mult > 1 else "f32",
                                "useful_flops_per_launch": flops, "useful_TFLOPs": tf,
                                "executed_TFLOPs": tf * mult, "peak_TFLOPs": peak, "frac": tf * mult / peak}
    return per_kernel


def run_order(cdf, w, P, dev, order, rho, phi, warmup, steps, profile):
    """Build the model in one order of the products, warm up, time `steps` steps."""
    import torch
    from paper_2408_00232_amd.workload import Model
    model = Model(w, dev, rho=rho, phi=phi, partition=P, order=order)
    for t in range(warmup):
        model.step(t)
    torch.cuda.synchronize()
    if profile:
        cdf.cdf_profile_enable(True)
    elapsed, step_ms = time_steps(model, warmup, steps)
    if profile:
        cdf.cdf_profile_enable(False)
    res = {"ms_per_step": elapsed / steps * 1e3, "ms_per_step_median": statistics.median(step_ms),
           "per_kernel_events": bool(profile),
           "value": model.edges_per_step() / (elapsed / steps) / 1e9,
           "value_median": model.edges_per_step() / (statistics.median(step_ms) * 1e-3) / 1e9,
           "order_per_layer": ["transform-first" if t else "aggregate-first" for t in model.tf]}
    return model, res


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="share", help="tiny | mid | large | wide | share")
    ap.add_argument("--rho", type=float, default=0.37, help="fraction of halo rows refreshed per step (imposed by the inputs)")
    ap.add_argument("--phi", type=float, default=0.01, help="fraction of local rows whose gradient changes")
    ap.add_argument("--order", default="aggregate", choices=["aggregate", "auto"],
                    help="aggregate: every layer computes (A X) W, the generic layer step (headline); "
                         "auto: layers with f_out < f_in compute A (X W)")
    ap.add_argument("--no-optimised", action="store_true", help="skip the second timing in the other order")
    ap.add_argument("--no-rho-sweep", action="store_true", help="skip the timings at other send fractions")
    ap.add_argument("--epochs", type=int, default=10,
                    help="after the timed region: this many steps on drifting inputs from zero caches, with the cache hit "
                         "rate and the step time of every epoch (0 to skip)")
    ap.add_argument("--graph", action="store_true",
                    help="also time the same steps replayed from captured HIP graphs (reported beside the eager figures)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run the library's plain copy kernel on 1 GiB (for scaling hardware counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        log("bench.py: this build runs on one GPU only (no collectives are part of it); use --gpus 1")
        sys.exit(2)

    import torch
    from cdfgen import configs
    import paper_2408_00232_amd as cdf
    from paper_2408_00232_amd import build as cdf_build

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    cdf.binding.load()
    dev = "cuda:0"
    w = configs.ALL[args.workload]
    t_setup = time.time()
    log(f"[bench] building workload '{w.name}' on {dev} ...")
    P = configs.build_partition(w, device=dev)
    if args.copy_calibration:
        src = torch.ones(1 << 28, dtype=torch.float32, device=dev)
        dst = torch.zeros_like(src)
        for _ in range(3):
            cdf.cdf_profile_copy(dst, src)
        torch.cuda.synchronize()
        del src, dst
    model, head = run_order(cdf, w, P, dev, args.order, args.rho, args.phi, args.warmup, args.steps, profile=True)
    log(f"[bench] partition: n_loc={model.n_loc} n_halo={model.n_halo} nnz={model.nnz} layers={w.layers()} "
        f"order={args.order} setup+run {time.time() - t_setup:.1f}s mem {torch.cuda.memory_allocated() / 2**30:.1f} GiB")
    log(f"[bench] {head['ms_per_step']:.3f} ms/step (median {head['ms_per_step_median']:.3f}) = {head['value']:.3f} GE/s")

    kernels, positions = kernel_report(cdf, model, w, args.steps)
    # the same steps once more without the library's per-kernel events (two event records per launch
    # cost nothing on millisecond kernels and up to half of a launch-bound step)
    e2, ms2 = time_steps(model, args.warmup + args.steps, args.steps)
    head["ms_per_step_without_kernel_events"] = statistics.median(ms2)
    head["value_without_kernel_events"] = model.edges_per_step() / (statistics.median(ms2) * 1e-3) / 1e9
    log(f"[bench] without per-kernel events: {head['ms_per_step_without_kernel_events']:.3f} ms/step")
    traffic, tinfo = read_traffic(w.name, args.order, cdf_build.sources_sha())
    roof = roofline(positions, traffic, tinfo)
    per_kernel = kernel_rooflines(model, w, kernels)

    # per layer shape: forward and backward time of the layer step (a separate, untimed pass of the
    # same steps with an event pair around every layer call), median over the passes
    fw, bw = [], []
    t_next = args.warmup + 2 * args.steps
    for t in range(t_next, t_next + max(4, min(args.steps, 10))):
        a_ms, b_ms = model.step_timed_per_layer(t)
        fw.append(a_ms)
        bw.append(b_ms)
    per_layer = []
    for li, (f_in, f_out) in enumerate(w.layers()):
        tf_ms = statistics.median(x[li] for x in fw)
        tb_ms = statistics.median(x[li] for x in bw)
        per_layer.append({"f_in": f_in, "f_out": f_out, "order": "transform-first" if model.tf[li] else "aggregate-first",
                          "fwd_ms": tf_ms, "bwd_ms": tb_ms, "GE_per_s": model.nnz / ((tf_ms + tb_ms) * 1e-3) / 1e9})

    graph_replay = None
    if args.graph:
        # launch-bound workloads (tiny, mid): the same steps as two captured graphs, one per input version
        model.capture()
        t_next += 12
        for t in range(t_next, t_next + 2):
            model.step(t)
        eg, g_ms = time_steps(model, t_next + 2, args.steps)
        graph_replay = {"ms_per_step": eg / args.steps * 1e3, "ms_per_step_median": statistics.median(g_ms),
                        "value": model.edges_per_step() / (eg / args.steps) / 1e9, "unit": "GE/s"}

    rho_f = [int(L.n_sent.item()) / max(model.n_halo, 1) for L in model.layers]
    rho_b = [int(L.gn_sent.item()) / max(model.n_halo, 1) for L in model.layers]
    n, h, nnz = model.n_loc, model.n_halo, model.nnz
    edges = model.edges_per_step()

    cpu = None
    if not args.no_cpu_baseline:
        log("[bench] timing the CPU oracle on a sample ...")
        cpu = cpu_baseline(model)

    # the threshold at work: epochs on drifting inputs from zero caches (hit rate per epoch is a result here,
    # not an input as in the stationary step above)
    epochs = None
    if args.epochs > 0:
        eps_run = model.run_epochs(args.epochs)
        for e in eps_run:
            e["GE_per_s"] = edges / (e["ms"] * 1e-3) / 1e9
        epochs = {"eps": w.eps, "drift": "halo rows and upstream gradients x (1 + eta_t u_r g), eta_t = 0.2 * 0.6^t, "
                                         "u_r log-uniform in [0.1, 10] per row, g ~ N(0,1) per element; caches start at zero",
                  "per_epoch": eps_run}
        log("[bench] epochs from zero caches: hit rate fwd " +
            " ".join(f"{sum(e['hit_rate_fwd']) / len(e['hit_rate_fwd']):.2f}" for e in eps_run) +
            " | ms " + " ".join(f"{e['ms']:.1f}" for e in eps_run))

    # measured streaming ceiling: the library's plain copy kernel on 1 GiB (read + write bytes)
    src = torch.ones(1 << 28, dtype=torch.float32, device=dev)
    dst = torch.zeros_like(src)
    cdf.cdf_profile_copy(dst, src)
    torch.cuda.synchronize()
    tc = time.perf_counter()
    for _ in range(10):
        cdf.cdf_profile_copy(dst, src)
    torch.cuda.synchronize()
    copy_gbs = 10 * 2 * (1 << 30) / (time.perf_counter() - tc) / 1e9
    del src, dst

    # the same workload at other send fractions, and in the other order of the products
    del model
    torch.cuda.empty_cache()
    sweep = None
    if not args.no_rho_sweep:
        sweep = [{"rho": args.rho, "ms_per_step": head["ms_per_step_without_kernel_events"],
                  "value": head["value_without_kernel_events"]}]   # like the other points: no per-kernel events
        for rho in (0.05, 1.0):
            m2, r2 = run_order(cdf, w, P, dev, args.order, rho, args.phi, 3, max(4, args.steps // 2), profile=False)
            sweep.append({"rho": rho, "ms_per_step": r2["ms_per_step_median"], "value": r2["value_median"]})
            del m2
            torch.cuda.empty_cache()
        sweep.sort(key=lambda x: x["rho"])
    optimised = None
    if not args.no_optimised:
        other = "auto" if args.order == "aggregate" else "aggregate"
        m2, optimised = run_order(cdf, w, P, dev, other, args.rho, args.phi, args.warmup, args.steps, profile=False)
        optimised["order"] = other
        optimised["unit"] = "GE/s"
        optimised["note"] = ("layers whose output is narrower than their input compute A (X W): same layer, same "
                             "steps, narrower rows in the messages and in the aggregation"
                             if other == "auto" else "every layer computes (A X) W")
        log(f"[bench] order={other}: {optimised['ms_per_step']:.3f} ms/step = {optimised['value']:.3f} GE/s")
        del m2
        torch.cuda.empty_cache()

    out = {
        "metric": "GCN layer fwd+bwd edges/sec (GE/s) per partition; % of HBM roofline",
        "value": head["value"], "unit": "GE/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": w.dtype, "data": "synthetic",
        "ms_per_step_median": head["ms_per_step_median"], "value_median": head["value_median"],
        "ms_per_step_without_kernel_events": head["ms_per_step_without_kernel_events"],
        "value_without_kernel_events": head["value_without_kernel_events"],
        "config": {"workload": f"{w.name}: {w.kind} graph, {w.n_vertices} vertices, partition {w.part} of "
                               f"{w.parts} ({w.partitioner}), n_loc={n}, n_halo={h}, nnz={nnz}, layers "
                               f"{'-'.join(str(d) for d in w.dims)}, {w.bits}-bit {w.qscheme} messages, "
                               f"eps={w.eps} ({w.norm})",
                   "order": args.order, "order_per_layer": head["order_per_layer"],
                   "edges_per_step": edges,
                   "send_fraction": {"imposed_by_inputs": True, "rho": args.rho, "phi": args.phi,
                                     "fwd": rho_f, "bwd": rho_b}},
        "roofline": roof,
        "cpu_baseline": cpu,
        "optimised_order": optimised,
        "rho_sweep": sweep,
        "epochs_from_zero_caches": epochs,
        "aggregation_by_position": positions,
        "kernels": kernels,
        "kernel_rooflines": per_kernel,
        "per_layer": per_layer,
        "copy_ceiling_GBps": copy_gbs,
        "graph_replay": graph_replay,
        "kernels_sha": cdf_build.sources_sha(),
    }
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
