"""Benchmark of the spiking-network timestep on one MI355X.

Default workload: the batched conductance-scaling sweep, 256 independent
instances of uneven size (A ~ LU[200, 1000] Poisson sources at 20 Hz,
B ~ LU[2000, 20000] and C ~ LU[100, 1000] Traub-Miles neurons, A->B p = 0.2,
B->C p = 0.5, C->C all-to-all inhibitory; g_scale ~ LU[0.1, 10] per
instance; about 612 M synapses), stepped together, dt = 0.1 ms with 3 Euler
substeps.  A "step" is one timestep of every instance: propagation of the
previous step's spikes, the neuron update and spike compaction.

Prints ONE JSON line: value = Traub-Miles neuron-steps per second over the
timed steps (graph replays, inputs already resident in HBM), synaptic events
per second, the roofline of the dominant kernel (per-launch durations from
event-stamped launches over live steps after the timed region), the same
instances stepped one at a time on the same kernels (per-instance loop), and
the FP64 oracle timed on a bounded sample on the host cores.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, GB/s
# VALU issue peak: 256 CUs x 4 SIMDs x 16 lanes per cycle x 2.4 GHz; fp64 FMA
# issues at this full rate (78.6 fp64 TFLOP/s = 2 flops x 3.93e13)
VALU_PEAK_TLANE = 256 * 4 * 16 * 2.4e9 / 1e12

# Algorithmic work per unit (the method's own data, not this library's
# representation of it):
#  - propagation: 8 B per synaptic event (col_idx + fp32 weight) + 12 B per
#    spiking row (its two row-start entries and its spike id)
#  - neuron update: per Traub-Miles neuron-step, V, m, h, n in fp32 read and
#    written (32 B), the V compensation word read and written (8 B), and 8 B
#    per incoming projection (fp32 conductance read and written); and about
#    500 VALU lane-instructions (3 substeps of 6 exponentials, 4 divisions
#    and about 50 other operations)
#  - potentiation: per column entry of a post neuron that spiked, its CRS
#    position and pre index (8 B), the weight read and written (8 B) and the
#    pre-synaptic trace read (4 B)
PROP_BYTES_PER_EVENT = 8
PROP_BYTES_PER_ROW = 12
NEURON_ALG_STATE_BYTES = 32
NEURON_ALG_VLO_BYTES = 8
NEURON_ALG_G_BYTES = 8
NEURON_VALU_PER_STEP = 500
#  - Izhikevich neuron-step: v and u in fp32 read and written (16 B), its
#    a, b, c, d read (16 B), and 8 B per incoming projection
NEURON_ALG_IZH_BYTES = 32
POT_BYTES_PER_ENTRY = 20
# What this library stores per unit (double-float state, 64-bit conductances,
# 16 B per spiking row including its work item): bytes a launch moves beyond
# the algorithmic ones
NEURON_REPR_STATE_BYTES = 64
NEURON_REPR_G_BYTES = 16
PROP_REPR_BYTES_PER_ROW = 16

WORKLOADS = {
    1: "A=100 Poisson @20 Hz, B=1000 HH, C=100 HH; A->B p=0.5, B->C and C->C all-to-all; dt=0.1 ms, 3 Euler substeps",
    2: "A=1000 Poisson @20 Hz, B=20000 HH, C=1000 HH; A->B p=0.2, B->C p=0.5, C->C all-to-all "
       "inhibitory; dt=0.1 ms, 3 Euler substeps",
    3: "A=2000 Poisson @30 Hz, B=100000 HH, C=1000 HH; A->B p=0.2, B->C p=0.5 with pair STDP, C->C all-to-all; "
       "dt=0.1 ms, 3 Euler substeps",
    4: "256 instances, A~LU[200,1000], B~LU[2000,20000], C~LU[100,1000], g_scale~LU[0.1,10], p=0.2/0.5; "
       "dt=0.1 ms, 3 Euler substeps",
    5: "64 x (A=500, B=5000, C=200), p=0.2/0.5; loss = MSE of time-averaged C voltage to a seeded target; "
       "dt=0.1 ms, 3 Euler substeps",
}


STEP_KERNEL_SOURCES = ("snn_device.h", "snn_internal.h", "snn_kernels.hip")


def kernel_sources_sha256():
    """Hash of the device sources the step kernels (neuron update,
    propagation, potentiation) are compiled from; the host runtime and the
    adjoint kernels live in other files."""
    import hashlib
    d = os.path.join(ROOT, "paper_1412_0595_amd", "csrc")
    h = hashlib.sha256()
    for f in STEP_KERNEL_SOURCES:
        h.update(f.encode())
        with open(os.path.join(d, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def profiled_values(kernel, workload, what):
    """The key: value lines of the committed counter summary
    profiles/<kernel>_<workload>_<what>.txt, or None when there is none or the
    kernel sources changed since its counters were taken."""
    name = f"workload{workload}" if isinstance(workload, int) else str(workload)
    path = os.path.join(ROOT, "profiles", f"{kernel}_{name}_{what}.txt")
    if not os.path.exists(path):
        return None
    vals = {}
    with open(path) as fh:
        for line in fh:
            if ":" in line and not line.startswith((" ", "#")):
                k, v = line.split(":", 1)
                vals[k.strip()] = v.strip()
    if vals.get("sources_sha256") != kernel_sources_sha256():
        return None
    return vals


def profiled_traffic(kernel, workload):
    """HBM bytes per launch of `kernel` on `workload` from the committed
    counter summary (rocprofv3 FETCH_SIZE and WRITE_SIZE passes, each scaled
    by the same counter's reading for a plain copy of known size), or None
    when there is none or the kernel sources changed since it was taken."""
    vals = profiled_values(kernel, workload, "traffic")
    if vals is None:
        return None
    try:
        return int(float(vals["traffic_bytes_per_launch"]))
    except (KeyError, ValueError):
        return None


def sub_spec(spec, k):
    return dict(dt=spec["dt"], substeps=spec["substeps"], instances=[spec["instances"][k]])


def time_loop(spec, steps, warmup, tune_cache=None):
    """Every instance alone on the same kernels (autotuned, graph replays),
    one after the other: `warmup` untimed steps and one untimed run of the
    timed length (graph capture), then `steps` timed.  Returns the summed
    step time (hipEvents around each instance's timed steps) and the synaptic
    events of those steps."""
    import numpy as np
    import torch
    from paper_1412_0595_amd import snn
    total_ms = 0.0
    events = 0
    for k in range(len(spec["instances"])):
        if k % 64 == 0:
            note(f"per-instance loop: instance {k} of {len(spec['instances'])}")
        sub = sub_spec(spec, k)
        net = snn.Network(sub, autotune=True, tune_cache=tune_cache)
        net.step(warmup)
        net.step(steps)
        deg = out_degree_table(sub)
        c0 = spike_totals(net, sub)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s = torch.cuda.current_stream()
        e0.record(s)
        net.step(steps)
        e1.record(s)
        e1.synchronize()
        total_ms += e0.elapsed_time(e1)
        c1 = spike_totals(net, sub)
        events += sum(int(((c1[0][p] - c0[0][p]) * deg[0][p]).sum()) for p in range(len(c0[0])))
        net.close()
        del net
    return total_ms, events


def adjoint_bench(args):
    """Recorded forward + reverse pass of workload 5 (gradient of the MSE of
    the time-averaged output voltage w.r.t. every weight and g_scale),
    batched, and the same per instance in a loop."""
    import numpy as np
    import torch
    from paper_1412_0595_amd import netgen, snn
    spec = netgen.make_config(args.workload, n_instances=args.instances)
    T, K = args.steps, args.ckpt_every
    y = torch.tensor(np.concatenate(spec["target"]), device="cuda")
    sizes = [inst["pops"][2]["n"] for inst in spec["instances"]]
    w = torch.tensor(np.concatenate([np.full(n, 1.0 / n) for n in sizes]), device="cuda")

    def run(sp, yy, ww, reps=2):
        net = snn.Network(sp, record_vbar=("C",))
        best = None
        for _ in range(reps):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
            s = torch.cuda.current_stream()
            e[0].record(s)
            vb = net.forward_record(2, T, K)
            e[1].record(s)
            dv = 2 * ww * (vb - yy)
            dg, ds, _ = net.backward(dv)
            e[2].record(s)
            e[2].synchronize()
            f, b = e[0].elapsed_time(e[1]), e[1].elapsed_time(e[2])
            if best is None or f + b < best[0] + best[1]:
                best = (f, b)
        n_hh = sum(p["n"] for inst in sp["instances"] for p in inst["pops"] if p["kind"] == "hh")
        net.close()
        return best, n_hh

    (fb, bb), n_hh = run(spec, y, w)
    loop_f = loop_b = 0.0
    off = 0
    if args.loop == 0:
        sizes_loop = []          # batched pass only (profiling runs)
    else:
        sizes_loop = sizes
    for k, n in enumerate(sizes_loop):
        (f, b), _ = run(sub_spec(spec, k), y[off:off + n], w[off:off + n], reps=1)
        loop_f += f
        loop_b += b
        off += n
    rec = {"metric": "adjoint (recorded forward + reverse) time, batched vs plain per-instance loop",
           "value": (loop_f + loop_b) / (fb + bb) if sizes_loop else None, "unit": "x speedup",
           "higher_is_better": True,
           "n_gpus": 1, "steps": T, "ckpt_every": K, "dtype": "f64", "data": "synthetic",
           "config": {"workload": WORKLOADS.get(args.workload), "instances": len(sizes), "hh_neurons": n_hh},
           "batched_ms": {"forward_record": fb, "backward": bb},
           "loop_ms": {"forward_record": loop_f, "backward": loop_b},
           "neuron_steps_per_s_forward": n_hh * T / (fb * 1e-3)}
    print(json.dumps(rec))


def live_roofline(net, spec, n_hh, deg, profile_steps, workload):
    """Roofline of the dominant kernel over `profile_steps` further live steps
    (advances the network).

    Per-kernel launch duration: every kernel of those steps is launched
    directly with a start/stop hipEvent pair that the HIP runtime stamps with
    that dispatch's own begin and end.  The algorithmic work of those launches
    is counted exactly: the propagation launches deliver the spikes pending at
    the start plus those emitted during the window, less those still pending
    at its end.  A kernel's roofline is the tighter of its HBM bound
    (algorithmic bytes / duration against 8 TB/s) and its VALU bound
    (algorithmic lane-instructions / duration against the issue peak); the
    dominant kernel is the one with the most time."""
    import numpy as np
    pend0 = [[net.last_spikes(b, p).astype(np.int64) for p in range(len(spec["instances"][b]["pops"]))]
             for b in range(len(spec["instances"]))]
    ca = spike_totals(net, spec)
    prof = net.profile_steps(profile_steps)
    cb = spike_totals(net, spec)
    pend_events = 0
    pend_rows = 0
    for b in range(len(spec["instances"])):
        for p in range(len(spec["instances"][b]["pops"])):
            delivered = pend0[b][p] + (cb[b][p] - ca[b][p]) - net.last_spikes(b, p).astype(np.int64)
            n_out = sum(1 for q in spec["instances"][b]["projs"] if q["pre"] == p)
            pend_events += int((delivered * deg[b][p]).sum())
            pend_rows += int(delivered.sum()) * n_out
    n_in = sum(len([q for q in inst["projs"] if q["post"] == k]) * inst["pops"][k]["n"]
               for inst in spec["instances"] for k in range(len(inst["pops"])))
    n_launch = prof["neuron"][1]
    neuron_alg = neuron_alg_bytes(spec)
    neuron_repr = NEURON_REPR_STATE_BYTES * n_hh + NEURON_REPR_G_BYTES * n_in
    prop_alg = PROP_BYTES_PER_EVENT * pend_events + PROP_BYTES_PER_ROW * pend_rows
    prop_repr = PROP_BYTES_PER_EVENT * pend_events + PROP_REPR_BYTES_PER_ROW * pend_rows
    kern = {
        "propagate": dict(ms=prof["propagate"][0], n=prof["propagate"][1], bytes=prop_alg, repr=prop_repr, valu=0),
        "neuron": dict(ms=prof["neuron"][0], n=n_launch, bytes=neuron_alg * n_launch,
                       repr=neuron_repr * n_launch, valu=NEURON_VALU_PER_STEP * n_hh * n_launch),
    }
    if kern["propagate"]["n"] == 0:
        # fused delivery: the neuron update walks the rows itself
        kern["neuron"]["bytes"] += prop_alg
        kern["neuron"]["repr"] += prop_repr
        del kern["propagate"]
    if prof["potentiate"][1]:
        # the potentiation launches walk the columns of the post neurons whose
        # spikes were pending at the start or emitted in the window, less
        # those still pending at its end
        pot_entries = 0
        for b, inst in enumerate(spec["instances"]):
            for q in inst["projs"]:
                if not q.get("stdp"):
                    continue
                k = q["post"]
                cdeg = np.bincount(np.asarray(q["col_idx"]), minlength=inst["pops"][k]["n"]).astype(np.int64)
                delivered = pend0[b][k] + (cb[b][k] - ca[b][k]) - net.last_spikes(b, k).astype(np.int64)
                pot_entries += int((delivered * cdeg).sum())
        kern["potentiate"] = dict(ms=prof["potentiate"][0], n=prof["potentiate"][1],
                                  bytes=POT_BYTES_PER_ENTRY * pot_entries, repr=POT_BYTES_PER_ENTRY * pot_entries,
                                  valu=0)

    def fracs(k):
        sec = kern[k]["ms"] * 1e-3
        hbm = kern[k]["bytes"] / sec / 1e9
        alu = kern[k]["valu"] / sec / 1e12
        return hbm, alu

    dom = max(kern, key=lambda k: kern[k]["ms"])
    hbm, alu = fracs(dom)
    per = lambda v: int(v / max(kern[dom]["n"], 1))
    if alu / VALU_PEAK_TLANE > hbm / HBM_PEAK_GBS:
        roof = {"kernel": "k_" + dom, "bound": "alu", "achieved": round(alu, 4), "peak": round(VALU_PEAK_TLANE, 3),
                "unit": "T VALU lane-instructions/s", "frac": round(alu / VALU_PEAK_TLANE, 6),
                "work_per_launch": per(kern[dom]["valu"]),
                "work_per_unit": f"{NEURON_VALU_PER_STEP} VALU lane-instructions per Traub-Miles neuron-step"}
    else:
        roof = {"kernel": "k_" + dom, "bound": "hbm", "achieved": round(hbm, 3), "peak": HBM_PEAK_GBS,
                "unit": "GB/s", "frac": round(hbm / HBM_PEAK_GBS, 6)}
    roof["traffic"] = profiled_traffic("k_" + dom, workload) if workload is not None else None
    if roof["bound"] == "alu" and workload is not None:
        # the issue rate the counters measured (all instructions the kernel
        # runs, not only the method's arithmetic), from the committed summary
        v = profiled_values("k_" + dom, workload, "valu")
        if v is not None:
            roof["valu_issue_counted"] = {"frac": float(v["valu_issue_frac"]),
                                          "instructions_per_wave": float(v["valu_instructions_per_wave"]),
                                          "source": f"profiles/k_{dom}_workload{workload}_valu.txt"}
    roof["hbm"] = {"algorithmic_bytes_per_launch": per(kern[dom]["bytes"]),
                   "achieved_GBs": round(hbm, 3), "frac": round(hbm / HBM_PEAK_GBS, 6),
                   "stored_bytes_per_launch": per(kern[dom]["repr"])}
    roof["profiled_steps"] = profile_steps
    roof["ms_per_launch"] = {k: round(v["ms"] / max(v["n"], 1), 6) for k, v in kern.items()}
    roof["algorithmic_bytes_per_launch"] = {k: int(v["bytes"] / max(v["n"], 1)) for k, v in kern.items()}
    roof["share_of_kernel_time"] = {k: round(v["ms"] / sum(x["ms"] for x in kern.values()), 4)
                                    for k, v in kern.items()}
    if "propagate" in kern and dom != "propagate":
        h, _ = fracs("propagate")
        roof["propagate"] = {"achieved_GBs": round(h, 3), "frac": round(h / HBM_PEAK_GBS, 6),
                             "events_per_launch": int(pend_events / max(kern["propagate"]["n"], 1)),
                             "traffic": profiled_traffic("k_propagate", workload) if workload is not None else None}
    return roof


def calibrate_bench(args):
    """The calibration of Section 5.1 (Fig. 1) end to end: each (nConn,
    gScale) sweep stepped as one batched network, then the selection against
    the reference run (gScale 1 at the smallest nConn) and the fit of
    gScale = k1 / (k2 + nConn) + k3.

    layered: nConn = 100..1000 (step 50) x 25 gScale in [0.1, 10], A = nConn /
    0.2 Poisson inputs at 20 Hz, B = 1000, C = 100.
    lhi: the LHI variant, PN = 100..1000 (step 50) x 25 scales, KC = 1000,
    DN = 100, with 20 and 40 LHI, the PN->KC and the PN->LHI scale each swept.
    izh: the 4:1 Izhikevich network of Section 5.1 (800 excitatory, 200
    inhibitory neurons, 1000 Poisson inputs at 20 Hz), nConn = 100..1000
    (step 50) recurrent connections per neuron x 26 scales of the recurrent
    weights, 10^-1.5 .. 10 in tenths of a decade, criterion the excitatory
    avgSpike."""
    import numpy as np
    import torch
    from paper_1412_0595_amd import calibrate as cal
    from paper_1412_0595_amd import netgen, snn
    gs = 10.0 ** np.linspace(-1.0, 1.0, 25)
    if args.model == "layered":
        sweeps = [("layered: A->B scale, B spiking",
                   netgen.calibration_config(np.arange(100.0, 1001.0, 50.0), gs, n_b=1000, n_c=100,
                                             ref_n_conn=100.0, steps=args.steps))]
        workload = ("calibration sweep: nConn 100..1000 step 50 x 25 gScale in [0.1, 10]; "
                    "A = nConn/0.2 Poisson at 20 Hz, B = 1000 HH, C = 100 HH, p = 0.2/0.5")
    elif args.model == "izh":
        gi = 10.0 ** (np.arange(-15, 11) / 10.0)     # 10^-1.5 .. 10 in tenths of a decade, 1 included
        sweeps = [("Izhikevich 4:1 network: recurrent scale, E spiking",
                   netgen.izhikevich_calibration_config(np.arange(100.0, 1001.0, 50.0), gi, steps=args.steps))]
        workload = ("Izhikevich calibration sweep (Section 5.1): nConn 100..1000 step 50 x 26 recurrent scales "
                    "10^-1.5..10^1; 800 E + 200 I Izhikevich neurons, 1000 Poisson inputs at 20 Hz (p 0.1)")
    else:
        n_pn = np.arange(100, 1001, 50)
        sweeps = [(f"LHI variant, {nl} LHI: PN->{sw.upper()} scale, {sw.upper()} spiking",
                   netgen.mushroom_body_calibration_config(n_pn, gs, swept=sw, n_lhi=nl, n_kc=1000, n_dn=100,
                                                           ref_n_pn=100, steps=args.steps))
                  for nl in (20, 40) for sw in ("kc", "lhi")]
        workload = ("LHI-variant calibration sweeps: PN 100..1000 step 50 x 25 scales in [0.1, 10]; PN Poisson at "
                    "20 Hz, LHI 20 or 40, KC 1000, DN 100 HH; PN->KC p 0.2, PN->LHI p 0.5; PN->KC and PN->LHI "
                    "scale each swept")
    out, total_ns, total_ms, roof, launch = [], 0.0, 0.0, None, None
    for label, spec in sweeps:
        ref = cal.reference_run(spec, spec["n_conn"][0], 1.0)
        n_hh = sum(p["n"] for inst in spec["instances"] for p in inst["pops"] if p["kind"] == "hh")
        n_state = sum(p["n"] for inst in spec["instances"] for p in inst["pops"] if p["kind"] != "poisson")
        n_syn = sum(int(np.asarray(q["col_idx"]).size) for inst in spec["instances"] for q in inst["projs"])
        t_make = time.perf_counter()
        net = snn.Network(spec, autotune=bool(args.autotune), tune_cache=args.tune_cache)
        t_make = time.perf_counter() - t_make
        stream = torch.cuda.current_stream()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        net.step(args.steps)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1)
        t_fit = time.perf_counter()
        res = cal.calibrate(net, spec, ref)
        t_fit = time.perf_counter() - t_fit
        if roof is None:
            # after the table is read: the profiled steps continue the runs
            roof = live_roofline(net, spec, n_hh, out_degree_table(spec), args.profile_steps,
                                 "calibration_sweep" if args.model == "layered" else None)
            launch = net.launch
        net.close()
        total_ns += n_state * args.steps
        total_ms += ms
        out.append({"sweep": label, "runs": len(spec["instances"]), "neurons": n_state, "synapses": n_syn,
                    "sweep_ms": ms, "ms_per_step": ms / args.steps, "create_s": t_make,
                    "table_select_fit_ms": t_fit * 1e3,
                    "reference": {"n_conn": spec["n_conn"][0], "g_scale": 1.0,
                                  "avg_spike": float(res["avg_spike"][ref])},
                    "n_nans_total": int(res["n_nans"].sum()),
                    "points": [[float(x), float(res["g_scale"][i]) if i >= 0 else None]
                               for x, i in zip(res["groups"], res["picked"])],
                    "k": [float(v) for v in res["k"]], "mape_percent": res["mape"]})
    rec = {"metric": "calibration sweep (Fig. 1) neuron-steps/s", "value": total_ns / (total_ms * 1e-3),
           "unit": "neuron-steps/s", "higher_is_better": True, "n_gpus": 1, "steps": args.steps,
           "dtype": "f64", "data": "synthetic", "config": {"workload": workload, "sweeps": len(sweeps)},
           "sweeps": out, "launch": launch, "roofline": roof}
    if not args.no_cpu:
        from oracle import oracle
        spec = sweeps[0][1]
        mid = len(spec["instances"]) // 2
        inst = spec["instances"][mid]
        orc = oracle.OracleNet(inst)
        nh = sum(p["n"] for p in inst["pops"] if p["kind"] != "poisson")
        t0, steps = time.perf_counter(), 0
        while time.perf_counter() - t0 < args.cpu_seconds:
            orc.step(50)
            steps += 50
        dt = time.perf_counter() - t0
        rec["cpu_baseline"] = {"value": nh * steps / dt, "unit": "neuron-steps/s", "cores": 1, "kind": "oracle",
                               "sample": f"one run of the first sweep (nConn {spec['n_conn'][mid]:.0f}), "
                                         f"{steps} steps, {dt:.1f} s"}
    print(json.dumps(rec), flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=100)
    ap.add_argument("--preroll", type=int, default=1000,
                    help="untimed steps before the warmup that leave the start-up transient of a network at rest")
    ap.add_argument("--workload", type=int, default=4)
    ap.add_argument("--instances", type=int, default=None, help="trim a batched workload")
    ap.add_argument("--autotune", type=int, default=1)
    ap.add_argument("--tune-cache", default=None,
                    help="JSON file of tuned launch shapes per network signature (read, and written after tuning)")
    ap.add_argument("--cpu-seconds", type=float, default=24.0, help="budget of the oracle sample")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-sweep", action="store_true",
                    help="leave out the forced-activity delivery points of a batched workload's line")
    ap.add_argument("--profile-steps", type=int, default=500)
    ap.add_argument("--sweep", action="store_true",
                    help="forced-activity sweep of the propagation kernel instead of the step benchmark")
    ap.add_argument("--sweep-workload", type=int, default=3)
    ap.add_argument("--loop", type=int, default=None,
                    help="1: also time every instance alone on the same kernels (per-instance loop); "
                         "default: on for batched workloads")
    ap.add_argument("--adjoint", action="store_true",
                    help="time the recorded forward + reverse pass (gradient) instead of plain steps")
    ap.add_argument("--ckpt-every", type=int, default=100)
    ap.add_argument("--calibrate", action="store_true",
                    help="the calibration of Fig. 1: (nConn, gScale) sweep, selection and law fit")
    ap.add_argument("--model", choices=("layered", "lhi", "izh"), default="layered",
                    help="calibration network: the layered model, its LHI variant (two swept scales), or the "
                         "4:1 Izhikevich network")
    ap.add_argument("--sources-sha", action="store_true", help="print the kernel sources hash and exit")
    ap.add_argument("--calib-copy", type=int, default=0,
                    help="MiB of a plain device copy to run first (counter calibration)")
    return ap.parse_args()


def out_degree_table(spec):
    """Per instance, per population: total outgoing row length of each neuron."""
    import numpy as np
    tabs = []
    for inst in spec["instances"]:
        t = [np.zeros(p["n"], np.int64) for p in inst["pops"]]
        for q in inst["projs"]:
            t[q["pre"]] += np.diff(np.asarray(q["row_ptr"], np.int64))
        tabs.append(t)
    return tabs


def spike_totals(net, spec):
    import numpy as np
    return [[net.spikes(b, p).astype(np.int64) for p in range(len(inst["pops"]))]
            for b, inst in enumerate(spec["instances"])]


def copy_bandwidth(nbytes=1 << 30, reps=10):
    """Achievable device-to-device copy bandwidth on this GPU (bytes read plus
    bytes written per second), the practical ceiling a streaming kernel is
    compared with besides the HBM peak."""
    import torch
    a = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    b = torch.empty_like(a)
    for _ in range(2):
        b.copy_(a)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        b.copy_(a)
    e1.record()
    torch.cuda.synchronize()
    gbs = 2 * nbytes * reps / (e0.elapsed_time(e1) * 1e-3) / 1e9
    del a, b
    torch.cuda.empty_cache()
    return gbs


def sweep_points(spec, fractions, configs, seed=7):
    """Propagation alone on a network's connectivity with seeded synthetic
    spike sets: every input (A) row and a fraction of the hidden (B) rows
    spiking, C silent, plasticity off (pure delivery); one hipEvent pair
    around back-to-back launches of one step's delivery per launch shape."""
    import numpy as np
    from paper_1412_0595_amd import netgen, snn
    spec = dict(spec, instances=[dict(inst, projs=[dict(q, stdp=None) for q in inst["projs"]])
                                 for inst in spec["instances"]])
    net = snn.Network(spec, autotune=False)
    rng = np.random.default_rng(seed)
    deg = out_degree_table(spec)
    out = []
    for frac in fractions:
        ev = rows = 0
        for b, inst in enumerate(spec["instances"]):
            n_a, n_b = inst["pops"][0]["n"], inst["pops"][1]["n"]
            fa = np.ones(n_a, np.uint8)
            fb = np.zeros(n_b, np.uint8)
            fb[netgen.forced_spikes(rng, n_b, frac)] = 1
            net.set_last_spikes(b, 0, fa)
            net.set_last_spikes(b, 1, fb)
            net.set_last_spikes(b, 2, np.zeros(inst["pops"][2]["n"], np.uint8))
            ev += int(deg[b][0].sum() + deg[b][1][fb.astype(bool)].sum())
            rows += n_a + int(fb.sum())
        for L in configs:
            net.set_launch(**L)
            launches = 20 if ev > 1e7 else 200
            ms = net.time_kernel(0, launches)
            byt = PROP_BYTES_PER_EVENT * ev + PROP_BYTES_PER_ROW * rows
            gbs = byt / (ms * 1e-3) / 1e9
            out.append({"hidden_fraction": frac, "events_per_launch": ev, "rows": rows, "ms_per_launch": ms,
                        "launch": net.launch, "events_per_s": ev / (ms * 1e-3), "achieved_GBs": gbs,
                        "frac_of_hbm": gbs / HBM_PEAK_GBS})
    net.close()
    return out


def sweep(args):
    """Forced-activity sweep of the propagation on a workload's connectivity
    (every input row and 0.1 / 1 / 10 / 100% of the hidden rows spiking), in
    both delivery modes and several launch shapes; one JSON line per point."""
    from paper_1412_0595_amd import netgen
    copy_gbs = copy_bandwidth()
    print(json.dumps({"sweep": "copy", "bytes": 1 << 30, "copy_GBs": copy_gbs,
                      "frac_of_hbm": copy_gbs / HBM_PEAK_GBS}), flush=True)
    spec = netgen.make_config(args.sweep_workload, n_instances=args.instances)
    configs = (dict(mode=0, prop_blocks=1024, prop_block=256), dict(mode=0, prop_blocks=4096, prop_block=256),
               dict(mode=1, prop_blocks=1024), dict(mode=1, prop_blocks=2048), dict(mode=1, prop_blocks=4096))
    for pt in sweep_points(spec, (0.001, 0.01, 0.1, 1.0), configs):
        print(json.dumps(dict({"sweep": "propagation", "workload": args.sweep_workload}, **pt,
                              frac_of_copy=pt["achieved_GBs"] / copy_gbs)), flush=True)


def note(msg):
    """Progress line on stderr (the result stays the one JSON line on stdout)."""
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def host_cpu():
    """Cores this process may use (capped at 16, the host share of one GPU)
    and the CPU model, read from the OS."""
    try:
        avail = len(os.sched_getaffinity(0))
    except AttributeError:
        avail = os.cpu_count() or 1
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"nproc": os.cpu_count(), "affinity": avail, "threads": max(1, min(16, avail)), "cpu_model": model}


def cpu_baseline(spec, seconds, max_instances=32):
    """The FP64 oracle on the host cores, on a bounded sample of the same
    workload: up to `max_instances` instances spread over the batch (all of a
    single-instance workload), S steps each.  Single-thread runs step the
    sample serially; all-core runs step the instances on a thread pool (a
    batch) or run the neuron loop on OpenMP threads (one instance).  Median
    of 3 runs each; S is sized so that the six runs take about `seconds`."""
    import numpy as np
    from oracle import oracle as O
    hc = host_cpu()
    n_inst = len(spec["instances"])
    pick = sorted(set(np.linspace(0, n_inst - 1, min(max_instances, n_inst)).round().astype(int).tolist()))
    nets = [O.OracleNet(spec["instances"][k]) for k in pick]
    n_hh = sum(p["n"] for k in pick for p in spec["instances"][k]["pops"] if p["kind"] == "hh")
    deg = out_degree_table(dict(instances=[spec["instances"][k] for k in pick]))
    t0 = time.perf_counter()
    O.step_many(nets, 5, 1)
    per_step = (time.perf_counter() - t0) / 5
    S = int(min(2000, max(10, seconds / 3.0 / 2.0 / per_step)))

    def counts():
        return [[net.counts(p).astype(np.int64) for p in range(len(net.pops))] for net in nets]

    def run(threads):
        if len(nets) == 1:
            nets[0].set_threads(threads)
        c0 = counts()
        t = time.perf_counter()
        O.step_many(nets, S, threads if len(nets) > 1 else 1)
        el = time.perf_counter() - t
        c1 = counts()
        ev = sum(int(((c1[b][p] - c0[b][p]) * deg[b][p]).sum()) for b in range(len(nets)) for p in range(len(c0[b])))
        return n_hh * S / el, ev / el

    single = sorted(run(1) for _ in range(3))
    multi = sorted(run(hc["threads"]) for _ in range(3))
    for net in nets:
        net.set_threads(1)
    how = ("instances on a thread pool" if len(nets) > 1 else "neuron loop on OpenMP threads")
    return {"value": multi[1][0], "unit": "neuron-steps/s", "cores": hc["threads"], "kind": "oracle",
            "sample": f"{len(nets)} of {n_inst} instances ({n_hh} HH neurons), {S} steps per run after 5, "
                      f"median of 3 runs; all-core: {how}",
            "synaptic_events_per_s": multi[1][1],
            "single_thread": {"value": single[1][0], "synaptic_events_per_s": single[1][1], "cores": 1},
            "runs_neuron_steps_per_s": {"all_core": [r[0] for r in multi], "single": [r[0] for r in single]},
            "host": hc}


def neuron_alg_bytes(spec):
    """Algorithmic bytes of one neuron-update launch: per Traub-Miles neuron,
    V, m, h, n (fp32) read and written, the V compensation word read and
    written, and each incoming projection's fp32 conductance read and written."""
    tot = 0
    for inst in spec["instances"]:
        for k, p in enumerate(inst["pops"]):
            if p["kind"] == "poisson":
                continue
            n_in = sum(1 for q in inst["projs"] if q["post"] == k)
            own = (NEURON_ALG_STATE_BYTES + NEURON_ALG_VLO_BYTES) if p["kind"] == "hh" else NEURON_ALG_IZH_BYTES
            tot += p["n"] * (own + NEURON_ALG_G_BYTES * n_in)
    return tot


def step_bench(args):
    import numpy as np
    import torch
    from paper_1412_0595_amd import netgen, snn

    t_gen = time.perf_counter()
    spec = netgen.make_config(args.workload, n_instances=args.instances)
    t_gen = time.perf_counter() - t_gen
    n_hh = sum(p["n"] for inst in spec["instances"] for p in inst["pops"] if p["kind"] == "hh")
    n_syn = sum(int(np.asarray(q["col_idx"]).size) for inst in spec["instances"] for q in inst["projs"])
    note(f"workload {args.workload}: {len(spec['instances'])} instances, {n_hh} HH neurons, {n_syn} synapses "
         f"drawn in {t_gen:.1f} s")
    t_make = time.perf_counter()
    net = snn.Network(spec, autotune=bool(args.autotune), tune_cache=args.tune_cache)
    t_make = time.perf_counter() - t_make
    note(f"created (autotune {args.autotune}) in {t_make:.1f} s: launch {net.launch}")
    stream = torch.cuda.current_stream()

    # untimed: the pre-roll leaves the start-up transient of a network started
    # at rest; the warmup steps follow; one untimed run of the timed length
    # captures the graphs the timed run replays
    net.step(args.preroll)
    net.step(args.warmup)
    net.step(args.steps)
    net.sync()
    t_start = net.t
    deg = out_degree_table(spec)
    c0 = spike_totals(net, spec)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t_wall = time.perf_counter()
    e0.record(stream)
    net.step(args.steps)
    e1.record(stream)
    torch.cuda.synchronize()
    t_wall = time.perf_counter() - t_wall
    net.sync()
    ms = e0.elapsed_time(e1)
    c1 = spike_totals(net, spec)
    events = 0
    spikes = 0
    for b in range(len(spec["instances"])):
        for p in range(len(c0[b])):
            d = c1[b][p] - c0[b][p]
            spikes += int(d.sum())
            events += int((d * deg[b][p]).sum())
    nan_total = int(net.nan_counts().sum())
    sec = ms * 1e-3
    neuron_steps = n_hh * args.steps / sec
    events_s = events / sec

    note(f"timed {args.steps} steps: {ms / args.steps * 1e3:.2f} us per step")
    roof = live_roofline(net, spec, n_hh, deg, args.profile_steps, args.workload)
    note(f"profiled {args.profile_steps} live steps: {roof['ms_per_launch']}")
    launch = net.launch
    net.close()

    rec = {
        "metric": "neuron-steps/s + synaptic events/s (1 GPU); batched/adjoint vs plain loop",
        "value": neuron_steps,
        "unit": "neuron-steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": WORKLOADS.get(args.workload, f"workload {args.workload}"),
                   "instances": len(spec["instances"]), "hh_neurons": n_hh, "synapses": n_syn,
                   "preroll_steps": args.preroll,
                   "timed_steps_start_at": t_start,
                   "untimed_before_timed": "pre-roll (leaves the rest transient), warmup, and one run of the "
                                           "timed length that captures the replayed graphs",
                   "timed_region": "captured hipGraphs of whole steps (64-step graphs and one of the remainder); "
                                   "resident launches of many steps for a network that fits"},
        "synaptic_events_per_s": events_s,
        "spikes": spikes,
        "nan_neurons_total": nan_total,
        "wall_s": t_wall,
        "netgen_s": t_gen,
        "create_s": t_make,
        "launch": launch,
        "roofline": roof,
    }
    if args.loop is None:
        args.loop = len(spec["instances"]) > 1
    if args.loop and len(spec["instances"]) > 1:
        note("per-instance loop")
        loop_ms, loop_events = time_loop(spec, args.steps, args.preroll + args.warmup, args.tune_cache)
        note(f"per-instance loop: {loop_ms:.2f} ms for {args.steps} steps")
        rec["per_instance_loop"] = {"ms": loop_ms, "neuron_steps_per_s": n_hh * args.steps / (loop_ms * 1e-3),
                                    "synaptic_events_per_s": loop_events / (loop_ms * 1e-3),
                                    "batched_speedup": loop_ms / ms,
                                    "how": "every instance alone on the same kernels (autotuned, graphs), "
                                           "one after the other, same pre-roll and step count; step time only"}
    if len(spec["instances"]) > 1 and not args.no_sweep:
        # the propagation target (>= 60% of HBM peak) on this workload's own
        # connectivity: forced activity at the 10% and 100% hidden points
        note("forced-activity delivery on this workload's connectivity")
        pts = sweep_points(spec, (0.1, 1.0), (dict(mode=1, prop_blocks=4096),))
        rec["propagation_sweep"] = {
            "how": "every input row and a seeded fraction of the hidden rows spiking, one step's delivery timed "
                   "20 times back to back (hipEvent pair), tile mode with pull, 4096 blocks; bytes are the "
                   "method's CSR bytes, 8 B per synaptic event + 16 B per spiking row",
            "points": [{"hidden_fraction": p["hidden_fraction"], "events_per_launch": p["events_per_launch"],
                        "ms_per_launch": round(p["ms_per_launch"], 6), "achieved_GBs": round(p["achieved_GBs"], 1),
                        "frac_of_hbm": round(p["frac_of_hbm"], 4)} for p in pts]}
    if not args.no_cpu:
        note("oracle sample on the host cores")
    rec["cpu_baseline"] = None if args.no_cpu else cpu_baseline(spec, args.cpu_seconds)
    print(json.dumps(rec), flush=True)


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU only; multi-GPU sharding is a design note",
                          "n_gpus": args.gpus}))
        sys.exit(2)
    if args.sources_sha:
        print(kernel_sources_sha256())
        return
    if args.calib_copy:
        import torch
        a = torch.ones(args.calib_copy * (1 << 18), dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        del a, b
    if args.sweep:
        sweep(args)
        return
    if args.adjoint:
        adjoint_bench(args)
        return
    if args.calibrate:
        calibrate_bench(args)
        return
    step_bench(args)


if __name__ == "__main__":
    main()
