"""Benchmark: makespan and inferences/s of the attention DAG under coarse- and fine-grained
schedules on one MI355X, BF16 beside FP32, with a roofline figure for the dominant kernel and the
CPU oracle's throughput beside it.

Default workload (--config mha1024x12): 12 stacked multi-head attention layers, n = d_model = 1024,
16 heads of dim 64, BF16 GEMM operands with FP32 accumulation, FP32 softmax input (1,356 kernels:
per layer and head three projection GEMMs, a transpose, the score GEMM, a row softmax and the P*V
GEMM; then the output projection).  A step is one pass of the whole DAG over device-resident inputs
(``value``); the makespan from the first upload to the last read-back (inputs and weights from
page-locked memory) is reported beside it for every schedule.  ``value`` is inferences/s of the
fine-grained schedule the schedule autotuner picks among stream counts, mappers (clustering: one
task component per head on a stream; round robin), enqueue threads and the two dispatchers (AQL
packets on the GPU's own HSA queues with barrier-AND packets on completion signals, or HIP streams
and events).  The coarse schedule (one in-order queue) is timed with both dispatchers; the device
executor (one persistent kernel) is reported as a separate row, never as ``value``.  The same DAG
with FP32 GEMMs is timed after it (``fp32_same_dag``).  GEMM tiles are autotuned first.

--config mha512: one layer, n = d = 512, 8 heads, FP32 (57 kernels).
--config kernels: standalone softmax / transpose / add against HBM bandwidth and GEMMs against the
matrix-core peak, at large sizes.
--config batch64: 64 instances of log-uniform length, 6 layers, BF16 (21,888 kernels), inferences/s
and per-instance latency p50/p99, eager streams vs one hipGraph, untuned vs autotuned.
--config costmodel: the learned cost model at full scale.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--config mha1024x12|mha512|batch64|kernels|costmodel]
"""
import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK = {"mfma_f32": 157.3e12, "mfma_bf16": 2.5e15, "hbm": 8.0e12}


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=None)
    p.add_argument("--warmup", type=int, default=None)
    p.add_argument("--config", default="mha1024x12")
    p.add_argument("--no-fp32", action="store_true", help="skip the FP32 run of the 12-layer DAG")
    p.add_argument("--streams", type=int, default=4)
    p.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    p.add_argument("--no-tune", action="store_true", help="skip the GEMM tile autotuner")
    p.add_argument("--cpu-seconds", type=float, default=10.0)
    p.add_argument("--graph", action="store_true", help="also time the schedule launched as one hipGraph")
    p.add_argument("--variants", action="store_true", help="also time other fine-grained variants")
    p.add_argument("--kernel-iters", type=int, default=200)
    p.add_argument("--heldout", type=int, default=20, help="--config costmodel: held-out DAGs")
    p.add_argument("--epochs", type=int, default=100, help="--config costmodel: training passes")
    p.add_argument("--dump-samples", default=None, help="--config costmodel: save the samples (.npz)")
    p.add_argument("--kernel-profile", choices=["dominant", "executor", "timeline"], default=None,
                   help="launch sequence for rocprofv3 runs (no timing line): the dominant kernel of the "
                        "stream schedule, or the device executor, then a calibration copy; or "
                        "(timeline) runs of one fine schedule, device-resident and with host copies")
    p.add_argument("--fine-opts", default=None,
                   help="--kernel-profile timeline: the fine schedule's options as JSON (default: "
                        "the schedule autotuner's choice)")
    p.add_argument("--profile-tile", type=int, default=0,
                   help="with --kernel-profile: GEMM tile of the shape --profile-shape (0 = autotune)")
    p.add_argument("--profile-shape", default="512x64x512", help="MxNxK pinned by --profile-tile")
    p.add_argument("--gemm-tile", type=int, default=0,
                   help="--config kernels: run the large GEMMs (above 1e10 MNK) on this tile, untuned")
    a = p.parse_args()
    big = a.config in ("mha1024x12", "batch64")
    if a.steps is None:
        a.steps = {"mha1024x12": 50, "batch64": 5}.get(a.config, 300)
    if a.warmup is None:
        a.warmup = 2 if a.config == "batch64" else (5 if big else 30)
    return a


def workload(name):
    import workloads
    if name == "forkjoin":
        spec = workloads.forkjoin_spec(256)
        return spec, workloads.forkjoin_inputs(0, 256), {"workload": "fork-join DAG (Fig. 1 shape), 3 GEMMs 256^3 + add, FP32",
                                                         "gemm_dtype": "f32"}
    if name == "mha512":
        n, d, h, L, dt = 512, 512, 8, 1, "f32"
    elif name == "mha1024x12":
        n, d, h, L, dt = 1024, 1024, 16, 12, "bf16"
    else:
        raise SystemExit(f"unknown config {name}")
    spec = workloads.mha_spec(n, d, h, L, gemm_dtype=dt)
    inp = workloads.mha_inputs(0, n, d, L)
    desc = {"workload": f"multi-head attention inference DAG, {L} layer(s), n={n}, d_model={d}, "
                        f"{h} heads of dim {d // h}, GEMM {dt.upper()}" + (" (FP32 accumulation)" if dt == "bf16" else ""),
            "seq_len": n, "d_model": d, "heads": h, "layers": L, "gemm_dtype": dt,
            "kernels": len(spec["kernels"])}
    return spec, inp, desc


def kernel_class(spec, k):
    by = {b["name"]: b for b in spec["buffers"]}
    ker = spec["kernels"][k]
    ins = [by[b] for b in ker["inputs"]]
    out = by[ker["outputs"][0]]
    if ker["kind"] == "gemm":
        m, kk, n = ins[0]["rows"], ins[0]["cols"], ins[1]["cols"]
        return (f"gemm {m}x{n}x{kk} {ins[0]['dtype']}->{out['dtype']}",
                2.0 * m * n * kk, "mfma", ins[0]["dtype"])
    es = {"f32": 4, "bf16": 2}
    nbytes = sum(b["rows"] * b["cols"] * es[b["dtype"]] for b in ins) + out["rows"] * out["cols"] * es[out["dtype"]]
    shape = "x".join(str(v) for v in (ins[0]["rows"], ins[0]["cols"]))
    return (f"{ker['kind']} {shape} {ins[0]['dtype']}->{out['dtype']}", float(nbytes), "hbm", None)


def gemm_bytes(spec, k):
    """Algorithmic bytes of a GEMM: A, B and C each moved once."""
    by = {b["name"]: b for b in spec["buffers"]}
    ker = spec["kernels"][k]
    es = {"f32": 4, "bf16": 2}
    return float(sum(b["rows"] * b["cols"] * es[b["dtype"]] for b in [by[n] for n in ker["inputs"] + ker["outputs"]]))


def timed(runner, steps, warmup):
    import paper_2009_07482_amd as psc
    for _ in range(warmup):
        runner.run(with_inputs=False, with_outputs=False)
    psc.psc_device_sync(0)
    mk = []
    t0 = time.perf_counter()
    for _ in range(steps):
        st = runner.run(with_inputs=False, with_outputs=False)
        mk.append(st["makespan_ms"])
    psc.psc_device_sync(0)
    wall = time.perf_counter() - t0
    return wall, np.array(mk), st


def cpu_baseline(spec, inp, seconds):
    from oracle import dag as odag
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count() or 1
    n = 0
    t0 = time.perf_counter()
    while True:
        odag.run_dag(spec, inp)
        n += 1
        el = time.perf_counter() - t0
        if el >= seconds or n >= 1000:
            break
    return {"value": n / el, "unit": "inferences/s", "cores": int(cores), "kind": "oracle",
            "sample": f"{n} full run(s) of the same DAG in FP64 (numpy), {el:.1f} s"}


def overlap(times):
    """Mean number of ops in flight over the busy time of a per-op timeline."""
    ivals = sorted((t[2], t[3]) for t in times if t[3] > t[2])
    busy, cs, ce = 0.0, None, None
    for s0, e0 in ivals:
        if ce is None or s0 > ce:
            if ce is not None:
                busy += ce - cs
            cs, ce = s0, e0
        else:
            ce = max(ce, e0)
    if ce is not None:
        busy += ce - cs
    return sum(e - s for s, e in ivals) / busy if busy > 0 else 0.0


def dominant_roofline(spec, r, kernel_iters):
    """Dominant kernel: per kernel class, the mean duration of back-to-back launches on the
    class's own stream (HIP events around the launches, on that stream) times its launches per
    step; the class with the largest product dominates the step."""
    import paper_2009_07482_amd as psc
    kers = {}
    for k in range(len(spec["kernels"])):
        key, work, bound, dt = kernel_class(spec, k)
        kers.setdefault(key, {"work": work, "bound": bound, "dtype": dt, "ids": []})["ids"].append(k)
    for key, c in kers.items():
        psc.psc_kernel_time(r.sched, c["ids"][0], 10)
        c["avg_us"] = psc.psc_kernel_time(r.sched, c["ids"][0], kernel_iters)
        c["total_us"] = c["avg_us"] * len(c["ids"])
        if c["bound"] == "mfma":
            c["tile"] = psc.psc_sched_kernel_tile(r.sched, c["ids"][0])
    print("# kernel classes (isolated mean us per launch x launches per step), top 12:", file=sys.stderr)
    for key, c in sorted(kers.items(), key=lambda kv: -kv[1]["total_us"])[:12]:
        print(f"#   {key}: {c['avg_us']:.2f} us x {len(c['ids'])}" + (f" (tile {c['tile']})" if "tile" in c else ""),
              file=sys.stderr)
    dom_key = max(kers, key=lambda k: kers[k]["total_us"])
    dom = kers[dom_key]
    avg_us = dom["avg_us"]
    achieved = dom["work"] / (avg_us * 1e-6)
    extra = {}
    bound = dom["bound"]
    if bound == "mfma":
        # a GEMM whose arithmetic intensity is below the ridge (matrix-core peak / HBM bandwidth)
        # is bound by memory on the roofline: reported in bytes, with the FLOP rate beside it
        peak = PEAK["mfma_bf16"] if dom["dtype"] == "bf16" else PEAK["mfma_f32"]
        nbytes = gemm_bytes(spec, dom["ids"][0])
        ai = dom["work"] / nbytes
        extra = {"flop_per_byte": ai, "ridge_flop_per_byte": peak / PEAK["hbm"],
                 "mfma_tflops": achieved / 1e12, "mfma_frac": achieved / peak}
        if ai < peak / PEAK["hbm"]:
            bound, achieved, dom = "hbm", nbytes / (avg_us * 1e-6), dict(dom, work=nbytes)
    if bound == "mfma":
        roof = {"bound": "mfma", "achieved": achieved / 1e12, "peak": peak / 1e12, "unit": "TFLOP/s",
                "frac": achieved / peak, "traffic": None}
    else:
        roof = {"bound": "hbm", "achieved": achieved / 1e9, "peak": PEAK["hbm"] / 1e9, "unit": "GB/s",
                "frac": achieved / PEAK["hbm"], "traffic": None}
    roof.update(extra)
    roof.update({"kernel": dom_key, "avg_us": avg_us, "launches_per_step": len(dom["ids"]),
                 "work_per_launch": dom["work"], "tile": dom.get("tile"),
                 "timing": f"{kernel_iters} back-to-back launches, HIP events on its stream"})
    roof["traffic"] = stored_traffic(dom_key, dom.get("tile"))
    return roof


CAL_N = 4096   # calibration: an FP32 4096 x 4096 transpose reads and writes 64 MiB each


def source_digest(executor=False):
    """Hash of the kernel sources; a stored counter profile applies only to the code it measured:
    the standalone kernels' sources, and for the device executor also its own and the runtime that
    plans its task lists."""
    import hashlib
    h = hashlib.sha256()
    files = ("tiles.hpp", "kernels.hip", "kernels.hpp")
    if executor:
        files += ("persistent.hip", "persistent.hpp", "runtime.cpp")
    for f in files:
        with open(os.path.join(ROOT, "paper_2009_07482_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def kernel_profile(a):
    """Dispatches for hardware-counter runs (rocprofv3 --pmc): the profiled kernel 100 times, then
    the calibration transpose 20 times; prints which kernel (name, grid) to read."""
    import paper_2009_07482_amd as psc
    import workloads
    spec, inp, desc = workload(a.config)
    if not a.no_tune:
        d0 = psc.build_dag(spec)
        psc.psc_autotune_dag(d0, iters=20)
        psc.psc_dag_destroy(d0)
    info = {"config": a.config, "target": a.kernel_profile, "source_digest": source_digest(a.kernel_profile == "executor")}
    if a.profile_tile:
        # every counter pass must profile the same kernel instance: pin the tile of every GEMM
        # shape whose autotuned choice would otherwise vary from run to run
        by = {b["name"]: b for b in spec["buffers"]}
        for k in spec["kernels"]:
            if k["kind"] == "gemm":
                A_, B_, C_ = by[k["inputs"][0]], by[k["inputs"][1]], by[k["outputs"][0]]
                if (A_["rows"], B_["cols"], A_["cols"]) == tuple(int(v) for v in a.profile_shape.split("x")):
                    psc.psc_tile_cache_set(A_["rows"], B_["cols"], A_["cols"], A_["dtype"], C_["dtype"], a.profile_tile)
    if a.kernel_profile == "executor":
        # --fine-opts may set the executor's options (e.g. {"exec_per_cu": 1})
        r = psc.SpecRunner(spec, "device", **(json.loads(a.fine_opts) if a.fine_opts else {}))
        r.set_inputs(inp)
        r.run()
        for _ in range(100):
            r.run(with_inputs=False, with_outputs=False)
        w, pcu, grp = psc.psc_sched_executor_info(r.sched)
        info.update({"kernel": "exec_kernel (whole DAG, one launch)", "match": "exec_kernel",
                     "work_per_launch": workloads.spec_flops(spec), "launches": 100,
                     "executor": {"workers": w, "per_cu": pcu, "groups": grp}})
    else:
        r = psc.SpecRunner(spec, "fine", n_streams=4, mapper="component")
        r.set_inputs(inp)
        r.run()
        kers = {}
        for k in range(len(spec["kernels"])):
            key, work, bound, dt = kernel_class(spec, k)
            kers.setdefault(key, {"work": work, "ids": []})["ids"].append(k)
        for c in kers.values():
            c["total"] = psc.psc_kernel_time(r.sched, c["ids"][0], 20) * len(c["ids"])
        key = max(kers, key=lambda k: kers[k]["total"])
        kid = kers[key]["ids"][0]
        psc.psc_kernel_time(r.sched, kid, 100)
        info.update({"kernel": key, "kernel_id": kid, "tile": psc.psc_sched_kernel_tile(r.sched, kid)
                     if spec["kernels"][kid]["kind"] == "gemm" else None, "work_per_launch": kers[key]["work"],
                     "launches": 100})
    r.close()
    import numpy as np
    cal = {"buffers": [{"name": "A", "dtype": "f32", "rows": CAL_N, "cols": CAL_N, "view_of": None, "row_off": 0, "col_off": 0},
                       {"name": "C", "dtype": "f32", "rows": CAL_N, "cols": CAL_N, "view_of": None, "row_off": 0, "col_off": 0}],
           "kernels": [{"name": "cal", "kind": "transpose", "inputs": ["A"], "outputs": ["C"], "alpha": 1.0, "tile": 0}],
           "edges": [], "component": [0]}
    c = psc.SpecRunner(cal, "coarse")
    c.set_inputs({"A": np.zeros((CAL_N, CAL_N), np.float32)})
    c.run()
    psc.psc_kernel_time(c.sched, 0, 20)
    c.close()
    info["calibration"] = {"kernel": f"transpose {CAL_N}x{CAL_N} f32", "match": "transpose",
                           "grid": (CAL_N // 64) * (CAL_N // 64), "read_bytes": CAL_N * CAL_N * 4,
                           "write_bytes": CAL_N * CAL_N * 4, "launches": 20}
    print(json.dumps(info), flush=True)


def timeline_profile(a):
    """Runs for a kernel and memory-copy trace of one fine schedule: 3 device-resident runs, then
    3 runs that upload the inputs and weights and read the output back (page-locked memory)."""
    import paper_2009_07482_amd as psc
    spec, inp, desc = workload(a.config)
    if not a.no_tune:
        d0 = psc.build_dag(spec)
        psc.psc_autotune_dag(d0, iters=20)
        psc.psc_dag_destroy(d0)
    if a.fine_opts:
        opts = dict(json.loads(a.fine_opts), copy_roots=True)   # may name a "policy" (default fine)
    else:
        d1 = psc.build_dag(spec)
        bi, _ = psc.psc_autotune_schedule(d1, "fine", FINE_CANDIDATES, iters=5)
        psc.psc_dag_destroy(d1)
        opts = FINE_CANDIDATES[bi]
    policy = opts.pop("policy", "fine")
    # the device executor runs its copies inside its one kernel: a kernel trace shows one launch,
    # so its per-op device clocks are recorded and summarised instead
    r = psc.SpecRunner(spec, policy, **opts, **({"record_ops": True} if policy == "device" else {}))
    r.set_inputs(inp)
    r.run()
    res = {"resident_ms": [], "with_copies_ms": []}
    for _ in range(3):
        res["resident_ms"].append(r.run(with_inputs=False, with_outputs=False)["makespan_ms"])
    for _ in range(3):
        res["with_copies_ms"].append(r.run()["makespan_ms"])
    if policy == "device":
        # the last run with copies: per-op start/end (us from the executor's reset) by type
        ops = psc.psc_sched_export(r.sched)
        t = {o: (a_, b_) for (o, _, a_, b_) in psc.psc_sched_op_times(r.sched)}
        iv = {k: [t[o["id"]] for o in ops if o["type"] == k and t[o["id"]][1] > 0] for k in ("h2d", "kernel", "d2h")}
        ups, kers = iv["h2d"], iv["kernel"]
        res["device_ops"] = {
            "uploads": len(ups), "upload_span_us": [min(u[0] for u in ups), max(u[1] for u in ups)] if ups else None,
            "kernel_span_us": [min(k[0] for k in kers), max(k[1] for k in kers)],
            "kernels_started_before_last_upload_ended": sum(1 for k in kers if ups and k[0] < max(u[1] for u in ups)),
            "upload_kernel_overlapping_pairs": sum(1 for u in ups for k in kers if u[0] < k[1] and k[0] < u[1]),
            "readback_span_us": [min(d[0] for d in iv["d2h"]), max(d[1] for d in iv["d2h"])] if iv["d2h"] else None}
        res["executor"] = dict(zip(("workers", "per_cu", "groups"), psc.psc_sched_executor_info(r.sched)))
    r.close()
    print(json.dumps({"config": a.config, "target": "timeline", "policy": policy, "fine_opts": opts,
                      "schedule": describe(opts) if policy == "fine" else policy,
                      "source_digest": source_digest(), **res}), flush=True)


def stored_traffic(kernel_key, tile):
    """HBM bytes per launch from a committed counter profile of this kernel (profiles/*.md),
    or None if there is none for this kernel, tile and kernel source."""
    import glob
    import re
    digest = source_digest(kernel_key.startswith("exec_kernel"))
    for f in sorted(glob.glob(os.path.join(ROOT, "profiles", "*.md"))):
        # one entry per block of "- key: `value`" lines (a file may hold several tiles)
        for block in re.split(r"\n\s*\n", open(f).read()):
            kv = dict(re.findall(r"^- (\w+): `([^`]*)`", block, re.M))
            if kv.get("kernel") == kernel_key and kv.get("source_digest") == digest and \
                    kv.get("tile", "None") == str(tile):
                try:
                    return float(kv["traffic_bytes_per_launch"])
                except (KeyError, ValueError):
                    return None
    return None


def environment():
    import paper_2009_07482_amd as psc
    env = {"device": psc.psc_device_info(0)}
    try:
        with open("/opt/rocm/.info/version") as fh:
            env["rocm"] = fh.read().strip()
    except OSError:
        pass
    return env


def dag_bound_us(spec):
    """Whole-DAG lower bound with every kernel at its roofline and no overlap lost: GEMM FLOPs at
    the matrix-core peak of their operand type plus the other kernels' bytes at HBM bandwidth."""
    t = 0.0
    for k in range(len(spec["kernels"])):
        _, work, bound, dt = kernel_class(spec, k)
        t += work / (PEAK["mfma_bf16"] if dt == "bf16" else PEAK["mfma_f32"]) if bound == "mfma" else work / PEAK["hbm"]
    return t * 1e6


def one_kernel(kind, shapes, dtypes, tile=0, alpha=1.0):
    names = ["A", "B"][: len(shapes) - 1] + ["C"]
    bufs = [{"name": n, "dtype": d, "rows": r, "cols": c, "view_of": None, "row_off": 0, "col_off": 0}
            for n, (r, c), d in zip(names, shapes, dtypes)]
    ker = {"name": "k", "kind": kind, "inputs": names[:-1], "outputs": ["C"], "alpha": alpha, "tile": tile}
    return {"buffers": bufs, "kernels": [ker], "edges": [], "component": [0]}


_LIBREF = r"""
import json, torch
out = []
for n in (4096, 8192):
    g = torch.Generator(device="cuda").manual_seed(0)
    a = (torch.rand((n, n), device="cuda", generator=g) * 2 - 1).to(torch.bfloat16)
    b = (torch.rand((n, n), device="cuda", generator=g) * 2 - 1).to(torch.bfloat16)
    for _ in range(5):
        c = a @ b
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    it = 50 if n == 4096 else 20
    e0.record()
    for _ in range(it):
        c = a @ b
    e1.record()
    torch.cuda.synchronize()
    us = e0.elapsed_time(e1) / it * 1e3
    out.append({"kernel": f"torch.matmul {n}x{n}x{n} bf16->bf16 (vendor library)", "avg_us": us,
                "achieved": 2 * n ** 3 / (us * 1e-6) / 1e12, "unit": "TFLOP/s", "peak": 2500.0,
                "frac": 2 * n ** 3 / (us * 1e-6) / 2.5e15})
print(json.dumps(out))
"""


def library_reference():
    """The vendor GEMM library (torch.matmul on hipBLASLt) on the same large BF16 shapes, random
    operands, in a child process (torch's HIP runtime cannot share this process): context for
    what the matrix cores sustain on this part, not a product path."""
    import subprocess
    try:
        r = subprocess.run([sys.executable, "-c", _LIBREF], capture_output=True, text=True, timeout=300)
        return json.loads(r.stdout.strip().splitlines()[-1]) if r.returncode == 0 else {"error": r.stderr[-300:]}
    except Exception as e:   # context only: report why it is missing
        return {"error": str(e)}


def kernels_main(a):
    """Standalone kernel rates at sizes large enough to reach the hardware's asymptotes: row
    softmax and transpose against HBM bandwidth (algorithmic bytes: input and output once), GEMMs
    against the matrix-core peak (2MNK).  Each kernel: seeded device-resident operands, the mean of
    back-to-back launches timed with HIP events on its stream; GEMM tiles autotuned."""
    import paper_2009_07482_amd as psc
    es = {"f32": 4, "bf16": 2}
    # element-wise working sets of 1.5 GiB and more: several times the 256 MiB last-level cache, so
    # back-to-back launches cannot serve each other from it
    cases = [("softmax", (262144, 1024), "f32", "f32"), ("softmax", (131072, 2048), "f32", "bf16"),
             ("softmax", (262144, 2048), "bf16", "bf16"), ("transpose", (16384, 16384), "f32", "f32"),
             ("transpose", (16384, 16384), "bf16", "bf16"), ("transpose1", (16384, 16384), "f32", "f32"),
             ("transpose1", (16384, 16384), "bf16", "bf16"), ("transpose2", (16384, 16384), "f32", "f32"),
             ("transpose2", (16384, 16384), "bf16", "bf16"), ("add", (16384, 16384), "f32", "f32"),
             ("gemm", (4096, 4096, 4096), "bf16", "f32"), ("gemm", (8192, 8192, 8192), "bf16", "bf16"),
             ("gemm", (4096, 4096, 4096), "f32", "f32"), ("gemm", (1024, 64, 1024), "bf16", "bf16"),
             ("gemm", (512, 64, 512), "f32", "f32")]
    out = []

    def seeded_inputs(spec):
        # seeded operands (uniform in [-1, 1); softmax rows standard normal): matrix-core power,
        # and with it the clock, depends on the data, so zeros would overstate the rate
        g = np.random.default_rng(0)
        ins = {}
        for b in spec["buffers"][:-1]:
            shape = (b["rows"], b["cols"])
            ins[b["name"]] = (g.standard_normal(shape, dtype=np.float32) if spec["kernels"][0]["kind"] == "softmax"
                              else g.random(shape, dtype=np.float32) * 2 - 1)
        return ins

    for kind, shp, idt, odt in cases:
        if kind == "gemm":
            m, n, k = shp
            tile = 0
            if a.gemm_tile and m * n * k > 1e10:
                tile = a.gemm_tile
            elif not a.no_tune and m * n * k <= 1e10:
                tile, _, _ = psc.psc_autotune_gemm(m, n, k, idt, odt, iters=20)
            elif not a.no_tune:
                # large shapes: only the large-tile kernels are candidates (the K-split ones are
                # for few output tiles and would take seconds each here), each timed on the
                # seeded operands of the measurement below
                best = None
                ins = seeded_inputs(one_kernel("gemm", [(m, k), (k, n), (m, n)], [idt, idt, odt]))
                for t in (1, 2, 4, 5, 16, 20, 21):
                    rr = psc.SpecRunner(one_kernel("gemm", [(m, k), (k, n), (m, n)], [idt, idt, odt], tile=t), "coarse")
                    rr.set_inputs(ins)
                    rr.run(with_inputs=True, with_outputs=False)
                    psc.psc_kernel_time(rr.sched, 0, 2)
                    u = psc.psc_kernel_time(rr.sched, 0, 5)
                    rr.close()
                    print(f"#   tile {t}: {u:.1f} us", file=sys.stderr, flush=True)
                    if best is None or u < best[1]:
                        best = (t, u)
                tile = best[0]
            spec = one_kernel("gemm", [(m, k), (k, n), (m, n)], [idt, idt, odt], tile=tile)
            work, unit, peak = 2.0 * m * n * k, "TFLOP/s", PEAK["mfma_bf16"] if idt == "bf16" else PEAK["mfma_f32"]
            label = f"gemm {m}x{n}x{k} {idt}->{odt}"
        else:
            r_, c_ = shp
            if kind.startswith("transpose"):
                # transpose1 / transpose2 / transpose3 / transpose4: the 64 x 64, 64 x 128,
                # 128 x 64 and 64 x 256 tiles
                spec = one_kernel("transpose", [(r_, c_), (c_, r_)], [idt, odt], tile=int(kind[9:] or 0))
                work = r_ * c_ * (es[idt] + es[odt])
            elif kind == "add":
                spec = one_kernel(kind, [(r_, c_), (r_, c_), (r_, c_)], [idt, idt, odt])
                work = r_ * c_ * (2 * es[idt] + es[odt])
            else:
                spec = one_kernel(kind, [(r_, c_), (r_, c_)], [idt, odt])
                work = r_ * c_ * (es[idt] + es[odt])
            unit, peak = "GB/s", PEAK["hbm"]
            label = f"{kind} {r_}x{c_} {idt}->{odt}"
            if kind.startswith("transpose"):
                label = f"transpose {r_}x{c_} {idt}->{odt} " + {"": "(automatic tile)", "1": "(64x64 tiles)",
                                                                "2": "(64x128 tiles)", "3": "(128x64 tiles)",
                                                                "4": "(64x256 tiles)"}[kind[9:]]
        r = psc.SpecRunner(spec, "coarse")
        ins = seeded_inputs(spec)
        r.set_inputs(ins)
        del ins
        r.run(with_inputs=True, with_outputs=False)
        big = work > 1e11
        psc.psc_kernel_time(r.sched, 0, 3)
        us = psc.psc_kernel_time(r.sched, 0, 10 if big else 100)
        rate = work / (us * 1e-6)
        row = {"kernel": label, "avg_us": us, "achieved": rate / (1e12 if unit == "TFLOP/s" else 1e9),
               "unit": unit, "peak": peak / (1e12 if unit == "TFLOP/s" else 1e9), "frac": rate / peak}
        if kind == "gemm":
            row["tile"] = psc.psc_sched_kernel_tile(r.sched, 0)
        r.close()
        out.append(row)
        print(f"# {json.dumps(row)}", file=sys.stderr, flush=True)
    print(json.dumps({"metric": "standalone kernel rates vs roofline", "kernels": out,
                      "library_reference": library_reference()}), flush=True)


def costmodel_main(a):
    """Learned cost model at full scale: ~20k op timings recorded by the runtime from random
    layered DAGs (50-500 nodes, widths 1-16, dims 64-4096, FP32 or BF16; each op's time the median
    of three runs), the MLP trained on the
    GPU, then on held-out DAGs: op-time error of the MLP vs the roofline heuristic, and the
    measured makespan of EFT schedules (4 streams) under each model, beside round robin."""
    import paper_2009_07482_amd as psc
    import workloads
    from paper_2009_07482_amd import costmodel
    t0 = time.perf_counter()
    xs, ts = [], []
    seed = 0
    while sum(len(t) for t in ts) < 20000 and seed < 200:
        # every 8th DAG is drawn with dims up to 1024 and also times its host copies (H2D / D2H
        # samples); the others are full-size and device-resident
        if seed % 8 == 0:
            spec = workloads.random_dag_spec(seed, dim=(64, 1024))
            inp = workloads.random_dag_inputs(seed, spec)
        else:
            spec = workloads.random_dag_spec(seed)
            inp = None
        x, t = costmodel.record_samples(spec, inp, n_streams=(1, 2, 4, 8)[seed % 4], runs=3, reduce="median")
        xs.append(x)
        ts.append(t)
        seed += 1
        if seed % 10 == 0:
            print(f"# recorded {sum(len(t) for t in ts)} samples from {seed} DAGs "
                  f"({time.perf_counter() - t0:.0f} s)", file=sys.stderr, flush=True)
    X, T = np.concatenate(xs), np.concatenate(ts)
    if a.dump_samples:
        np.savez(a.dump_samples, X=X, T=T)
    t1 = time.perf_counter()
    cm = costmodel.fit(X, T, epochs=a.epochs, batch=256, lr=2e-3, seed=0)
    train_s = time.perf_counter() - t1
    print(f"# trained on {len(T)} samples in {train_s:.1f} s; loss {cm.losses[0]:.3f} -> {cm.losses[-1]:.3f}",
          file=sys.stderr, flush=True)
    held = []
    e_mlp, e_heu = [], []
    for hs in range(1000, 1000 + a.heldout):
        spec = workloads.random_dag_spec(hs)
        x, t = costmodel.record_samples(spec, None, n_streams=4, runs=3, reduce="median")
        if a.dump_samples:
            np.savez(a.dump_samples.replace(".npz", f"_heldout{hs}.npz"), X=x, T=t)
        e_mlp.append(costmodel.mape(cm.predict_us(x), t))
        e_heu.append(costmodel.mape(psc.psc_cost_predict(x), t))
        ms = {}
        for name, kw in (("rr", dict(mapper="rr")), ("eft_heuristic", dict(mapper="eft")),
                         ("eft_mlp", dict(mapper="eft", cost=cm.handle))):
            r = psc.SpecRunner(spec, "fine", n_streams=4, host_threads=1, **kw)
            psc.psc_sched_prepare(r.sched)
            r.run(with_inputs=False, with_outputs=False)
            mk = [r.run(with_inputs=False, with_outputs=False)["makespan_ms"] for _ in range(5)]
            ms[name] = float(np.median(mk))
            r.close()
        held.append({"seed": hs, "kernels": len(spec["kernels"]), "dtype": spec["dtype"], "makespan_ms": ms,
                     "mape_mlp": e_mlp[-1], "mape_heuristic": e_heu[-1]})
        print(f"# held-out {hs}: {len(spec['kernels'])} kernels {spec['dtype']}: " +
              ", ".join(f"{k} {v:.2f} ms" for k, v in ms.items()) +
              f"; op-time MAPE mlp {e_mlp[-1]:.3f} heuristic {e_heu[-1]:.3f}", file=sys.stderr, flush=True)
    cm.close()
    ratio = [h["makespan_ms"]["eft_mlp"] / h["makespan_ms"]["eft_heuristic"] for h in held]
    ratio_rr = [h["makespan_ms"]["eft_mlp"] / h["makespan_ms"]["rr"] for h in held]
    gm = lambda v: float(np.exp(np.mean(np.log(v))))
    line = {"metric": "learned cost model: op-time error and EFT makespan vs the roofline heuristic",
            "training_samples": int(len(T)), "training_dags": seed, "train_seconds": train_s,
            "loss_first_last": [float(cm.losses[0]), float(cm.losses[-1])],
            "heldout_dags": len(held), "op_time_mape": {"mlp": float(np.mean(e_mlp)), "heuristic": float(np.mean(e_heu))},
            "makespan_ratio_mlp_over_heuristic_geomean": gm(ratio),
            "makespan_ratio_mlp_over_rr_geomean": gm(ratio_rr),
            "mlp_faster_on": int(sum(r < 1.0 for r in ratio)), "per_dag": held,
            "data": "synthetic random layered DAGs (seeded), device-resident timings plus copies on every 8th DAG"}
    print(json.dumps(line), flush=True)


def batch_main(a):
    """64 attention instances of log-uniform length in [64, 2048] (d = 512, 8 heads, 6 layers,
    BF16 GEMMs), one task component each, in one DAG of 21,888 kernels.  A step is one batch.
    Reports inferences/s = 64 / batch time and per-instance completion latency (device-clock
    marks after each instance's last kernel), untuned vs autotuned, eager vs one hipGraph."""
    import paper_2009_07482_amd as psc
    import workloads
    lengths = workloads.batch_lengths(0)
    d, h, L = 512, 8, 6
    spec = workloads.batch_spec(lengths, d, h, L, gemm_dtype="bf16")
    inp = workloads.batch_inputs(0, lengths, d, L)
    print(f"# batch: {len(lengths)} instances, n in [{min(lengths)}, {max(lengths)}], "
          f"{len(spec['kernels'])} kernels", file=sys.stderr, flush=True)
    res, keep = {}, {}

    def measure(name, policy, keep_runner=False, **kw):
        t0 = time.perf_counter()
        r = psc.SpecRunner(spec, policy, mark_components=(policy != "device"), **kw)
        r.set_inputs(inp)
        st_io = r.run()
        setup = time.perf_counter() - t0
        wall, mk, st = timed(r, a.steps, a.warmup)
        done = psc.psc_sched_component_times(r.sched) / 1000.0
        res[name] = {"ms_per_batch": wall / a.steps * 1e3, "makespan_ms_median": float(np.median(mk)),
                     "latency_ms_p50": float(np.percentile(done, 50)),
                     "latency_ms_p99": float(np.percentile(done, 99)),
                     "makespan_with_copies_ms": st_io["makespan_ms"], "host_enqueue_ms": st["host_enqueue_ms"],
                     "first_run_s": setup, "opts": {"policy": policy, **kw}}
        print(f"# {name}: {json.dumps(res[name])}", file=sys.stderr, flush=True)
        if keep_runner:
            keep[name] = r
        else:
            r.close()

    measure("coarse_default", "coarse")
    measure("fine_default", "fine", n_streams=4, mapper="component")
    measure("graph_default", "fine", n_streams=4, mapper="component", use_graph=True)
    tuned = 0
    if not a.no_tune:
        d0 = psc.build_dag(spec)
        t0 = time.perf_counter()
        tuned = psc.psc_autotune_dag(d0, iters=10)
        psc.psc_dag_destroy(d0)
        print(f"# tile autotuner: {tuned} GEMM shapes in {time.perf_counter() - t0:.1f} s", file=sys.stderr,
              flush=True)
    cands = ([dict(n_streams=s_, mapper="component", use_graph=g_, copy_roots=True) for s_ in (4, 8, 16)
              for g_ in (False, True)]
             + [dict(n_streams=s_, mapper="component", dispatch="aql", copy_roots=True) for s_ in (2, 4)])
    d1 = psc.build_dag(spec)
    bi, cms = psc.psc_autotune_schedule(d1, "fine", cands, iters=3)
    psc.psc_dag_destroy(d1)
    best = cands[bi]
    print("# schedule autotuner: " + ", ".join(
        f"{c.get('dispatch', 'hip')}/{c['n_streams']}{'g' if c.get('use_graph') else 'e'}={m:.2f}"
        for c, m in zip(cands, cms)) + f" -> {best}", file=sys.stderr, flush=True)
    if not a.no_tune:
        d2 = psc.build_dag(spec)
        changed = psc.psc_autotune_dag_in_schedule(d2, "fine", top_k=3, iters=2, max_classes=4, **best)
        psc.psc_dag_destroy(d2)
        print(f"# tiles by makespan: {changed} shape class(es) changed", file=sys.stderr, flush=True)
    measure("coarse", "coarse")
    measure("tuned", "fine", keep_runner=True, **best)
    if best.get("dispatch") == "aql":
        measure("tuned_hip_eager", "fine", n_streams=4, mapper="component", copy_roots=True)
        measure("tuned_hip_graph", "fine", n_streams=4, mapper="component", use_graph=True, copy_roots=True)
    else:
        other = dict(best, use_graph=not best["use_graph"])
        measure("tuned_" + ("eager" if best["use_graph"] else "graph"), "fine", **other)
    roof = dominant_roofline(spec, keep["tuned"], a.kernel_iters)
    keep["tuned"].close()
    chosen = "tuned"
    t = res[chosen]
    line = {
        "metric": "batched inference: inferences/s and per-instance latency p50/p99",
        "value": len(lengths) / (t["ms_per_batch"] / 1e3), "unit": "inferences/s", "n_gpus": 1,
        "steps": a.steps, "warmup": a.warmup, "ms_per_step": t["ms_per_batch"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) inputs, N(0,1/d) weights, log-uniform lengths)",
        "config": {"workload": f"batch of {len(lengths)} attention instances, n log-uniform in [64, 2048], "
                               f"d_model={d}, {h} heads, {L} layers, GEMM BF16 (FP32 accumulation)",
                   "kernels": len(spec["kernels"]),
                   "schedule": best if chosen == "tuned" else "device executor (one persistent kernel)",
                   "inputs": "device-resident",
                   "gemm_tiles": "autotuned" if tuned else "size heuristic"},
        "latency_ms": {"p50": t["latency_ms_p50"], "p99": t["latency_ms_p99"]},
        "by_schedule": res,
        "roofline": roof,
    }
    if not a.no_cpu:
        line["cpu_baseline"] = batch_cpu_baseline(lengths, d, h, L, inp, a.cpu_seconds)
    print(json.dumps(line), flush=True)


def batch_cpu_baseline(lengths, d, h, L, inp, seconds):
    """The oracle on instances taken shortest first until the time is used, scaled to the whole
    batch by floating-point work (the oracle's time is dominated by its matrix products)."""
    import workloads
    from oracle import dag as odag
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count() or 1
    order = sorted(range(len(lengths)), key=lambda i: lengths[i])
    total = sum(workloads.spec_flops(workloads.mha_spec(n, d, h, L, "bf16")) for n in lengths)
    done, el, t0 = 0.0, 0.0, time.perf_counter()
    count = 0
    for i in order[::max(1, len(order) // 16)]:
        sub = workloads.mha_spec(lengths[i], d, h, L, "bf16", prefix=f"i{i}_", weight_prefix="")
        odag.run_dag(sub, {k: inp[k] for k in workloads.host_inputs_of(sub)})
        done += workloads.spec_flops(sub)
        count += 1
        el = time.perf_counter() - t0
        if el >= seconds:
            break
    batch_s = el * total / done
    return {"value": len(lengths) / batch_s, "unit": "inferences/s", "cores": int(cores), "kind": "oracle",
            "sample": f"{count} instance(s) spread over the length range in FP64 (numpy), {el:.1f} s, "
                      f"scaled to the batch by FLOPs"}


# every schedule uploads a read-only weight matrix as one dense copy (copy_roots), not one
# strided rectangle per attention head
FINE_CANDIDATES = [dict(n_streams=s_, mapper=m_, host_threads=t_, dispatch=d_, copy_roots=True)
                   for d_ in ("aql", "hip") for s_ in (2, 4, 8, 16) for m_ in ("component", "rr") for t_ in (1, 0)]


def measure_runner(r, steps, warmup, copies_runs=5, copies_warmup=15):
    """Device-resident timing (the value) and the PCIe-inclusive makespan (inputs uploaded and the
    output read back inside the run, from page-locked memory: first H2D to last D2H).  The first runs
    with copies on new HIP streams take several times the later ones, a dozen of them on eight streams
    (the runtime sets up its copy engines): the median is over steady runs, the first is given too.
    plan_waits and plan_streams describe the exported schedule, aql_packets what a run writes."""
    first = r.run()["makespan_ms"]
    for _ in range(copies_warmup):
        r.run()
    io = [r.run()["makespan_ms"] for _ in range(copies_runs)]
    wall, mk, st = timed(r, steps, warmup)
    return {"ms_per_step": wall / steps * 1e3, "makespan_ms_median": float(np.median(mk)),
            "makespan_ms_p5": float(np.percentile(mk, 5)), "makespan_ms_p95": float(np.percentile(mk, 95)),
            "host_enqueue_ms": st["host_enqueue_ms"], "makespan_with_copies_ms": float(np.median(io)),
            "first_run_with_copies_ms": first,
            "plan_waits": st["n_waits"], "plan_streams": st["n_streams"], "aql_packets": st["aql_packets"]}


def describe(opts):
    if opts is None:
        return "device executor (one persistent kernel)"
    how = ("AQL packets on HSA queues, barrier-AND packets on completion signals"
           if opts.get("dispatch") == "aql" else "HIP streams and events")
    if opts.get("n_streams", 1) == 1 and not opts.get("mapper"):
        return f"coarse: one in-order queue ({how})"
    m = {"component": "clustering (one task component per head per stream)", "rr": "round robin per kernel",
         "eft": "EFT list scheduling"}[opts.get("mapper", "rr")]
    th = "one enqueue thread" if opts.get("host_threads") == 1 else "one enqueue thread per stream"
    q = ("out-of-order queues (kernels of one queue run concurrently; every precedence a barrier-AND)"
         if opts.get("out_of_order") else "in-order queues")
    return f"fine: {opts['n_streams']} streams, {m}, {th}; {how}; {q}"


def dag_bench(spec, inp, a, tune=True, with_device=True, label=""):
    """Coarse (both dispatchers), the autotuned fine schedule, the best HIP-stream fine schedule
    and the device executor on one DAG; returns (results, fine opts, runners kept for the roofline)."""
    import paper_2009_07482_amd as psc
    tuned = 0
    if tune and not a.no_tune:
        d0 = psc.build_dag(spec)
        tuned = psc.psc_autotune_dag(d0, iters=20)
        psc.psc_dag_destroy(d0)
    d1 = psc.build_dag(spec)
    bi, cms = psc.psc_autotune_schedule(d1, "fine", FINE_CANDIDATES, iters=max(5, a.steps // 4))
    psc.psc_dag_destroy(d1)
    fine_opts = FINE_CANDIDATES[bi]
    if tune and not a.no_tune:
        # then the GEMM tiles again, by the chosen schedule's makespan (isolated times do not
        # predict a kernel's time beside the schedule's concurrent kernels)
        d2 = psc.build_dag(spec)
        changed = psc.psc_autotune_dag_in_schedule(d2, "fine", top_k=3, iters=5, **fine_opts)
        psc.psc_dag_destroy(d2)
        print(f"# {label} tiles by makespan: {changed} shape class(es) changed from the isolated choice",
              file=sys.stderr, flush=True)
    hip_idx = [i for i, c in enumerate(FINE_CANDIDATES) if c["dispatch"] == "hip"]
    hip_opts = FINE_CANDIDATES[min(hip_idx, key=lambda i: cms[i] if cms[i] > 0 else 1e30)]
    print(f"# {label} schedule autotuner: chose {fine_opts} ({cms[bi]:.3f} ms/run); " +
          ", ".join(f"{c['dispatch']}{'-ooo' if c.get('out_of_order') else ''}/{c['n_streams']}/{c['mapper'][0]}/"
                    f"{'1t' if c['host_threads'] == 1 else 'mt'}={m:.3f}"
                    for c, m in zip(FINE_CANDIDATES, cms)), file=sys.stderr, flush=True)
    plan = {"coarse_hip": ("coarse", dict(dispatch="hip", copy_roots=True)),
            "coarse_aql": ("coarse", dict(dispatch="aql", copy_roots=True)),
            "fine": ("fine", fine_opts), "fine_hip": ("fine", hip_opts),
            # the same fine schedule with every upload on a copy stream of its own, issued ahead
            # (its uploads overlap the first layers' kernels)
            "fine_copy_stream": ("fine", dict(fine_opts, copy_stream=True))}
    if with_device:
        # the executor with the most resident workgroups its instance allows, and with one per CU
        # (which is faster depends on the DAG); the row reports the faster
        plan["device_executor_most"] = ("device", dict(copy_roots=True))
        plan["device_executor_1cu"] = ("device", dict(copy_roots=True, exec_per_cu=1))
    res, keep = {}, {}
    for name, (policy, kw) in plan.items():
        r = psc.SpecRunner(spec, policy, **kw)
        r.set_inputs(inp)
        res[name] = measure_runner(r, a.steps, a.warmup)
        if policy == "device":
            w, pcu, grp = psc.psc_sched_executor_info(r.sched)
            res[name]["schedule"] = describe(None) + f": {w} workgroups, {pcu} per CU, tile-function groups {grp:#x}"
        else:
            res[name]["schedule"] = describe(kw) if policy != "coarse" else describe(dict(kw, n_streams=1))
        print(f"# {label} {name}: {json.dumps(res[name])}", file=sys.stderr, flush=True)
        if name == "fine":
            keep[name] = r
        else:
            r.close()
    res["coarse"] = min((res["coarse_hip"], res["coarse_aql"]), key=lambda v: v["ms_per_step"])
    if with_device:
        res["device_executor"] = min((res["device_executor_most"], res["device_executor_1cu"]),
                                     key=lambda v: v["ms_per_step"])
    return res, fine_opts, keep, tuned


def kernel_timeline(spec, inp, opts):
    """Kernels in flight and per-class in-DAG durations from one recorded run of the fine schedule
    (AQL: the queues' profiler timestamps; HIP: event pairs)."""
    import paper_2009_07482_amd as psc
    rec = psc.SpecRunner(spec, "fine", record_ops=True, **opts)
    rec.set_inputs(inp)
    rec.run()
    rec.run(with_inputs=False, with_outputs=False)
    times = psc.psc_sched_op_times(rec.sched)
    ops = psc.psc_sched_export(rec.sched)
    rec.close()
    kern = [t for t, o in zip(times, ops) if o["type"] == "kernel" and t[3] > t[2]]
    by_class, by_q = {}, {}
    for t, o in zip(times, ops):
        if o["type"] == "kernel" and t[3] > t[2]:
            key = kernel_class(spec, o["kernel"])[0]
            by_class.setdefault(key, []).append(t[3] - t[2])
            by_q.setdefault(o["stream"], []).append((t[2], t[3]))
    span = max(t[3] for t in kern) - min(t[2] for t in kern) if kern else 0.0
    queues = {}
    for q, iv in sorted(by_q.items()):
        iv.sort()
        gaps = [max(0.0, b[0] - a[1]) for a, b in zip(iv, iv[1:])]
        queues[str(q)] = {"kernels": len(iv), "busy_frac": sum(b - a for a, b in iv) / span if span else 0.0,
                          "gap_median_us": float(np.median(gaps)) if gaps else 0.0}
    return overlap(kern), {k: float(np.mean(v)) for k, v in by_class.items()}, queues


def dynamic_rows(spec, inp, a, static_opts):
    """The paper's dynamic coarse-grained baselines (eager, HEFT: one kernel per task component,
    host callbacks on completion, Sec. V) beside the static fine-grained schedule: makespan and
    the median gap between consecutive kernels of one stream, which is where the callbacks show."""
    import paper_2009_07482_amd as psc

    def gaps(r):
        times = psc.psc_sched_op_times(r.sched)
        ops = r.export()["ops"]
        by = {}
        for t, o in zip(times, ops):
            if o["type"] == "kernel" and t[3] > t[2]:
                by.setdefault(o["stream"], []).append((t[2], t[3]))
        g = []
        for iv in by.values():
            iv.sort()
            g += [b[0] - a_[1] for a_, b in zip(iv, iv[1:])]
        return float(np.median(g)) if g else 0.0

    out = {}
    for name, policy, kw in (("eager", "eager", dict(n_streams=4)), ("heft", "heft", dict(n_streams=4)),
                             ("static_fine", "fine", dict(static_opts))):
        kw = dict(kw, copy_roots=True)
        r = psc.SpecRunner(spec, policy, **kw)
        r.set_inputs(inp)
        r.run()
        steps = max(3, min(a.steps, 10))
        mk = [r.run(with_inputs=False, with_outputs=False)["makespan_ms"] for _ in range(steps)]
        r.close()
        rec = psc.SpecRunner(spec, policy, record_ops=True, **kw)
        rec.set_inputs(inp)
        rec.run()
        rec.run(with_inputs=False, with_outputs=False)
        g = gaps(rec)
        rec.close()
        out[name] = {"makespan_ms": float(np.median(mk)), "median_gap_between_kernels_us": g}
        print(f"# dynamic {name}: {json.dumps(out[name])}", file=sys.stderr, flush=True)
    return out


def main():
    a = parse()
    if a.gpus != 1:
        print(json.dumps({"error": "this build runs on one GPU; --gpus must be 1 (how the DAG would shard is "
                                   "described in the design notes, not built)"}))
        sys.exit(2)
    import paper_2009_07482_amd as psc

    if a.config == "batch64":
        batch_main(a)
        return
    if a.config == "kernels":
        kernels_main(a)
        return
    if a.config == "costmodel":
        costmodel_main(a)
        return
    if a.kernel_profile == "timeline":
        timeline_profile(a)
        return
    if a.kernel_profile:
        kernel_profile(a)
        return
    spec, inp, desc = workload(a.config)
    res, fine_opts, keep, tuned = dag_bench(spec, inp, a, label=desc.get("gemm_dtype", ""))
    fine = res["fine"]
    roof = dominant_roofline(spec, keep["fine"], a.kernel_iters)
    keep["fine"].close()
    in_flight, in_dag_us, queues = kernel_timeline(spec, inp, fine_opts)
    roof["in_dag_avg_us"] = in_dag_us.get(roof["kernel"])
    line = {
        "metric": "DAG makespan (ms) + inferences/s, fine vs coarse schedule, BF16 vs FP32",
        "value": 1e3 / fine["ms_per_step"], "unit": "inferences/s", "n_gpus": 1, "steps": a.steps,
        "warmup": a.warmup, "ms_per_step": fine["ms_per_step"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": desc.get("gemm_dtype", "f32"),
        "data": "synthetic (seeded N(0,1) inputs, N(0,1/d) weights)",
        "config": dict(desc, schedule=fine["schedule"], inputs="device-resident",
                       gemm_tiles="autotuned" if tuned else "size heuristic"),
        "makespan_ms": {k: v["makespan_ms_median"] for k, v in res.items()},
        "ms_per_step_by_schedule": {k: v["ms_per_step"] for k, v in res.items()},
        "makespan_with_copies_ms": {k: v["makespan_with_copies_ms"] for k, v in res.items()},
        "schedules": {k: v["schedule"] for k, v in res.items()},
        "fine_vs_coarse_speedup": res["coarse"]["ms_per_step"] / fine["ms_per_step"],
        "fine_vs_coarse_speedup_same_dispatch": {
            "hip": res["coarse_hip"]["ms_per_step"] / res["fine_hip"]["ms_per_step"],
            "aql": res["coarse_aql"]["ms_per_step"] / fine["ms_per_step"] if fine_opts["dispatch"] == "aql" else None},
        "dynamic_baselines": dynamic_rows(spec, inp, a, fine_opts),
        "fine_kernels_in_flight_mean": in_flight,
        "fine_queues": queues,
        "fine_in_dag_kernel_us": in_dag_us,
        "dag_bound_us": dag_bound_us(spec),
        "makespan_over_dag_bound": fine["makespan_ms_median"] * 1e3 / dag_bound_us(spec),
        "roofline": roof,
        "environment": environment(),
    }
    if a.config == "mha1024x12" and not a.no_fp32:
        # the same DAG with FP32 GEMMs (and FP32 storage throughout): the other half of the metric
        import workloads
        spec32 = workloads.mha_spec(1024, 1024, 16, 12, gemm_dtype="f32")
        res32, opts32, keep32, _ = dag_bench(spec32, inp, a, with_device=False, label="f32")
        keep32["fine"].close()
        line["fp32_same_dag"] = {
            "inferences_per_s": 1e3 / res32["fine"]["ms_per_step"],
            "makespan_ms": {k: v["makespan_ms_median"] for k, v in res32.items()},
            "ms_per_step_by_schedule": {k: v["ms_per_step"] for k, v in res32.items()},
            "makespan_with_copies_ms": {k: v["makespan_with_copies_ms"] for k, v in res32.items()},
            "schedule": res32["fine"]["schedule"],
            "fine_vs_coarse_speedup": res32["coarse"]["ms_per_step"] / res32["fine"]["ms_per_step"]}
        line["bf16_vs_fp32_speedup"] = res32["fine"]["ms_per_step"] / fine["ms_per_step"]
    if not a.no_cpu:
        if a.config == "mha1024x12":
            # bounded sample: the first 2 of the 12 identical-shape layers, scaled to 12
            import workloads
            sub = workloads.mha_spec(1024, 1024, 16, 2, gemm_dtype="bf16")
            sub_inp = {k: v for k, v in inp.items() if k in set(workloads.host_inputs_of(sub))}
            cb = cpu_baseline(sub, sub_inp, a.cpu_seconds)
            cb["value"] *= 2.0 / 12.0
            cb["sample"] += "; first 2 of 12 layers, rate scaled by 2/12"
            line["cpu_baseline"] = cb
        else:
            line["cpu_baseline"] = cpu_baseline(spec, inp, a.cpu_seconds)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
