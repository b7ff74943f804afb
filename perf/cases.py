"""The workloads whose speed this repository is held to, as plain cases.

A case is a dict of plain values that names a DAG family with its sizes, the schedule policy and the
dispatcher.  ``listed()`` gives the fixed cases, ``draw(rng)`` one more of the same families and
ranges; ``prepare`` builds what a program holds before it runs (inputs on the device or in
page-locked host memory, the DAG and its prepared schedule), ``run`` is one pass (one ``psc_run``,
or one training of the cost model), ``work`` the bytes and operations of a pass that no
implementation can avoid, and ``exact`` the pass's result in 64 bits.

torch is imported first: libpsc.so then resolves its HIP runtime to the one torch has loaded (both
carry the same soname), so tensors and schedules share one runtime and one device context.
"""
import math

import numpy as np
import torch

import paper_2009_07482_amd as psc
import workloads

TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "bf16": 2}


def listed():
    return [
        # The smallest call: the paper's four-kernel fork-join (Fig. 1) with every default of
        # psc_schedule (four HIP streams, round robin).  Launches, events and the wait count.
        dict(name="forkjoin_256_f32", family="forkjoin", n=256, dtype="f32", policy="fine", dispatch="hip",
             mapper="rr", streams=4),
        # One attention layer of the size the benchmark's small configuration runs, FP32, on the
        # GPU's own queues with one task component per head (the schedule the benchmark selects).
        dict(name="mha_512_f32_fine", family="mha", n=512, d=512, heads=8, layers=1, dtype="f32", policy="fine",
             dispatch="aql", mapper="component", streams=4),
        # The same layer on the persistent device executor.
        dict(name="mha_512_f32_device", family="mha", n=512, d=512, heads=8, layers=1, dtype="f32",
             policy="device", dispatch="hip", mapper="rr", streams=4),
        # The benchmark's main shape (n = d = 1024, 16 heads, BF16 operands) as a whole call of four
        # stacked layers: 452 kernels.
        dict(name="mha_1024x4_bf16_fine", family="mha", n=1024, d=1024, heads=16, layers=4, dtype="bf16",
             policy="fine", dispatch="aql", mapper="component", streams=4),
        dict(name="mha_1024x4_bf16_device", family="mha", n=1024, d=1024, heads=16, layers=4, dtype="bf16",
             policy="device", dispatch="hip", mapper="rr", streams=4),
        # A served layer whose input and weights come from page-locked host memory on every call
        # and whose output goes back there: uploads on copy streams beside the kernels.
        dict(name="mha_1024_bf16_hostio", family="mha", n=1024, d=1024, heads=16, layers=1, dtype="bf16",
             policy="fine", dispatch="aql", mapper="component", streams=4, hostio=True),
        # Batched serving: sixteen attention DAGs of uneven, mostly odd length over shared weights,
        # joined by psc_schedule_batch, on HIP streams.
        dict(name="batch_16x2_bf16", family="batch", count=16, lo=64, hi=2048, lengths_seed=5, d=512, heads=8,
             layers=2, dtype="bf16", policy="fine", dispatch="hip", mapper="component", streams=4),
        # An application DAG of mixed kernels and arbitrary (mostly odd) sizes, mapped by earliest
        # finish time: rows of these matrices have no common alignment.
        dict(name="random_60_bf16", family="random", nodes=60, dag_seed=11, dim_lo=64, dim_hi=1024, dtype="bf16",
             policy="fine", dispatch="hip", mapper="eft", streams=4),
        # Large single kernels, as the benchmark's kernel table has them: the biggest matrix
        # product, a ragged FP32 one, and the streaming kernels (transpose, softmax, add) in a row.
        dict(name="gemm_4096_bf16", family="gemm", m=4096, n=4096, k=4096, dtype="bf16", out="f32",
             policy="coarse", dispatch="hip", mapper="rr", streams=1),
        dict(name="gemm_ragged_f32", family="gemm", m=1777, n=2050, k=1001, dtype="f32", out="f32",
             policy="coarse", dispatch="hip", mapper="rr", streams=1),
        dict(name="elementwise_16384x2048_f32", family="elementwise", rows=16384, cols=2048, dtype="f32",
             policy="coarse", dispatch="hip", mapper="rr", streams=1),
        # Training the learned cost model: two passes of mini-batch Adam over as many op timings as
        # the benchmark's corpus holds (forward, backward and update of every step).
        dict(name="costmodel_20000x2", family="costmodel", samples=20000, batch=256, epochs=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["forkjoin", "mha", "mha", "mha", "batch", "random", "gemm", "gemm", "elementwise", "costmodel"])
    dtype = rng.choice(["f32", "bf16"])
    sched = rng.choice([("fine", "hip", "rr"), ("fine", "aql", "component"), ("fine", "aql", "rr"),
                        ("coarse", "hip", "rr"), ("device", "hip", "rr")])
    common = dict(dtype=dtype, policy=sched[0], dispatch=sched[1], mapper=sched[2], streams=4)
    if family == "forkjoin":
        return dict(family=family, n=_log_int(rng, 64, 1024), **dict(common, dtype="f32"))
    if family == "mha":
        d = rng.choice([256, 512, 1024])
        c = dict(family=family, n=_log_int(rng, 64, 1024), d=d, heads=d // 64, layers=rng.choice([1, 2]), **common)
        if sched[0] == "fine" and rng.random() < 0.3:
            c["hostio"] = True
        return c
    if family == "batch":
        return dict(family=family, count=rng.randint(2, 12), lo=64, hi=1024, lengths_seed=rng.randint(0, 10 ** 6),
                    d=512, heads=8, layers=rng.choice([1, 2]), **common)
    if family == "random":
        return dict(family=family, nodes=rng.randint(50, 60), dag_seed=rng.randint(0, 10 ** 6), dim_lo=64,
                    dim_hi=rng.choice([512, 1024]), **dict(common, mapper=rng.choice(["rr", "eft"])))
    if family == "gemm":
        return dict(family=family, m=_log_int(rng, 64, 4096), n=_log_int(rng, 64, 4096), k=_log_int(rng, 64, 4096),
                    out=rng.choice(["f32", dtype]), **dict(common, policy="coarse", dispatch="hip", streams=1))
    if family == "elementwise":
        return dict(family=family, rows=_log_int(rng, 256, 16384), cols=_log_int(rng, 64, 2048),
                    **dict(common, policy="coarse", dispatch="hip", streams=1))
    return dict(family="costmodel", samples=_log_int(rng, 500, 20000), batch=rng.choice([64, 200, 256, 1000]),
                epochs=rng.choice([1, 2]))


# --- DAG families ---------------------------------------------------------------------------------

def _specs(case):
    """The DAG specs of a case, one per schedule member, and the buffers its pass returns."""
    f = case["family"]
    if f == "forkjoin":
        sp = workloads.forkjoin_spec(case["n"], case["dtype"])
        return [sp], [["C3"]]
    if f == "mha":
        sp = workloads.mha_spec(case["n"], case["d"], case["heads"], case["layers"], case["dtype"],
                                final_dtype=case["dtype"])
        return [sp], [[f"Y{case['layers'] - 1}"]]
    if f == "batch":
        lengths = workloads.batch_lengths(case["lengths_seed"], case["count"], case["lo"], case["hi"])
        sps = [workloads.mha_spec(n, case["d"], case["heads"], case["layers"], case["dtype"],
                                  final_dtype=case["dtype"]) for n in lengths]
        for sp in sps:   # one task component per instance
            sp["component"] = [0] * len(sp["kernels"])
        return sps, [[f"Y{case['layers'] - 1}"]] * len(sps)
    if f == "random":
        sp = workloads.random_dag_spec(case["dag_seed"], n_nodes=(case["nodes"], case["nodes"]),
                                       dim=(case["dim_lo"], case["dim_hi"]), dtype=case["dtype"])
        return [sp], [workloads.host_outputs_of(sp)]
    if f == "gemm":
        bufs = [_buf("A", case["dtype"], case["m"], case["k"]), _buf("B", case["dtype"], case["k"], case["n"]),
                _buf("C", case["out"], case["m"], case["n"])]
        kers = [{"name": "gemm", "kind": "gemm", "inputs": ["A", "B"], "outputs": ["C"], "alpha": 1.0}]
        return [{"buffers": bufs, "kernels": kers, "edges": [], "component": [0]}], [["C"]]
    # elementwise: T = A^T, P = softmax(T), Y = P + B
    r, c, dt = case["rows"], case["cols"], case["dtype"]
    bufs = [_buf("A", dt, c, r), _buf("T", dt, r, c), _buf("P", dt, r, c), _buf("B", dt, r, c), _buf("Y", dt, r, c)]
    kers = [{"name": "t", "kind": "transpose", "inputs": ["A"], "outputs": ["T"], "alpha": 1.0},
            {"name": "p", "kind": "softmax", "inputs": ["T"], "outputs": ["P"], "alpha": 1.0},
            {"name": "y", "kind": "add", "inputs": ["P", "B"], "outputs": ["Y"], "alpha": 1.0}]
    edges = [(0, "T", 1, "T"), (1, "P", 2, "P")]
    return [{"buffers": bufs, "kernels": kers, "edges": edges, "component": [0, 0, 0]}], [["P", "Y"]]


def _buf(name, dtype, rows, cols):
    return {"name": name, "dtype": dtype, "rows": rows, "cols": cols, "view_of": None, "row_off": 0, "col_off": 0}


def _inputs(case, specs, seed):
    """Device tensors of every host input, one dict per spec.  Attention: X ~ N(0, 1), weights ~
    N(0, 1/d), shared by the members of a batch.  Others: uniform in [-1, 1), a GEMM's B operand
    in a chain at variance 1/K."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    out, weights = [], {}
    for sp in specs:
        by = {b["name"]: b for b in sp["buffers"]}
        b_operand = {k["inputs"][1] for k in sp["kernels"] if k["kind"] == "gemm"}
        have = {}
        for name in workloads.host_inputs_of(sp):
            b = by[name]
            shape = (b["rows"], b["cols"])
            if case["family"] in ("mha", "batch"):
                if name == "X":
                    t = torch.randn(shape, generator=g, device="cuda")
                elif name in weights:
                    have[name] = weights[name]
                    continue
                else:
                    t = torch.randn(shape, generator=g, device="cuda") / math.sqrt(case["d"])
            else:
                r = math.sqrt(3.0 / b["rows"]) if case["family"] == "random" and name in b_operand else 1.0
                t = (torch.rand(shape, generator=g, device="cuda") * 2.0 - 1.0) * r
            have[name] = t.to(TORCH_DT[b["dtype"]]).contiguous()
            if case["family"] in ("mha", "batch") and name != "X":
                weights[name] = have[name]
        out.append(have)
    return out


def _options(case):
    return dict(n_streams=case["streams"], mapper=case["mapper"], dispatch=case["dispatch"])


class _Resident:
    """A prepared schedule over device-resident inputs and outputs (torch tensors bound as the
    DAG's buffers)."""

    def __init__(self, case, seed):
        specs, outs = _specs(case)
        inputs = _inputs(case, specs, seed)
        self.keep, self.outputs, self.dags, self.sched = [inputs], [], [], None
        for sp, names, have in zip(specs, outs, inputs):
            by = {b["name"]: b for b in sp["buffers"]}
            mine = {n: torch.zeros((by[n]["rows"], by[n]["cols"]), dtype=TORCH_DT[by[n]["dtype"]], device="cuda")
                    for n in names}
            self.outputs += [mine[n] for n in names]
            bind = {n: (t.data_ptr(), t.numel() * t.element_size()) for n, t in {**have, **mine}.items()}
            self.dags.append(psc.build_dag(sp, bind))
        if case["family"] == "batch":
            self.sched = psc.psc_schedule_batch(self.dags, case["policy"], **_options(case))
        else:
            self.sched = psc.psc_schedule(self.dags[0], case["policy"], **_options(case))
        psc.psc_sched_prepare(self.sched)
        torch.cuda.synchronize()   # the schedule's streams do not order behind torch's

    def run(self):
        psc.psc_run(self.sched)
        return list(self.outputs)

    def __del__(self):
        if self.sched is not None:
            psc.psc_sched_destroy(self.sched)
        for d in self.dags:
            psc.psc_dag_destroy(d)


class _HostIO:
    """A scheduled DAG whose inputs and outputs lie in page-locked host memory (torch tensors)."""

    def __init__(self, case, seed):
        specs, outs = _specs(case)
        by = {b["name"]: b for b in specs[0]["buffers"]}
        self.sched, self.dag = None, psc.build_dag(specs[0])
        self.sched = psc.psc_schedule(self.dag, case["policy"], copy_stream=True, copy_roots=True, **_options(case))
        psc.psc_sched_prepare(self.sched)
        host = {n: t.cpu().pin_memory() for n, t in _inputs(case, specs, seed)[0].items()}
        self.outputs = [torch.zeros((by[n]["rows"], by[n]["cols"]), dtype=TORCH_DT[by[n]["dtype"]], pin_memory=True)
                        for n in outs[0]]
        host.update(zip(outs[0], self.outputs))
        self.host = host
        self.io = [(n, t.data_ptr(), t.numel() * t.element_size()) for n, t in host.items()]
        torch.cuda.synchronize()

    def run(self):
        psc.psc_run(self.sched, self.io)
        return list(self.outputs)

    def __del__(self):
        if self.sched is not None:
            psc.psc_sched_destroy(self.sched)
        psc.psc_dag_destroy(self.dag)


# --- cost model -----------------------------------------------------------------------------------

def _timings(case, seed):
    """Feature rows and ln-microsecond targets as recorded op timings look: a kind, log2 sizes,
    log2 bytes, the operand type and the streams in flight."""
    g = np.random.default_rng(int(seed))
    n = case["samples"]
    x = np.zeros((n, psc.PSC_FEATURES), np.float32)
    kind = g.choice(6, n, p=[0.45, 0.15, 0.15, 0.15, 0.05, 0.05])
    x[np.arange(n), kind] = 1.0
    x[:, 6:9] = g.uniform(6.0, 12.0, (n, 3))
    x[kind != 0, 8] = 0.0
    x[:, 10] = g.integers(0, 2, n)
    es = np.where(x[:, 10] > 0, 1.0, 2.0)
    x[:, 9] = x[:, 6] + x[:, 7] + es + 1.0
    x[:, 11] = g.integers(0, 8, n)
    bytes_us = np.exp2(x[:, 9]) / 4.0e6
    flops_us = np.where(kind == 0, np.exp2(x[:, 6:9].sum(1) + 1.0) / np.where(x[:, 10] > 0, 5e8, 6e7), 0.0)
    t = np.log(4.0 + bytes_us + flops_us) + 0.05 * x[:, 11] + 0.3 * g.standard_normal(n)
    return x, t.astype(np.float32)


def _mlp_start(case, seed):
    x, t = _timings(case, seed)
    std = x.std(axis=0)
    std = np.where(std > 1e-6, std, 1.0).astype(np.float32)
    params = workloads.mlp_init(int(seed) % 1000, psc.PSC_FEATURES)
    params["b3"] = np.array([t.mean()], np.float32)
    return x, t, x.mean(axis=0), std, psc.mlp_flatten(params)


class _CostModel:
    LR = 2e-3

    def __init__(self, case, seed):
        self.x, self.t, mean, std, self.flat = _mlp_start(case, seed)
        self.epochs, self.batch = case["epochs"], case["batch"]
        self.model = psc.psc_mlp_create(0)
        psc.psc_mlp_set_norm(self.model, mean, std)

    def run(self):
        psc.psc_mlp_set_params(self.model, self.flat)
        losses = psc.psc_mlp_train(self.model, self.x, self.t, epochs=self.epochs, batch=self.batch, lr=self.LR)
        return [psc.psc_mlp_get_params(self.model), losses]

    def __del__(self):
        psc.psc_mlp_destroy(self.model)


# --- the interface --------------------------------------------------------------------------------

def prepare(case, seed):
    if case["family"] == "costmodel":
        return _CostModel(case, seed)
    return _HostIO(case, seed) if case.get("hostio") else _Resident(case, seed)


def run(state):
    return state.run()


def work(case):
    if case["family"] == "costmodel":
        # per sample and pass: forward, backward (twice the forward) and the forward of the epoch's
        # loss, 2 * 5057 operations each; samples read twice per pass, parameters once in and out
        n, e = case["samples"], case["epochs"]
        return {"bytes": float(n * (psc.PSC_FEATURES + 1) * 4 + 2 * psc.PSC_MLP_PARAMS * 4),
                "flops": float(2 * psc.PSC_MLP_PARAMS * 4 * n * e)}
    specs, outs = _specs(case)
    total, flops, seen = 0, 0.0, set()
    for i, (sp, names) in enumerate(zip(specs, outs)):
        by = {b["name"]: b for b in sp["buffers"]}
        for n in workloads.host_inputs_of(sp) + list(names):
            key = n if n.startswith("W") else (i, n)   # a batch's weights are shared
            if key not in seen:
                seen.add(key)
                total += by[n]["rows"] * by[n]["cols"] * BYTES[by[n]["dtype"]]
        for k in sp["kernels"]:
            a, o = by[k["inputs"][0]], by[k["outputs"][0]]
            elems = o["rows"] * o["cols"]
            flops += {"gemm": 2.0 * elems * a["cols"], "softmax": 4.0 * elems, "add": 1.0 * elems,
                      "transpose": 0.0}[k["kind"]]
    return {"bytes": float(total), "flops": float(flops)}


def exact(case, seed):
    if case["family"] == "costmodel":
        return _exact_costmodel(case, seed)
    specs, outs = _specs(case)
    inputs = _inputs(case, specs, seed)
    got = []
    for sp, names, have in zip(specs, outs, inputs):
        by = {b["name"]: b for b in sp["buffers"]}
        store = {}

        def at(name):
            b, r0, c0 = by[name], 0, 0
            rows, cols = b["rows"], b["cols"]
            while b["view_of"] is not None:
                r0, c0, b = r0 + b["row_off"], c0 + b["col_off"], by[b["view_of"]]
            if b["name"] not in store:
                t = have.get(b["name"])
                store[b["name"]] = (torch.zeros((b["rows"], b["cols"]), dtype=torch.float64, device="cuda")
                                    if t is None else t.double())
            return store[b["name"]][r0:r0 + rows, c0:c0 + cols]

        last = {}   # the last kernel that touches a root, so that its storage can be let go
        for i, k in enumerate(sp["kernels"]):
            for n in k["inputs"] + k["outputs"]:
                b = by[n]
                while b["view_of"] is not None:
                    b = by[b["view_of"]]
                last[b["name"]] = i
        for i, k in enumerate(sp["kernels"]):
            a = at(k["inputs"][0])
            if k["kind"] == "gemm":
                r = (a @ at(k["inputs"][1])) * k.get("alpha", 1.0)
            elif k["kind"] == "transpose":
                r = a.t()
            elif k["kind"] == "softmax":
                r = torch.softmax(a, dim=1)
            else:
                r = a + at(k["inputs"][1])
            at(k["outputs"][0]).copy_(r)
            for n in [n for n, j in last.items() if j == i and n not in names]:
                store.pop(n, None)
        got += [store[n] for n in names]
    return got


def _exact_costmodel(case, seed):
    x, t, mean, std, flat = _mlp_start(case, seed)
    # the scale of a feature is the 32-bit reciprocal of its deviation, as the model keeps it
    inv = (np.float32(1.0) / std).astype(np.float64)
    xn = torch.from_numpy((x.astype(np.float64) - mean.astype(np.float64)) * inv)
    y = torch.from_numpy(t.astype(np.float64))
    p = {k: torch.from_numpy(v.astype(np.float64)) for k, v in psc.mlp_unflatten(flat).items()}
    order = [k for k, _ in psc.MLP_LAYOUT]
    m = {k: torch.zeros_like(v) for k, v in p.items()}
    v2 = {k: torch.zeros_like(v) for k, v in p.items()}
    b1, b2, eps = 0.9, 0.999, 1e-8
    lr, b1, b2, eps = (float(np.float32(v)) for v in (_CostModel.LR, b1, b2, eps))

    def forward(a):
        z1 = a @ p["W1"].t() + p["b1"]
        z2 = z1.clamp(min=0) @ p["W2"].t() + p["b2"]
        return z1, z2, z2.clamp(min=0) @ p["W3"].t()[:, 0] + p["b3"]

    losses, step, n, batch = [], 0, case["samples"], case["batch"]
    for _ in range(case["epochs"]):
        for s in range(0, n, batch):
            a, tt = xn[s:s + batch], y[s:s + batch]
            z1, z2, out = forward(a)
            dy = (2.0 / len(tt)) * (out - tt)
            dz2 = dy[:, None] * p["W3"] * (z2 > 0)
            dz1 = (dz2 @ p["W2"]) * (z1 > 0)
            g = {"W1": dz1.t() @ a, "b1": dz1.sum(0), "W2": dz2.t() @ z1.clamp(min=0), "b2": dz2.sum(0),
                 "W3": (dy[None, :] @ z2.clamp(min=0)), "b3": dy.sum()[None]}
            step += 1
            for k in order:
                m[k] = b1 * m[k] + (1 - b1) * g[k]
                v2[k] = b2 * v2[k] + (1 - b2) * g[k] * g[k]
                p[k] = p[k] - lr * (m[k] / (1 - b1 ** step)) / ((v2[k] / (1 - b2 ** step)).sqrt() + eps)
        losses.append(((forward(xn)[2] - y) ** 2).mean())
    return [torch.cat([p[k].reshape(-1) for k in order]).numpy(), torch.stack(losses).numpy()]
