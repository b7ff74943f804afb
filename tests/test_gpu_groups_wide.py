"""GPU tests of shared launches beyond the small attention DAGs: products that walk K in steps (the
other summation order), eight streams on both dispatchers, members at the size where a kernel stops
sharing, and that launches are shared at all."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
import workloads
from gpu_helpers import uniform
from test_gpu_groups import _run_all

pytestmark = pytest.mark.gpu


def _buf(name, dt, r, c):
    return dict(name=name, dtype=dt, rows=r, cols=c, view_of=None, row_off=0, col_off=0)


def products(dt):
    """Products of one level that fill the GPU by themselves (64 x 64 to 128 x 128 tiles), of unlike
    shapes, and ones of the other summation order beside them."""
    spec = {"buffers": [], "kernels": [], "edges": [], "component": []}
    inp = {}
    for i, (m, n, k) in enumerate([(1024, 1024, 64), (1024, 1024, 64), (1000, 1100, 96), (2048, 1024, 33), (900, 1300, 256),
                                   (1024, 1024, 64), (200, 200, 512), (100, 300, 700), (1200, 1030, 65)]):
        spec["buffers"] += [_buf(f"A{i}", dt, m, k), _buf(f"B{i}", dt, k, n), _buf(f"C{i}", "f32", m, n)]
        spec["kernels"].append(dict(name=f"k{i}", kind="gemm", inputs=[f"A{i}", f"B{i}"], outputs=[f"C{i}"], alpha=0.5,
                                    tile=0))
        spec["component"].append(i)
        inp[f"A{i}"], inp[f"B{i}"] = uniform(i, (m, k)), uniform(50 + i, (k, n))
    return spec, inp


def limits(dt):
    """Element-wise kernels of 2,047 workgroups, the most that shares, of 2,048 and of one."""
    spec = {"buffers": [], "kernels": [], "edges": [], "component": []}
    inp = {}
    for i, (kind, r, c) in enumerate([("add", 2047, 2048), ("add", 2047, 2048), ("add", 2048, 2048), ("add", 1, 3),
                                      ("add", 2047, 2048), ("softmax", 8188, 64), ("softmax", 8189, 64),
                                      ("softmax", 5, 60), ("softmax", 8185, 64), ("transpose", 64 * 89, 64 * 23),
                                      ("transpose", 64 * 32, 64 * 64), ("transpose", 70, 1)]):
        o = (c, r) if kind == "transpose" else (r, c)
        spec["buffers"] += [_buf(f"A{i}", dt, r, c), _buf(f"Y{i}", dt, *o)]
        ins = [f"A{i}"]
        if kind == "add":
            spec["buffers"].append(_buf(f"B{i}", dt, r, c))
            ins.append(f"B{i}")
            inp[f"B{i}"] = uniform(70 + i, (r, c))
        spec["kernels"].append(dict(name=f"k{i}", kind=kind, inputs=ins, outputs=[f"Y{i}"], alpha=1.0, tile=0))
        spec["component"].append(i)
        inp[f"A{i}"] = uniform(i, (r, c))
    return spec, inp


SPECS = {
    "products": products, "limits": limits,
    "mha": lambda dt: (workloads.mha_spec(1024, 256, 4, 2, dt), workloads.mha_inputs(3, 1024, 256, 2)),
    "random": lambda dt: (lambda s: (s, workloads.random_dag_inputs(9, s)))(
        workloads.random_dag_spec(9, (50, 50), dim=(16, 500), dtype=dt)),
}


@pytest.mark.parametrize("dispatch", ["hip", "aql"])
@pytest.mark.parametrize("name,dt,mapper,copy,streams", [
    ("products", "bf16", "component", False, 2), ("products", "f32", "rr", True, 8), ("products", "bf16", "eft", False, 8),
    ("mha", "bf16", "component", False, 8), ("mha", "f32", "rr", False, 8), ("mha", "bf16", "rr", True, 8),
    ("random", "bf16", "component", False, 8), ("random", "f32", "eft", True, 6), ("limits", "f32", "rr", False, 1),
    ("limits", "bf16", "component", False, 2)])
def test_shared_launches_match_single_ones(name, dt, mapper, copy, streams, dispatch):
    print(f"{name} {dt} {mapper} copy {copy} {streams} streams {dispatch}", flush=True)
    spec, inp = SPECS[name](dt)
    opts = dict(n_streams=streams, mapper=mapper, copy_stream=copy, copy_roots=True, dispatch=dispatch)
    want = _run_all(spec, inp, record_ops=True, **opts)
    got = _run_all(spec, inp, **opts)
    for w, g in zip(want, got):
        for n in w:
            np.testing.assert_array_equal(g[n], w[n], err_msg=n)
            np.testing.assert_array_equal(g[n], want[0][n], err_msg=n)


@pytest.mark.parametrize("streams", [1, 3, 8])
def test_launches_are_shared(streams):
    """452 kernels, 13 launches a layer at best: far fewer packets than one dispatch per kernel."""
    spec, inp = workloads.mha_spec(256, 256, 16, 4, "bf16"), workloads.mha_inputs(1, 256, 256, 4)
    packets = []
    for record in (True, False):
        r = psc.SpecRunner(spec, "fine", n_streams=streams, mapper="component", copy_roots=True, dispatch="aql",
                           record_ops=record)
        r.set_inputs(inp)
        r.run()
        packets.append(r.run(with_inputs=False, with_outputs=False)["aql_packets"])
        r.close()
    assert packets[0] >= len(spec["kernels"]) == 452
    assert packets[1] <= packets[0] // 2
