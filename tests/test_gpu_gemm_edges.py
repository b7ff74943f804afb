"""GPU tests of the GEMM tiles' edge path: every K around a step and a vector and every N around a
vector, exact, with NaN around the operand windows (nothing outside a window may reach a sum), and
the time of short products beside longer ones."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
from gpu_helpers import one_kernel_spec

pytestmark = pytest.mark.gpu

KS = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 100, 127, 129, 191, 257, 300]
NS = [1, 3, 4, 5, 7, 8, 9, 17, 33, 65, 70]


def _window(name, dt, rows, cols):
    """A window at (1, 3) that ends with its matrix's last row and column."""
    return [{"name": name + "r", "dtype": dt, "rows": rows + 1, "cols": cols + 3, "view_of": None, "row_off": 0,
             "col_off": 0},
            {"name": name, "dtype": dt, "rows": rows, "cols": cols, "view_of": name + "r", "row_off": 1, "col_off": 3}]


def _embed(value):
    out = np.full((value.shape[0] + 1, value.shape[1] + 3), np.nan, np.float32)
    out[1:, 3:] = value
    return out


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("policy,tile", [("coarse", t) for t in range(1, 13)] + [("device", 0)])
def test_products_are_exact_at_every_edge(policy, tile, dt):
    g = np.random.default_rng(200 + tile)
    cases = [(int(g.integers(1, 140)), NS[i % len(NS)], k) for i, k in enumerate(KS * 2)] + \
        [(1, 1, 1), (200, 3, 130), (129, 70, 64), (5, 7, 500)]
    spec = {"buffers": [], "kernels": [], "edges": [], "component": [0] * len(cases)}
    inp, want = {}, {}
    for i, (m, n, k) in enumerate(cases):
        spec["buffers"] += _window(f"A{i}", dt, m, k) + _window(f"B{i}", dt, k, n) + \
            [{"name": f"C{i}", "dtype": "f32", "rows": m, "cols": n, "view_of": None, "row_off": 0, "col_off": 0}]
        spec["kernels"].append({"name": f"k{i}", "kind": "gemm", "inputs": [f"A{i}", f"B{i}"], "outputs": [f"C{i}"],
                                "alpha": 1.0, "tile": tile})
        a, b = g.integers(-1, 2, (m, k)).astype(np.float32), g.integers(-1, 2, (k, n)).astype(np.float32)
        inp[f"A{i}r"], inp[f"B{i}r"] = _embed(a), _embed(b)
        want[f"C{i}"] = a.astype(np.float64) @ b.astype(np.float64)
    print(f"gemm {dt} tile {tile} {policy}: {len(cases)} products", flush=True)
    out, _ = psc.run_spec(spec, inp, policy)
    for i, c in enumerate(cases):
        np.testing.assert_array_equal(out[f"C{i}"], want[f"C{i}"], err_msg=str(c))


def _timed_in_turn(specs, rounds=12):
    """Microseconds of each one-kernel spec, the least of several rounds that take them in turn (the clock
    of a GPU that has just started to work still rises)."""
    dags = [psc.build_dag(sp) for sp in specs]
    scheds = [psc.psc_schedule(d, "coarse") for d in dags]
    for s in scheds:
        psc.psc_sched_prepare(s)
        psc.psc_kernel_time(s, 0, 2000)
    us = [min(t) for t in zip(*[[psc.psc_kernel_time(s, 0, 100) for s in scheds] for _ in range(rounds)])]
    for s, d in zip(scheds, dags):
        psc.psc_sched_destroy(s)
        psc.psc_dag_destroy(d)
    return us


@pytest.mark.parametrize("m,n,k,longer", [(64, 64, 64, 256), (512, 64, 40, 256), (64, 64, 200, 256)])
def test_a_short_product_takes_no_longer_than_a_longer_one(m, n, k, longer):
    """Four wavefronts take a 64-deep chunk each: a product of fewer or partial chunks does less.  With a
    branch per vector it took 1.35 to 1.37 times the longer one; the masks of a partial chunk cost a
    tenth of these few microseconds (1.05 to 1.14 on different cards)."""
    short, full = _timed_in_turn([one_kernel_spec("gemm", [(m, kk), (kk, n), (m, n)], ["bf16", "bf16", "f32"])
                                  for kk in (k, longer)])
    print(f"{m}x{n}x{k}: {short:.2f} us, {m}x{n}x{longer}: {full:.2f} us", flush=True)
    assert short <= 1.25 * full
