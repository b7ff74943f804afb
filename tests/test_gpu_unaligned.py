"""Kernels on operands of no common alignment: odd leading dimensions and windows that start at odd
rows and columns, at widths around a 16-byte vector and a tile.  Every GEMM tile and dtype, against
exact results (ternary operands), and softmax, transpose and add."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
from oracle.bf16 import round_bf16, round_f32
from gpu_helpers import normwise, oracle_outputs, uniform

pytestmark = pytest.mark.gpu


def _window(name, dt, rows, cols, pad):
    """A root of odd width and the rows x cols window of it at an odd offset."""
    width = cols + 2 * pad + 1
    return [{"name": name + "r", "dtype": dt, "rows": rows + pad, "cols": width, "view_of": None, "row_off": 0,
             "col_off": 0},
            {"name": name, "dtype": dt, "rows": rows, "cols": cols, "view_of": name + "r", "row_off": pad,
             "col_off": pad}]


def _embed(value, spec, name):
    b = {x["name"]: x for x in spec["buffers"]}
    v, r = b[name], b[name + "r"]
    out = np.full((r["rows"], r["cols"]), 7.0, np.float32)   # what lies around a window must not matter
    out[v["row_off"]:v["row_off"] + v["rows"], v["col_off"]:v["col_off"] + v["cols"]] = value
    return out


SHAPES = [(5, 1, 3), (33, 7, 9), (70, 9, 65), (64, 65, 64), (130, 66, 127), (257, 129, 200)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("tile", list(range(1, psc.psc_gemm_tile_count())))
def test_gemm_windows_exact(dt, tile):
    g = np.random.default_rng(40 + tile)
    for m, n, k in SHAPES:
        for pad in (1, 3):
            print(f"gemm {dt} {m}x{n}x{k} tile {tile} pad {pad}", flush=True)
            spec = {"buffers": _window("A", dt, m, k, pad) + _window("B", dt, k, n, pad) + _window("C", "f32", m, n, pad),
                    "kernels": [{"name": "k", "kind": "gemm", "inputs": ["A", "B"], "outputs": ["C"], "alpha": 1.0,
                                 "tile": tile}], "edges": [], "component": [0]}
            a = g.integers(-1, 2, (m, k)).astype(np.float32)
            b = g.integers(-1, 2, (k, n)).astype(np.float32)
            out, _ = psc.run_spec(spec, {"Ar": _embed(a, spec, "A"), "Br": _embed(b, spec, "B")}, "coarse")
            np.testing.assert_array_equal(out["C"], a.astype(np.float64) @ b.astype(np.float64))


@pytest.mark.parametrize("out_dt", ["f32", "bf16"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("policy,tile", [("coarse", t) for t in range(psc.psc_gemm_tile_count())] + [("device", 0)])
def test_gemm_stores_stay_in_their_columns(policy, tile, dt, out_dt):
    """Products into neighbouring column windows of one matrix, of every width modulo the four
    columns that a lane stores: exact, so no store reaches into the window to its right."""
    g = np.random.default_rng(70 + tile)
    m, k, widths = 37, 9, (67, 1, 66, 2, 65, 3, 4)    # sums of nine ternary products: exact in bf16
    spec = {"buffers": [{"name": "A", "dtype": dt, "rows": m, "cols": k, "view_of": None, "row_off": 0, "col_off": 0},
                        {"name": "C", "dtype": out_dt, "rows": m, "cols": sum(widths), "view_of": None, "row_off": 0,
                         "col_off": 0}],
            "kernels": [], "edges": [], "component": [0] * len(widths)}
    a = g.integers(-1, 2, (m, k)).astype(np.float32)
    inp, at = {"A": a}, 0
    for i, n in enumerate(widths):
        spec["buffers"] += [{"name": f"B{i}", "dtype": dt, "rows": k, "cols": n, "view_of": None, "row_off": 0,
                             "col_off": 0},
                            {"name": f"C{i}", "dtype": out_dt, "rows": m, "cols": n, "view_of": "C", "row_off": 0,
                             "col_off": at}]
        spec["kernels"].append({"name": f"k{i}", "kind": "gemm", "inputs": ["A", f"B{i}"], "outputs": [f"C{i}"],
                                "alpha": 1.0, "tile": tile})
        inp[f"B{i}"] = g.integers(-1, 2, (k, n)).astype(np.float32)
        at += n
    print(f"gemm {dt} -> {out_dt} tile {tile} {policy}", flush=True)
    out, _ = psc.run_spec(spec, inp, policy)
    for i in range(len(widths)):
        np.testing.assert_array_equal(out[f"C{i}"], a.astype(np.float64) @ inp[f"B{i}"].astype(np.float64))


@pytest.mark.parametrize("policy", ["coarse", "device"])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("r,c,pad", [(3, 1, 1), (65, 7, 3), (9, 257, 1), (66, 515, 3), (5, 1001, 1), (4, 2047, 3)])
def test_elementwise_windows(policy, dt, r, c, pad):
    print(f"elementwise {dt} {r}x{c} pad {pad} {policy}", flush=True)
    names = [("A", r, c), ("B", r, c), ("S", r, c), ("P", r, c), ("T", c, r)]
    spec = {"buffers": [b for n, h, w in names for b in _window(n, dt, h, w, pad)],
            "kernels": [{"name": "s", "kind": "add", "inputs": ["A", "B"], "outputs": ["S"], "alpha": 1.0, "tile": 0},
                        {"name": "p", "kind": "softmax", "inputs": ["A"], "outputs": ["P"], "alpha": 1.0, "tile": 0},
                        {"name": "t", "kind": "transpose", "inputs": ["A"], "outputs": ["T"], "alpha": 1.0, "tile": 0}],
            "edges": [], "component": [0, 0, 0]}
    a, b = uniform(51, (r, c), -3, 3), uniform(52, (r, c))
    inp = {"Ar": _embed(a, spec, "A"), "Br": _embed(b, spec, "B")}
    out, _ = psc.run_spec(spec, inp, policy)
    if dt == "bf16":
        a, b = round_bf16(a), round_bf16(b)
    s = a.astype(np.float64) + b.astype(np.float64)
    np.testing.assert_array_equal(out["S"], round_bf16(round_f32(s)) if dt == "bf16" else round_f32(s))
    np.testing.assert_array_equal(out["T"], np.asarray(a, np.float64).T)
    # FP32 exponentials and sums (~1e-7 each), and for BF16 output the rare rounding they flip
    assert normwise(out["P"], oracle_outputs(spec, inp, emulate=True)["P"]) < (1e-5 if dt == "f32" else 1e-3)


@pytest.mark.parametrize("out_dt", ["f32", "bf16"])
@pytest.mark.parametrize("m,n,k", [(128, 128, 64), (129, 127, 1), (257, 130, 65), (64, 300, 255), (130, 1, 128),
                                   (256, 384, 200)])
def test_executor_short_products_exact(m, n, k, out_dt):
    """Products of K < 256 on the device executor, in DAGs narrow and wide enough that its tiles are
    the smallest and the largest: exact."""
    g = np.random.default_rng(90)
    for width in (1, 96):
        spec = {"buffers": [], "kernels": [], "edges": [], "component": list(range(width))}
        inp, want = {}, {}
        for i in range(width):
            pad = i % 2
            spec["buffers"] += _window(f"A{i}", "bf16", m, k, pad) + _window(f"B{i}", "bf16", k, n, pad) + \
                _window(f"C{i}", out_dt, m, n, pad)
            spec["kernels"].append({"name": f"k{i}", "kind": "gemm", "inputs": [f"A{i}", f"B{i}"],
                                    "outputs": [f"C{i}"], "alpha": 1.0, "tile": 0})
            a = g.integers(-1, 2, (m, k)).astype(np.float32)
            b = g.integers(-1, 2, (k, n)).astype(np.float32)
            inp[f"A{i}r"], inp[f"B{i}r"] = _embed(a, spec, f"A{i}"), _embed(b, spec, f"B{i}")
            want[f"C{i}"] = a.astype(np.float64) @ b.astype(np.float64)   # |sums| <= 255: exact in bf16
        print(f"executor {m}x{n}x{k} -> {out_dt}, {width} kernels", flush=True)
        out, _ = psc.run_spec(spec, inp, "device")
        for name, w in want.items():
            np.testing.assert_array_equal(out[name], w)


@pytest.mark.parametrize("dt,out_dt", [("f32", "f32"), ("f32", "bf16"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("c", [256, 512, 1024, 2048])
def test_executor_softmax_of_whole_rows(c, dt, out_dt):
    """Rows that fill the executor's registers exactly and rows one short of it, over whole and partial
    tasks of 16 rows, with entries of -inf: the same as each row by itself (another matrix, whose
    rows start elsewhere in their task)."""
    for r in (16, 33):
        for cols in (c, c - 1):
            print(f"executor softmax {r}x{cols} {dt} -> {out_dt}", flush=True)
            spec = {"buffers": [], "kernels": [], "edges": [], "component": [0, 1]}
            x = uniform(91, (r, cols), -8, 8)
            x[::3, 5] = -np.inf
            inp = {}
            for n, v in (("A", x), ("B", x[::-1])):
                spec["buffers"] += _window(n, dt, r, cols, 1) + _window("P" + n, out_dt, r, cols, 3)
                spec["kernels"].append({"name": "k" + n, "kind": "softmax", "inputs": [n], "outputs": ["P" + n],
                                        "alpha": 1.0, "tile": 0})
                inp[n + "r"] = _embed(v, spec, n)
            out, _ = psc.run_spec(spec, inp, "device")
            np.testing.assert_array_equal(out["PA"], out["PB"][::-1])
            xr = (round_bf16(x) if dt == "bf16" else x).astype(np.float64)
            e = np.exp(xr - xr.max(axis=1, keepdims=True))
            # FP32 exponentials and a sum of up to 2048 terms; BF16 output: half a unit of 2^-8
            err = np.abs(out["PA"] - e / e.sum(axis=1, keepdims=True)) / (e / e.sum(axis=1, keepdims=True)).max()
            assert err.max() < (1e-5 if out_dt == "f32" else 2.0 ** -8)
