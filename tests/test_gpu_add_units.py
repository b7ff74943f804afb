"""GPU tests of the add kernel's units of eight columns: rows shorter and longer than a unit and than a
block, results exact and inside their window, and the time of ragged rows beside whole ones."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
from gpu_helpers import one_kernel_spec, uniform
from oracle.bf16 import round_bf16, round_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policy", ["coarse", "device"])
@pytest.mark.parametrize("dt,out_dt", [("f32", "f32"), ("f32", "bf16"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("r,widths", [(1, (1, 3, 2)), (5, (7, 8, 9)), (300, (15, 17, 1)), (33, (2047, 2049, 5)),
                                      (9, (2040, 2056, 2171)), (1000, (4, 6, 1)), (257, (248, 255, 256)),
                                      (2011, (9, 100, 4104))])
def test_sums_are_exact_and_stay_in_their_window(r, widths, dt, out_dt, policy):
    """Sums into neighbouring column windows of one matrix: a store beyond a row's end would land in
    the next window, and one that starts late would leave a gap."""
    print(f"add {r}x{widths} {dt} -> {out_dt} {policy}", flush=True)
    spec = {"buffers": [{"name": "C", "dtype": out_dt, "rows": r, "cols": sum(widths), "view_of": None, "row_off": 0,
                         "col_off": 0}], "kernels": [], "edges": [], "component": [0] * len(widths)}
    inp, want, at = {}, {}, 0
    for i, n in enumerate(widths):
        for x in "AB":
            # operands are windows that end with their matrix's last row: nothing lies behind them
            spec["buffers"] += [{"name": f"{x}{i}r", "dtype": dt, "rows": r, "cols": n + 1, "view_of": None,
                                 "row_off": 0, "col_off": 0},
                                {"name": f"{x}{i}", "dtype": dt, "rows": r, "cols": n, "view_of": f"{x}{i}r",
                                 "row_off": 0, "col_off": 1}]
            inp[f"{x}{i}r"] = uniform(10 * i + ord(x), (r, n + 1), -3, 3)
        spec["buffers"].append({"name": f"C{i}", "dtype": out_dt, "rows": r, "cols": n, "view_of": "C", "row_off": 0,
                                "col_off": at})
        spec["kernels"].append({"name": f"k{i}", "kind": "add", "inputs": [f"A{i}", f"B{i}"], "outputs": [f"C{i}"],
                                "alpha": 1.0, "tile": 0})
        a, b = inp[f"A{i}r"][:, 1:], inp[f"B{i}r"][:, 1:]
        if dt == "bf16":
            a, b = round_bf16(a), round_bf16(b)
        s = round_f32(a.astype(np.float64) + b.astype(np.float64))
        want[f"C{i}"] = round_bf16(s) if out_dt == "bf16" else s
        at += n
    out, _ = psc.run_spec(spec, inp, policy)
    for name, w in want.items():
        np.testing.assert_array_equal(out[name], w, err_msg=name)


def _timed_in_turn(specs, rounds=6):
    """Microseconds of each one-kernel spec, the least of several rounds that take them in turn."""
    dags = [psc.build_dag(sp) for sp in specs]
    scheds = [psc.psc_schedule(d, "coarse") for d in dags]
    for s in scheds:
        psc.psc_sched_prepare(s)
        psc.psc_kernel_time(s, 0, 200)
    us = [min(t) for t in zip(*[[psc.psc_kernel_time(s, 0, 30) for s in scheds] for _ in range(rounds)])]
    for s, d in zip(scheds, dags):
        psc.psc_sched_destroy(s)
        psc.psc_dag_destroy(d)
    return us


@pytest.mark.parametrize("r,c,dt", [(6472, 2171, "f32"), (7240, 12, "bf16"), (5846, 164, "f32")])
def test_ragged_rows_take_the_time_of_long_ones(r, c, dt):
    """As many elements in rows of 2048, which fill every block."""
    ragged, even = _timed_in_turn([one_kernel_spec("add", [shape] * 3, [dt, dt, "f32"])
                                   for shape in ((r, c), ((r * c + 2047) // 2048, 2048))])
    print(f"add {r}x{c}: {ragged:.2f} us, in rows of 2048: {even:.2f} us", flush=True)
    assert ragged <= 1.3 * even
