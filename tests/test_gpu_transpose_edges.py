"""GPU tests of the transpose kernels' edge tiles: every tile shape at matrices narrower, shorter and
just larger than it, exact and inside their window, and the time of large matrices that are all edge."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
from gpu_helpers import one_kernel_spec, uniform
from oracle.bf16 import round_bf16

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 70), (70, 3), (15, 300), (300, 15), (64, 65), (65, 64), (129, 257), (63, 130), (200, 5),
          (64, 256), (128, 64), (7, 8), (9, 4)]


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("policy,tile", [("coarse", t) for t in range(5)] + [("device", 0)])
def test_edges_are_exact_and_stay_in_their_window(policy, tile, dt):
    """Transposes into neighbouring column windows of one matrix, from windows that end with their
    matrix's last row."""
    print(f"transpose {dt} tile {tile} {policy}", flush=True)
    height = max(c for _, c in SHAPES)
    spec = {"buffers": [{"name": "T", "dtype": dt, "rows": height, "cols": sum(r for r, _ in SHAPES), "view_of": None,
                         "row_off": 0, "col_off": 0}], "kernels": [], "edges": [], "component": [0] * len(SHAPES)}
    inp, want, at = {}, {}, 0
    for i, (r, c) in enumerate(SHAPES):
        spec["buffers"] += [{"name": f"A{i}r", "dtype": dt, "rows": r + 1, "cols": c + 1, "view_of": None,
                             "row_off": 0, "col_off": 0},
                            {"name": f"A{i}", "dtype": dt, "rows": r, "cols": c, "view_of": f"A{i}r", "row_off": 1,
                             "col_off": 1},
                            {"name": f"T{i}", "dtype": dt, "rows": c, "cols": r, "view_of": "T", "row_off": height - c,
                             "col_off": at}]
        spec["kernels"].append({"name": f"k{i}", "kind": "transpose", "inputs": [f"A{i}"], "outputs": [f"T{i}"],
                                "alpha": 1.0, "tile": tile})
        inp[f"A{i}r"] = uniform(60 + i, (r + 1, c + 1), -3, 3)
        a = inp[f"A{i}r"][1:, 1:]
        want[f"T{i}"] = (round_bf16(a) if dt == "bf16" else a).T
        at += r
    out, _ = psc.run_spec(spec, inp, policy)
    for name, w in want.items():
        np.testing.assert_array_equal(out[name], w, err_msg=name)


def _us(kind, shapes, dtypes):
    dag = psc.build_dag(one_kernel_spec(kind, shapes, dtypes))
    s = psc.psc_schedule(dag, "coarse")
    psc.psc_sched_prepare(s)
    psc.psc_kernel_time(s, 0, 2)
    us = min(psc.psc_kernel_time(s, 0, 5) for _ in range(3))
    psc.psc_sched_destroy(s)
    psc.psc_dag_destroy(dag)
    return us


@pytest.mark.parametrize("r,c", [(4500000, 15), (15, 4500000), (4500000, 16), (5000003, 17)])
def test_long_narrow_matrices_take_the_time_of_a_copy(r, c):
    """Of at least 256 MiB, where the rectangular tiles would be nearly all outside the matrix: within
    four times what an add of two matrices half as large takes (which moves three quarters of the bytes)."""
    moved = _us("transpose", [(r, c), (c, r)], ["f32"] * 2)
    add = _us("add", [(r * c // 4096, 2048)] * 3, ["f32"] * 3)
    print(f"transpose {r}x{c}: {moved:.1f} us, add of half as many: {add:.1f} us", flush=True)
    assert moved <= 4 * add
