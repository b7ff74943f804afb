"""GPU test: a fine schedule on AQL queues whose launches all together exceed what one hardware queue
holds still runs, on more queues, with and without host copies."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc

pytestmark = pytest.mark.gpu


def ladder(levels, n=4):
    """Two chains that wait for each other at every level, an add on one and a transpose on the other
    (no two kernels of a level share a function): one queue is the predicted best."""
    buf = lambda name: dict(name=name, dtype="f32", rows=n, cols=n, view_of=None, row_off=0, col_off=0)
    bufs, kers, edges, comp = [buf("x"), buf("y")], [], [], []
    a, b = "x", "y"
    for i in range(levels):
        kers.append(dict(name=f"a{i}", kind="add", inputs=[a, b], outputs=[f"p{i}"]))
        kers.append(dict(name=f"t{i}", kind="transpose", inputs=[a], outputs=[f"q{i}"]))
        bufs += [buf(f"p{i}"), buf(f"q{i}")]
        if i:
            edges += [(2 * i - 2, a, 2 * i, a), (2 * i - 1, b, 2 * i, b), (2 * i - 2, a, 2 * i + 1, a)]
        a, b = f"p{i}", f"q{i}"
        comp += [0, 1]
    return {"buffers": bufs, "kernels": kers, "edges": edges, "component": comp}


# four packets bound a launch, 131,072 is the largest queue: 34,000 launches do not fit one queue
@pytest.mark.parametrize("levels", [40, 17000])
def test_more_launches_than_one_queue_holds(levels):
    r = psc.SpecRunner(ladder(levels), "fine", n_streams=2, mapper="component", dispatch="aql", copy_roots=True)
    # (any other values grow past the range of the type: a' = a + b, b' = a^T)
    zero = np.zeros((4, 4), np.float32)
    r.set_inputs({"x": zero, "y": zero})
    st = r.run()
    assert st["n_kernels"] == 2 * levels
    for n in r.out_names:
        np.testing.assert_array_equal(r.result(n), zero)
    r.run(with_inputs=False, with_outputs=False)
    r.close()
