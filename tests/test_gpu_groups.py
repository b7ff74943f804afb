"""GPU tests of grouped launches: a fine schedule that groups them gives bit-identical results to
the same schedule run kernel by kernel (record_ops), with and without host copies, on both
dispatchers and every mapper."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
import workloads

pytestmark = pytest.mark.gpu


def _run_all(spec, inp, **opts):
    """Outputs of a run with host copies, then of a device-resident one."""
    r = psc.SpecRunner(spec, "fine", **opts)
    r.set_inputs(inp)
    r.run()
    first = {n: r.result(n) for n in r.out_names}
    for n in r.out_names:
        r.outputs[n].array[...] = 0
    r.run(with_inputs=False)
    second = {n: r.result(n) for n in r.out_names}
    r.run(with_inputs=False, with_outputs=False)
    third = {n: r.read_device(n) for n in r.out_names}
    r.close()
    return first, second, third


SPECS = {
    "mha": lambda dt: (workloads.mha_spec(160, 256, 4, 2, dt), workloads.mha_inputs(3, 160, 256, 2)),
    "mha_odd": lambda dt: (workloads.mha_spec(97, 128, 2, 1, dt), workloads.mha_inputs(4, 97, 128, 1)),
    "batch": lambda dt: (workloads.batch_spec([17, 64, 130, 75, 33], 128, 2, 2, dt),
                         workloads.batch_inputs(5, [17, 64, 130, 75, 33], 128, 2)),
    "random": lambda dt: (lambda s: (s, workloads.random_dag_inputs(6, s)))(
        workloads.random_dag_spec(6, (40, 40), dim=(16, 200), dtype=dt)),
}


@pytest.mark.parametrize("dispatch", ["hip", "aql"])
@pytest.mark.parametrize("name,dt,mapper,copy", [
    ("mha", "bf16", "component", False), ("mha", "f32", "rr", True), ("mha", "bf16", "eft", True),
    ("mha_odd", "f32", "component", True), ("mha_odd", "bf16", "rr", False), ("batch", "bf16", "component", False),
    ("batch", "f32", "eft", True), ("random", "bf16", "eft", False), ("random", "f32", "rr", True),
    ("random", "bf16", "component", True)])
def test_grouped_launches_match_single_ones(name, dt, mapper, copy, dispatch):
    print(f"{name} {dt} {mapper} copy {copy} {dispatch}", flush=True)
    spec, inp = SPECS[name](dt)
    opts = dict(n_streams=3, mapper=mapper, copy_stream=copy, copy_roots=True, dispatch=dispatch)
    want = _run_all(spec, inp, record_ops=True, **opts)
    got = _run_all(spec, inp, **opts)
    for w, g in zip(want, got):
        for n in w:
            np.testing.assert_array_equal(g[n], w[n], err_msg=n)
            np.testing.assert_array_equal(g[n], want[0][n], err_msg=n)
