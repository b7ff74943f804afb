"""GPU tests of the two tile choices of a GEMM shape: tuning launches of several kernels leaves the
choice for one kernel alone near its isolated best, and tuning kernels alone does not slow the
launches of several."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
import workloads

pytestmark = pytest.mark.gpu

N, D, H = 1024, 1024, 16
OPTS = dict(n_streams=2, mapper="component", dispatch="aql", copy_roots=True)


@pytest.fixture(autouse=True)
def clean_cache():
    psc.psc_tile_cache_clear()
    yield
    psc.psc_tile_cache_clear()


def _runner(spec):
    r = psc.SpecRunner(spec, "fine", **OPTS)
    r.set_inputs(workloads.mha_inputs(1, N, D, 4))
    r.run()
    return r


def _tuned(spec, tune):
    dag = psc.build_dag(spec)
    tune(dag)
    psc.psc_dag_destroy(dag)


def test_tuning_in_a_grouping_schedule_keeps_the_tiles_of_single_launches():
    """The sixteen 1024 x 64 x 1024 products of a layer share launches, where tiles 2, 6 and 7 win;
    one such product alone on a 64 x 64 tile (sixteen blocks) takes about twice its best time."""
    spec = workloads.mha_spec(N, D, H, 1, "bf16")
    _tuned(spec, lambda dag: psc.psc_autotune_dag_in_schedule(dag, "fine", top_k=3, iters=3, **OPTS))
    tile = psc.psc_tile_cache_get(N, D // H, D, "bf16", "bf16")
    dag = psc.build_dag(spec)
    s = psc.psc_schedule(dag, "coarse")
    psc.psc_sched_prepare(s)
    used = [psc.psc_sched_kernel_tile(s, i) for i, k in enumerate(spec["kernels"]) if k["kind"] == "gemm"]
    psc.psc_sched_destroy(s)
    psc.psc_dag_destroy(dag)
    assert tile in used
    _, best_us, us = psc.psc_autotune_gemm(N, D // H, D, "bf16", "bf16", iters=50)
    print(f"single launches: tile {tile}, {us[tile]:.2f} us, best {best_us:.2f} us", flush=True)
    assert us[tile] <= 1.35 * best_us


def test_tuning_kernels_alone_does_not_slow_shared_launches():
    spec = workloads.mha_spec(N, D, H, 4, "bf16")
    runners = [_runner(spec)]   # (a schedule takes its tiles when it is prepared)
    _tuned(spec, lambda dag: psc.psc_autotune_dag(dag, iters=20))
    runners.append(_runner(spec))
    ms = zip(*[[r.run(with_inputs=False, with_outputs=False)["makespan_ms"] for r in runners] for _ in range(25)])
    untuned, tuned = (sorted(t)[12] for t in ms)
    for r in runners:
        r.close()
    print(f"fine schedule: {untuned:.3f} ms, after tuning the kernels alone {tuned:.3f} ms", flush=True)
    assert tuned <= 1.15 * untuned


def test_results_do_not_depend_on_copies_after_tuning():
    spec, inp = workloads.mha_spec(160, 256, 4, 2, "bf16"), workloads.mha_inputs(3, 160, 256, 2)
    _tuned(spec, lambda dag: psc.psc_autotune_dag_in_schedule(dag, "fine", top_k=6, iters=2, **dict(OPTS, n_streams=3)))
    r = psc.SpecRunner(spec, "fine", **dict(OPTS, n_streams=3))
    r.set_inputs(inp)
    r.run()
    first = {n: r.result(n).copy() for n in r.out_names}
    r.run(with_inputs=False, with_outputs=False)
    for n in r.out_names:
        np.testing.assert_array_equal(r.read_device(n), first[n], err_msg=n)
    r.close()
