"""GPU test of the summation order of the device executor's FP32 products: a long K is summed by parts,
so that what one part rounds away is not lost in every other."""
import numpy as np
import pytest

import paper_2009_07482_amd as psc
from gpu_helpers import one_kernel_spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1023, 513), (1024, 512), (130, 70)])
@pytest.mark.parametrize("k", [63, 64, 65, 256, 511, 513, 1001, 2050])
def test_small_terms_are_kept_from_the_second_part_on(m, n, k):
    """1 + 2^-27 + 2^-27 + ...: each small term alone is less than half an ulp of 1 and is rounded away
    where it is added to the first one; summed apart from it they are exact.  A quarter of K (in steps
    of 16) may be lost that way, and each of the sums of the parts rounds once more."""
    a = np.ones((m, k), np.float32)
    b = np.full((k, n), 2.0 ** -27, np.float32)
    b[0] = 1.0
    want = 1.0 + (k - 1) * 2.0 ** -27
    quarter = ((k + 3) // 4 + 15) // 16 * 16
    bound = quarter * 2.0 ** -27 + max(4, -(-k // 128)) * 2.0 ** -24
    out, _ = psc.run_spec(one_kernel_spec("gemm", [(m, k), (k, n), (m, n)], ["f32"] * 3), {"A": a, "B": b}, "device")
    off = np.abs(out["C"].astype(np.float64) - want).max()
    print(f"{m}x{n}x{k}: off by {off:.2e}, bound {bound:.2e}, every small term {(k - 1) * 2.0 ** -27:.2e}", flush=True)
    assert off <= bound
