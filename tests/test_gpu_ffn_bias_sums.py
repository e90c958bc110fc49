"""The bias gradients' column sums are not one long chain of fp32 additions: a large entry that a later one cancels
costs the small entries near it, not all of them."""
import numpy as np
import pytest

from paper_2301_08984_amd.workloads import make_ffn_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,dm,dh", [(8192, 1536, 1536), (4096, 2304, 1152)])
def test_large_entries_that_cancel(T, dm, dh):
    import torch
    from paper_2301_08984_amd.runner import FfnCase
    print(f"bias sums {T} {dm} {dh}", flush=True)
    inp = make_ffn_inputs(seed=5, T=T, dm=dm, dh=dh, lo=0, hi=dh, act="relu")
    small, big = 2.0 ** -9, 2.0 ** 16   # fp32 holds 2^16 in steps of 2^-7: two small entries are half a step
    dY = np.full((T, dm), small, np.float32)
    dY[0], dY[T - 16] = big, -big
    inp["dY"] = dY
    fc = FfnCase(inp, act="relu")
    fc.bwd(fc.desc(0, dh, 1))
    torch.cuda.synchronize()
    want = small * (T - 2)
    # each large entry costs the small ones of its own turn of the ring at most (192 rows, half of them in its
    # lane), and the result is rounded to bf16
    bound = 2 * 96 * small + want * 2.0 ** -8
    got = fc.host("db2")
    assert np.max(np.abs(got - want)) <= bound, (want, float(got.min()), float(got.max()))
