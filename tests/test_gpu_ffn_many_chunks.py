"""As many chunks as there are units of 16 hidden columns: how many of them share a pass through the library's
scratch is computed, not searched for, and every pass fits.  Weight and bias gradients are the bits of one chunk."""
import pytest

from paper_2301_08984_amd.workloads import make_ffn_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,dh,k", [(3000, 4808, 301), (3000, 4808, 150), (1100, 16 * 977, 977), (17, 4000, 250)])
def test_many_chunks(T, dh, k):
    import torch
    from paper_2301_08984_amd.runner import FfnCase
    print(f"many chunks {T} {dh} {k}", flush=True)
    fc = FfnCase(make_ffn_inputs(seed=T + k, T=T, dm=40, dh=dh, lo=0, hi=dh, act="gelu"), act="gelu")
    outs = {}
    for n in (1, k):
        d = fc.desc(0, dh, n, 1)  # fp32 partial sums: the same bits for every k
        fc.fwd(d, poison=True)
        fc.bwd(d, poison=True)
        torch.cuda.synchronize()
        outs[n] = {o: getattr(fc, o).clone() for o in ("Y", "dX", "dW1", "db1", "dW2", "db2")}
    for o, x in outs[1].items():
        assert bool(x.isfinite().all()) and torch.equal(x, outs[k][o]), o
