"""Few tokens against weights too large for the few-rows kernel: the 64 x 128 tile at the edges of its rows and of the five stages of its ring, with chunks (of
which all but the first continue a sum with the larger tile) and exact sums.  Against the oracle, and bit for bit with a captured call, which has no scratch for the parts."""
import numpy as np
import pytest

from oracle import ffn as orc
from paper_2301_08984_amd.workloads import make_ffn_inputs
from parity import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,dm,dh,k,flags", [(1, 4616, 3720, 1, 0), (16, 8008, 2120, 1, 0), (33, 4104, 4104, 2, 0), (64, 3080, 5512, 1, 0), (17, 4616, 3720, 3, 1)])
def test_forward(T, dm, dh, k, flags):
    import torch
    from paper_2301_08984_amd.runner import FfnCase
    inp = make_ffn_inputs(seed=4100 + T, T=T, dm=dm, dh=dh, lo=0, hi=dh, act="gelu")
    fc = FfnCase(inp, act="gelu")
    d = fc.desc(0, dh, k, flags)
    print(f"large weights {T} x {dm} x {dh} k={k}", flush=True)
    fc.fwd(d, poison=True)
    torch.cuda.synchronize()
    p = orc.FfnProblem(inp["X"], inp["W1"], inp["b1"], inp["W2"], inp["b2"], orc.ACT_GELU_TANH)
    assert rel_err(fc.host("Y"), orc.ffn_forward(p, 0, dh)) <= 2e-2
    eager = fc.Y.clone()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        fc.fwd(d)
    for rep in range(2):
        fc.Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(fc.Y, eager), rep
