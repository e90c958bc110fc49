"""Split contractions under graph capture, where the library's buffer is not taken: a workspace with room for the
parts' sums carries them (its end is written), one without does them in turn, and the bits are the same."""
import pytest

from paper_2301_08984_amd.workloads import make_ffn_inputs

pytestmark = pytest.mark.gpu
NAMES = ("Y", "dX", "dW1", "db1", "dW2", "db2")


@pytest.mark.parametrize("T,dm,dh,k,flags", [(16, 4104, 3080, 1, 0), (100, 1032, 1544, 2, 0), (2056, 136, 200, 1, 0), (40, 1800, 4104, 1, 1)])
def test_captured_call_with_room_for_the_parts(T, dm, dh, k, flags):
    import torch
    from paper_2301_08984_amd import ffn_binding as fb
    from paper_2301_08984_amd.runner import FfnCase
    print(f"captured parts {T} {dm} {dh}", flush=True)
    fc = FfnCase(make_ffn_inputs(seed=60 + T, T=T, dm=dm, dh=dh, lo=0, hi=dh, act="gelu"), act="gelu")
    d = fc.desc(0, dh, k, flags)
    fc.fwd(d, poison=True)
    fc.bwd(d, poison=True)
    torch.cuda.synchronize()
    eager = {n: getattr(fc, n).clone() for n in NAMES}
    need = fc.ws.numel()
    for extra in (fb.SS_FFN_PARTS_BYTES, 0):
        fc.ws = torch.full((need + extra,), 0xFF, dtype=torch.uint8, device=fc.dev)
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            fc.fwd(d)
            fc.bwd(d)
        for rep in range(3):
            for n in NAMES:
                getattr(fc, n).fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for n in NAMES:
                assert torch.equal(getattr(fc, n), eager[n]), (n, rep, extra)
        used = int((fc.ws[need:] != 0xFF).sum())
        assert (used > 4096) == (extra == fb.SS_FFN_PARTS_BYTES), (used, extra)
