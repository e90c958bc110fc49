"""Attention at head size 128 with two blocks per work-group.  The forward's order of every sum is that of the kernel with one,
which a share of fewer heads takes, so their results are the same bits; the backward (causal or without a mask) has two groups
where that one has four and is compared with the oracle.  Lengths with an odd number of 32-row blocks, a last block of one row
and of 31, fewer blocks than groups."""
import pytest

from paper_2301_08984_amd.workloads import make_inputs
from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,S", [(1, 12, 1985), (1, 12, 2047), (2, 23, 513), (1, 12, 2016)])
def test_two_query_blocks_give_the_bits_of_one(B, H, S):
    import torch
    cfg = dict(seed=890 + S, B=B, H=H, S=S, D=128, dtype="bf16", mask="causal", axis="head")
    print(f"query block pairs {B} x {H} x {S}", flush=True)
    inp = make_inputs(**cfg)
    whole, _ = run_case(cfg, inputs=inp)
    few, _ = run_case(cfg, inputs=inp, lo=3, hi=6)
    a, b = whole.Y[:, :, 3:6], few.Y[:, :, 3:6]
    assert bool(a.isfinite().all()) and torch.equal(a, b)
    assert torch.equal(whole.lse[:, 3:6], few.lse[:, 3:6])


# the share's work-groups: 768, 768, 864, 768, 432, 900 (causal from 544; without a mask where the last of the rounds of 512 is half full)
@pytest.mark.parametrize("B,H,S,mask,layout", [(4, 32, 65, "causal", "bshd"), (4, 32, 95, "causal", "sbhd"), (2, 16, 513, "causal", "bshd"),
                                               (4, 32, 97, None, "bshd"), (1, 16, 513, None, "bshd"), (6, 10, 289, None, "sbhd")])
def test_backward_of_two_blocks(B, H, S, mask, layout):
    print(f"backward of two blocks {B} x {H} x {S} {mask}", flush=True)
    check_against_oracle(dict(seed=895 + S, B=B, H=H, S=S, D=128, dtype="bf16", mask=mask, axis="head", layout=layout), k=2)


# shares that begin at another head or row than the first, with the forward's statistics and without
@pytest.mark.parametrize("use_lse", [False, True])
@pytest.mark.parametrize("B,H,axis", [(6, 9, "head"), (7, 8, "row")])
def test_shares_that_begin_later(B, H, axis, use_lse):
    print(f"two blocks from {axis} 1 on, statistics kept: {use_lse}", flush=True)
    check_against_oracle(dict(seed=899, B=B, H=H, S=513, D=128, dtype="bf16", mask="causal", axis=axis), lo=1, use_lse=use_lse)


@pytest.mark.parametrize("use_lse", [False, True])
@pytest.mark.parametrize("B,H,axis,mask", [(6, 9, "head", "causal"), (7, 8, "row", "causal"), (6, 10, "head", None)])
def test_chunks_one_by_one_give_the_bits_of_all_at_once(B, H, axis, mask, use_lse):
    """A captured call runs its chunks one by one, each with scratch of its own origin; an eager one runs them together."""
    import torch
    S = 513 if mask else 289
    print(f"two blocks in chunks {B} x {H} {axis} {mask}, statistics kept: {use_lse}", flush=True)
    dc, _ = run_case(dict(seed=898, B=B, H=H, S=S, D=128, dtype="bf16", mask=mask, axis=axis), lo=1, k=3, use_lse=use_lse)
    d = dc.desc(axis, 1, H if axis == "head" else B, 3)
    names = ("dQ", "dK", "dV")
    first = {n: getattr(dc, n).clone() for n in names}
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        dc.bwd(d, use_lse=use_lse)
    for rep in range(2):
        for n in names:
            getattr(dc, n).fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for n in names:
            assert torch.equal(getattr(dc, n).nan_to_num(nan=12345.0), first[n].nan_to_num(nan=12345.0)), (rep, n)
