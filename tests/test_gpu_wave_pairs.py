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
