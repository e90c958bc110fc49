"""Causal attention at head size 128 with two query blocks per work-group: the order of every sum is that of the kernel with
one, which a share of fewer heads takes, so their results are the same bits.  Lengths with an odd number of 32-row blocks,
a last block of one row and of 31, and fewer key blocks than key groups for the first queries (all causal shapes)."""
import pytest

from paper_2301_08984_amd.workloads import make_inputs
from parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,S", [(1, 12, 1985), (1, 12, 2047), (2, 23, 513), (1, 12, 2016)])
def test_two_query_blocks_give_the_bits_of_one(B, H, S):
    import torch
    cfg = dict(seed=890 + S, B=B, H=H, S=S, D=128, dtype="bf16", mask="causal", axis="head")
    print(f"query block pairs {B} x {H} x {S}", flush=True)
    inp = make_inputs(**cfg)
    whole, _ = run_case(cfg, inputs=inp)
    few, _ = run_case(cfg, inputs=inp, lo=3, hi=6)
    for n in ("Y", "dQ", "dK", "dV"):
        a, b = getattr(whole, n)[:, :, 3:6], getattr(few, n)[:, :, 3:6]
        assert bool(a.isfinite().all()) and torch.equal(a, b), n
    assert torch.equal(whole.lse[:, 3:6], few.lse[:, 3:6])
