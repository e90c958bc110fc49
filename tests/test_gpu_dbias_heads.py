"""Bias gradient of two heads per work-group: from 256 such work-groups on (here 450, 400, and 400 in four groups of rows)."""
import pytest

from parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,S,layout", [(3, 4, 901, "sbhd"), (2, 8, 640, "bshd"), (32, 8, 300, "bshd")])
def test_two_heads_per_work_group(B, H, S, layout):
    print(f"bias gradient {B} x {H} x {S}", flush=True)
    check_against_oracle(dict(seed=910 + S, B=B, H=H, S=S, D=32, dtype="bf16", bias="dense", mask=None, gated=True, axis="row", layout=layout))
