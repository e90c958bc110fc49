"""Large shares at head size 128 without a bias: edges of the 128-token blocks, 64-token tiles and 32-token steps, kept statistics, a gate, transposed
storage."""
import pytest

from parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,S,kw", [(6, 28, 65, {}), (4, 42, 96, dict(mask="causal")), (3, 56, 97, dict(mask="causal", use_lse=True)),
                                      (2, 42, 129, dict(mask="causal", layout="sbhd")), (2, 32, 160, dict(use_lse=True)), (2, 28, 257, dict(mask="causal", gated=True)),
                                      (2, 21, 385, dict(mask="causal", use_lse=True)), (2, 20, 511, {})],
                         ids=["65", "96c", "97c_lse", "129c_sbhd", "160_lse", "257c_gated", "385c_lse", "511"])
def test_against_the_oracle(B, H, S, kw):
    kw = dict(kw)
    lse = kw.pop("use_lse", False)
    print(f"large share {B} x {H} x {S} {kw}", flush=True)
    check_against_oracle(dict(dict(seed=1600 + S, B=B, H=H, S=S, D=128, dtype="bf16", mask=None, axis="head"), **kw), k=2, use_lse=lse)
