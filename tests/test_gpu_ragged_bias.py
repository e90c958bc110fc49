"""Dense bias with a sequence length that is no multiple of 4: the rows of the bias start at any
2-byte boundary and, for an odd length, the matrix ends inside a dword.  Lengths around the edges of
the 64-column bias tiles, every head size, both masks, both work-group shapes, against the oracle
and bit for bit across k."""
import numpy as np
import pytest

from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def _cfg(S, D=32, mask=None, B=3, H=2, **kw):
    return dict(seed=900 + S, B=B, H=H, S=S, D=D, dtype="bf16", bias="dense", mask=mask, gated=True, axis="row", **kw)


@pytest.mark.parametrize("mask", [None, "causal"])
@pytest.mark.parametrize("S,D", [(65, 32), (66, 32), (95, 32), (127, 32), (129, 32), (193, 32), (322, 32), (131, 64), (67, 128)])
def test_matches_oracle(S, D, mask):
    print(f"ragged bias S={S} D={D} mask={mask}", flush=True)
    check_against_oracle(_cfg(S, D, mask), k=2)


@pytest.mark.parametrize("cfg", [_cfg(201, layout="sbhd"), _cfg(131, B=70, H=1), _cfg(515, 64, "causal", B=2, H=1), _cfg(577, B=14, H=4)],
                         ids=["transposed", "row_groups", "long_small_share", "long_mid_share"])
def test_same_bits_for_every_k_and_the_oracle(cfg):
    ref = None
    for k in (1, 2):
        print(f"ragged bias S={cfg['S']} k={k}", flush=True)
        dc, _ = run_case(cfg, k=k)
        outs = {n: getattr(dc, n).detach().float().cpu().numpy() for n in ("Y", "dQ", "dK", "dV", "dG", "dBias", "lse")}
        ref = ref or outs
        for n in outs:
            assert np.array_equal(outs[n], ref[n], equal_nan=True), (k, n)
    check_against_oracle(cfg, k=2)
