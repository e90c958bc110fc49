"""Short rows where the last group of eight tokens begins or ends: up to 56 tokens the kernels leave out the registers of the last group."""
import pytest

from parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [31, 33, 48, 55, 56, 57, 64])
@pytest.mark.parametrize("mask", [None, "causal"])
def test_dense_bias(S, mask):
    print(f"short rows of {S} tokens", flush=True)
    check_against_oracle(dict(seed=1500 + S, B=9, H=3, S=S, D=32, dtype="bf16", bias="dense", mask=mask, axis="row"), k=2)


@pytest.mark.parametrize("win,mask", [((7, 8), None), ((3, 19), None), ((7, 7), "region"), ((8, 8), "region")])
def test_windows(win, mask):
    print(f"windows of {win}", flush=True)
    check_against_oracle(dict(seed=1520 + win[0], B=20, H=2, S=win[0] * win[1], D=32, dtype="bf16", bias="relpos", win=win, mask=mask, axis="row"), k=3)
