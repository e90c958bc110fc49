"""Windows of 65 to 160 tokens (head size 32): kernels whose scores start from the bias, here (small shares) a strip of it held in
registers; from a copy in accumulator layout see test_gpu_bias_copy.py.  Sizes at the edges of the 32-token blocks, every bias kind with and without the
region mask, gating, both split axes and transposed storage, against the oracle; bit for bit across k,
with row groups of the bias gradient that a chunk boundary cuts."""
import numpy as np
import pytest

from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def _cfg(win, B=11, H=2, mask="region", bias="relpos", **kw):
    return dict(seed=700 + win[0] * win[1], B=B, H=H, S=win[0] * win[1], D=32, dtype="bf16", bias=bias, win=win, mask=mask,
                **{"axis": "row", **kw})


CASES = {
    "9x9": _cfg((9, 9)),
    "9x9_no_mask": _cfg((9, 9), mask=None),
    "5x13_one_over_a_block": _cfg((5, 13), mask=None),
    "8x12_whole_blocks": _cfg((8, 12), mask=None),
    "10x10_heads": _cfg((10, 10), axis="head", H=3),
    "8x16_whole_blocks": _cfg((8, 16), mask=None),
    "12x12": _cfg((12, 12)),
    "12x12_gated": _cfg((12, 12), gated=True),
    "12x12_transposed": _cfg((12, 12), layout="sbhd"),
    "10x16_largest": _cfg((10, 16), mask=None),
    "11x11_dense_bias": _cfg((11, 11), bias="dense"),
    "9x9_no_bias": _cfg((9, 9), bias=None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_matches_oracle_and_same_bits_for_every_k(name):
    cfg = CASES[name]
    ref = None
    for k in (1, 3):
        print(f"window {name} k={k}", flush=True)
        check_against_oracle(cfg, k=k, use_lse=k == 3)
        dc, _ = run_case(cfg, k=k)
        outs = {n: getattr(dc, n).detach().float().cpu().numpy() for n in ("Y", "dQ", "dK", "dV", "dG", "dBias", "lse")
                if getattr(dc, n) is not None}
        ref = ref or outs
        for n in outs:
            assert np.array_equal(outs[n], ref[n], equal_nan=True), (k, n)


def test_sub_range_of_many_rows():
    """Enough rows for groups of several rows, a share that starts inside a group."""
    cfg = _cfg((9, 9), B=70, H=64, mask=None)
    print("window sub-range", flush=True)
    check_against_oracle(cfg, lo=3, hi=67, k=5)
