"""Gradient of the relative-position table from the groups' partial sums: windows whose S x S sums are reduced whole, in two and in four parts, at
the edges of those, one token wide, with several slices of groups.  Reference: the fp64 oracle at the bf16
tolerances of parity.py; bit for bit the same in one chunk and in five."""
import numpy as np
import pytest

from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("win", [(1, 1), (1, 3), (2, 2), (3, 5), (4, 4), (1, 16), (5, 7), (8, 8), (1, 64), (5, 13), (1, 67), (11, 11), (1, 160)],
                         ids=lambda w: f"{w[0]}x{w[1]}")
def test_tables(win):
    cfg = dict(seed=1400 + win[0] * win[1], B=70, H=2, S=win[0] * win[1], D=32, dtype="bf16", bias="relpos", win=win, mask=None, axis="row")
    print(f"table of {win}", flush=True)
    dc, _ = check_against_oracle(cfg, k=1)
    again, _ = run_case(cfg, k=5)
    assert np.array_equal(dc.host("dBias"), again.host("dBias"))
