"""The one-kernel backward of windows at the edges of its 16-token blocks: every count of wavefronts, whole and one token over, with the row
statistics kept and without, groups of one row and of several, gated or not.  Reference: the fp64 oracle at the bf16 tolerances of parity.py."""
import numpy as np
import pytest

from paper_2301_08984_amd.workloads import make_inputs
from parity import check_against_oracle

pytestmark = pytest.mark.gpu

# windows of 17, 32, 33, 48, 49, 64, 66, 80, 84, 96, 98, 112, 114, 128, 130, 144, 147, 160 tokens: 2 to 10 wavefronts
WINS = [(1, 17), (4, 8), (3, 11), (6, 8), (7, 7), (8, 8), (6, 11), (8, 10), (7, 12), (8, 12), (7, 14), (8, 14), (6, 19), (8, 16), (10, 13), (9, 16), (7, 21), (10, 16)]


@pytest.mark.parametrize("win", WINS, ids=lambda w: f"{w[0]}x{w[1]}")
@pytest.mark.parametrize("form", ["relpos", "dense_gated", "none_heads"])
def test_edges_of_blocks(win, form):
    S = win[0] * win[1]
    kw = {"relpos": dict(bias="relpos", axis="row"), "dense_gated": dict(bias="dense", gated=True, axis="row"), "none_heads": dict(bias=None, axis="head")}[form]
    cfg = dict(seed=1200 + S, B=9, H=3, S=S, D=32, dtype="bf16", win=win, mask=None, **kw)
    inp = make_inputs(**cfg)
    if form != "relpos":  # rows of one region, of two and of three in turn
        inp["region_ids"] = (np.arange(S)[None] * np.arange(1, 4)[:, None] // S).astype(np.int32)
        cfg["mask"] = "region"
    print(f"window backward {win} {form}", flush=True)
    check_against_oracle(cfg, k=2, use_lse=form == "relpos", inputs=inp)


def test_groups_of_several_rows_with_tokens_past_the_end():
    """More rows than work-groups fit the chip at once: a group walks both buffers several times, an odd number of rows in the last."""
    cfg = dict(seed=1300, B=333, H=8, S=130, D=32, dtype="bf16", bias="relpos", win=(10, 13), mask=None, axis="row")
    print("window backward, many rows", flush=True)
    check_against_oracle(cfg, k=1)


def test_short_rows_with_a_dense_bias_and_cut_groups():
    """Dense bias of up to 64 tokens, groups of rows that chunk boundaries cut."""
    for S, k in ((17, 3), (50, 4), (64, 5)):
        cfg = dict(seed=1500 + S, B=611, H=5, S=S, D=32, dtype="bf16", bias="dense", mask=None, axis="row")
        print(f"short rows {S}", flush=True)
        check_against_oracle(cfg, lo=3, hi=600, k=k)


@pytest.mark.parametrize("win", [(8, 11), (8, 12), (7, 15), (9, 15), (12, 12), (7, 21), (10, 16)], ids=lambda w: f"{w[0]}x{w[1]}")
@pytest.mark.parametrize("gated", [True, False], ids=["gated", "plain"])
def test_several_rows_with_bias_and_regions(win, gated):
    """Blocks that are finished one at a time (AT_ONCE, DP_AGAIN): several rows a work-group, through both buffers, with masked and unmasked rows in turn."""
    S = win[0] * win[1]
    cfg = dict(seed=1700 + S, B=335, H=4, S=S, D=32, dtype="bf16", bias="relpos", win=win, mask=None, gated=gated, axis="row")
    inp = make_inputs(**cfg)
    inp["region_ids"] = (np.arange(S)[None] * np.arange(1, 4)[:, None] // S).astype(np.int32)
    cfg["mask"] = "region"
    print(f"window backward, several rows {win} {gated}", flush=True)
    check_against_oracle(cfg, k=3, inputs=inp)
