"""Short rows where a block of 16 tokens, or a group of eight, begins or ends.  With a causal mask, with a bias in fp32 next to bf16 tensors and up to
16 tokens, one wavefront takes a row (small_kernels.hip) and leaves out the registers of the last group of eight up to 56 tokens; with no mask or
regions, and a bf16 bias, a wavefront takes 16 tokens (win_fwd.hip, win_bwd.hip)."""
import numpy as np
import pytest

from oracle import attention as orc
from paper_2301_08984_amd import binding as ss
from paper_2301_08984_amd.runner import DeviceCase
from paper_2301_08984_amd.workloads import make_inputs
from parity import AXIS, TOL, assert_close, check_against_oracle, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [31, 33, 48, 55, 56, 57, 64])
@pytest.mark.parametrize("mask", [None, "causal"])
def test_dense_bias(S, mask):
    print(f"short rows of {S} tokens", flush=True)
    check_against_oracle(dict(seed=1500 + S, B=9, H=3, S=S, D=32, dtype="bf16", bias="dense", mask=mask, axis="row"), k=2)


@pytest.mark.parametrize("win,mask", [((7, 8), None), ((3, 19), None), ((7, 7), "region"), ((8, 8), "region"), ((3, 3), "region"), ((4, 4), "region")])
def test_windows(win, mask):
    print(f"windows of {win}", flush=True)
    check_against_oracle(dict(seed=1520 + win[0], B=20, H=2, S=win[0] * win[1], D=32, dtype="bf16", bias="relpos", win=win, mask=mask, axis="row"), k=3)


@pytest.mark.parametrize("regions", [False, True])
@pytest.mark.parametrize("S,win", [(15, (3, 5)), (16, None), (16, (4, 4)), (49, (7, 7)), (56, None), (57, None), (64, (8, 8)), (64, None)])
def test_a_bias_in_fp32(S, win, regions):
    """A bias in fp32 (of values that bf16 holds too) with bf16 tensors; three regions in odd rows, one in even ones, of which some begin a
    wavefront's rows."""
    cfg = dict(seed=1540 + S, B=20, H=2, S=S, D=32, dtype="bf16", bias="relpos" if win else "dense", win=win, axis="row")
    inp = make_inputs(**cfg)
    if regions:
        ids = np.zeros((4, S), np.int32)
        ids[1::2] = np.arange(S) * 3 // S
        inp["region_ids"], cfg["mask"] = ids, "region"
    dc = DeviceCase(inp, dtype="bf16", bias=cfg["bias"], mask=cfg.get("mask"), win=win)
    dc.bias = dc.bias.float()
    p = oracle_problem(inp, cfg)
    Y, lse = orc.attn_forward(p, AXIS["row"], 0, cfg["B"])
    ref = dict(orc.attn_backward(p, inp["dY"].astype(np.float64), AXIS["row"], 0, cfg["B"]), Y=Y)
    for k in (1, 3):
        print(f"fp32 bias, {S} tokens, window {win}, regions {regions}, k={k}", flush=True)
        d = dc.desc("row", 0, cfg["B"], k)
        d.bias_dtype = ss.SS_F32
        dc.fwd(d)
        dc.bwd(d, poison=True)
        assert float(np.max(np.abs(dc.host("lse") - lse))) <= 4 * TOL["bf16"]
        for n in ("Y", "dQ", "dK", "dV", "dBias"):
            assert_close(n, dc.host(n), ref[n], TOL["bf16"])
