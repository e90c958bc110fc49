"""Pair attention and windows with and without the library's copies of the bias in accumulator layout: shares large enough
for a copy give the same bits in a captured graph, which does without it (the forward of pair attention then takes one row
per wavefront instead of two, windows hold the bias in registers).  And the row maximum that is raised only when a block's sum of probabilities asks for it."""
import numpy as np
import pytest

from paper_2301_08984_amd.workloads import make_inputs, round_to_bf16
from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def _cfg(B, H, S, **kw):
    return dict(dict(seed=870 + S, B=B, H=H, S=S, D=32, dtype="bf16", bias="dense", mask=None, gated=True, axis="row"), **kw)


def _win(B, H, win, **kw):
    return _cfg(B, H, win[0] * win[1], **dict(dict(bias="relpos", win=win, gated=False), **kw))


# an odd number of rows; lengths that end right after a 64-key tile, after a 32-key block, and one entry short of it
@pytest.mark.parametrize("cfg,k", [(_cfg(901, 8, 193), 3), (_cfg(301, 6, 416, layout="sbhd"), 2), (_cfg(301, 6, 415, gated=False), 1),
                                   (_cfg(401, 5, 384, axis="head", lo=1), 2), (_win(70, 8, (12, 12), mask="region"), 2),
                                   (_win(130, 4, (10, 16), gated=True), 1), (_win(100, 6, (9, 9), mask="region"), 3),
                                   (_win(90, 6, (11, 11), bias="dense", mask="region"), 2)],
                         ids=["193", "416_sbhd", "415", "384_heads", "12x12", "10x16_gated", "9x9", "11x11_dense"])
def test_copies_give_the_same_bits(cfg, k):
    import torch
    cfg = dict(cfg)
    lo = cfg.pop("lo", 0)
    print(f"bias copies {cfg['B']} x {cfg['H']} x {cfg['S']}", flush=True)
    dc, _ = run_case(cfg, lo=lo, k=k)
    names = [n for n in ("Y", "lse", "dQ", "dK", "dV", "dG", "dBias") if getattr(dc, n) is not None]
    first = {n: getattr(dc, n).clone() for n in names}
    d = dc.desc(cfg["axis"], lo, dc.H if cfg["axis"] == "head" else dc.B, k)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        dc.fwd(d)
        dc.bwd(d)
    for rep in range(2):
        for n in names:
            getattr(dc, n).fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for n in names:
            a, b = getattr(dc, n), first[n]
            assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num()), (rep, n)


@pytest.mark.parametrize("S", [200, 257])
def test_maxima_that_grow_along_the_keys(S):
    """Scores that rise by up to 2^40 from block to block for some queries and fall for others."""
    cfg = _cfg(3, 2, S)
    inp = make_inputs(**cfg)
    rise = np.linspace(0, 4, S)[None, :, None, None]
    inp["K"] = round_to_bf16((inp["K"] * rise).astype(np.float32))
    inp["Q"] = round_to_bf16((inp["Q"] * 3).astype(np.float32))
    print(f"growing maxima S={S}", flush=True)
    # peaked rows: one probability near 1, its bf16 rounding against V and dP of the one key; the bound of the other tests holds
    check_against_oracle(cfg, inputs=inp)


@pytest.mark.parametrize("cfg", [_win(5, 2, (9, 9)), _cfg(3, 2, 130)], ids=["9x9", "130"])
def test_a_scale_that_the_bias_cannot_be_divided_by(cfg):
    """The fast kernels start a score from bias / scale, here beyond fp32 for a bias above 4: these calls go elsewhere."""
    from oracle import attention as orc
    from parity import AXIS, TOL, assert_close, oracle_problem
    inp = make_inputs(**cfg)
    inp["bias"] = round_to_bf16((inp["bias"] * (6 / np.max(np.abs(inp["bias"])))).astype(np.float32))
    print(f"scale 1.2e-38, {cfg['S']} tokens", flush=True)
    dc, _ = run_case(cfg, inputs=inp, scale=1.2e-38)
    Y, _ = orc.attn_forward(oracle_problem(inp, cfg, 1.2e-38), AXIS[cfg["axis"]], 0, cfg["B"])
    assert_close("Y", dc.host("Y"), Y, TOL["bf16"])
    for n in ("dQ", "dK", "dV", "dBias"):
        assert bool(getattr(dc, n).isfinite().all()), n
