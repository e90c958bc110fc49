"""Pair attention and windows with and without the library's copies of the bias in accumulator layout: shares large enough
for a copy give the same bits in a captured graph, which does without it (the forward of pair attention then takes one row
per wavefront instead of two, windows gather the bias).  And the row maximum that is raised only when a block's sum of probabilities asks for it: by a
scaling where the sum is moderate, by forming the block again beyond 2^26, by a look at the maximum on the blocks after that."""
import numpy as np
import pytest

from oracle import attention as orc
from paper_2301_08984_amd import binding as ss
from paper_2301_08984_amd.workloads import make_inputs, round_to_bf16
from parity import AXIS, TOL, assert_close, check_against_oracle, oracle_problem, run_case

pytestmark = pytest.mark.gpu


def _cfg(B, H, S, **kw):
    return dict(dict(seed=870 + S, B=B, H=H, S=S, D=32, dtype="bf16", bias="dense", mask=None, gated=True, axis="row"), **kw)


def _win(B, H, win, **kw):
    return _cfg(B, H, win[0] * win[1], **dict(dict(bias="relpos", win=win, gated=False), **kw))


def _table_launches(call):
    import torch
    ss.ss_attn_profile_enable(True)
    call()
    torch.cuda.synchronize()
    ss.ss_attn_profile_enable(False)
    return {n: ss.ss_attn_profile_read(i)[1] for i, n in enumerate(ss.KERNEL_NAMES)}["table_reduce"]  # (reading a slot clears it)


def _eager_and_captured(cfg, lo, k, inputs=None):
    """The outputs of an eager step, which takes the copies, and of two replays of a captured one, bit for bit."""
    import torch
    dc, _ = run_case(cfg, lo=lo, k=k, inputs=inputs)
    d = dc.desc(cfg["axis"], lo, dc.H if cfg["axis"] == "head" else dc.B, k)
    # the forward's only launch beside the attention kernel is the copy's (none of a table, or where a window has up to 128 tokens);
    # the backward makes a copy of a dense bias, and has two launches that reduce the slices of a table's gradient
    window = cfg.get("win") is not None or cfg["mask"] is not None
    rows, heads = (dc.B, dc.H - lo) if cfg["axis"] == "head" else (dc.B - lo, dc.H)
    assert _table_launches(lambda: dc.fwd(d)) == (0 if window and (cfg["bias"] == "relpos" or cfg["S"] <= 128) else 1)
    if window:
        assert _table_launches(lambda: dc.bwd(d)) == (2 if cfg["bias"] == "relpos" else 1)
    else:
        assert rows * heads * cfg["S"] ** 2 >= 2 ** 28
    names = [n for n in ("Y", "lse", "dQ", "dK", "dV", "dG", "dBias") if getattr(dc, n) is not None]
    first = {n: getattr(dc, n).clone() for n in names}
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
    return dc


# an odd number of rows; lengths that end right after a 64-key tile, after a 32-key block, and one entry short of it; shares that begin
# at another head than the first
@pytest.mark.parametrize("cfg,k", [(_cfg(901, 8, 193), 3), (_cfg(301, 6, 416, layout="sbhd"), 2), (_cfg(301, 6, 415, gated=False), 1),
                                   (_cfg(457, 5, 384, axis="head", lo=1), 2), (_win(70, 8, (12, 12), mask="region"), 2),
                                   (_win(130, 4, (10, 16), gated=True), 1), (_win(180, 6, (9, 9), mask="region"), 3),
                                   (_win(175, 6, (11, 11), bias="dense", mask="region"), 2), (_win(70, 8, (12, 12), bias="dense", mask="region"), 2),
                                   (_win(130, 5, (12, 12), mask="region", axis="head", lo=1), 2)],
                         ids=["193", "416_sbhd", "415", "384_heads", "12x12", "10x16_gated", "9x9", "11x11_dense", "12x12_dense", "12x12_heads"])
def test_copies_give_the_same_bits(cfg, k):
    cfg = dict(cfg)
    lo = cfg.pop("lo", 0)
    print(f"bias copies {cfg['B']} x {cfg['H']} x {cfg['S']}", flush=True)
    _eager_and_captured(cfg, lo, k)


@pytest.mark.parametrize("cfg", [_cfg(301, 6, 416), _cfg(457, 4, 385, layout="sbhd", gated=False), _win(131, 4, (12, 12), mask=None)],
                         ids=["416", "385_sbhd", "12x12"])
def test_maxima_that_grow_in_some_rows(cfg):
    """Scores that rise along the first half of the keys by 12 bits a block of 32 in every other row and by 40 in every third, and fall in
    the others: of two rows that a wavefront takes together one raises its maxima, by either means, and the other does not."""
    inp = make_inputs(**cfg)
    print(f"growing maxima of some rows {cfg['B']} x {cfg['H']} x {cfg['S']}", flush=True)
    rows, along = np.arange(cfg["B"]), np.minimum(np.arange(cfg["S"]), cfg["S"] // 2) / 32.0
    bits = np.where(rows % 2 == 0, 12.0, np.where(rows % 3 == 0, 40.0, -5.0))
    inp["Q"][..., 0] = 4.0
    rise = bits[:, None] * along[None] * np.log(2) * 32 ** 0.5 / 4
    inp["K"][..., 0] = round_to_bf16((inp["K"][..., 0] + rise[:, :, None]).astype(np.float32))
    dc = _eager_and_captured(cfg, 0, 1, inputs=inp)
    some = [0, 1, 2, 3, cfg["B"] // 2, cfg["B"] - 2, cfg["B"] - 1]
    part = {n: (a[some] if n in ("Q", "K", "V", "dY", "G") else a) for n, a in inp.items()}
    p = oracle_problem(part, cfg)
    Y, lse = orc.attn_forward(p, AXIS["row"], 0, len(some))
    g = orc.attn_backward(p, part["dY"].astype(np.float64), AXIS["row"], 0, len(some))
    # an LSE of up to 180: scores of up to 1020 before the scale, three fp32 roundings of 6e-5 each times 0.177, the rounding of scale * log2(e),
    # 6e-8 of it, that of the result, 8e-6, and that of exponents of up to 26 bits, 1e-6.  2-norms of the others: operands rounded to bf16
    # leave 1.8e-3 (twice that in dQ, see test_gpu_offset_data.py), the result's rounding 1.1e-3, a gate's as much again
    assert float(np.max(np.abs(dc.host("lse")[some] - lse))) <= 6e-5
    for n, ref in [("Y", Y)] + [(n, g[n]) for n in ("dQ", "dK", "dV") + (("dG",) if cfg["gated"] else ())]:
        e = float(np.linalg.norm(dc.host(n)[some] - ref) / np.linalg.norm(ref))
        print(n, e, flush=True)
        assert e <= 6e-3, (n, e)


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
    inp = make_inputs(**cfg)
    inp["bias"] = round_to_bf16((inp["bias"] * (6 / np.max(np.abs(inp["bias"])))).astype(np.float32))
    print(f"scale 1.2e-38, {cfg['S']} tokens", flush=True)
    dc, _ = run_case(cfg, inputs=inp, scale=1.2e-38)
    Y, _ = orc.attn_forward(oracle_problem(inp, cfg, 1.2e-38), AXIS[cfg["axis"]], 0, cfg["B"])
    assert_close("Y", dc.host("Y"), Y, TOL["bf16"])
    for n in ("dQ", "dK", "dV", "dBias"):
        assert bool(getattr(dc, n).isfinite().all()), n
