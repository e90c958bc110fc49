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


@pytest.mark.parametrize("B,H,S", [(1030, 8, 81), (1100, 15, 97), (1030, 16, 112), (777, 16, 113), (519, 32, 128), (300, 8, 144)])
def test_runs_of_rows_of_every_length(B, H, S):
    """Forward: a row's results do not depend on how many rows its work-group walks, nor in how many rounds the launch runs them."""
    import torch
    from paper_2301_08984_amd import binding as ss
    gen = torch.Generator(device="cuda").manual_seed(S)
    q, k, v, g = (torch.randn((B, S, H, 32), generator=gen, device="cuda").bfloat16() for _ in range(4))
    bias = torch.randn((H, S, S), generator=gen, device="cuda").bfloat16()
    ids = torch.stack([torch.arange(S, dtype=torch.int32, device="cuda") * n // S for n in (1, 2, 3)]).contiguous()
    print(f"runs of rows {B} x {H} x {S}", flush=True)
    for gated in (False, True):
        out = []
        for lo, hi in ((0, B), (B // 2, B // 2 + 7), (B - 3, B)):
            y, lse = torch.full_like(q, float("nan")), torch.full((B, H, S), float("nan"), device="cuda")
            d = ss.make_desc(B, H, S, 32, ss.SS_BF16, 32 ** -0.5, ss.SS_AXIS_ROW, lo, hi, 1, stride_b=S * H * 32, stride_s=H * 32, stride_h=32,
                             bias_kind=ss.SS_BIAS_DENSE, mask_kind=ss.SS_MASK_REGION, mask_period=3, gated=gated)
            ss.ss_attn_fwd(d, q, k, v, bias, ids, g if gated else None, y, lse, None, 0, torch.cuda.current_stream().cuda_stream)
            out.append((lo, hi, y, lse))
        torch.cuda.synchronize()
        for lo, hi, y, lse in out[1:]:
            assert not torch.isnan(y[lo:hi]).any() and not torch.isnan(lse[lo:hi]).any()
            assert torch.equal(y[lo:hi], out[0][2][lo:hi]) and torch.equal(lse[lo:hi], out[0][3][lo:hi])
        b = B - 2  # one row in fp32
        s = torch.einsum("ihd,jhd->hij", q[b].float(), k[b].float()) * 32 ** -0.5 + bias.float()
        s.masked_fill_(ids[b % 3][:, None] != ids[b % 3][None], float("-inf"))
        ref = torch.einsum("hij,jhd->ihd", torch.softmax(s, -1), v[b].float())
        ref = ref * torch.sigmoid(g[b].float()) if gated else ref
        assert ((out[0][2][b].float() - ref).norm() / ref.norm()).item() <= 1e-2  # bf16 probabilities and results


@pytest.mark.parametrize("win", [(5, 13), (5, 16), (9, 9), (8, 12)], ids=lambda w: f"{w[0]}x{w[1]}")
@pytest.mark.parametrize("form", ["regions", "bias", "both"])
def test_gates_of_several_rows(win, form):
    """A work-group walks several rows, whose gates some kernels ask for before the next row and some after it; without a bias in two rounds."""
    from paper_2301_08984_amd.workloads import make_inputs
    cfg = _cfg(win, **(dict(B=601, H=8, bias=None) if form == "regions" else dict(B=401, H=6)), mask=None, gated=True)
    inp = make_inputs(**cfg)
    if form != "bias":
        inp["region_ids"] = (np.arange(cfg["S"])[None] * np.arange(1, 4)[:, None] // cfg["S"]).astype(np.int32)
        cfg["mask"] = "region"
    print(f"gates {win} {form}", flush=True)
    check_against_oracle(cfg, inputs=inp)
