"""Transposed storage in which the slice of one (row, head) pair spans more than 4 GiB, at head size 128: 32-bit offsets into it would wrap."""
import math

import pytest
import torch

from paper_2301_08984_amd import binding as ss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", ["causal", None])
def test_a_slice_of_more_than_4_gib(mask):
    H, S, D, stride = (6 if mask else 4), 8320, 128, 1 << 18  # 8320 rows of 512 KiB; large shares: from 304 work-groups of 128 tokens on, 192 without a mask
    assert (S - 1) * stride * 2 > 1 << 32
    gen = torch.Generator(device="cuda").manual_seed(88)

    def tensor(fill):
        x = torch.empty((S, stride), dtype=torch.bfloat16, device="cuda")
        x[:, : H * D] = torch.randn((S, H * D), generator=gen, device="cuda").bfloat16() if fill else float("nan")
        return x

    t = {n: tensor(n in ("Q", "K", "V", "dY")) for n in ("Q", "K", "V", "dY", "Y", "dQ", "dK", "dV")}
    d = ss.make_desc(1, H, S, D, ss.SS_BF16, 1.0 / math.sqrt(D), ss.SS_AXIS_HEAD, 0, H, 1, stride_b=stride, stride_s=stride, stride_h=D,
                     mask_kind=ss.SS_MASK_CAUSAL if mask else ss.SS_MASK_NONE)
    ws = torch.empty(ss.ss_attn_workspace_bytes(d)[1], dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    print(f"long slice, mask={mask}: forward and backward", flush=True)
    ss.ss_attn_fwd(d, t["Q"], t["K"], t["V"], None, None, None, t["Y"], None, None, 0, stream)
    ss.ss_attn_bwd(d, t["Q"], t["K"], t["V"], None, None, None, t["dY"], None, t["dQ"], t["dK"], t["dV"], None, None, ws, ws.numel(), stream)
    torch.cuda.synchronize()
    for h in range(H):
        q, k, v, g = (t[n][:, h * D : (h + 1) * D].float() for n in ("Q", "K", "V", "dY"))
        s = q @ k.T / math.sqrt(D)
        if mask:
            s.masked_fill_(torch.ones((S, S), dtype=torch.bool, device="cuda").triu_(1), float("-inf"))
        p = torch.softmax(s, -1)
        o = p @ v
        ds = p * (g @ v.T - (g * o).sum(-1, keepdim=True)) / math.sqrt(D)
        for n, ref in (("Y", o), ("dQ", ds @ k), ("dK", ds.T @ q), ("dV", p.T @ g)):
            x = t[n][:, h * D : (h + 1) * D].float()
            assert ((x - ref).norm() / ref.norm()).item() <= 1e-2, (n, h)  # products of bf16 operands
            assert ((x[8192:] - ref[8192:]).norm() / ref[8192:].norm()).item() <= 1e-2, (n, h, "last rows")
