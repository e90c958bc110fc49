"""The bias gradient's partial sums where the workspace holds fewer of them than the share has: the caller's
workspace alone (under graph capture), the library's buffer, and the built-in buffer run different numbers of
chunks and give the same bits; and sums that go on in the result, without partial sums."""
import pytest

from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def _cfg(B, H, win, **kw):
    return dict(seed=850 + B, B=B, H=H, S=win[0] * win[1], D=32, dtype="bf16", bias="relpos", win=win,
                mask="region" if win[0] == win[1] else None,
                **{"axis": "row", **kw})


@pytest.mark.parametrize("cfg,k", [(_cfg(120, 8, (12, 12)), 1), (_cfg(8, 128, (10, 12), axis="head"), 2), (_cfg(300, 16, (8, 8)), 1),
                                   (dict(_cfg(60, 8, (3, 101)), bias="dense", mask=None), 1)],
                         ids=["12x12", "10x12_heads", "8x8", "dense_303"])
def test_workspace_library_buffer_and_built_in_buffer_agree(cfg, k):
    import torch
    from paper_2301_08984_amd import binding as ss
    print(f"partial sums S={cfg['S']} k={k}", flush=True)
    dc, _ = run_case(cfg, k=k)
    names = [n for n in ("dQ", "dK", "dV", "dBias") if getattr(dc, n) is not None]
    first = {n: getattr(dc, n).clone() for n in names}
    ext = dc.H if cfg["axis"] == "head" else dc.B
    d = dc.desc(cfg["axis"], 0, ext, k)

    def check(what):
        torch.cuda.synchronize()
        for n in names:
            assert bool(getattr(dc, n).isfinite().all()) and torch.equal(getattr(dc, n), first[n]), (what, n)
            getattr(dc, n).fill_(float("nan"))

    dc.ws.fill_(0xFF)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        dc.bwd(d)
    for n in names:
        getattr(dc, n).fill_(float("nan"))
    for rep in range(2):
        graph.replay()
        check(f"captured {rep}")
    ss.ss_attn_bwd_static(d, dc.Q, dc.K, dc.V, dc.bias, dc.region, dc.G, dc.dY, None, dc.dQ, dc.dK, dc.dV, dc.dBias, dc.dG,
                          torch.cuda.current_stream().cuda_stream)
    check("built-in buffer")
    big = torch.full((64 << 20,), 0xFF, dtype=torch.uint8, device=dc.dev)
    dc.ws = big
    dc.bwd(d)
    check("large workspace")


@pytest.mark.parametrize("cfg", [_cfg(2, 300, (9, 9)), _cfg(1, 3, (12, 12)), dict(_cfg(3, 700, (7, 13)), axis="head")],
                         ids=["two_rows", "one_row", "heads"])
def test_sums_without_partial_sums(cfg):
    for k in (1, 2) if cfg["B"] > 1 or cfg["axis"] == "head" else (1,):
        print(f"in place S={cfg['S']} k={k}", flush=True)
        check_against_oracle(cfg, k=k)
