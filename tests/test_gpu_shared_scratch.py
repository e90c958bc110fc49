"""Chunks of a small share run together in the library's own scratch when nobody else is using it, and one
by one in the caller's workspace otherwise: under graph capture, and on a second stream while the first
one's work is under way.  Both ways give the same bits."""
import pytest

from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu
OUTS = ("dQ", "dK", "dV", "dG", "dBias")


@pytest.mark.parametrize("name,k", [("gpt_like", 2), ("tri_like", 3), ("swin_like", 4), ("f32_all", 2)])
def test_chunked_and_merged_runs_agree(name, k):
    import torch
    from paper_2301_08984_amd.runner import DeviceCase
    from paper_2301_08984_amd.workloads import make_inputs
    cfg = SMALL[name]
    inp = make_inputs(**cfg)
    dc, other = (DeviceCase(inp, dtype=cfg["dtype"], bias=cfg.get("bias"), mask=cfg.get("mask"), gated=cfg.get("gated", False),
                            win=cfg.get("win"), layout=cfg.get("layout", "bshd")) for _ in range(2))
    ext = dc.H if cfg["axis"] == "head" else dc.B
    d = dc.desc(cfg["axis"], 0, ext, min(k, ext))
    dc.bwd(d, poison=True)
    torch.cuda.synchronize()
    names = [n for n in OUTS if getattr(dc, n) is not None]
    merged = {n: getattr(dc, n).clone() for n in names}

    def check(case, what):
        torch.cuda.synchronize()
        for n in names:
            assert torch.equal(torch.nan_to_num(getattr(case, n), nan=12345.0), torch.nan_to_num(merged[n], nan=12345.0)), (what, n)
            getattr(case, n).fill_(float("nan"))

    dc.ws.fill_(0xFF)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        dc.bwd(d)
    for n in names:
        getattr(dc, n).fill_(float("nan"))
    graph.replay()
    check(dc, "captured")
    # two streams at a time, several calls deep
    other.workspace(d)
    torch.cuda.synchronize()
    for _ in range(8):
        dc.bwd(d)
        with torch.cuda.stream(side):
            other.bwd(d)
    check(dc, "first stream")
    check(other, "second stream")


@pytest.mark.parametrize("name,k", [("gpt_like", 2), ("swin_like", 4)])
def test_two_host_threads_on_two_streams(name, k):
    """Whoever holds the buffer, and whoever does without, gets the results of a run alone."""
    import threading
    import torch
    from paper_2301_08984_amd.runner import DeviceCase
    from paper_2301_08984_amd.workloads import make_inputs
    cfg = SMALL[name]
    inp = make_inputs(**cfg)
    cases = [DeviceCase(inp, dtype=cfg["dtype"], bias=cfg.get("bias"), mask=cfg.get("mask"), gated=cfg.get("gated", False),
                        win=cfg.get("win"), layout=cfg.get("layout", "bshd")) for _ in range(3)]
    ext = cases[0].H if cfg["axis"] == "head" else cases[0].B
    d = cases[0].desc(cfg["axis"], 0, ext, k)
    for c in cases:
        c.workspace(d)
    cases[2].bwd(d, poison=True)
    streams, errors = [torch.cuda.Stream(), torch.cuda.Stream()], []
    print(f"attention two threads {name}", flush=True)
    torch.cuda.synchronize()

    def work(i):
        try:
            for _ in range(20):
                cases[i].bwd(d, stream=streams[i].cuda_stream)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i in range(2):
        for n in OUTS:
            ref = getattr(cases[2], n)
            if ref is not None:
                assert torch.equal(torch.nan_to_num(getattr(cases[i], n), nan=12345.0), torch.nan_to_num(ref, nan=12345.0)), (i, n)


def test_a_forward_leaves_room_for_the_chunks_of_another_stream():
    """Beside a forward of pair attention (about 300 us), whose copy of the bias is in the library's buffer, the 16 chunks of a small share
    still run together."""
    import torch
    from paper_2301_08984_amd import binding as ss
    from paper_2301_08984_amd.runner import DeviceCase
    from paper_2301_08984_amd.workloads import make_inputs
    print("attention beside a forward", flush=True)
    cases = [DeviceCase(make_inputs(B=B, H=H, S=S, D=32, dtype="bf16", bias="dense", gated=True, seed=S), dtype="bf16", bias="dense", gated=True)
             for B, H, S in ((256, 4, 1024), (18, 8, 200))]
    long, small = cases[0].desc("row", 0, 256, 1), cases[1].desc("row", 0, 18, 16)
    side = torch.cuda.Stream()
    cases[1].workspace(small)
    for _ in range(2):  # what a first call does once
        cases[0].fwd(long)
        cases[1].bwd(small)
        torch.cuda.synchronize()
    alone = {n: getattr(cases[1], n).clone() for n in OUTS if getattr(cases[1], n) is not None}
    cases[0].fwd(long)
    cases[0].fwd(long)
    ss.ss_attn_profile_enable(True)
    with torch.cuda.stream(side):
        cases[1].bwd(small)
    torch.cuda.synchronize()
    ss.ss_attn_profile_enable(False)
    launches = {n: ss.ss_attn_profile_read(i)[1] for i, n in enumerate(ss.KERNEL_NAMES)}
    assert launches["dkdv"] + launches["dq_dkdv"] == 1, launches
    for n, ref in alone.items():
        assert torch.equal(getattr(cases[1], n), ref), n
