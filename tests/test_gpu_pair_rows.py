"""Pair attention over rows of 65 to 160 tokens, whose backward takes the kernel that holds a row's scores in registers: sizes at the edges of its blocks and
of the rules that choose it, with and without bias and gate, both split axes, transposed storage, groups of rows that chunk boundaries cut, a share
that begins inside a group; and captured, where the library's buffer is not used.  Reference: the fp64 oracle at the tolerances of parity.py."""
import pytest

from paper_2301_08984_amd.workloads import make_inputs
from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def _cfg(B, H, S, **kw):
    return dict(dict(seed=1600 + S, B=B, H=H, S=S, D=32, dtype="bf16", bias="dense", mask=None, gated=True, axis="row"), **kw)


@pytest.mark.parametrize("S", [65, 79, 80, 96, 97, 112, 113, 128, 129, 144, 145, 160, 161])
@pytest.mark.parametrize("form", ["gated", "plain", "no_bias", "sbhd_heads"])
def test_lengths(S, form):
    kw = {"gated": {}, "plain": dict(gated=False), "no_bias": dict(bias=None), "sbhd_heads": dict(layout="sbhd", axis="head")}[form]
    print(f"pair rows {S} {form}", flush=True)
    check_against_oracle(_cfg(11, 4, S, **kw), k=2, use_lse=form == "plain")


@pytest.mark.parametrize("S", [16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("form", ["dense", "no_bias", "sbhd_heads"])
def test_short_gated_rows(S, form):
    kw = {"dense": {}, "no_bias": dict(bias=None), "sbhd_heads": dict(layout="sbhd", axis="head")}[form]
    print(f"short gated rows {S} {form}", flush=True)
    check_against_oracle(_cfg(37, 4, S, **kw), k=3, use_lse=form == "dense")


@pytest.mark.parametrize("win", [(5, 5), (6, 7), (7, 7), (8, 8)], ids=lambda w: f"{w[0]}x{w[1]}")
def test_short_gated_windows(win):
    print(f"short gated windows {win}", flush=True)
    check_against_oracle(_cfg(67, 3, win[0] * win[1], bias="relpos", win=win, mask="region" if win[0] == win[1] else None), k=4, lo=1)


@pytest.mark.parametrize("B,H,S,k", [(301, 8, 100, 5), (257, 4, 129, 3), (64, 8, 128, 1), (150, 5, 144, 4)])
def test_groups_of_rows(B, H, S, k):
    print(f"pair rows in groups {B} x {H} x {S}", flush=True)
    check_against_oracle(_cfg(B, H, S), lo=3, hi=B - 2, k=k)


@pytest.mark.parametrize("S", [129, 144, 145, 160])
@pytest.mark.parametrize("B", [32, 33])
def test_forward_on_both_sides_of_its_line(B, S):
    """Up to 128 (row, head) pairs a forward with a bias takes the tiled kernels, beyond them the kernel that holds a row's scores."""
    print(f"pair rows, forward {B} x 4 x {S}", flush=True)
    check_against_oracle(_cfg(B, 4, S, gated=S % 2 == 0))


@pytest.mark.parametrize("B,H,S,axis,gated", [(9, 62, 160, "row", False), (14, 76, 144, "head", True)])
def test_many_heads_in_two_groups(B, H, S, axis, gated):
    """Groups of rows whose sums take the place of the transposed bias; the same bits for every k."""
    import torch
    cfg = _cfg(B, H, S, axis=axis, gated=gated)
    print(f"pair rows, many heads {B} x {H} x {S}", flush=True)
    dc, _ = check_against_oracle(cfg, k=1)
    want = {n: getattr(dc, n).clone() for n in ("dQ", "dK", "dV", "dBias")}
    for k in (2, 5):
        dc.ws = None
        dc.bwd(dc.desc(axis, 0, H if axis == "head" else B, k), poison=True)
        torch.cuda.synchronize()
        for n, x in want.items():
            assert torch.equal(getattr(dc, n), x), (k, n)


def test_captured_and_eager_calls_agree():
    import torch
    cfg = _cfg(130, 4, 132)
    print("pair rows, captured", flush=True)
    dc, _ = run_case(cfg, k=3, inputs=make_inputs(**cfg))
    d = dc.desc("row", 0, dc.B, 3)
    names = ("Y", "dQ", "dK", "dV", "dG", "dBias")
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
            assert torch.equal(getattr(dc, n), first[n]), (rep, n)
