"""Bias gradient with 64 queries x 64 keys of two heads per work-group (from 256 such work-groups in a launch on, with a causal mask those below the
diagonal): edges of its tiles, odd lengths,
transposed storage, the causal mask, groups of rows, sums that go on from chunk to chunk, and, on fewer work-groups, one head at a time with
the same bits."""
import os
import subprocess

import pytest
import torch

from paper_2301_08984_amd import build as B
from parity import check_against_oracle
from test_wave_isa import pending_read_violations

CASES = {  # rows, heads, tokens
    "groups_65_causal": dict(B=300, H=12, S=65, mask="causal"),
    "groups_193": dict(B=70, H=16, S=193),
    "groups_129_causal": dict(B=40, H=16, S=129, mask="causal"),
    "groups_193_causal": dict(B=70, H=24, S=193, mask="causal"),
    "sbhd_191": dict(B=40, H=12, S=191, layout="sbhd"),
    "one_row_1000": dict(B=1, H=4, S=1000),
    "odd_833": dict(B=3, H=4, S=833),
    "heads_320": dict(B=34, H=8, S=320, axis="head"),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_against_the_oracle_and_every_k(name):
    print(f"paired bias gradient {name}", flush=True)
    cfg = dict(dict(seed=1400 + CASES[name]["S"], D=32, dtype="bf16", bias="dense", mask=None, gated=True, axis="row"), **CASES[name])
    dc, _ = check_against_oracle(cfg)
    want = dc.dBias.clone()
    n = cfg["H"] if cfg["axis"] == "head" else cfg["B"]
    for k in sorted({min(3, n), n}):  # in a captured graph the chunks run one by one, small ones with fewer work-groups
        dc.ws = None
        d = dc.desc(cfg["axis"], 0, n, k)
        dc.workspace(d)
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            dc.bwd(d)
        for rep in range(2):
            dc.dBias.fill_(float("nan"))
            dc.ws.fill_(0xFF)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(dc.dBias, want), (k, rep)


def test_no_register_is_touched_between_a_read_and_its_wait(tmp_path):
    out = os.path.join(tmp_path, "k.s")
    subprocess.run(["hipcc", *B.FLAGS, *B.EXTRA_FLAGS["pair_dbias.hip"], "--cuda-device-only", "-S", os.path.join(B.CSRC, "pair_dbias.hip"), "-o", out], check=True,
                   capture_output=True)
    lines = open(out).read().splitlines()
    assert any("ds_read_b128" in l for l in lines)
    assert pending_read_violations(lines) == []
