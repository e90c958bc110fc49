"""fp32 operators of head size up to 64 on the fp32 matrix instructions: block edges of 16 rows, rounds of
128 / 256 / 512 keys and more than one round, head sizes that are no multiple of 16 (and one that is no
multiple of 4: plain kernels), every bias and mask kind, gating, transposed storage, against the oracle at
an fp32 bar; bit for bit across k."""
import numpy as np
import pytest

from parity import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def _cfg(S, D, B=2, H=2, **kw):
    return dict(seed=900 + S + D, B=B, H=H, S=S, D=D, dtype="f32", **{"axis": "row", **kw})


CASES = {
    "one_token": _cfg(1, 4),
    "one_short_of_a_block": _cfg(15, 16, mask="causal"),
    "one_block": _cfg(16, 20, bias="dense"),
    "one_over_a_block": _cfg(17, 32, bias="dense", mask="causal", gated=True),
    "one_round": _cfg(128, 24, B=3),
    "one_over_a_round": _cfg(129, 64, bias="dense", gated=True),
    "two_rounds_transposed": _cfg(257, 48, mask="causal", layout="sbhd", gated=True),
    "four_blocks_a_wavefront": _cfg(512, 64, H=1, mask="causal"),
    "more_than_one_round": _cfg(530, 16, H=1, bias="dense"),
    "more_than_one_round_causal": _cfg(1100, 8, B=1, mask="causal", bias="dense"),
    "window": _cfg(49, 32, B=7, bias="relpos", win=(7, 7), mask="region"),
    "heads": _cfg(70, 40, H=5, axis="head", bias="dense"),
    "plain_kernels": _cfg(33, 6, bias="dense"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_matches_oracle(name):
    cfg = CASES[name]
    n = cfg["H"] if cfg["axis"] == "head" else cfg["B"]
    ref = None
    for k in sorted({1, n}):
        print(f"f32 case {name} k={k}", flush=True)
        check_against_oracle(cfg, k=k, use_lse=k > 1, tol=2e-5)
        dc, _ = run_case(cfg, k=k)
        outs = {o: dc.host(o) for o in ("Y", "lse", "dQ", "dK", "dV", "dG", "dBias") if dc.host(o) is not None}
        ref = ref or outs
        for o, x in outs.items():
            assert np.array_equal(x, ref[o], equal_nan=True), (o, k)


def test_the_flag_for_plain_kernels_is_honoured_and_slots_count_launches():
    """SS_FLAG_GENERIC_KERNELS takes an fp32 operator to the plain kernels (recompute, dQ, dK/dV, dBias: four
    launches a chunk); without it there are two, and no time slot counts a launch that does not exist."""
    import torch
    from paper_2301_08984_amd import binding as ss
    from paper_2301_08984_amd.runner import DeviceCase
    from paper_2301_08984_amd.workloads import make_inputs
    cfg = _cfg(70, 32, bias="dense")
    dc = DeviceCase(make_inputs(**cfg), dtype="f32", bias="dense")
    print("f32 launches", flush=True)
    for flags, want in ((0, {"fwd": 1, "recompute_dq": 1, "dkdv": 1}),
                        (ss.SS_FLAG_GENERIC_KERNELS, {"fwd": 1, "recompute": 1, "dq": 1, "dkdv": 1, "dbias": 1})):
        d = dc.desc("row", 0, dc.B, 1, flags)
        ss.ss_attn_profile_enable(True)
        dc.fwd(d)
        dc.bwd(d)
        torch.cuda.synchronize()
        ss.ss_attn_profile_enable(False)
        got = {n: ss.ss_attn_profile_read(i)[1] for i, n in enumerate(ss.KERNEL_NAMES)}
        assert {n: c for n, c in got.items() if c} == want, (flags, got)
