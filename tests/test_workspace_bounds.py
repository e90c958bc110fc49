"""The partial sums of the bias gradient in the backward's workspace are bounded, and never push a share past the
built-in buffer of ss_attn_bwd_static that fits it without them.  Host arithmetic only, no GPU."""
import ctypes as C
import random

import pytest

from paper_2301_08984_amd import binding as ss

MIB = 1 << 20


def _desc(B, H, S, k, *, D=32, bias=ss.SS_BIAS_RELPOS, win=None, gated=False, axis=ss.SS_AXIS_ROW, lo=0, hi=None):
    ext = B if axis == ss.SS_AXIS_ROW else H
    return ss.make_desc(B, H, S, D, ss.SS_BF16, 0.17, axis, lo, ext if hi is None else hi, k, bias_kind=bias,
                        win=win or (0, 0), gated=gated)


def _bytes(d):
    return ss.ss_attn_workspace_bytes(d)[1]


def _static_takes(d):
    """Whether ss_attn_bwd_static gets past its size check (Q = NULL: nothing can be enqueued)."""
    one = 256
    rc = ss.lib().ss_attn_bwd_static(C.byref(d), None, one, one, one, None, one, one, None, one, one, one, one, one, None)
    assert rc < 0
    return rc != ss.SS_ERR_STATIC_SCRATCH


def _up(x):
    return (x + 255) // 256 * 256


def _least(d):
    """Bytes of the backward with the fewest partial sums: none where the bias gradient's sum can go on in the
    result, groups of 8 rows for windows of up to 64 tokens, of 64 for dense biases of a length divisible by 4."""
    n = d.hi - d.lo
    row = d.shard_axis == ss.SS_AXIS_ROW
    nmax = -(-n // d.k)
    Bc, Hc = (nmax, d.H) if row else (d.B, nmax)
    total = 2 * _up(Bc * Hc * d.S * 4) + (_up(Bc * d.S * Hc * d.D * 2) if d.gated else 0)
    if d.bias_kind == ss.SS_BIAS_RELPOS:
        total += _up(d.H * d.S * d.S * 4)
    if d.bias_kind == ss.SS_BIAS_DENSE:
        total += _up(d.H * d.S * d.S * 2)
    short = d.D == 32 and d.S <= 64 and not d.gated
    gw = 8 if short else 64 if d.bias_kind == ss.SS_BIAS_DENSE and d.S > 64 and d.S % 4 == 0 and (-(-d.S // 64)) ** 2 * d.H < 512 else 0
    if gw:
        lo, hi = (d.lo, d.hi) if row else (0, d.B)
        groups = (hi - 1) // gw - lo // gw + 1
        slices = min(max(groups // 16, 1), 32)
        ring, hs = (min(slices + -(-nmax // gw) + 1, groups), d.H) if row else (groups, nmax)
        total += _up(ring * hs * d.S * d.S * 4)
    return total


@pytest.mark.parametrize("B,H,win,k,most", [(512, 8, (12, 12), 1, 16), (512, 8, (12, 12), 2, 16), (512, 8, (12, 12), 4, 10),
                                            (256, 6, (9, 9), 1, 9), (512, 16, (8, 8), 1, 24), (128, 8, (7, 7), 1, 10)])
def test_windows_fit_the_built_in_buffer(B, H, win, k, most):
    d = _desc(B, H, win[0] * win[1], k, win=win)
    assert _bytes(d) <= most * MIB, _bytes(d) / MIB
    assert _static_takes(d)


def test_partial_sums_are_bounded_and_never_cost_the_built_in_buffer():
    rng = random.Random(7)
    worst = 0.0
    limit, shorter, more_chunks, refused = ss.SS_ATTN_STATIC_SCRATCH_BYTES, 0, 0, 0
    for _ in range(4000):
        B, H = int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 7))
        axis = rng.choice((ss.SS_AXIS_ROW, ss.SS_AXIS_HEAD))
        ext = B if axis == ss.SS_AXIS_ROW else H
        lo = rng.randint(0, ext - 1)
        hi = rng.randint(lo + 1, ext)
        k = min(hi - lo, int(2 ** rng.uniform(0, 6)))
        if rng.random() < 0.5:
            w = (rng.randint(2, 16), rng.randint(2, 10))
            d = _desc(B, H, w[0] * w[1], k, win=w, axis=axis, lo=lo, hi=hi, gated=rng.random() < 0.2)
        else:
            d = _desc(B, H, int(2 ** rng.uniform(4, 10)), k, bias=ss.SS_BIAS_DENSE, axis=axis, lo=lo, hi=hi,
                      D=rng.choice((32, 32, 64)), gated=rng.random() < 0.5)
        got, least = _bytes(d), _least(d)
        # 12 MiB, or a few groups where each of them is large
        over = (got - least - 12 * MIB) / (d.H * d.S * d.S * 4)
        worst = max(worst, over)
        assert _static_takes(d) == (least <= limit), (got / MIB, least / MIB)
        shorter += got > least
        more_chunks += least <= limit < got
        refused += least > limit
    assert worst <= 4, worst
    assert shorter > 300 and more_chunks >= 1 and refused > 200, (shorter, more_chunks, refused)


def test_library_device_memory_is_what_the_header_says():
    """The sizes in the header, in the binding and (a static assertion) in the library are the same."""
    import os
    import re
    text = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "ss_attn.h")).read()
    macros = dict(re.findall(r"#define (SS_\w+_BYTES) (.+)", text))
    value = lambda name: eval(re.sub(r"SS_\w+", lambda m: str(value(m.group(0))), macros[name]).replace("u", ""))
    assert value("SS_ATTN_STATIC_SCRATCH_BYTES") == ss.SS_ATTN_STATIC_SCRATCH_BYTES
    assert value("SS_LIBRARY_DEVICE_BYTES") == ss.SS_LIBRARY_DEVICE_BYTES


@pytest.mark.parametrize("B,H,S,gated", [(100, 62, 160, False), (300, 64, 157, False), (100, 76, 144, True), (33, 90, 144, True), (50, 100, 144, False)])
def test_many_heads_keep_groups_of_rows(B, H, S, gated):
    """One work-group per head and group of rows: one group would leave most of the chip idle.  Two groups' sums take the place of the transposed bias
    and no more than the spare beside it."""
    d = _desc(B, H, S, 1, bias=ss.SS_BIAS_DENSE, gated=gated)
    transposed = _up(H * S * S * 2)
    assert _bytes(d) == _least(d) - transposed + _up(2 * H * S * S * 4)
    finest = _desc(B, H, S, B, bias=ss.SS_BIAS_DENSE, gated=gated)
    assert _least(finest) < _bytes(finest) <= _least(finest) + 12 * MIB
