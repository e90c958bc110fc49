"""Host-side arithmetic model of the one-walk recompute + dQ kernel (head size 32, large shares),
checked against the fp64 oracle.

The kernel cannot form dS = P (dP - Delta) while it walks the keys, because Delta is known only
after the last key.  It accumulates A1 = sum_j bf16(p~ dP) K_j and A2 = sum_j bf16(p~) K_j over the
unnormalised probabilities p~ and combines them at the end: dQ = scale / l' (A1 - Delta' A2).  The
two terms cancel on peaked rows, so which mean is subtracted matters: the kernel takes
Delta' = sum_j bf16(p~ dP) / sum_j bf16(p~), the mean of the operands the products saw.  This file
models that arithmetic in numpy (bf16 rounding of the operands, everything else in fp64) and pins
  * that the formula reproduces the oracle's dQ to the accuracy of forming dS directly, and
  * that the mean of the unrounded values (Delta itself) would be several times worse on peaked rows,
so that a change of the kernel's reading of Delta' has a failing test on the CPU.
No GPU, no HIP library: the oracle and the seeded input generator only."""
import math

import numpy as np
import pytest

from oracle import attention as orc
from paper_2301_08984_amd.workloads import make_inputs, round_to_bf16


def _bf(x):
    return round_to_bf16(np.asarray(x, dtype=np.float32)).astype(np.float64)


def _model(Q, K, V, dO, bias, causal, scale):
    """dQ of one (row, head) three ways: dS rounded directly; the two-product formula with the mean of
    the rounded operands; the same with the exact Delta."""
    S = Q.shape[0]
    x = scale * Q @ K.T + (bias if bias is not None else 0.0)
    if causal:
        x = np.where(np.tril(np.ones((S, S), bool)), x, -np.inf)
    p = np.exp(x - x.max(1, keepdims=True))    # unnormalised, largest entry 1
    l = p.sum(1, keepdims=True)
    P = p / l
    dP = dO @ V.T
    delta = (P * dP).sum(1, keepdims=True)
    direct = scale * _bf(P * (dP - delta)) @ K
    pb, wb = _bf(p), _bf(p * dP)
    a1, a2 = wb @ K, pb @ K
    lp = pb.sum(1, keepdims=True)
    fused = scale * (a1 - (wb.sum(1, keepdims=True) / lp) * a2) / lp
    exact_mean = scale * (a1 - delta * a2) / l
    return direct, fused, exact_mean


def _case(S, D, bias, causal, peak, seed):
    inp = make_inputs(B=1, H=1, S=S, D=D, dtype="bf16", bias="dense" if bias else None,
                      mask="causal" if causal else None, seed=seed)
    inp["Q"] = _bf(inp["Q"] * peak).astype(np.float32)   # larger queries: peaked softmax rows
    sc = float(np.float32(1.0 / math.sqrt(D)))
    prob = orc.AttnProblem(inp["Q"], inp["K"], inp["V"], sc,
                           ("dense", inp["bias"].astype(np.float64)) if bias else None,
                           ("causal",) if causal else None, None)
    ref = orc.attn_backward(prob, inp["dY"].astype(np.float64))["dQ"][0, :, 0, :]
    f64 = lambda a: a[0, :, 0, :].astype(np.float64)
    got = _model(f64(inp["Q"]), f64(inp["K"]), f64(inp["V"]), f64(inp["dY"]),
                 inp["bias"][0].astype(np.float64) if bias else None, causal, sc)
    den = np.max(np.abs(ref))
    return [float(np.max(np.abs(g - ref)) / den) for g in got]


@pytest.mark.parametrize("S,D,bias,causal,peak", [(384, 32, True, False, 1.0), (384, 32, True, False, 4.0),
                                                    (200, 32, True, True, 4.0), (130, 32, False, False, 2.0)])
def test_two_product_formula_matches_the_oracle(S, D, bias, causal, peak):
    direct, fused, _ = _case(S, D, bias, causal, peak, seed=11)
    assert direct <= 6e-3 and fused <= 6e-3, (direct, fused)
    assert fused <= 2.0 * direct + 1e-3, (direct, fused)   # as accurate as dS formed directly


def test_mean_of_the_unrounded_values_is_worse_on_peaked_rows():
    ratios = []
    for seed in (11, 12, 13):
        _, fused, exact_mean = _case(384, 32, True, False, 4.0, seed=seed)
        ratios.append(exact_mean / fused)
    assert min(ratios) >= 1.5 and sum(ratios) / len(ratios) >= 2.0, ratios


def test_one_hot_row_cancels_exactly():
    """One key carries all the weight: dS = 0, and the two products cancel to the last bit because the
    mean is the very operand that entered A1."""
    rng = np.random.default_rng(5)
    D, S = 32, 64
    K = _bf(rng.standard_normal((S, D)))
    V = _bf(rng.standard_normal((S, D)))
    dO = _bf(rng.standard_normal((1, D)))
    p = np.zeros((1, S))
    p[0, 17] = 1.0
    dP = dO @ V.T
    pb, wb = _bf(p), _bf(p * dP)
    a1, a2 = wb @ K, pb @ K
    dmean = wb.sum(1, keepdims=True) / pb.sum(1, keepdims=True)
    assert np.array_equal(a1 - dmean * a2, np.zeros((1, D)))
    # ... and does not with the exact mean, which is not a bf16 number
    assert np.max(np.abs(a1 - dP[:, 17:18] * a2)) > 0


def _two_products(Q, K, V, dO, bias, scale, shifted):
    """dQ of one (row, head) by the kernel's formula, with or without the constant that it subtracts from every dP of a
    query: the weighted mean of dP over the blocks of 32 keys so far, the present one included, taken anew in the first
    block and when the weight seen by a half-wave (keys whose index has bit 2 clear, or set) has grown fourfold for
    any of the 32 queries of a wavefront."""
    S, D = Q.shape[0], Q.shape[1]
    x = (scale * Q @ K.T + bias) / math.log(2)
    dP = dO @ V.T
    out = np.zeros((S, D))
    for q in range(0, S, 32):
        xq, dq = x[q:q + 32], dP[q:q + 32]
        n = xq.shape[0]
        top, c = np.full(n, -1e30), np.zeros(n)
        a1, a2, ls, ds, due = np.zeros((n, D)), np.zeros((n, D)), np.zeros((2, n)), np.zeros((2, n)), np.zeros((2, n))
        for k in range(0, S, 32):
            xb, db = xq[:, k:k + 32], dq[:, k:k + 32]
            half = [(np.arange(xb.shape[1]) >> 2 & 1) == i for i in (0, 1)]
            peak = xb.max(1)
            if np.any(peak > top + 8):
                raised = np.maximum(top, peak)
                alpha = np.exp2(top - raised)
                top = raised
                a1, a2 = a1 * alpha[:, None], a2 * alpha[:, None]
                ls, ds, due = ls * alpha, ds * alpha, due * alpha
            p = np.exp2(xb - top[:, None])
            pb = _bf(p)
            weight = ls + np.stack([pb[:, h].sum(1) for h in half])
            if shifted and np.any(weight > due):
                seen = weight.sum(0)
                move = (ds.sum(0) + (p * db).sum(1) - c * (weight - ls).sum(0)) / np.where(seen > 0, seen, 1.0)
                a1 -= move[:, None] * a2
                ds -= move * ls
                c += move
                due = 4 * weight
            wb = _bf(p * (db - c[:, None]))
            ls, ds = weight, ds + np.stack([wb[:, h].sum(1) for h in half])
            a1 += wb @ K[k:k + 32]
            a2 += pb @ K[k:k + 32]
        l = ls.sum(0)[:, None]
        out[q:q + 32] = scale * (a1 - (ds.sum(0)[:, None] / l) * a2) / l
    return out


def _errors(Q, K, V, dO, bias):
    """Relative 2-norm errors of dQ: dS rounded directly, two products without and with the constant."""
    scale = float(np.float32(1.0 / math.sqrt(Q.shape[1])))
    x = scale * Q @ K.T + bias
    P = np.exp(x - x.max(1, keepdims=True))
    P /= P.sum(1, keepdims=True)
    dP = dO @ V.T
    dS = P * (dP - (P * dP).sum(1, keepdims=True))
    ref = scale * dS @ K
    err = lambda a: float(np.linalg.norm(a - ref) / np.linalg.norm(ref))
    return tuple(err(a) for a in (scale * _bf(dS) @ K, _two_products(Q, K, V, dO, bias, scale, False),
                                  _two_products(Q, K, V, dO, bias, scale, True)))


@pytest.mark.parametrize("S", [144, 901])
@pytest.mark.parametrize("offset", [0.0, 0.5, 1.0, 2.0])
def test_common_offset_of_values_and_gradients(offset, S):
    """V and dO with a mean of their own, `offset` standard deviations: dP is then nearly the same for every key of
    a query, and only the constant keeps the two products as accurate as dS formed directly."""
    g = np.random.default_rng(S)
    D = 32
    Q, K, V, dO = (_bf(g.standard_normal((S, D)) + o) for o in (0.0, 0.0, offset, offset))
    bias = _bf(g.standard_normal((S, S)))
    direct, plain, shifted = _errors(Q, K, V, dO, bias)
    print(f"S={S} offset={offset}: direct {direct:.2e}, two products {plain:.2e}, with the constant {shifted:.2e}")
    assert shifted <= 1.25 * direct + 2e-4, (direct, plain, shifted)
    assert shifted <= 1.05 * plain, (plain, shifted)   # nor does it cost anything where there is no offset
    if offset >= 1.0:
        assert plain >= 2.5 * direct, (direct, plain)  # these data do show the difference


@pytest.mark.parametrize("S", [144, 384])
@pytest.mark.parametrize("what", ["first", "first_-4", "first_-8", "first_-20", "first_-60", "half", "rising"])
def test_offset_of_some_keys(what, S):
    """V offset for some of the keys, with a bias of its own: the constant follows the weight, and the rounding of the products
    is at most twice that of dS formed directly."""
    g = np.random.default_rng(S + 1)
    D, at = 32, np.arange(S)
    Q, K, V, dO = (_bf(g.standard_normal((S, D)) + o) for o in (0.0, 0.0, 0.0, 1.0))
    bias = _bf(g.standard_normal((S, S)))
    if what.startswith("first"):
        V = _bf(V + np.where(at < 32, 4.0, 0.0)[:, None])
        bias = bias + np.where(at < 32, float(what[6:] or 0), 0.0)
    elif what == "half":
        V = _bf(V + np.where(at >= S // 2, 4.0, 0.0)[:, None])
    else:
        V = _bf(V + np.linspace(0, 8, S)[:, None])
        bias = bias + np.linspace(0, 40, S)
    direct, plain, shifted = _errors(Q, K, V, dO, bias)
    print(f"S={S} {what}: direct {direct:.2e}, two products {plain:.2e}, with the constant {shifted:.2e}")
    assert shifted <= 2.0 * direct, (direct, plain, shifted)
