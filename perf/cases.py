"""Performance cases: the calls that users of this package make, over the sizes they make them at.

Attention is called through `binding.ss_attn_fwd` / `ss_attn_bwd`, the feed-forward operator through
`ffn_binding.ss_ffn_fwd` / `ss_ffn_bwd`, with tensors, outputs and workspace that stay on the GPU, as a
training loop or a server holds them.  A case is a dict of plain values:

  op         "attn" or "ffn"
  what       "fwd" (inference, or the first half of a step), "bwd", or "step" (forward, then backward)
  attention  B, H, S, D, dtype ("bf16", "f32"), bias ("", "dense", "relpos"), win (side of a window),
             mask ("", "causal", "region"), gated, layout ("bshd", or "sbhd": attention along the first
             storage axis), axis (the axis that is cut into chunks: "head" or "row"), k (chunks),
             keep_lse (the caller keeps the softmax statistics of the forward for the backward)
  ffn        T (tokens), dm, dh (hidden columns of this GPU's share), k, act ("gelu", "relu"),
             exact (partial sums in fp32, equal bits for every k)
"""
import math

import numpy as np
import torch

from paper_2301_08984_amd import binding as ss
from paper_2301_08984_amd import ffn_binding as fb
from paper_2301_08984_amd.workloads import shifted_window_region_ids

DEVICE = "cuda:0"
_DTYPE = {"bf16": (torch.bfloat16, ss.SS_BF16), "f32": (torch.float32, ss.SS_F32)}
_BIAS = {"": ss.SS_BIAS_NONE, "dense": ss.SS_BIAS_DENSE, "relpos": ss.SS_BIAS_RELPOS}
_MASK = {"": ss.SS_MASK_NONE, "causal": ss.SS_MASK_CAUSAL, "region": ss.SS_MASK_REGION}


def _attn(what, B, H, S, D, *, dtype="bf16", bias="", win=0, mask="", gated=False, layout="bshd", axis="row", k=1,
          keep_lse=False):
    return {"op": "attn", "what": what, "B": B, "H": H, "S": S, "D": D, "dtype": dtype, "bias": bias, "win": win,
            "mask": mask, "gated": gated, "layout": layout, "axis": axis, "k": k, "keep_lse": keep_lse}


def _ffn(what, T, dm, dh, *, k=1, act="gelu", exact=False):
    return {"op": "ffn", "what": what, "T": T, "dm": dm, "dh": dh, "k": k, "act": act, "exact": exact}


def listed():
    cases = {
        # the smallest call: a small fp32 operator, where launches and host time count
        "tiny_f32_step": _attn("step", 1, 4, 128, 32, dtype="f32", axis="head", k=2),
        # one GPU's 12 heads of a GPT layer under tensor parallelism, one training sequence
        "gpt_step": _attn("step", 1, 12, 2048, 128, mask="causal", axis="head", k=2),
        # long documents: the setting in which the plan's memory argument is made
        "gpt_long_step": _attn("step", 1, 12, 12288, 128, mask="causal", axis="head", k=2, keep_lse=True),
        # serving two prompts of an arbitrary length, heads of 64
        "gpt_prefill_ragged": _attn("fwd", 2, 12, 1531, 64, mask="causal", axis="head"),
        # shifted-window attention over a batch of feature maps: 4096 windows of 7 x 7
        "window_step": _attn("step", 4096, 16, 49, 32, bias="relpos", win=7, mask="region", k=4),
        # larger windows
        "window12_step": _attn("step", 512, 8, 144, 32, bias="relpos", win=12, mask="region", k=4),
        # row-wise gated attention with a pair bias over a multiple alignment
        "msa_row_step": _attn("step", 512, 8, 384, 32, bias="dense", gated=True, k=4),
        # triangle attention over a pair representation of 1024 residues
        "triangle_step": _attn("step", 1024, 4, 1024, 32, bias="dense", gated=True, k=16),
        # the same around the ending node (transposed storage) for a molecule of an arbitrary length
        "triangle_ragged_step": _attn("step", 901, 4, 901, 32, bias="dense", gated=True, layout="sbhd", k=16),
        # a feed-forward share serving a few tokens at a time: bound by reading the weights
        "ffn_decode": _ffn("fwd", 16, 12288, 6144),
        # the feed-forward share of the same GPT layer, one training sequence
        "ffn_step": _ffn("step", 2048, 12288, 6144, k=2),
        # and its backward with a micro-batch of four sequences
        "ffn_bwd_mb4": _ffn("bwd", 8192, 12288, 6144),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["fwd", "bwd", "step", "step"])
    kind = rng.choice(["gpt", "gpt", "window", "pair", "pair", "ffn", "ffn", "f32"])
    if kind == "gpt":
        H = rng.randint(1, 16)
        S = _log(rng, 128, 12288)
        B = rng.choice([1, 1, 2, 4])
        while B * H * S * S > 12 * 12288 ** 2:
            S = S * 3 // 4
        return _attn(what, B, H, S, rng.choice([128, 128, 64]), mask=rng.choice(["causal", "causal", "causal", ""]), axis="head",
                     k=min(H, rng.choice([1, 2, 4])), keep_lse=rng.random() < 0.5)
    if kind == "window":
        win = rng.choice([7, 7, 7, 8, 9, 12])
        H = rng.choice([3, 4, 6, 8, 12, 16, 24, 32])
        B = _log(rng, 16, 4096)
        while B * H * win ** 4 > 4096 * 16 * 49 ** 2:
            B = B * 2 // 3
        return _attn(what, B, H, win * win, 32, bias="relpos", win=win, mask=rng.choice(["region", ""]),
                     axis=rng.choice(["row", "row", "head"]), k=min(B, H, rng.choice([1, 2, 4])))
    if kind == "pair":
        H, S, B = rng.choice([4, 8]), _log(rng, 64, 1024), _log(rng, 16, 1024)
        while B * H * S * S > 901 * 4 * 901 ** 2:
            B = B * 2 // 3
        return _attn(what, B, H, S, 32, bias=rng.choice(["dense", "dense", ""]), gated=True, layout=rng.choice(["bshd", "sbhd"]),
                     k=min(B, rng.choice([1, 4, 16])), keep_lse=rng.random() < 0.25)
    if kind == "f32":
        return _attn(what, rng.randint(1, 4), rng.randint(1, 8), _log(rng, 32, 512), rng.choice([16, 24, 32, 64]), dtype="f32",
                     bias=rng.choice(["", "dense"]), mask=rng.choice(["", "causal"]), gated=rng.random() < 0.25,
                     axis="row", k=1, keep_lse=rng.random() < 0.25)
    dm, dh, T = 8 * _log(rng, 96, 1536), 8 * _log(rng, 96, 768), _log(rng, 1, 8192)
    act = rng.choice(["gelu", "gelu", "relu"])
    if T < 128:  # a few tokens are served, not trained on, and have no memory to save
        return _ffn("fwd", T, dm, dh, act=act)
    return _ffn(what, T, dm, dh, k=rng.choice([1, 1, 2, 4]), act=act, exact=rng.random() < 0.2)


def _normal(gen, shape, dtype, scale=1.0):
    """Standard normal values times `scale`, rounded once to the run's type."""
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)
    return (x if scale == 1.0 else x.mul_(scale)).to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    return _prepare_attn(case, gen) if case["op"] == "attn" else _prepare_ffn(case, gen)


def _prepare_attn(case, gen):
    B, H, S, D = case["B"], case["H"], case["S"], case["D"]
    torch_type, ss_type = _DTYPE[case["dtype"]]
    stored = (S, B, H, D) if case["layout"] == "sbhd" else (B, S, H, D)
    sb, st = (H * D, B * H * D) if case["layout"] == "sbhd" else (S * H * D, H * D)
    state = {"op": "attn", "what": case["what"], "keep_lse": case["keep_lse"]}
    for name in ("Q", "K", "V", "dY") + (("G",) if case["gated"] else ()):
        state[name] = _normal(gen, stored, torch_type)
    for name in ("Y", "dQ", "dK", "dV") + (("dG",) if case["gated"] else ()):
        state[name] = torch.zeros(stored, dtype=torch_type, device=DEVICE)
    state["lse"] = torch.zeros((B, H, S), dtype=torch.float32, device=DEVICE) if case["keep_lse"] else None
    if case["bias"]:
        w = case["win"]
        shape = (H, S, S) if case["bias"] == "dense" else (H, (2 * w - 1) ** 2)
        state["bias"] = _normal(gen, shape, torch_type, 1.0 if case["bias"] == "dense" else 0.02)
        state["dBias"] = torch.zeros(shape, dtype=torch.float32, device=DEVICE)
    period = 0
    if case["mask"] == "region":
        ids = shifted_window_region_ids(16 * case["win"], case["win"], case["win"] // 2)
        state["region"], period = torch.from_numpy(np.ascontiguousarray(ids)).to(DEVICE), ids.shape[0]
    head = case["axis"] == "head"
    desc = ss.make_desc(B, H, S, D, ss_type, 1.0 / math.sqrt(D), ss.SS_AXIS_HEAD if head else ss.SS_AXIS_ROW, 0,
                        H if head else B, case["k"], stride_b=sb, stride_s=st, stride_h=D, bias_kind=_BIAS[case["bias"]],
                        win=(case["win"], case["win"]), mask_kind=_MASK[case["mask"]], mask_period=period,
                        gated=case["gated"])
    need = ss.ss_attn_workspace_bytes(desc)[1]
    state["desc"] = desc
    state["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEVICE)
    if case["what"] == "bwd" and case["keep_lse"]:  # the statistics that the forward left
        _attn_fwd(state, torch.cuda.current_stream().cuda_stream)
    return state


def _attn_fwd(s, stream):
    ss.ss_attn_fwd(s["desc"], s["Q"], s["K"], s["V"], s.get("bias"), s.get("region"), s.get("G"), s["Y"], s["lse"], None, 0,
                   stream)


def _prepare_ffn(case, gen):
    T, dm, dh = case["T"], case["dm"], case["dh"]
    bf16 = torch.bfloat16
    state = {"op": "ffn", "what": case["what"], "X": _normal(gen, (T, dm), bf16), "dY": _normal(gen, (T, dm), bf16),
             "W1": _normal(gen, (dm, dh), bf16, dm ** -0.5), "W2": _normal(gen, (dh, dm), bf16, dh ** -0.5),
             "b1": _normal(gen, (dh,), bf16, 0.02), "b2": _normal(gen, (dm,), bf16, 0.02)}
    for name, like in (("Y", "X"), ("dX", "X"), ("dW1", "W1"), ("db1", "b1"), ("dW2", "W2"), ("db2", "b2")):
        state[name] = torch.zeros_like(state[like])
    desc = fb.make_desc(T, dm, dh, 0, dh, case["k"], act=fb.SS_ACT_GELU_TANH if case["act"] == "gelu" else fb.SS_ACT_RELU,
                        flags=fb.SS_FFN_FLAG_EXACT_SUM if case["exact"] else 0)
    state["desc"] = desc
    state["workspace"] = torch.empty(max(256, *fb.ss_ffn_workspace_bytes(desc)), dtype=torch.uint8, device=DEVICE)
    return state


def run(state):
    s, ws, what = state, state["workspace"], state["what"]
    stream = torch.cuda.current_stream().cuda_stream
    out = []
    if s["op"] == "attn":
        if what != "bwd":
            _attn_fwd(s, stream)
            out += ["Y", "lse"]
        if what != "fwd":
            ss.ss_attn_bwd(s["desc"], s["Q"], s["K"], s["V"], s.get("bias"), s.get("region"), s.get("G"), s["dY"], s["lse"],
                           s["dQ"], s["dK"], s["dV"], s.get("dBias"), s.get("dG"), ws, ws.numel(), stream)
            out += ["dQ", "dK", "dV", "dG", "dBias"]
    else:
        if what != "bwd":
            fb.ss_ffn_fwd(s["desc"], s["X"], s["W1"], s["b1"], s["W2"], s["b2"], s["Y"], ws, ws.numel(), stream)
            out += ["Y"]
        if what != "fwd":
            fb.ss_ffn_bwd(s["desc"], s["X"], s["W1"], s["b1"], s["W2"], s["dY"], s["dX"], s["dW1"], s["db1"], s["dW2"],
                          s["db2"], ws, ws.numel(), stream)
            out += ["dX", "dW1", "db1", "dW2", "db2"]
    return {name: s[name] for name in out if s.get(name) is not None}


def work(case):
    fwd, bwd = case["what"] != "bwd", case["what"] != "fwd"
    if case["op"] == "ffn":
        T, dm, dh = case["T"], case["dm"], case["dh"]
        act, weights, vecs = 2.0 * T * dm, 4.0 * dm * dh, 2.0 * (dm + dh)
        # forward: read X and the weights, write Y; backward: read X and dY too, write dX and the gradients
        moved = (2 * act + weights + vecs if fwd else 0) + (3 * act + 2 * weights + 2 * vecs if bwd else 0)
        return {"bytes": moved, "flops": 4.0 * T * dm * dh * fwd + 8.0 * T * dm * dh * bwd}
    B, H, S, D = case["B"], case["H"], case["S"], case["D"]
    size = 2 if case["dtype"] == "bf16" else 4
    act, stats = float(B) * S * H * D * size, 4.0 * B * H * S * case["keep_lse"]
    entries = {"": 0, "dense": H * S * S, "relpos": H * (2 * case["win"] - 1) ** 2}[case["bias"]]
    gate = 1 if case["gated"] else 0
    moved = 0.0
    if fwd:  # Q, K, V, G and the bias in; Y and the statistics out
        moved += (4 + gate) * act + entries * size + stats
    if bwd:  # Q, K, V, dY, G, bias and statistics in; dQ, dK, dV, dG and the bias gradient out
        moved += (7 + 2 * gate) * act + entries * (size + 4) + stats
    pairs = float(B) * H * S * S * (0.5 * (1 + 1.0 / S) if case["mask"] == "causal" else 1.0)
    # two products forward, five backward
    return {"bytes": moved, "flops": 2.0 * D * pairs * (2 * fwd + 5 * bwd)}


def tolerance(case):
    # fp32 operators carry 32-bit sums throughout; the others multiply bf16 operands
    return {"rel": 1e-5} if case.get("dtype") == "f32" else {"rel": 1e-2}
