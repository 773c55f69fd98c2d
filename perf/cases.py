"""The attention calls whose speed this library stands for: forward, split-KV forward, backward, and a layer's
forward + backward, over the sizes, element types and options that its entry points take.

A case is a dict of plain values:
    call    "fwd" (attn_fwd / attn_fwd_f16), "splitkv" (attn_fwd_splitkv[_f16]), "bwd" (attn_bwd[_f16] on the tensors a
            forward call left), "train" (forward, then backward: one attention layer of a training step)
    dtype   "bf16" or "f16"
    B, H, S_q, S_kv, D, causal
    n_split key ranges of a split-KV call, 0 otherwise
    sharp   every row of Q and K also gets an offset drawn from N(0, 4): a peaked softmax whose maximum keeps moving
"""
import math

import torch

from paper_2512_18134_amd import binding

_DTYPE = {"bf16": torch.bfloat16, "f16": torch.float16}
_FWD = {"bf16": binding.attn_fwd, "f16": binding.attn_fwd_f16}
_SPLITKV = {"bf16": binding.attn_fwd_splitkv, "f16": binding.attn_fwd_splitkv_f16}
_BWD = {"bf16": binding.attn_bwd, "f16": binding.attn_bwd_f16}

_DEVICE = "cuda"
_MAX_S = 16384            # longest square sequence: the library's largest benchmark workload
_MAX_KV = 131072          # longest key sequence of a split-KV call
_MAX_FLOPS = 2.2e12       # a drawn case costs no more than the largest listed ones


def _case(name, call, dtype, B, H, S_q, S_kv, D, causal=False, n_split=0, sharp=False):
    return {"name": name, "call": call, "dtype": dtype, "B": B, "H": H, "S_q": S_q, "S_kv": S_kv, "D": D,
            "causal": causal, "n_split": n_split, "sharp": sharp}


def listed():
    return [
        # the five benchmark workloads: one head, where the launch itself counts; many short heads; causal
        # training length; the long-context headline; wide heads with a peaked softmax
        _case("fwd_one_head", "fwd", "bf16", 1, 1, 128, 128, 64),
        _case("fwd_short_heads", "fwd", "bf16", 4, 16, 1024, 1024, 64),
        _case("fwd_causal_4k", "fwd", "bf16", 2, 16, 4096, 4096, 128, causal=True),
        _case("fwd_long_16k", "fwd", "bf16", 1, 16, 16384, 16384, 128),
        _case("fwd_wide_sharp", "fwd", "bf16", 1, 8, 8192, 8192, 256, causal=True, sharp=True),
        # prefill of a single prompt whose length is no multiple of anything
        _case("fwd_prompt_777", "fwd", "bf16", 1, 16, 777, 777, 128, causal=True),
        # a batch of the paper's evaluation shape (32 heads of 128, fp16)
        _case("fwd_f16_2k", "fwd", "f16", 4, 32, 2048, 2048, 128),
        # decode: one new query per sequence against its cache of keys
        _case("decode_8k", "splitkv", "bf16", 4, 16, 1, 8191, 128, n_split=8),
        # few queries against a very long context
        _case("long_context", "splitkv", "bf16", 1, 8, 256, 131072, 128, n_split=32),
        # training steps: a small ragged one, an ordinary causal one
        _case("train_ragged_f16", "train", "f16", 2, 8, 515, 515, 64),
        _case("train_causal_2k", "train", "bf16", 2, 16, 2048, 2048, 128, causal=True),
        # backward alone, at the paper's batch and head count
        _case("bwd_4k", "bwd", "bf16", 4, 32, 4096, 4096, 128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _pairs(case):
    """(query, key) pairs that are not masked, of one head."""
    S_q, S_kv = case["S_q"], case["S_kv"]
    if not case["causal"]:
        return S_q * S_kv
    n = min(S_q, S_kv)
    return n * (n + 1) // 2 + (S_q - n) * S_kv


def draw(rng):
    """One more case of the ranges above: sizes log-uniform, most of them no multiple of a tile."""
    while True:
        call = rng.choice(["fwd", "fwd", "splitkv", "bwd", "train"])
        case = {"call": call, "dtype": rng.choice(["bf16", "f16"]), "n_split": 0, "sharp": False,
                "B": _log_int(rng, 1, 8), "H": rng.choice([1, 2, 4, 8, 12, 16, 32])}
        if call == "splitkv":
            case.update(D=rng.choice([64, 128]), causal=False, n_split=rng.choice([2, 3, 4, 8, 16, 32, 64]),
                        S_q=rng.choice([1, 1, _log_int(rng, 2, 512)]), S_kv=_log_int(rng, 1024, _MAX_KV))
        else:
            case.update(D=rng.choice([64, 128, 256] if call == "fwd" else [64, 128]), causal=rng.random() < 0.5)
            s = _log_int(rng, 64, _MAX_S)
            if rng.random() < 0.3:
                s = max(64, s // 64 * 64)
            case.update(S_q=s, S_kv=s)
            if rng.random() < 0.25:   # cross attention, or a chunk of a prompt
                case["S_q"] = _log_int(rng, 1 if call == "fwd" else 64, s)
            case["sharp"] = rng.random() < 0.15
        w = work(case)
        # (one entry of the state is at most a few GB: three states and their outputs fit the card many times over)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= 8e9:
            return case


def _scale(case):
    return 1.0 / math.sqrt(case["D"])


def _inputs(case, seed):
    """q, k, v (and d_o) on the GPU, from the seed alone."""
    g = torch.Generator(device=_DEVICE)
    g.manual_seed(int(seed) * 7919 + 17)
    B, H, D = case["B"], case["H"], case["D"]
    dt = _DTYPE[case["dtype"]]

    def normal(S, offset):
        x = torch.empty((B, H, S, D), dtype=torch.float32, device=_DEVICE).normal_(generator=g)
        if offset:
            x += torch.empty((B, H, S, 1), dtype=torch.float32, device=_DEVICE).normal_(0.0, 2.0, generator=g)
        return x.to(dt)

    q = normal(case["S_q"], case["sharp"])
    k = normal(case["S_kv"], case["sharp"])
    v = normal(case["S_kv"], False)
    d_o = normal(case["S_q"], False) if case["call"] in ("bwd", "train") else None
    return q, k, v, d_o


def prepare(case, seed):
    q, k, v, d_o = _inputs(case, seed)
    state = {"case": case, "q": q, "k": k, "v": v, "d_o": d_o}
    if case["call"] == "bwd":   # the forward call of the same step has been made
        state["o"], state["lse"] = _FWD[case["dtype"]](q, k, v, causal=case["causal"])
    return state


def run(state):
    case = state["case"]
    q, k, v = state["q"], state["k"], state["v"]
    call, dt, causal = case["call"], case["dtype"], case["causal"]
    if call == "splitkv":
        o, lse = _SPLITKV[dt](q, k, v, case["n_split"])
        return {"o": o, "lse": lse}
    if call == "bwd":
        dq, dk, dv = _BWD[dt](q, k, v, state["o"], state["d_o"], state["lse"], causal=causal)
        return {"dq": dq, "dk": dk, "dv": dv}
    o, lse = _FWD[dt](q, k, v, causal=causal)
    if call == "fwd":
        return {"o": o, "lse": lse}
    dq, dk, dv = _BWD[dt](q, k, v, o, state["d_o"], lse, causal=causal)
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def work(case):
    """Every input read once, every output written once; 4 D operations per unmasked pair forward, 10 D backward."""
    heads = case["B"] * case["H"]
    q = heads * case["S_q"] * case["D"] * 2
    kv = heads * case["S_kv"] * case["D"] * 2
    lse = heads * case["S_q"] * 4
    products = heads * _pairs(case) * case["D"]
    if case["call"] in ("fwd", "splitkv"):
        return {"bytes": 2 * q + 2 * kv + lse, "flops": 4 * products}
    if case["call"] == "bwd":       # q, o, d_o, dq; k, v, dk, dv; lse
        return {"bytes": 4 * q + 4 * kv + lse, "flops": 10 * products}
    return {"bytes": 4 * q + 4 * kv + lse, "flops": 14 * products}  # q, d_o, o, dq; k, v, dk, dv; lse


def tolerance(case):
    """16-bit P, dS and outputs: a call is 2.4e-3 (bf16) or 3e-4 (fp16) from the exact result, so two correct ones are
    up to 1.4 times that apart; about four times as much is allowed."""
    if case["dtype"] == "bf16":
        return {"rel": 1e-2}
    return {"rel": 2e-3}


def exact(case, seed):
    """The definition in 64 bits, head by head and in blocks of query rows."""
    q, k, v, d_o = _inputs(case, seed)
    B, H, S_q, S_kv, D = (case[n] for n in ("B", "H", "S_q", "S_kv", "D"))
    if B * H * S_q * S_kv > 6e9:
        return None
    scale = _scale(case)
    f64 = dict(dtype=torch.float64, device=_DEVICE)
    grads = d_o is not None
    o, lse = torch.empty((B * H, S_q, D), **f64), torch.empty((B * H, S_q), **f64)
    if grads:
        dq, dk, dv = torch.empty((B * H, S_q, D), **f64), torch.zeros((B * H, S_kv, D), **f64), torch.zeros((B * H, S_kv, D), **f64)
    q, k, v = q.view(B * H, S_q, D), k.view(B * H, S_kv, D), v.view(B * H, S_kv, D)
    step = max(1, min(S_q, (1 << 27) // S_kv))
    for h in range(B * H):
        kh, vh = k[h].double(), v[h].double()
        kt, vt = kh.t().contiguous(), vh.t().contiguous()
        for r0 in range(0, S_q, step):
            r1 = min(S_q, r0 + step)
            qh = q[h, r0:r1].double()
            s = torch.mm(qh, kt).mul_(scale)
            if case["causal"]:
                rows = torch.arange(r0, r1, device=_DEVICE)[:, None]
                s.masked_fill_(torch.arange(S_kv, device=_DEVICE)[None, :] > rows, float("-inf"))
            top = s.amax(dim=1, keepdim=True)
            p = s.sub_(top).exp_()
            total = p.sum(dim=1, keepdim=True)
            p.div_(total)
            lse[h, r0:r1] = (top + total.log())[:, 0]
            o[h, r0:r1] = torch.mm(p, vh)
            if grads:
                g = d_o.view(B * H, S_q, D)[h, r0:r1].double()
                dv[h] += torch.mm(p.t().contiguous(), g)
                ds = torch.mm(g, vt)
                ds.sub_((g * o[h, r0:r1]).sum(dim=1, keepdim=True)).mul_(p).mul_(scale)
                dq[h, r0:r1] = torch.mm(ds, kh)
                dk[h] += torch.mm(ds.t().contiguous(), qh)
    out = {"o": o.view(B, H, S_q, D), "lse": lse.view(B, H, S_q)}
    if not grads:
        return out
    grad = {"dq": dq.view(B, H, S_q, D), "dk": dk.view(B, H, S_kv, D), "dv": dv.view(B, H, S_kv, D)}
    return grad if case["call"] == "bwd" else {**out, **grad}
