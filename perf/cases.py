"""The work a user of this library has it do, case by case, for timing and for comparing results.

Every case goes through the public calls of ``paper_2406_07368_amd.binding`` the way a model's layer would: a prompt
(prefill), a generation or speculation step on a running state (decode, verify, tree verify, three-branch step), or a
training step (three-branch forward and its gradient).  Sizes are those of the repository's workloads -- the layers of
LLaMA-2-7B (32 heads of 128), GPT-2-small (12 heads of 64), the FLASH experiment (8 heads of 128, groups of 256, 63
taps) -- and ragged ones around them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2406_07368_amd import binding
from paper_2406_07368_amd.workloads import candidate_tree, conv_weights

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # one user's chat on one GPU: a token at a time, one layer per call; nothing but latency
        dict(name="decode_single", kind="verify", B=1, H=32, d=128, dv=128, Kc=3, k=1, dtype="bf16", phi="elu1", prefix=2048),
        # a serving batch with a draft model: eight drafts a step, each row keeps its own number of them
        dict(name="verify_batch", kind="verify", B=32, H=32, d=128, dv=128, Kc=3, k=8, dtype="bf16", phi="elu1", prefix=2048),
        # Medusa-style speculation: 64 candidates in a tree with 42 leaves, one path kept per row
        dict(name="tree_batch", kind="tree", B=32, H=32, d=128, dv=128, Kc=3, n=64, leaves=42, dtype="bf16", phi="elu1", prefix=2048),
        # generation with the three-branch block: one token per row, open groups at every stage of filling
        dict(name="three_branch_step", kind="step", B=32, H=32, d=128, dv=128, Kc=3, k=1, dtype="bf16", phi="elu1", prefix=2048),
        # fp32 rows: a small model, or a reference run next to a bf16 one
        dict(name="prefill_fp32", kind="prefill", B=1, H=4, L=256, d=64, dv=64, Kc=3, chunk=64, dtype="f32", phi="elu1", layout="bhld"),
        # a GPT-2-small layer on a small batch of prompts, projections written token-major
        dict(name="prefill_gpt2", kind="prefill", B=4, H=12, L=1024, d=64, dv=64, Kc=3, chunk=64, dtype="bf16", phi="elu1", layout="blhd"),
        # a LLaMA-2-7B layer on a batch of full prompts
        dict(name="prefill_llama", kind="prefill", B=8, H=32, L=4096, d=128, dv=128, Kc=3, chunk=64, dtype="bf16", phi="elu1", layout="blhd"),
        # one very long document
        dict(name="prefill_long", kind="prefill", B=1, H=32, L=65536, d=128, dv=128, Kc=5, chunk=128, dtype="bf16", phi="elu1", layout="bhld"),
        # value rows twice as wide as key rows, a prompt length that no tile divides
        dict(name="prefill_wide", kind="prefill", B=4, H=32, L=2047, d=64, dv=128, Kc=3, chunk=64, dtype="bf16", phi="elu1", layout="bhld"),
        # the three-branch block over the LLaMA layer's prompts
        dict(name="three_branch_llama", kind="grouped", B=8, H=32, L=4096, d=128, dv=128, Kc=3, chunk=64, dtype="bf16", phi="elu1", layout="blhd"),
        # training of the FLASH layer, forward and gradient: one short ragged sequence ...
        dict(name="train_short", kind="train", B=1, H=8, L=1000, d=128, dv=128, Kc=63, chunk=256, dtype="bf16", phi="elu1", layout="bhld"),
        # ... and a batch of the experiment's longest ones
        dict(name="train_batch", kind="train", B=8, H=8, L=8192, d=128, dv=128, Kc=63, chunk=256, dtype="bf16", phi="elu1", layout="bhld"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: any kind, sizes log-uniform (ragged ones among them by nature)."""
    kind = rng.choice(["verify", "verify", "tree", "step", "prefill", "prefill", "prefill", "grouped", "train", "train"])
    dtype = "bf16"
    if kind in ("prefill", "grouped") and rng.random() < 0.25:
        dtype = "f32"
    d = rng.choice([64, 128, 128])
    H = {64: 12, 128: 32}[d] if rng.random() < 0.5 else rng.choice([4, 8, 16])
    phi = "relu" if rng.random() < 0.15 else "elu1"
    case = dict(kind=kind, H=H, d=d, dv=d, dtype=dtype, phi=phi)
    if kind in ("verify", "tree", "step"):
        case.update(B=_log(rng, 1, 32), Kc=rng.choice([1, 3, 3, 4, 5]), prefix=_log(rng, 64, 8192))
        if kind == "tree":
            n = rng.randint(4, 64)
            case.update(n=n, leaves=rng.randint((n + 1) // 2, n))
        else:
            case.update(k=rng.choice([1, 1, 2, 4, 5, 8, 16]))
        if kind == "verify" and d == 64 and rng.random() < 0.3:
            case["dv"] = 128
        return case
    case["layout"] = rng.choice(["bhld", "blhd"])
    if kind == "train":
        case.update(H=rng.choice([4, 8, 12]), chunk=rng.choice([256, 256, 64]), Kc=rng.choice([63, 63, 31, 3]))
        room = 8 * 8 * 8192 * 128
    elif dtype == "f32":
        # a reference run is a small one
        case.update(chunk=64, Kc=rng.choice([3, 3, 5]))
        room = 2 * 32 * 1024 * 128
    else:
        long_taps = kind == "grouped" and rng.random() < 0.4
        case.update(chunk=256 if long_taps else 64, Kc=63 if long_taps else rng.choice([1, 3, 3, 4, 5]))
        room = 8 * 32 * 4096 * 128
        if kind == "prefill" and d == 64 and rng.random() < 0.3:
            case["dv"] = 128
    width = case["H"] * max(case["d"], case["dv"])
    L = _log(rng, 100, min(16384, room // width))
    case.update(L=L, B=_log(rng, 1, max(1, min(16, room // (width * L)))))
    return case


def _rows(g, B, H, L, d, dtype, scale, layout):
    if layout == "blhd":
        return (torch.randn((B, L, H, d), generator=g, device="cuda") * scale).to(dtype).transpose(1, 2)
    return (torch.randn((B, H, L, d), generator=g, device="cuda") * scale).to(dtype)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, H, d, dv, Kc, dt = case["B"], case["H"], case["d"], case["dv"], case["Kc"], DTYPES[case["dtype"]]
    s = dict(case=case, eps=1e-6 if case["phi"] == "relu" else 0.0)
    s["w"] = torch.from_numpy(conv_weights(np.random.default_rng(seed), H, dv, Kc)).cuda()
    kind = case["kind"]
    if kind in ("prefill", "grouped", "train"):
        lay, L = case["layout"], case["L"]
        s["q"] = _rows(g, B, H, L, d, dt, d ** -0.5, lay)
        s["k"] = _rows(g, B, H, L, d, dt, d ** -0.5, lay)
        s["v"] = _rows(g, B, H, L, dv, dt, d ** -0.5 if kind == "train" else 1.0, lay)
        if kind == "train":
            s["dout"] = _rows(g, B, H, L, dv, dt, 1.0, lay)
        return s
    # a running state of the size that a prefix of unit normals leaves behind
    n = case["n"] if kind == "tree" else case["k"]
    P = case["prefix"]
    s["q"] = _rows(g, B, H, n, d, dt, 1.0, "bhld")
    s["k"] = _rows(g, B, H, n, d, dt, 1.0, "bhld")
    s["v"] = _rows(g, B, H, n, dv, dt, 1.0, "bhld")
    S = torch.randn((B, H, d, dv), generator=g, device="cuda") * (1.6 * P) ** 0.5
    z = 0.95 * P + torch.randn((B, H, d), generator=g, device="cuda") * (0.5 * P) ** 0.5
    hist = torch.randn((B, H, Kc - 1, dv), generator=g, device="cuda").to(dt)
    if kind == "tree":
        parent = candidate_tree(n, case["leaves"], seed)
        inner = set(parent.tolist())
        leaves = torch.tensor([i for i in range(n) if i not in inner], dtype=torch.int32, device="cuda")
        pick = torch.randint(len(leaves), (B,), generator=g, device="cuda")
        s["parent"] = torch.from_numpy(parent).cuda()
        s["accept"] = leaves[pick].contiguous()
        s["state"] = (S, z, hist)
        return s
    # the rows of a batch keep different numbers of drafts; a single draft is always kept
    s["n_commit"] = torch.randint(1, n + 1, (B,), generator=g, device="cuda", dtype=torch.int32) if n > 1 else None
    if kind == "step":
        kwin = torch.randn((B, H, 64, d), generator=g, device="cuda").to(dt)
        vwin = torch.randn((B, H, 64, d), generator=g, device="cuda").to(dt)
        fill = torch.randint(0, 64, (B, 1), generator=g, device="cuda", dtype=torch.int32).expand(B, H).contiguous()
        s["state"] = (S, z, hist, kwin, vwin, fill)
    else:
        s["state"] = (S, z, hist)
    return s


def run(s):
    c, kind, eps, phi = s["case"], s["case"]["kind"], s["eps"], s["case"]["phi"]
    if kind == "verify":
        if c["k"] == 1:
            out = binding.decode(s["q"], s["k"], s["v"], s["w"], s["state"], eps=eps, phi=phi)
        else:
            out = binding.verify(s["q"], s["k"], s["v"], s["w"], s["state"], n_commit=s["n_commit"], eps=eps, phi=phi)
        return (out, *s["state"])
    if kind == "tree":
        out = binding.verify_tree(s["q"], s["k"], s["v"], s["parent"], s["w"], s["state"], accept=s["accept"], eps=eps, phi=phi)
        return (out, *s["state"])
    if kind == "step":
        out = binding.verify_grouped(s["q"], s["k"], s["v"], s["w"], s["state"], n_commit=s["n_commit"], eps=eps, phi=phi)
        return (out, *s["state"])
    if kind == "prefill":
        out, state = binding.prefill(s["q"], s["k"], s["v"], s["w"], chunk=c["chunk"], eps=eps, phi=phi)
        return (out, *state)
    if kind == "grouped":
        out, state = binding.prefill_grouped(s["q"], s["k"], s["v"], s["w"], eps=eps, phi=phi, group=c["chunk"])
        return (out, *state)
    out, _ = binding.prefill_grouped(s["q"], s["k"], s["v"], s["w"], eps=eps, want_state=False, phi=phi, group=c["chunk"])
    return (out, *binding.prefill_grouped_backward(s["q"], s["k"], s["v"], s["w"], s["dout"], eps=eps, phi=phi, group=c["chunk"]))


def work(case):
    B, H, d, dv, Kc = case["B"], case["H"], case["d"], case["dv"], case["Kc"]
    eb = 2 if case["dtype"] == "bf16" else 4
    BH, kind = B * H, case["kind"]
    state = BH * ((d * dv + d) * 4 + (Kc - 1) * dv * eb)
    taps = H * dv * Kc * 4
    if kind in ("prefill", "grouped", "train"):
        L = case["L"]
        N = BH * L
        row = N * (2 * d + 2 * dv) * eb                             # q, k, v in, out out
        keys = (min(case["chunk"], L) + 1) / 2                      # keys a token meets in its own group
        token = 4 * d * dv + 3 * d + 2 * Kc * dv                    # state read and update, normaliser, conv
        if kind != "prefill":
            token += keys * 2 * (d + dv)
        if kind != "train":
            return {"bytes": row + state + taps, "flops": N * token}
        # gradient: q, k, v, dout in, dq, dk, dv out; five products per key and query, five per token and state, the conv's two
        back = keys * 10 * d + 10 * d * d + 4 * Kc * d
        return {"bytes": row + N * 7 * d * eb + 3 * taps, "flops": N * (token + back)}
    n = case["n"] if kind == "tree" else case["k"]
    rows = BH * n * (2 * d + 2 * dv) * eb
    token = 4 * d * dv + 3 * d + 2 * Kc * dv
    if kind == "step":
        # the open group's rows (half full on average) and the drafts; the sums are read and only now and then written
        read = BH * ((d * dv + d) * 4 + 2 * (Kc - 1) * dv * eb + 32 * 2 * d * eb + n * 2 * d * eb)
        return {"bytes": rows + read + taps, "flops": BH * n * (2 * d * dv + 32 * 4 * d + 2 * Kc * dv)}
    inner = (n + 1) / 2 * 2 * (d + dv)
    return {"bytes": rows + 2 * state + taps, "flops": BH * n * (token + inner)}


def tolerance(case):
    """Four times what the library differs from the fp64 oracle by (2-norm, and largest element over the larger of itself
    and the result's root mean square), measured over these ranges."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}                                        # 3e-7 at 256 tokens; sums over up to 16384 tokens
    if case["Kc"] > 8:
        return {"rel": 9e-3, "max": 4.5e-2}                         # 2.3e-3 and 1e-2: the long taps' pass rounds to bf16 too
    return {"rel": 7e-3, "max": 4.5e-2}                             # 1.7e-3 (one rounding to bf16) and 1.1e-2
