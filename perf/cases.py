"""The attention calls a user of this package makes, as measured cases.

A training step of a video DiT calls ``varlen_attention`` on a packed batch and takes the
gradients of q, k and v; sampling calls ``attn_fwd`` alone; a caller that may not allocate
device memory calls ``t2v_attn_bwd_noalloc`` with its own buffers. Clips come from latent
grids (tokens = frames x height x width patches), so packs mix very different lengths, and
the head shapes are those of the models the package is written for (12, 24 and 40 heads of
128, 30 heads of 64), whole or as one GPU's share under head sharding. Values are N(0, 1)
in bf16, scale 1 / sqrt(head dim).

A case: ``mode`` ("train", "infer" or "noalloc"), ``heads``, ``head_dim``, ``lengths`` (query
tokens of each clip) and ``lengths_k`` (keys of each clip for cross-attention, "" for
self-attention), the lengths as comma-separated text.
"""
import math

import numpy as np
import torch

from paper_2607_01701_amd import _lib, attn_fwd, varlen_attention

# Latent grids and what they are.
IMAGE = 1 * 32 * 32          # 1,024 tokens: one image
SHORT_CLIP = 5 * 16 * 16     # 1,280
MID_CLIP = 9 * 24 * 32       # 6,912
LONG_CLIP = 13 * 30 * 52     # 20,280
LONGEST_CLIP = 21 * 45 * 80  # 75,600

# The heterogeneous training batch (six short, seven middle and three long clips, shuffled).
HETERO = [MID_CLIP, SHORT_CLIP, SHORT_CLIP, LONG_CLIP, MID_CLIP, SHORT_CLIP, MID_CLIP, LONG_CLIP,
          MID_CLIP, MID_CLIP, SHORT_CLIP, MID_CLIP, SHORT_CLIP, LONG_CLIP, MID_CLIP, SHORT_CLIP]
# Text tokens of that batch's captions (32 to 256 each).
CAPTIONS = [77, 226, 32, 256, 120, 181, 45, 199, 128, 93, 250, 64, 143, 214, 109, 238]


def _case(name, mode, heads, head_dim, lengths, lengths_k=()):
    return {"name": name, "mode": mode, "heads": heads, "head_dim": head_dim,
            "lengths": ",".join(map(str, lengths)), "lengths_k": ",".join(map(str, lengths_k))}


def listed():
    return [
        # The smallest step: two few-second previews at 2 heads of 64; latency and launches count.
        _case("tiny_train", "train", 2, 64, [256, 384]),
        # Sampling one short clip with classifier-free guidance (two passes packed), 24 heads of 128.
        _case("short_clip_infer", "infer", 24, 128, [SHORT_CLIP, SHORT_CLIP]),
        # Image pre-training: a small batch of images, 12 heads of 128.
        _case("images_train", "train", 12, 128, [IMAGE] * 8),
        # Clips cropped to odd sizes, 30 heads of 64.
        _case("ragged_d64_train", "train", 30, 64, [4097, 333, 1280, 77, 6001, 2051, 911]),
        # Equal clips of 16 x 16 x 16 patches, 24 heads of 128.
        _case("uniform_train", "train", 24, 128, [4096] * 8),
        # The heterogeneous batch, 24 heads of 128: the ordinary training step.
        _case("hetero_train", "train", 24, 128, HETERO),
        # Cross-attention of that batch to its captions, 12 heads of 128: training and sampling.
        _case("cross_train", "train", 12, 128, HETERO, CAPTIONS),
        _case("cross_infer", "infer", 12, 128, [LONG_CLIP, LONG_CLIP], [226, 31]),
        # One middle clip, one GPU's three heads of 24 under eight-way head sharding.
        _case("clip_share_train", "train", 3, 128, [MID_CLIP]),
        # The longest clip, the same share.
        _case("longest_share_train", "train", 3, 128, [LONGEST_CLIP]),
        # Sampling a long clip, 24 heads of 128.
        _case("long_clip_infer", "infer", 24, 128, [LONG_CLIP]),
        # The backward pass of a small batch for a caller that may not allocate.
        _case("noalloc_backward", "noalloc", 12, 128, [SHORT_CLIP, 1999, IMAGE, 640]),
    ]


def _lengths(case):
    lq = [int(x) for x in case["lengths"].split(",")]
    lk = [int(x) for x in case["lengths_k"].split(",")] if case["lengths_k"] else lq
    return lq, lk


def _pairs(case):
    return sum(a * b for a, b in zip(*_lengths(case)))


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any mode, head shape and clip lengths of the same ranges, at most the cost
    of the heterogeneous training step."""
    top = next(c for c in listed() if c["name"] == "hetero_train")
    limit, tokens = work(top)["flops"], sum(_lengths(top)[0]) * 24 * 128
    while True:
        kind = rng.choice(["train", "train", "infer", "noalloc", "cross_train", "cross_infer"])
        heads, dim = rng.choice([(2, 64), (30, 64), (15, 64), (3, 128), (5, 128), (6, 128), (12, 128), (24, 128),
                                 (40, 128)])
        n = _log_int(rng, 1, 24)
        longest = _log_int(rng, 256, LONGEST_CLIP)
        lq = [min(longest, _log_int(rng, max(40, longest // 32), longest * 2)) for _ in range(n)]
        lk = [rng.randint(16, 256) for _ in lq] if kind.startswith("cross") else []
        case = _case("drawn", kind.replace("cross_", ""), heads, dim, lq, lk)
        del case["name"]
        rows = sum(lq) * heads
        if work(case)["flops"] > limit or rows * dim > tokens or rows < 600:
            continue
        if case["mode"] == "noalloc" and rows > 6_000_000:  # its scratch is 8 bytes a row, 64 MiB with the work lists
            continue
        return case


def _cu(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


def _inputs(case, seed):
    lq, lk = _lengths(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    h, d = case["heads"], case["head_dim"]
    return [torch.randn((rows, h, d), generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)
            for rows in (sum(lq), sum(lk), sum(lk), sum(lq))]


def prepare(case, seed):
    lq, lk = _lengths(case)
    q, k, v, dout = _inputs(case, seed)
    st = {"mode": case["mode"], "q": q, "k": k, "v": v, "dout": dout, "cu": _cu(lq),
          "cu_k": _cu(lk) if case["lengths_k"] else None, "scale": 1.0 / math.sqrt(case["head_dim"])}
    if case["mode"] == "train":
        for n in ("q", "k", "v"):
            st[n].requires_grad_(True)
    elif case["mode"] == "noalloc":
        st["out"], st["lse"] = attn_fwd(q, k, v, st["cu"], st["scale"])
        st["dq"], st["dk"], st["dv"] = (torch.empty_like(q) for _ in range(3))
    return st


def run(st):
    q, k, v = st["q"], st["k"], st["v"]
    if st["mode"] == "infer":
        return attn_fwd(q, k, v, st["cu"], st["scale"], cu_seqlens_k=st["cu_k"])
    if st["mode"] == "train":
        out, lse = varlen_attention(q, k, v, st["cu"], st["scale"], cu_seqlens_k=st["cu_k"])
        dq, dk, dv = torch.autograd.grad(out, (q, k, v), st["dout"])
        return out.detach(), lse, dq, dk, dv
    status = _lib.t2v_attn_bwd_noalloc(
        q.data_ptr(), k.data_ptr(), v.data_ptr(), st["out"].data_ptr(), st["lse"].data_ptr(), st["cu"],
        len(st["cu"]) - 1, q.shape[1], q.shape[2], st["scale"], st["dout"].data_ptr(), st["dq"].data_ptr(),
        st["dk"].data_ptr(), st["dv"].data_ptr(), torch.cuda.current_stream().cuda_stream)
    if status != 0:
        raise RuntimeError(_lib.t2v_last_error())
    return st["dq"], st["dk"], st["dv"]


def work(case):
    """Inputs read once and outputs written once; the forward's two matrix products and the
    backward's five (scores, dP, dV, dK, dQ), 2 flops per multiply-add."""
    lq, lk = _lengths(case)
    h, d = case["heads"], case["head_dim"]
    tq, tk = sum(lq) * h, sum(lk) * h
    product = 2 * h * d * _pairs(case)
    fwd_bytes = 2 * d * (2 * tq + 2 * tk) + 4 * tq       # q, k, v in; out and lse out
    bwd_bytes = 2 * d * (4 * tq + 4 * tk) + 4 * tq       # q, k, v, out, lse, dout in; dq, dk, dv out
    if case["mode"] == "infer":
        return {"bytes": fwd_bytes, "flops": 2 * product}
    if case["mode"] == "noalloc":
        return {"bytes": bwd_bytes, "flops": 5 * product}
    # A training step passes out and lse from the forward to the backward; dout comes in, the rest is read once.
    return {"bytes": 2 * d * (4 * tq + 4 * tk) + 4 * tq, "flops": 7 * product}


def tolerance(case):
    """bf16 inputs and results with P and dS in bf16 between the products: measured against
    float64, out, dq, dk and dv are off by 2e-3 to 3e-3 of their norm."""
    return {"rel": 1e-2}


def exact(case, seed):
    """The definition in float64 (blocks of whole score rows), laid out as ``run`` returns it."""
    if 7 * 2 * case["heads"] * case["head_dim"] * _pairs(case) > 1.2e14:
        return None
    lq, lk = _lengths(case)
    q, k, v, dout = (x.permute(1, 0, 2).contiguous() for x in _inputs(case, seed))
    scale = 1.0 / math.sqrt(case["head_dim"])
    cq, ck = _cu(lq), _cu(lk)
    out, lse = torch.empty_like(q, dtype=torch.float64), torch.empty(q.shape[:2], dtype=torch.float64, device=q.device)
    grads = case["mode"] != "infer"
    dq, dk, dv = (torch.zeros_like(x, dtype=torch.float64) for x in ((q, k, v) if grads else (q[:, :0],) * 3))
    for s in range(len(lq)):
        for h in range(case["heads"]):
            kk, vv = k[h, ck[s]:ck[s + 1]].double(), v[h, ck[s]:ck[s + 1]].double()
            kt, vt = kk.t().contiguous(), vv.t().contiguous()
            step = max(1, (1 << 27) // max(1, lk[s]))
            for a in range(int(cq[s]), int(cq[s + 1]), step):
                b = min(a + step, int(cq[s + 1]))
                qq = q[h, a:b].double()
                x = (qq @ kt) * scale
                lse[h, a:b] = torch.logsumexp(x, dim=1)
                p = torch.exp(x - lse[h, a:b, None])
                o = p @ vv
                out[h, a:b] = o
                if grads:
                    g = dout[h, a:b].double()
                    ds = p * (g @ vt - (g * o).sum(1, keepdim=True)) * scale
                    dv[h, ck[s]:ck[s + 1]] += p.t() @ g
                    dk[h, ck[s]:ck[s + 1]] += ds.t() @ qq
                    dq[h, a:b] = ds @ kk
    out, dq, dk, dv = (x.permute(1, 0, 2) for x in (out, dq, dk, dv))
    if case["mode"] == "infer":
        return out, lse
    return (dq, dk, dv) if case["mode"] == "noalloc" else (out, lse, dq, dk, dv)
