"""The work that is timed: attention-layer calls of a video-DiT sampler through the package's public entry points.

A sampler builds the mask, its visit lists and a workspace once per latent grid, keeps the layer's weights on the GPU, and
then calls the layer once per block and timestep with new activations.  `prepare` makes what exists before such a call,
`run` is the call.
"""
import math

import torch

from paper_2601_16515_amd import binding as sb
from paper_2601_16515_amd import workloads as wl

BLOCK = 64


def _case(name, B, H, d, grid, sparsity, dtype="bf16", option="plain", **more):
    return dict(name=name, B=B, H=H, d=d, T=grid[0], Hh=grid[1], W=grid[2], dtype=dtype, sparsity=sparsity, option=option, **more)


def listed():
    return [
        # the fp32 layer of a debugging or reference run: a handful of small kernels, launches count
        _case("tiny f32", 1, 2, 64, (4, 16, 16), 0.75, dtype="f32"),
        # a preview at low resolution: odd grid, ragged last block, fewer tiles than the chip has compute units
        _case("preview", 1, 12, 128, (5, 15, 26), 0.75),
        # a short clip, heads of different magnitude
        _case("clip 75%", 1, 12, 128, (8, 30, 52), 0.75, head_magnitudes=True),
        # guided sampling: the conditional and the unconditional sample in one call, grid with odd sides
        _case("guided pair 90%", 2, 12, 128, (13, 31, 51), 0.90),
        # the 480p layer at the sparsity that it is deployed with
        _case("480p 90%", 1, 12, 128, (21, 30, 52), 0.90),
        # the same layer before any block is dropped, as in the first sampling steps and for quality control
        _case("480p dense", 1, 12, 128, (21, 30, 52), 0.0),
        # branch dropping after tuning: the gate decides on the GPU that the linear branch is pruned
        _case("480p 90% pruned", 1, 12, 128, (21, 30, 52), 0.90, option="pruned"),
        # the static scale as the full projection across heads, its weights laid out once per layer
        _case("480p 90% projection", 1, 12, 128, (21, 30, 52), 0.90, option="proj"),
        # the linear branch with rotary position embedding
        _case("480p 90% rotary", 1, 12, 128, (21, 30, 52), 0.90, option="rope"),
        # the dynamic block mask in place of the window: 4 of 40 key blocks per query token
        _case("480p top-k", 1, 12, 128, (21, 30, 52), 0.90, option="topk", topk=4, key_block=832),
        # a model of the same width with 64-wide heads
        _case("480p 90% d64", 1, 24, 64, (21, 30, 52), 0.90),
        # the 720p layer of the large model, the largest call
        _case("720p 90%", 1, 40, 128, (21, 45, 80), 0.90),
    ]


def draw(rng):
    """Grids from a thumbnail to 720p, sizes over their logarithm, every option and data type that the layer call takes."""
    limit = work(listed()[-1])
    while True:
        f32 = rng.random() < 0.12
        n = math.exp(rng.uniform(math.log(256), math.log(4096 if f32 else 75600)))
        T = rng.randint(1, min(21, max(1, int(n) // 64)))
        aspect = rng.uniform(0.5, 2.0)
        Hh = max(4, round(math.sqrt(n / T * aspect)))
        W = max(4, round(n / T / Hh))
        d = 64 if f32 or rng.random() < 0.2 else 128
        H = rng.choice((2, 4, 6) if f32 else (2, 5, 8, 12, 16, 24, 40))
        c = dict(B=rng.choice((1, 1, 2)), H=H, d=d, T=T, Hh=Hh, W=W, dtype="f32" if f32 else "bf16",
                 sparsity=round(rng.choice((0.0, rng.uniform(0.5, 0.8), rng.uniform(0.8, 0.95), rng.uniform(0.8, 0.95))), 3),
                 option=rng.choice(("plain", "plain", "plain", "pruned", "proj", "rope", "topk")))
        if (f32 or d == 64) and c["option"] not in ("plain", "pruned"):
            c["option"] = "plain"
        if c["option"] == "topk":
            blocks = rng.randint(6, 64)
            c["key_block"] = BLOCK * max(1, -(-T * Hh * W // (BLOCK * blocks)))
            c["topk"] = rng.randint(1, 6)
            c["sparsity"] = round(max(0.0, 1.0 - c["topk"] * c["key_block"] / (T * Hh * W)), 3)
        w = work(c)
        if w["flops"] <= limit["flops"] and w["bytes"] <= limit["bytes"]:
            return c


def _kinds(c):
    return [h % 2 for h in range(c["H"])]       # odd heads in the temporal token order


def _kept(c):
    nb = -(-c["T"] * c["Hh"] * c["W"] // BLOCK)
    return nb, min(nb, max(1, math.floor((1.0 - c["sparsity"]) * nb + 0.5)))


def prepare(case, seed):
    c = case
    B, H, d, T, Hh, W = (c[k] for k in ("B", "H", "d", "T", "Hh", "W"))
    N, D = T * Hh * W, H * d
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=dt)

    q, k, v = (normal(B, H, N, d) for _ in range(3))
    if c.get("head_magnitudes"):
        for t in (q, k, v):
            t.mul_((torch.rand(H, generator=g, device="cuda") * 1.5 + 0.5).to(dt)[None, :, None, None])
    s = dict(q=q, k=k, v=v, grid=(T, Hh, W), kinds=_kinds(c), out=torch.empty_like(q))
    kw = dict(lam=1.0, eps=1e-6, x_t=normal(B, N, D), w_gate=torch.randn(D, generator=g, device="cuda") * 0.02,
              s_out=torch.empty(B, device="cuda"))
    s["row_ptr"] = s["col_idx"] = None
    if c["option"] == "topk":
        kw.update(topk=c["topk"], topk_key_block=c["key_block"])
    else:
        nb, kept = _kept(c)
        s["row_ptr"], s["col_idx"] = sb.salad_block_mask(T, Hh, W, BLOCK, [kept] * H)
        if c["dtype"] == "bf16":
            kw["tile_lists"] = sb.salad_tile_lists(s["row_ptr"], s["col_idx"], H, nb)
    if c["option"] == "proj":
        w = (torch.randn(D, D, generator=g, device="cuda") / D ** 0.5).to(dt)
        kw["w_proj_packed"] = sb.salad_proj_pack(w, H, d)
        s["w_proj"] = w
    else:
        kw["head_scale"] = torch.rand(H, generator=g, device="cuda")
    if c["option"] == "pruned":
        kw["drop_threshold"] = 0.75            # the mean of sigmoids of small logits lies near one half
        kw["dropped_out"] = torch.empty(B, dtype=torch.int32, device="cuda")
    if c["option"] == "rope":
        cos, sin = wl.rope_tables(T, Hh, W, d)
        kw["rope_cos"], kw["rope_sin"] = torch.from_numpy(cos).cuda(), torch.from_numpy(sin).cuda()
    code = sb.SALAD_F32 if c["dtype"] == "f32" else sb.SALAD_BF16
    kw["workspace"] = sb.Workspace(B, H, N, d, code, full_proj=c["option"] == "proj", topk=kw.get("topk", 0),
                                   rope=c["option"] == "rope")
    s["kw"] = kw
    return s


def run(state):
    s = state
    sb.salad_sparse_linear_attn_fwd(s["q"], s["k"], s["v"], s["grid"], s["row_ptr"], s["col_idx"], s["kinds"], out=s["out"], **s["kw"])
    got = {"out": s["out"], "s": s["kw"]["s_out"]}
    if "dropped_out" in s["kw"]:
        got["dropped"] = s["kw"]["dropped_out"]
    return got


def work(case):
    """Tensors in and out once; products of the kept block pairs, of the linear branch and of the projection."""
    c = case
    B, H, d = c["B"], c["H"], c["d"]
    N = c["T"] * c["Hh"] * c["W"]
    D, size = H * d, 4 if c["dtype"] == "f32" else 2
    if c["option"] == "topk":
        blocks = -(-N // c["key_block"])
        pairs = N * min(N, min(c["topk"], blocks) * c["key_block"])
    else:
        nb, kept = _kept(c)
        tail = N - (nb - 1) * BLOCK
        # rows that keep the short last block: those whose window ends there
        with_last = sum(BLOCK if i < nb - 1 else tail for i in range(nb) if min(max(i - kept // 2, 0), nb - kept) + kept == nb)
        pairs = N * kept * BLOCK - with_last * (BLOCK - tail)
    flops = 4 * B * H * d * pairs + 2 * B * N * D
    nbytes = size * (4 * B * H * N * d + B * N * D)
    if c["option"] != "pruned":
        flops += 4 * B * H * N * d * d
    if c["option"] == "topk":
        flops += 2 * B * H * N * d * (-(-N // c["key_block"]))
    if c["option"] == "proj":
        flops += 2 * B * N * D * D
        nbytes += size * D * D
    if c["option"] == "rope":
        nbytes += 4 * N * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times the distance from the 64-bit result: 32-bit sums, or bf16 operands of the products and one (projection
    and top-k: two) bf16 roundings of the result."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6}
    return {"rel": 1e-2}


def exact(case, seed):
    """The layer in 64 bits with plain torch, head by head and a run of query blocks at a time; None where that takes too long."""
    c = case
    B, H, d, T, Hh, W = (c[k] for k in ("B", "H", "d", "T", "Hh", "W"))
    N, D = T * Hh * W, H * d
    if work(c)["flops"] > 4e12:
        return None
    s = prepare(c, seed)
    kw, f64 = s["kw"], torch.float64
    gate = torch.sigmoid(kw["x_t"].to(f64) @ kw["w_gate"].to(f64)).mean(1)
    dropped = gate < kw.get("drop_threshold", 0.0)
    positions = torch.arange(N, device="cuda")
    orders = [positions, (positions % T) * (Hh * W) + positions // T]     # stored row of each position of a head's own order
    sparse, linear = (torch.empty(B, N, H, d, dtype=f64, device="cuda") for _ in range(2))
    for b in range(B):
        for h in range(H):
            order = orders[s["kinds"][h]]
            q, k, v = (s[t][b, h].to(f64)[order] for t in "qkv")
            o = torch.empty_like(q)
            if c["option"] == "topk":
                step = c["key_block"]
                means = torch.stack([k[i:i + step].mean(0) for i in range(0, N, step)])
                top = (q @ means.T).topk(min(c["topk"], len(means)), 1).indices
                for i in range(0, N, 2048):
                    keep = torch.zeros(len(q[i:i + 2048]), len(means), dtype=torch.bool, device="cuda").scatter_(1, top[i:i + 2048], True)
                    w = (q[i:i + 2048] @ k.T / math.sqrt(d)).masked_fill_(~keep.repeat_interleave(step, 1)[:, :N], -math.inf)
                    o[i:i + 2048] = torch.softmax(w, 1) @ v
            else:
                nb, kept = _kept(c)
                first = [min(max(i - kept // 2, 0), nb - kept) for i in range(nb)]
                for i in range(0, nb, 8):                                  # 8 query blocks share one stretch of keys
                    j = min(i + 8, nb)
                    lo, hi = first[i] * BLOCK, min((first[j - 1] + kept) * BLOCK, N)
                    rows = slice(i * BLOCK, min(j * BLOCK, N))
                    start = torch.tensor(first[i:j], device="cuda").repeat_interleave(BLOCK)[: rows.stop - rows.start, None] * BLOCK
                    key = torch.arange(lo, hi, device="cuda")[None]
                    w = (q[rows] @ k[lo:hi].T / math.sqrt(d)).masked_fill_((key < start) | (key >= start + kept * BLOCK), -math.inf)
                    o[rows] = torch.softmax(w, 1) @ v[lo:hi]
            sparse[b, order, h] = o
            if not dropped[b]:
                pq, pk = q.clamp(min=0), k.clamp(min=0)
                den = pq @ pk.sum(0) + kw["eps"]
                if c["option"] == "rope":
                    cos, sin = (kw[t].to(f64)[order] for t in ("rope_cos", "rope_sin"))
                    pq, pk = (torch.stack((x[:, ::2] * cos - x[:, 1::2] * sin, x[:, ::2] * sin + x[:, 1::2] * cos), 2).flatten(1) for x in (pq, pk))
                linear[b, order, h] = (pq @ (pk.T @ v)) / den[:, None]
    out = torch.empty(B, H, N, d, dtype=f64, device="cuda")
    for b in range(B):
        got = sparse[b]
        if not dropped[b]:
            if c["option"] == "proj":
                got = got + kw["lam"] * gate[b] * (linear[b].reshape(N, D) @ s["w_proj"].to(f64)).reshape(N, H, d)
            else:
                got = got + kw["lam"] * gate[b] * kw["head_scale"].to(f64)[:, None] * linear[b]
        out[b] = got.transpose(0, 1)
    res = {"out": out, "s": gate}
    if c["option"] == "pruned":
        res["dropped"] = dropped.to(torch.int32)
    return res
