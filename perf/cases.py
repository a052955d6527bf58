"""The cases that the framework's speed is measured on: what a program that generates video chunk by
chunk has this library do, through the public entry points of `paper_2605_31158_amd.la`.

A case is a dict of plain values; `what` names the call or calls that one pass makes:

  step     select_blocks (or select_blocks_topk) and sparse_attn_fwd: one attention layer of one
           denoising step, everything computed from q, k and v
  cached   pool_blocks of q, select_pooled and sparse_attn_fwd: the same layer in the later denoising
           steps of a chunk, with the key means pooled once when the context entered its buffer
  attn     sparse_attn_fwd on given lists (of an earlier selection, or every block: tau >= 1)
  grid     sparse_attn_3d: the whole 3-D block path on linear-order inputs
  denoise  the 3-D path of a later denoising step: Q-Prep, KV-Prep of the chunk region only, selection
           from the means, attention and Untile Scatter, on buffers that hold the context
  prep     KV-Prep of every region: the context of a new chunk entering its block-major buffers
  mse      the latent dynamics between two chunk latents

Sizes are those of the evaluated models' latent grids (480P: frames of 30 x 52 tokens, 720P: 45 x 80),
a small call, and ragged ones.
"""
import math

import numpy as np
import torch

from paper_2605_31158_amd import la

F480, F720 = 30 * 52, 45 * 80


def _flat(name, what, H, d, Lq, Lk, block, scene, frame, tau=0.0, r=0.0, B=1, n_text=0, causal=False, lse=False):
    """A 1-D case: tau > 0 selects by cumulative mass, else floor(r M) blocks are kept."""
    c = dict(what=what, B=B, H=H, d=d, Lq=Lq, Lk=Lk, block=block, n_text=n_text, scene=scene, frame=frame,
             tau=tau, r=r, causal=causal, lse=lse)
    return dict(name=name, **c) if name else c


def _grid(name, what, H, d, n_text, T_ctx, T_q, Hs, Ws, bt, bh, bw, block, window, related, r, B=1, lse=False):
    c = dict(what=what, B=B, H=H, d=d, n_text=n_text, T_ctx=T_ctx, T_q=T_q, Hs=Hs, Ws=Ws, bt=bt, bh=bh, bw=bw,
             block=block, window=window, related=related, r=r, lse=lse)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a preview-sized chunk, where launches and host time count
        _flat("step_tiny", "step", 2, 64, 256, 1024, 64, "blocks", 256, tau=0.9),
        # 480P with an 8-frame temporal window: the ordinary call of exploration
        _flat("step_480p_window", "step", 16, 128, 4 * F480, 12 * F480, 64, "walk", F480, tau=0.9),
        # 480P with 16 retrieved memory frames before the window, a later denoising step, the paper's rule
        _flat("cached_480p_memory", "cached", 16, 128, 4 * F480, 28 * F480, 64, "memory", F480, r=0.05),
        # 480P after a long trajectory: the most keys to pool and score for the attention that follows
        _flat("step_480p_long", "step", 16, 128, 4 * F480, 68 * F480, 64, "clusters", F480, tau=0.9),
        # 720P, the largest of the 1-D calls
        _flat("step_720p", "step", 24, 128, 4 * F720, 20 * F720, 128, "unrelated", F720, tau=0.85),
        # 720P, frame-causal inside the chunk, with the log-sum-exp a caller merges other context with
        _flat("attn_720p_causal", "attn", 24, 128, 4 * F720, 20 * F720, 128, "unrelated", F720, tau=0.85,
              causal=True, lse=True),
        # every block kept: the dense pass that full-attention layers run through the same call
        _flat("attn_480p_dense", "attn", 16, 128, 4 * F480, 28 * F480, 64, "memory", F480, tau=1.0),
        # ragged everywhere: two sequences, odd lengths, text tokens, 64-wide heads, both outputs
        _flat("step_ragged", "step", 5, 64, 1111, 9001, 128, "walk", 277, r=0.175, B=2, n_text=77, lse=True),
        # 3-D blocks at 480P, from linear-order inputs to linear-order outputs
        _grid("grid_480p", "grid", 16, 128, 300, 24, 4, 30, 52, 4, 8, 4, 128, 8, 3, 0.175),
        # 3-D blocks at 720P in a later denoising step: only the chunk is new
        _grid("denoise_720p", "denoise", 24, 128, 0, 16, 4, 45, 80, 4, 4, 8, 128, 4, 0, 0.175),
        # a new chunk's context enters the 3-D buffers at 480P
        _grid("prep_480p", "prep", 16, 128, 300, 24, 4, 30, 52, 4, 8, 4, 128, 8, 3, 0.175),
        # latent dynamics of a 4-frame 480P chunk
        dict(name="mse_480p", what="mse", n=4 * F480 * 64, bf16=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# a drawn case has at most the attention work and the keys of the listed 720P calls
_MOST_FLOPS = 2.6e12
_MOST_KV = 24 * 72000 * 128


def _fits(c):
    if c["what"] in ("prep", "grid", "denoise"):
        keys = c["n_text"] + (c["T_ctx"] + c["T_q"]) * c["Hs"] * c["Ws"]
    else:
        keys = c["Lk"]
    return work(c)["flops"] <= _MOST_FLOPS and c["B"] * c["H"] * keys * c["d"] <= _MOST_KV


def draw(rng):
    kind = rng.choice(["step", "step", "step", "cached", "cached", "attn", "attn", "attn", "grid", "denoise", "prep",
                       "mse"])
    if kind == "mse":
        return dict(what="mse", n=_log(rng, 4096, 16 << 20) | 1, bf16=rng.random() < 0.5)
    while True:
        B, H, d = rng.choice([1, 1, 1, 2]), _log(rng, 1, 24), rng.choice([64, 128, 128, 128])
        n_text = rng.choice([0, 0, _log(rng, 16, 600)])
        if kind in ("grid", "denoise", "prep"):
            if rng.random() < 0.5:
                Hs, Ws, e = rng.choice([(30, 52, (4, 8, 4)), (45, 80, (4, 4, 8))])
                block = 128
            else:
                Hs, Ws = _log(rng, 8, 48), _log(rng, 8, 80)
                e, block = rng.choice([((4, 8, 4), 128), ((4, 4, 8), 128), ((2, 4, 8), 64), ((1, 8, 8), 64),
                                       ((3, 5, 4), 64)])
            T_q = rng.randint(1, 5)
            T_ctx = _log(rng, 4, 32)
            c = _grid("", kind, H, d, n_text, T_ctx, T_q, Hs, Ws, *e, block, min(T_ctx, 4 * rng.randint(1, 2)),
                      rng.randint(0, 3), round(rng.uniform(0.1, 0.3), 3), B=B, lse=rng.random() < 0.3)
        else:
            block = rng.choice([64, 128])
            frame = rng.choice([F480, F720, _log(rng, 128, 3600)])
            if frame in (F480, F720) and rng.random() < 0.6:
                Lq, ctx = frame * rng.randint(1, 4), frame * _log(rng, 4, 64)
            else:
                Lq = _log(rng, 64, 14400)
                ctx = _log(rng, 512, 110000)
            scene = rng.choice(["walk", "memory", "unrelated", "clusters"])
            # 64-wide heads have flatter scores: they are drawn with the paper's Top-floor(rM) rule, or dense
            tau = 0.0 if d == 64 or kind == "cached" or rng.random() < 0.4 else round(rng.uniform(0.8, 0.92), 3)
            if kind == "attn" and rng.random() < 0.25:
                tau = 1.0
            c = _flat("", kind, H, d, Lq, n_text + ctx + Lq, block, scene, min(frame, Lq), tau=tau,
                      r=0.0 if tau else round(rng.uniform(0.03, 0.25), 3), B=B, n_text=n_text,
                      causal=kind != "cached" and rng.random() < 0.25, lse=rng.random() < 0.3)
            if c["Lk"] > 110000 or (ctx // block) > 4096:
                continue
        if _fits(c):
            return c


# ------------------------------------------------------------------------------------------------
# shapes and work

def _blocks(c):
    """(NQ, NK, first and past-the-last historical block) of a 1-D case."""
    b = c["block"]
    h0, h1 = -(-c["n_text"] // b), (c["Lk"] - c["Lq"]) // b
    return -(-c["Lq"] // b), -(-c["Lk"] // b), h0, max(h0, h1)


def _keep(c):
    """Historical blocks a query block keeps: floor(r M), or what the mass rule keeps of these scenes
    (4.7 to 8.1 blocks measured on the listed ones, whatever the context's length)."""
    M = (_blocks(c)[3] - _blocks(c)[2]) if "Lq" in c else _grid_of(c)[2]
    tau = c.get("tau", 0.0)
    if tau >= 1.0:
        return M
    return min(M, 5) if tau else int(c["r"] * M)


def _la_grid(c):
    return la.grid3d(c["B"], c["H"], c["d"], c["n_text"], c["T_ctx"], c["T_q"], c["Hs"], c["Ws"], c["bt"], c["bh"],
                     c["bw"], c["block"])


def _grid_of(c):
    """(NQ, text blocks, context blocks, tokens per frame) of a 3-D case."""
    per = -(-c["Hs"] // c["bh"]) * -(-c["Ws"] // c["bw"])
    return (-(-c["T_q"] // c["bt"]) * per, -(-c["n_text"] // c["block"]), -(-c["T_ctx"] // c["bt"]) * per,
            c["Hs"] * c["Ws"])


def work(c):
    if c["what"] == "mse":
        return {"bytes": 2 * c["n"] * (2 if c["bf16"] else 4) + 8, "flops": 3 * c["n"]}
    BH, d = c["B"] * c["H"], c["d"]
    row = 2 * d                                        # bytes of one token of one head
    if "Lq" in c:
        NQ, NK, h0, h1 = _blocks(c)
        M, keep = h1 - h0, _keep(c)
        forced = c["Lk"] - M * c["block"]
        seen = forced                                  # forced keys a query sees, on average
        if c["causal"]:
            F = c["frame"]
            vis = sum(min(t * F + F, c["Lq"]) * min(F, c["Lq"] - t * F) for t in range(-(-c["Lq"] // F)))
            seen = forced - c["Lq"] + vis / c["Lq"]
        flops = 4.0 * d * BH * c["Lq"] * (seen + keep * c["block"])
        lists = BH * NQ * (4 + 4 * (NK - M + keep))
        kv = forced + keep * c["block"]                # keys every head's attention reads at the least
        out = BH * c["Lq"] * (2 * row + (4 if c["lse"] else 0))
        if c["what"] == "attn":
            return {"bytes": out + BH * 2 * kv * row + lists, "flops": flops}
        lists += BH * NQ * NK
        if c["what"] == "cached":
            return {"bytes": out + BH * 2 * kv * row + BH * M * 4 * d + lists, "flops": flops + 2.0 * d * BH * NQ * M}
        return {"bytes": out + BH * (c["Lk"] + kv) * row + lists, "flops": flops + 2.0 * d * BH * NQ * M}
    NQ, NT, NC, F = _grid_of(c)
    slots, Lq = c["block"], c["T_q"] * F
    Lk = c["n_text"] + (c["T_ctx"] + c["T_q"]) * F
    NK = NT + NC + NQ
    if c["what"] == "prep":
        return {"bytes": BH * (2 * Lk * row + 2 * NK * slots * row + NK * 4 * d), "flops": float(BH * Lk * d)}
    keep = _keep(c)
    kept = c["n_text"] + Lq + keep * (c["T_ctx"] * F / max(1, NC))
    flops = 4.0 * d * BH * Lq * kept + 2.0 * d * BH * NQ * NC
    lists = BH * NQ * (NK + 4 + 4 * (NK - NC + keep))
    # linear q, k, v in (the whole keys, or the chunk's alone), linear o out; the context's kept blocks
    fresh = Lk if c["what"] == "grid" else Lq
    held = 0 if c["what"] == "grid" else 2 * (kept - Lq) * row + NC * 4 * d
    return {"bytes": BH * (2 * Lq * row + 2 * fresh * row + held + (4 * Lq if c["lse"] else 0)) + lists,
            "flops": flops}


def tolerance(c):
    if c["what"] in ("prep", "mse"):
        return {"rel": 1e-6}                           # fp32 means of up to 128 rows; fp64 sum of fp32 chunks
    # bf16 outputs of bf16 probabilities: 2.4e-3 to 2.9e-3 against fp64; a block that flips at the cut of
    # the selection moves its row only
    return {"rel": 1e-2, "max": 0.3, "differ": 1e-3}


# ------------------------------------------------------------------------------------------------
# inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _fields(c, g, n_ctx, n_q, *slots):
    """Centroid field of every frame, [BH, n_ctx + n_q, *slots, d]: the frames next to the chunk and the
    chunk itself are a random walk; what comes before depends on the scene."""
    BH, d = c["B"] * c["H"], c["d"]
    scene = c.get("scene", "memory")

    def std(n):
        return torch.randn((BH, n) + slots + (d,), generator=g, device="cuda")

    if scene == "clusters":                            # 8 revisited places; the chunk visits two of them
        places = std(8)
        pick = torch.randint(0, 8, (n_ctx,), generator=g, device="cuda")
        now = torch.arange(n_q, device="cuda") * 2 // n_q
        return torch.cat([places[:, pick], places[:, now]], 1) + 0.2 * std(n_ctx + n_q)
    near = c.get("window", {"walk": n_ctx, "memory": 8, "unrelated": 4, "blocks": 0}[scene])
    near = min(near, n_ctx)
    steps = std(near + n_q)
    steps[:, 1:] *= 0.2
    walk = steps.cumsum(1)
    early = std(n_ctx - near)
    related = min(c.get("related", 3 if scene == "memory" else 0), n_ctx - near)
    for m in torch.randperm(n_ctx - near, generator=g, device="cuda")[:related].tolist():
        early[:, m] = walk[:, near + m % n_q]          # a memory frame that shows what a chunk frame shows
    return torch.cat([early, walk], 1)


def _noisy(cent, g, scale=0.5):
    return (cent + scale * torch.randn(cent.shape, generator=g, device="cuda")).to(torch.bfloat16)


def _qkv_flat(c, seed):
    """q, k, v [B, H, L, d]: tokens are their block's centroid plus noise; query block i has the centroid of
    chunk block i (scene "blocks": of a random context block)."""
    g = _gen(seed)
    B, H, d, b = c["B"], c["H"], c["d"], c["block"]
    NQ, NK, h0, h1 = _blocks(c)
    F, BH = c["frame"], B * H
    j0 = (c["Lk"] - c["Lq"]) // b                      # the block the chunk starts in
    if c["scene"] == "blocks":
        kc = torch.randn((BH, NK, d), generator=g, device="cuda")
        pick = torch.randint(0, max(1, h1), (BH, NQ, 1), generator=g, device="cuda")
        qc = kc.gather(1, pick.expand(-1, -1, d))
    else:
        n_ctx, n_q, S = -(-j0 * b // F) + 1, -(-max(c["Lq"], (NK - j0) * b) // F), -(-F // b) + 1
        table = _fields(c, g, n_ctx, n_q, S)

        def centroids(jj):                             # of the blocks jj, counted from the chunk's first
            f = torch.div(jj * b, F, rounding_mode="floor")
            r = jj - torch.div(f * F + b - 1, b, rounding_mode="floor")
            return table[:, (f + n_ctx).clamp(max=n_ctx + n_q - 1), r.clamp(0, S - 1)]

        kc = centroids(torch.arange(NK, device="cuda") - j0)
        qc = centroids(torch.arange(NQ, device="cuda"))
    q = _noisy(qc[:, torch.arange(c["Lq"], device="cuda") // b], g).view(B, H, c["Lq"], d)
    k = _noisy(kc[:, torch.arange(c["Lk"], device="cuda") // b], g).view(B, H, c["Lk"], d)
    v = torch.randn((B, H, c["Lk"], d), generator=g, device="cuda").to(torch.bfloat16)
    return q, k, v


def _qkv_grid(c, seed):
    """q, k, v in linear order: visual tokens are the centroid of their region of their frame plus noise."""
    g = _gen(seed)
    B, H, d, nf = c["B"], c["H"], c["d"], c["T_ctx"] + c["T_q"]
    ry, rx, F = -(-c["Hs"] // c["bh"]), -(-c["Ws"] // c["bw"]), c["Hs"] * c["Ws"]
    table = _fields(c, g, c["T_ctx"], c["T_q"], ry, rx)
    y = torch.arange(c["Hs"], device="cuda") // c["bh"]
    x = torch.arange(c["Ws"], device="cuda") // c["bw"]
    cent = table[:, :, y][:, :, :, x].reshape(B, H, nf * F, d)
    q = _noisy(cent[:, :, c["T_ctx"] * F:], g)
    text = torch.randn((B, H, c["n_text"], d), generator=g, device="cuda").to(torch.bfloat16)
    k = torch.cat([text, _noisy(cent, g)], 2)
    v = torch.randn(k.shape, generator=g, device="cuda").to(torch.bfloat16)
    return q, k, v


def prepare(case, seed):
    c = dict(case)
    if c["what"] == "mse":
        g = _gen(seed)
        z = torch.randn(c["n"], generator=g, device="cuda")
        z2 = z + 0.3 * torch.randn(c["n"], generator=g, device="cuda")
        dt = torch.bfloat16 if c["bf16"] else torch.float32
        return dict(c=c, a=z.to(dt), b=z2.to(dt), out=torch.zeros(1, dtype=torch.float64, device="cuda"),
                    ws=torch.empty(la.LATENT_MSE_WS_BYTES, dtype=torch.uint8, device="cuda"))
    s = dict(c=c, keep=_keep(c))
    if "Lq" not in c:
        s["q"], s["k"], s["v"] = _qkv_grid(c, seed)
        g = s["g"] = _la_grid(c)
        s["shape"] = shape = la.grid3d_shape(g)
        s["kvalid"] = torch.from_numpy(la.grid3d_valid(g)[1]).cuda()
        if c["what"] in ("prep", "denoise"):
            s["kt"] = torch.zeros((c["B"], c["H"], shape.Lk, c["d"]), dtype=torch.bfloat16, device="cuda")
            s["vt"] = torch.zeros_like(s["kt"])
            s["kbar"] = torch.zeros((c["B"], c["H"], shape.Lk // c["block"], c["d"]), device="cuda")
        if c["what"] == "denoise":
            la.prep_kv_3d(g, s["k"], s["v"], la.LA_PART_ALL, s["kt"], s["vt"], s["kbar"])
            s["ws"] = torch.empty(la.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
            s["qt"] = torch.empty((c["B"], c["H"], shape.Lq, c["d"]), dtype=torch.bfloat16, device="cuda")
            s["ot"] = torch.empty_like(s["qt"])
            s["qbar"] = torch.empty((c["B"], c["H"], shape.Lq // c["block"], c["d"]), device="cuda")
            s["o"] = torch.empty_like(s["q"])
        return s
    s["q"], s["k"], s["v"] = q, k, v = _qkv_flat(c, seed)
    B, H, d, b = c["B"], c["H"], c["d"], c["block"]
    NQ, NK, _, _ = _blocks(c)
    s["frame"] = c["frame"] if c["causal"] else 0
    s["shape"] = shape = la.make_shape(B, H, c["Lq"], c["Lk"], d, b, c["n_text"], s["frame"])
    s["ws"] = torch.empty(la.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    s["o"] = torch.empty_like(q)
    s["lse"] = torch.empty((B, H, c["Lq"]), device="cuda") if c["lse"] else None
    lists = (torch.empty((B, H, NQ, NK), dtype=torch.uint8, device="cuda"),
             torch.empty((B, H, NQ), dtype=torch.int32, device="cuda"),
             torch.full((B, H, NQ, NK), -1, dtype=torch.int32, device="cuda"))
    s["lists"] = lists
    if c["what"] == "cached":
        s["kbar"] = la.pool_blocks(k, b, "k", shape)
        s["qbar"] = torch.empty((B, H, NQ, d), device="cuda")
    if c["what"] == "attn":
        _select(s)
    return s


# ------------------------------------------------------------------------------------------------
# one pass

def _select(s):
    c = s["c"]
    if c["tau"]:
        return la.select_blocks(s["q"], s["k"], c["block"], c["tau"], c["n_text"], ws=s["ws"], out=s["lists"])
    return la.select_blocks_topk(s["q"], s["k"], c["block"], s["keep"], c["n_text"], ws=s["ws"], out=s["lists"])


def _attend(s, counts, idx):
    c = s["c"]
    la.sparse_attn_fwd(s["q"], s["k"], s["v"], counts, idx, c["block"], n_text=c["n_text"], frame_tokens=s["frame"],
                       ws=s["ws"], out=s["o"], lse_out=s["lse"])
    return {"o": s["o"], "lse": s["lse"]}


def run(s):
    c = s["c"]
    what = c["what"]
    if what == "step":
        mask, counts, idx = _select(s)
        return dict(_attend(s, counts, idx), mask=mask, counts=counts, idx=idx)
    if what == "cached":
        la.pool_blocks(s["q"], c["block"], "q", s["shape"], out=s["qbar"])
        mask, counts, idx = la.select_pooled(s["shape"], s["qbar"], s["kbar"], keep_blocks=s["keep"], ws=s["ws"])
        return dict(_attend(s, counts, idx), mask=mask, counts=counts)
    if what == "attn":
        return _attend(s, s["lists"][1], s["lists"][2])
    if what == "grid":
        o, lse, mask, counts, _ = la.sparse_attn_3d(s["g"], s["q"], s["k"], s["v"], keep_blocks=s["keep"],
                                                    want_lse=c["lse"], kvalid=s["kvalid"])
        return {"o": o, "lse": lse, "mask": mask, "counts": counts}
    if what == "denoise":
        g, shape = s["g"], s["shape"]
        la.prep_q_3d(g, s["q"], s["qt"], s["qbar"])
        la.prep_kv_3d(g, s["k"], s["v"], la.LA_PART_CHUNK, s["kt"], s["vt"], s["kbar"])
        mask, counts, idx = la.select_pooled(shape, s["qbar"], s["kbar"], keep_blocks=s["keep"], ws=s["ws"])
        res = la.sparse_attn_fwd(s["qt"], s["kt"], s["vt"], counts, idx, c["block"], n_text=shape.n_text,
                                 want_lse=c["lse"], ws=s["ws"], out=s["ot"], kvalid=s["kvalid"])
        o, lse = la.untile_o_3d(g, s["ot"], res[1] if c["lse"] else None, s["o"])
        return {"o": o, "lse": lse, "mask": mask, "counts": counts}
    if what == "prep":
        kt, vt, kbar = la.prep_kv_3d(s["g"], s["k"], s["v"], la.LA_PART_ALL, s["kt"], s["vt"], s["kbar"])
        return {"k": kt, "v": vt, "kbar": kbar}
    return la.latent_mse(s["a"], s["b"], ws=s["ws"], out=s["out"])


# ------------------------------------------------------------------------------------------------
# the same results in 64 bits, from the definitions

def _blocks_of(c):
    """Token ids of the query blocks and of the key blocks, and whether a key block is forced."""
    b = c["block"]
    if "Lq" in c:
        NQ, NK, h0, h1 = _blocks(c)
        qs = [np.arange(i * b, min(c["Lq"], i * b + b)) for i in range(NQ)]
        ks = [np.arange(j * b, min(c["Lk"], j * b + b)) for j in range(NK)]
        return qs, ks, np.array([not h0 <= j < h1 for j in range(NK)])

    def cut(T, base):
        ids = base + np.arange(T * c["Hs"] * c["Ws"]).reshape(T, c["Hs"], c["Ws"])
        return [ids[t:t + c["bt"], y:y + c["bh"], x:x + c["bw"]].reshape(-1) for t in range(0, T, c["bt"])
                for y in range(0, c["Hs"], c["bh"]) for x in range(0, c["Ws"], c["bw"])]

    F = c["Hs"] * c["Ws"]
    text = [np.arange(j, min(c["n_text"], j + b)) for j in range(0, c["n_text"], b)]
    ctx, chunk = cut(c["T_ctx"], c["n_text"]), cut(c["T_q"], c["n_text"] + c["T_ctx"] * F)
    forced = np.array([True] * len(text) + [False] * len(ctx) + [True] * len(chunk))
    return cut(c["T_q"], 0), text + ctx + chunk, forced


def _mean(x, sets):
    """Means over the token sets, [L, d] -> [len(sets), d] fp64."""
    ids = torch.from_numpy(np.concatenate(sets)).cuda()
    n = torch.tensor([len(t) for t in sets], device="cuda")
    out = torch.zeros((len(sets), x.shape[1]), dtype=torch.float64, device="cuda")
    out.index_add_(0, torch.repeat_interleave(torch.arange(len(sets), device="cuda"), n), x[ids].double())
    return out / n[:, None]


def _kept(c, q, k, qs, ks, forced):
    """bool [NQ, NK] of one head: the forced blocks and the historical ones the rule keeps."""
    hist = np.flatnonzero(~forced)
    keep = torch.from_numpy(forced).cuda().expand(len(qs), -1).clone()
    if not len(hist):
        return keep
    s = _mean(q, qs) @ _mean(k, [ks[j] for j in hist]).t().contiguous() / math.sqrt(c["d"])
    val, order = torch.sort(s, dim=1, descending=True, stable=True)
    tau = float(np.float32(c.get("tau", 0.0)))
    rank = torch.arange(len(hist), device="cuda")
    if tau >= 1.0:
        n = torch.full((len(qs), 1), len(hist), device="cuda")
    elif tau:
        n = (torch.softmax(val, 1).cumsum(1) < tau).sum(1, keepdim=True) + 1
    else:
        n = torch.full((len(qs), 1), _keep(c), device="cuda")
    chosen = torch.zeros_like(s, dtype=torch.bool).scatter_(1, order, rank[None] < n)
    keep[:, torch.from_numpy(hist).cuda()] = chosen
    return keep


def exact(case, seed):
    c = dict(case)
    if c["what"] == "mse":
        s = prepare(c, seed)
        return (s["a"].double() - s["b"].double()).square().mean().reshape(1)
    flat = "Lq" in c
    q, k, v = _qkv_flat(c, seed) if flat else _qkv_grid(c, seed)
    B, H, d = c["B"], c["H"], c["d"]
    qs, ks, forced = _blocks_of(c)
    if c["what"] == "prep":
        b = c["block"]
        src = torch.full((len(ks) * b,), -1, dtype=torch.int64)
        for j, t in enumerate(ks):
            src[j * b:j * b + len(t)] = torch.from_numpy(t)
        src = src.cuda()
        kt, vt = (torch.where((src >= 0)[:, None], x[:, :, src.clamp(min=0)], torch.zeros((), dtype=x.dtype, device="cuda"))
                  for x in (k, v))
        kbar = torch.stack([_mean(x, ks) for x in k.view(B * H, -1, d)]).view(B, H, len(ks), d)
        return {"k": kt.double(), "v": vt.double(), "kbar": kbar}
    Lq, Lk = q.shape[2], k.shape[2]
    o = torch.zeros((B, H, Lq, d), dtype=torch.float64, device="cuda")
    lse = torch.full((B, H, Lq), -math.inf, dtype=torch.float64, device="cuda")
    causal = flat and c["causal"]
    key_block = torch.zeros(Lk, dtype=torch.int64, device="cuda")
    for j, t in enumerate(ks):
        key_block[torch.from_numpy(t).cuda()] = j
    for b in range(B):
        for h in range(H):
            keep = _kept(c, q[b, h], k[b, h], qs, ks, forced)
            kd, vd, qd = k[b, h].double(), v[b, h].double(), q[b, h].double()
            for i, rows in enumerate(qs):
                rows = torch.from_numpy(rows).cuda()
                if bool(c.get("tau", 0.0) >= 1.0):
                    ids, kk, vv = None, kd, vd
                else:
                    ids = keep[i][key_block].nonzero().squeeze(1)
                    kk, vv = kd[ids], vd[ids]
                z = (qd[rows] @ kk.t().contiguous()) / math.sqrt(d)
                if causal:
                    n = (torch.arange(Lk, device="cuda") if ids is None else ids) - (Lk - Lq)
                    late = torch.div(n, c["frame"], rounding_mode="floor")[None] > (rows // c["frame"])[:, None]
                    z = z.masked_fill(late & (n >= 0)[None], -math.inf)
                lse[b, h, rows] = torch.logsumexp(z, 1)
                o[b, h, rows] = torch.softmax(z, 1) @ vv
    return {"o": o, "lse": lse if c["lse"] else None}
