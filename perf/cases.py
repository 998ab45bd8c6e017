"""What a user of this package has it do, as measurable cases.

A case is one step of a video diffusion transformer's attention block (or of
its training, or of the VAE decoder's windowed attention) through the public
functions of the package, on inputs that lie in device memory.  Kinds:

  self         K rotated by rope3d, then attn_fwd with keys_prerotated: how a
               denoising step calls the self-attention; ``text`` trailing
               tokens make it the joint video+text attention
  fused        one attn_fwd call that rotates queries and keys itself
  cross        text cross-attention: unrotated, a padded text of valid
               lengths that differ between the sequences of the batch
  train        a training step's self-attention: rotation, forward with lse,
               backward, the gradients carried back through the rotation
  train_cross  the same for text cross-attention
  na           3D neighbourhood attention of the VAE decoder
  proj         Q/K/V projection with norm, gain and rotation in its epilogue
  norm         norm, gain and rotation of already projected queries and keys

Grids are patchified latent volumes (frames, height, width).  Shapes are those
of the package's own workloads (inputs.py) and of the ranges around them: one
latent frame to full clips, all heads of a model to a tensor-parallel shard.
"""

import math

import torch

import paper_2609_18077_amd as vx

D = 128
EPS = 1e-6


def listed():
    return [
        # the smallest call (the package's "tiny" workload): launch latency
        {"name": "tiny", "kind": "fused", "B": 1, "H": 2, "T": 2, "Hp": 16, "Wp": 16, "text": 0, "half": False},
        # one latent frame at 832x480 (image generation, or one frame of a
        # streaming model): a few workgroups on a large chip
        {"name": "image_480p", "kind": "self", "B": 1, "H": 12, "T": 1, "Hp": 30, "Wp": 52, "text": 0, "half": False},
        # a short clip with 256 text tokens, 76 of them padding, in the
        # half-split rotary convention; lengths no multiple of any tile
        {"name": "joint_clip", "kind": "self", "B": 1, "H": 24, "T": 5, "Hp": 30, "Wp": 52, "text": 256, "half": True},
        # the benchmark workload: 81 frames at 832x480, 12 heads
        {"name": "wan13b_480p", "kind": "self", "B": 1, "H": 12, "T": 21, "Hp": 30, "Wp": 52, "text": 0, "half": False},
        # the largest call: 129 frames at 1280x720 with text, 24 heads
        {"name": "hunyuan_joint", "kind": "self", "B": 1, "H": 24, "T": 33, "Hp": 45, "Wp": 80, "text": 256,
         "half": False},
        # text cross-attention of 81 frames at 832x480, guided and unguided
        # prompt in one batch (lengths 64 to 512)
        {"name": "cross_text", "kind": "cross", "B": 2, "H": 40, "Lq": 32760, "Lk": 512},
        # post-training steps: a short clip of odd sizes, the full clip, and
        # the text cross-attention
        {"name": "train_clip", "kind": "train", "B": 1, "H": 12, "T": 5, "Hp": 23, "Wp": 41},
        {"name": "train_480p", "kind": "train", "B": 1, "H": 12, "T": 21, "Hp": 30, "Wp": 52},
        {"name": "train_cross", "kind": "train_cross", "B": 2, "H": 40, "Lq": 32760, "Lk": 512},
        # a VAE decoder stage: 16 latent frames of 80 x 45, window 11^3
        {"name": "na_vae", "kind": "na", "B": 1, "H": 4, "T": 16, "Hp": 45, "Wp": 80, "win": 11, "border": "clip"},
        # the projection that makes the benchmark workload's inputs
        {"name": "proj_480p", "kind": "proj", "B": 1, "H": 12, "T": 21, "Hp": 30, "Wp": 52, "C": 1536, "half": False},
        # the same prologue behind a separate projection (HBM-bound)
        {"name": "norm_480p", "kind": "norm", "B": 1, "H": 12, "T": 21, "Hp": 30, "Wp": 52, "half": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# heads of one GPU: whole models (12, 24, 40) and tensor-parallel shards
HEADS = (2, 3, 4, 5, 6, 8, 10, 12, 20, 24, 40)


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("self", "self", "fused", "cross", "train", "train_cross", "na", "proj", "norm"))
        c = {"kind": kind, "B": rng.choice((1, 1, 1, 2)), "H": rng.choice(HEADS)}
        if kind in ("cross", "train_cross"):
            c.update(Lq=_log_int(rng, 1000, 40000), Lk=rng.randint(77, 512))
        else:
            c.update(T=_log_int(rng, 1, 33), Hp=rng.randint(16, 45), Wp=rng.randint(16, 80))
        if kind in ("self", "fused"):
            c["text"] = rng.choice((0, 0, 77, 256))
        if kind in ("self", "proj", "norm"):
            c["half"] = rng.choice((False, True))
        if kind == "fused":
            c["half"] = False  # the fused key rotation takes interleaved pairs
        if kind == "na":
            c.update(H=rng.choice((2, 4, 8)), T=rng.randint(4, 20), win=rng.choice((5, 7, 9, 11)),
                     border=rng.choice(("clip", "shift")))
        if kind == "proj":
            c["C"] = min(c["H"], 24) * 128  # hidden size: the heads' width (a shard keeps it within a model's)
        if _cost(c) <= limit:
            return c


# ---------------------------------------------------------------- sizes ----


def _tokens(c):
    return c["T"] * c["Hp"] * c["Wp"]


def _length(c):
    return _tokens(c) + c.get("text", 0)


def _lens(c):
    """Valid keys of every batch, or None (all)."""
    if c["kind"] in ("cross", "train_cross"):
        # the prompts of a batch differ in length; a lone one fills five eighths
        if c["B"] == 1:
            return [c["Lk"] * 5 // 8]
        return [c["Lk"] // 8 + 7, c["Lk"]]
    if c.get("text", 0):
        return [_tokens(c) + max(1, c["text"] * 180 // 256) - 7 * b for b in range(c["B"])]
    return None


def _axis_windows(n, k, border):
    """(start, length) of the window of every position of an axis."""
    r = (k - 1) // 2
    out = []
    for p in range(n):
        if border == "clip":
            lo, hi = max(0, p - r), min(n - 1, p + r)
        elif n <= k:
            lo, hi = 0, n - 1
        else:
            lo = min(max(p - r, 0), n - k)
            hi = lo + k - 1
        out.append((lo, hi - lo + 1))
    return out


def work(c):
    B, H = c["B"], c["H"]
    if c["kind"] == "proj":
        m, n = B * _tokens(c), 3 * H * D
        return {"bytes": 2 * (m * c["C"] + n * c["C"] + m * n), "flops": 2 * m * n * c["C"]}
    if c["kind"] == "norm":
        return {"bytes": 2 * 2 * 2 * B * _tokens(c) * H * D, "flops": 2 * 12 * B * _tokens(c) * H * D}
    if c["kind"] == "na":
        pairs = B * H
        for n in ("T", "Hp", "Wp"):
            pairs *= sum(l for _, l in _axis_windows(c[n], c["win"], c["border"]))
        return {"bytes": 4 * 2 * B * _tokens(c) * H * D, "flops": 4 * D * pairs}
    if c["kind"] in ("cross", "train_cross"):
        lq, lk = c["Lq"], c["Lk"]
    else:
        lq = lk = _length(c)
    lens = _lens(c) or [lk] * B
    q, k = B * lq * H * D * 2, sum(lens) * H * D * 2
    pairs = H * lq * sum(lens)
    if c["kind"] in ("train", "train_cross"):
        # q, dout in, o and dq out, lse; k, v in, dk and dv out
        return {"bytes": 4 * q + 4 * k + 4 * B * H * lq, "flops": 14 * D * pairs}
    return {"bytes": 2 * q + 2 * k, "flops": 4 * D * pairs}


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def tolerance(c):
    # Measured against exact() on these ranges: attention outputs 2.2e-3 to
    # 3.3e-3 (rotated operands, probabilities and outputs rounded to bf16),
    # gradients 2.4e-3 to 4.0e-3 (also dS); norm and projection outputs 1.7e-3
    # (the output rounding alone).  Four times that; the largest single
    # difference over the RMS is about twenty times the relative error.
    if c["kind"] in ("proj", "norm"):
        return {"rel": 7e-3, "max": 0.05}
    if c["kind"] in ("train", "train_cross"):
        return {"rel": 1.6e-2, "max": 0.3}
    return {"rel": 1.3e-2, "max": 0.25}


# --------------------------------------------------------------- inputs ----


def _rope(c, **kw):
    return vx.Rope(grid=(c["T"], c["Hp"], c["Wp"]), pair_mode=1 if c.get("half") else 0, **kw)


def _inputs(c, seed):
    """The tensors of a case, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, unit=False):
        x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
        if unit:  # RMS-normalised rows, as the models' queries and keys are
            x *= torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS)
        return x

    B, H = c["B"], c["H"]
    s = {}
    if c["kind"] == "proj":
        m, n, C = B * _tokens(c), 3 * H * D, c["C"]
        s["x"] = normal(m, C).bfloat16()
        s["w"] = (normal(n, C) / math.sqrt(C)).bfloat16()
        s["bias"] = 0.1 * normal(n)
        s["gain_q"], s["gain_k"] = 1 + 0.1 * normal(D), 1 + 0.1 * normal(D)
    elif c["kind"] == "norm":
        s["q"], s["k"] = (normal(B, _tokens(c), H, D).bfloat16() for _ in range(2))
        s["gain_q"], s["gain_k"] = 1 + 0.1 * normal(D), 1 + 0.1 * normal(D)
    elif c["kind"] in ("cross", "train_cross"):
        s["q"] = normal(B, c["Lq"], H, D).bfloat16()
        s["k"], s["v"] = (normal(B, c["Lk"], H, D).bfloat16() for _ in range(2))
    else:
        unit = c["kind"] != "na"
        L = _length(c)
        s["q"], s["k"] = (normal(B, L, H, D, unit=unit).bfloat16() for _ in range(2))
        s["v"] = normal(B, L, H, D).bfloat16()
    if c["kind"] in ("train", "train_cross"):
        s["dout"] = normal(*s["q"].shape).bfloat16()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    lens = _lens(case) if case["kind"] not in ("proj", "norm", "na") else None
    s["lens"] = torch.tensor(lens, dtype=torch.int32, device="cuda") if lens else None
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "self":
        k = vx.rope3d(s["k"], _rope(c))
        return vx.attn_fwd(s["q"], k, s["v"], kv_valid_len=s["lens"], rope=_rope(c, keys_prerotated=True))
    if kind == "fused":
        return vx.attn_fwd(s["q"], s["k"], s["v"], kv_valid_len=s["lens"], rope=_rope(c))
    if kind == "cross":
        return vx.attn_fwd(s["q"], s["k"], s["v"], kv_valid_len=s["lens"])
    if kind in ("train", "train_cross"):
        q, k, v = s["q"], s["k"], s["v"]
        if kind == "train":
            q, k = vx.rope3d(q, _rope(c)), vx.rope3d(k, _rope(c))
        o, lse = vx.attn_fwd(q, k, v, kv_valid_len=s["lens"], return_lse=True)
        dq, dk, dv = vx.attn_bwd(q, k, v, o, s["dout"], lse, kv_valid_len=s["lens"])
        if kind == "train":
            vx.rope3d_transpose(dq, _rope(c), out=dq)
            vx.rope3d_transpose(dk, _rope(c), out=dk)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "na":
        return vx.na3d_fwd(s["q"], s["k"], s["v"], (c["T"], c["Hp"], c["Wp"]), window=(c["win"],) * 3,
                           border=c["border"])
    if kind == "proj":
        q, k, v = vx.qkv_proj(s["x"], s["w"], c["B"], _tokens(c), c["H"], bias=s["bias"], gain_q=s["gain_q"],
                              gain_k=s["gain_k"], eps=EPS, rope=_rope(c))
        return {"q": q, "k": k, "v": v}
    if kind == "norm":
        return {"q": vx.qk_norm_rope(s["q"], _rope(c), gain=s["gain_q"], eps=EPS),
                "k": vx.qk_norm_rope(s["k"], _rope(c), gain=s["gain_k"], eps=EPS)}
    raise ValueError(kind)


# ---------------------------------------------------------------- exact ----

_DIMS, _THETA = (44, 42, 42), 10000.0


def _cos_sin(c):
    """cos and sin [tokens, 64] of every channel pair's angle."""
    dev = "cuda"
    n = torch.arange(_tokens(c), device=dev)
    pos = (n // (c["Hp"] * c["Wp"]), n // c["Wp"] % c["Hp"], n % c["Wp"])
    ang = []
    for p, da in zip(pos, _DIMS):
        w = _THETA ** (-2.0 * torch.arange(da // 2, device=dev, dtype=torch.float64) / da)
        ang.append(p.double()[:, None] * w)
    ang = torch.cat(ang, 1)
    return ang.cos(), ang.sin()


def _pairs(half):
    """Channels of the first and second member of every pair."""
    a, b, off = [], [], 0
    for da in _DIMS:
        for j in range(da // 2):
            a.append(off + (j if half else 2 * j))
            b.append(off + (j + da // 2 if half else 2 * j + 1))
        off += da
    return a, b


def _rotate(x, c, inverse=False):
    """x [..., L, H, 128] in 64 bits, the first tokens rotated."""
    cos, sin = _cos_sin(c)
    if inverse:
        sin = -sin
    n = cos.shape[0]
    a, b = _pairs(c.get("half", False))
    y = x.clone()
    xa, xb = x[..., :n, :, a], x[..., :n, :, b]
    y[..., :n, :, a] = xa * cos[:, None] - xb * sin[:, None]
    y[..., :n, :, b] = xa * sin[:, None] + xb * cos[:, None]
    return y


def _attention(q, k, v, lens, dout=None):
    """o, lse (and dq, dk, dv), head by head in 64 bits; q, k given rotated."""
    B, Lq, H, _ = q.shape
    scale = float(torch.tensor(1.0 / D ** 0.5, dtype=torch.float32))
    o = torch.empty_like(q, dtype=torch.float64 if dout is not None else torch.float32)
    lse = torch.empty((B, H, Lq), dtype=torch.float64, device=q.device)
    grads = [torch.zeros_like(x, dtype=torch.float64) for x in (q, k, v)] if dout is not None else None
    for b in range(B):
        n = k.shape[1] if lens is None else lens[b]
        rows = max(1, min(Lq, (1 << 28) // n))  # 2 GiB of scores at a time
        for h in range(H):
            kh, vh = k[b, :n, h].double().contiguous(), v[b, :n, h].double().contiguous()
            kt, vt = kh.t().contiguous(), vh.t().contiguous()
            for i in range(0, Lq, rows):
                qh = q[b, i:i + rows, h].double().contiguous()
                s = (qh @ kt).mul_(scale)
                m = s.amax(1, keepdim=True)
                p = s.sub_(m).exp_()
                l = p.sum(1, keepdim=True)
                oh = (p @ vh) / l
                o[b, i:i + rows, h] = oh
                lse[b, h, i:i + rows] = (m + l.log())[:, 0]
                if dout is None:
                    continue
                p.div_(l)
                gh = dout[b, i:i + rows, h].double().contiguous()
                grads[2][b, :n, h] += p.t() @ gh
                ds = (gh @ vt).sub_((gh * oh).sum(1, keepdim=True)).mul_(p)
                grads[0][b, i:i + rows, h] = (ds @ kh) * scale
                grads[1][b, :n, h] += (ds.t() @ qh) * scale
    return o, lse, grads


def _norm(x, gain):
    x = x.double()
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.double()


def _neighbourhood(q, k, v, c):
    """64-bit windowed attention, one window offset at a time."""
    B, _, H, _ = q.shape
    grid = (c["T"], c["Hp"], c["Wp"])
    q, k, v = (x.reshape(B, *grid, H, D).double() for x in (q, k, v))
    scale = float(torch.tensor(1.0 / D ** 0.5, dtype=torch.float32))
    win = [_axis_windows(n, c["win"], c["border"]) for n in grid]
    start = [torch.tensor([s for s, _ in w], device=q.device) for w in win]
    size = [torch.tensor([l for _, l in w], device=q.device) for w in win]
    most = [max(l for _, l in w) for w in win]

    def moved(x, axis, j):
        return x.index_select(axis + 1, (start[axis] + j).clamp(max=grid[axis] - 1))

    def over(x):
        for jt in range(most[0]):
            xt = moved(x, 0, jt)
            for jh in range(most[1]):
                xh = moved(xt, 1, jh)
                for jw in range(most[2]):
                    ok = ((jt < size[0])[:, None, None] & (jh < size[1])[None, :, None] & (jw < size[2])[None, None])
                    yield moved(xh, 2, jw), ok

    s = torch.stack([((q * x).sum(-1) * scale).masked_fill_(~ok[None, ..., None], -math.inf) for x, ok in over(k)])
    p = torch.softmax(s, 0)
    o = torch.zeros_like(q)
    for i, (x, _) in enumerate(over(v)):
        o.addcmul_(p[i][..., None], x)
    return o.reshape(B, -1, H, D)


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("self", "fused"):
        lens = _lens(case)
        # one head at a time: the rotated 64-bit copies of a large call stay small
        heads = [_attention(_rotate(s["q"][:, :, h:h + 1].double(), case), _rotate(s["k"][:, :, h:h + 1].double(), case),
                            s["v"][:, :, h:h + 1], lens)[0] for h in range(case["H"])]
        return torch.cat(heads, 2)
    if kind == "cross":
        return _attention(s["q"], s["k"], s["v"], _lens(case))[0]
    if kind in ("train", "train_cross"):
        q, k, v, dout = (s[n].double() for n in ("q", "k", "v", "dout"))
        if kind == "train":
            q, k = _rotate(q, case), _rotate(k, case)
        o, lse, (dq, dk, dv) = _attention(q, k, v, _lens(case), dout)
        if kind == "train":
            dq, dk = _rotate(dq, case, inverse=True), _rotate(dk, case, inverse=True)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "na":
        return _neighbourhood(s["q"], s["k"], s["v"], case)
    if kind == "proj":
        B, L, H = case["B"], _tokens(case), case["H"]
        y = s["x"].double() @ s["w"].double().t().contiguous() + s["bias"].double()
        q, k, v = y.reshape(B, L, 3, H, D).unbind(2)
        return {"q": _rotate(_norm(q, s["gain_q"]), case), "k": _rotate(_norm(k, s["gain_k"]), case), "v": v}
    if kind == "norm":
        return {n: _rotate(_norm(s[n], s["gain_" + n]), case) for n in ("q", "k")}
    return None
