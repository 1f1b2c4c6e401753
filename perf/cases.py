"""The work that a user of this library has it do, as a list of measurable cases.

A program that serves a video diffusion transformer calls the library for four things: self-attention on a latent
grid (one request or several packed ones), cross-attention onto the conditioning sequences, the dense projections
either side of them, and the q/k/v projection that leaves its keys and values ready for the attention.  The cases
below are such calls through paper_2601_20655_amd.binding, from a toy grid up to a full clip at the largest width
that the repository's workloads name, and draw() gives more of the same ranges.

Values: activations are N(0, 1) (rows behind a normalisation layer) or, where the call normalises q and k itself,
N(0, 1) times a per-token gain; weights are N(0, 1/K); normalisation weights 1 + N(0, 0.25^2).
"""
import math

import torch

from paper_2601_20655_amd import binding as dit

DEVICE = "cuda"
SPLITS = {64: (22, 20, 22), 128: (44, 42, 42)}  # channels per rotary axis (t, h, w)
ROPE_BASE = 10000.0
EPS = 1e-6


def listed():
    return [
        # The repository's toy grid in fp32: what a first integration test or a preview calls; all latency.
        dict(name="self_tiny", kind="self", B=1, T=4, Hg=8, Wg=8, H=4, D=64, dtype="f32", out="f32", norm="none",
             layout="blhd", lse=False),
        # Four heads of a short clip with the log-sum-exp asked for: a head shard of one request on one of several
        # GPUs, whose partial results are merged by their log-sum-exp.
        dict(name="self_shard", kind="self", B=1, T=4, Hg=30, Wg=52, H=4, D=128, dtype="bf16", out="f32",
             norm="none", layout="blhd", lse=True),
        # One high-resolution still image at 40 heads, q and k normalised per token, on the columns of a q/k/v
        # projection's output.
        dict(name="self_still_14b", kind="self", B=1, T=1, Hg=45, Wg=80, H=40, D=128, dtype="bf16", out="bf16",
             norm="token", layout="qkv", lse=False),
        # A full clip at 12 heads with q and k normalised per token.
        dict(name="self_clip_1p3b", kind="self", B=1, T=21, Hg=30, Wg=52, H=12, D=128, dtype="bf16", out="bf16",
             norm="token", layout="qkv", lse=False),
        # A full clip at 40 heads: the headline workload.
        dict(name="self_clip_14b", kind="self", B=1, T=21, Hg=30, Wg=52, H=40, D=128, dtype="bf16", out="bf16",
             norm="none", layout="blhd", lse=False),
        # A batch of requests of different resolution and length in one call at 12 heads.
        dict(name="packed_1p3b", kind="packed", grids="13x30x52 1x45x80 5x45x80 1x30x52 9x17x23", H=12, D=128,
             dtype="bf16", out="bf16", norm="head"),
        # Cross-attention of four full clips at 40 heads onto padded text and image keys with a byte mask.
        dict(name="cross_clip_14b", kind="cross", B=4, Lq=32760, n_text=512, n_image=257, text_len="169 281 104 319",
             keys="mask", two_softmax=False, resident=False, H=40, D=128, dtype="bf16", out="bf16", norm="none"),
        # One softmax each for text and image keys, lengths instead of a mask: image-to-video conditioning of one
        # clip at 40 heads.
        dict(name="cross_two_14b", kind="cross", B=1, Lq=32760, n_text=512, n_image=257, text_len="281",
             keys="lengths", two_softmax=True, resident=False, H=40, D=128, dtype="bf16", out="bf16", norm="none"),
        # A denoising step of a short clip at 12 heads: text keys packed by an earlier step, new queries.
        dict(name="cross_step_1p3b", kind="cross", B=1, Lq=7800, n_text=512, n_image=0, text_len="137",
             keys="lengths", two_softmax=False, resident=True, H=12, D=128, dtype="bf16", out="bf16", norm="token"),
        # Keys and values of the conditioning tokens of one request: a projection with few rows.
        dict(name="linear_cond_14b", kind="linear", M=769, N=10240, K=5120, bias=True, out="bf16"),
        # The output projection of a full clip at the width of 40 heads.
        dict(name="linear_out_14b", kind="linear", M=32760, N=5120, K=5120, bias=True, out="bf16"),
        # The front of a block at the width of 12 heads on a medium clip: the q/k/v projection that writes the
        # attention's tiles, then the attention.
        dict(name="block_1p3b", kind="block", T=9, Hg=30, Wg=52, H=12, K=1536, bias=True, out="bf16", norm="token"),
    ]


# ---- drawn cases ----

def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_grid(rng):
    return _log_int(rng, 1, 21), _log_int(rng, 6, 45), _log_int(rng, 6, 80)


def _draw_heads(rng):
    return _log_int(rng, 2, 40)


def _draw_once(rng):
    kind = rng.choice(["self", "self", "self", "packed", "cross", "cross", "cross", "linear", "linear", "block"])
    D = rng.choice([128, 128, 128, 64])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    out = dtype if rng.random() < 0.75 else "f32"
    norm = rng.choice(["none", "head", "token"])
    if kind == "self":
        T, Hg, Wg = _draw_grid(rng)
        return dict(kind=kind, B=rng.choice([1, 1, 2]), T=T, Hg=Hg, Wg=Wg, H=_draw_heads(rng), D=D, dtype=dtype,
                    out=out, norm=norm, layout=rng.choice(["blhd", "qkv", "bhld"]), lse=rng.random() < 0.25)
    if kind == "packed":
        grids = " ".join("%dx%dx%d" % _draw_grid(rng) for _ in range(rng.randint(2, 8)))
        return dict(kind=kind, grids=grids, H=_draw_heads(rng), D=D, dtype=dtype, out=out, norm=norm)
    if kind == "cross":
        B = rng.randint(1, 4)
        n_text = _log_int(rng, 32, 512)
        n_image = rng.choice([0, 257])
        return dict(kind=kind, B=B, Lq=_log_int(rng, 64, 32760), n_text=n_text, n_image=n_image,
                    text_len=" ".join(str(rng.randint(16, n_text)) for _ in range(B)),
                    keys=rng.choice(["mask", "lengths"]), two_softmax=n_image > 0 and rng.random() < 0.4,
                    resident=rng.random() < 0.4, H=_draw_heads(rng), D=D, dtype=dtype, out=out, norm=norm)
    if kind == "linear":
        return dict(kind=kind, M=_log_int(rng, 16, 32760), N=8 * _log_int(rng, 32, 1920), K=64 * _log_int(rng, 4, 80),
                    bias=rng.random() < 0.75, out=rng.choice(["bf16", "bf16", "f32"]))
    T, Hg, Wg = _draw_grid(rng)
    H = 2 * _log_int(rng, 1, 20)
    return dict(kind=kind, T=T, Hg=Hg, Wg=Wg, H=H, K=128 * H, bias=rng.random() < 0.75, out="bf16", norm=norm)


def draw(rng):
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= 8e12 and w["bytes"] <= 1.5e9:
            return case


# ---- helpers on a case ----

def _ints(text):
    return [int(x) for x in text.split()]


def _grids(case):
    if case["kind"] == "packed":
        return [tuple(int(x) for x in g.split("x")) for g in case["grids"].split()]
    return [(case["T"], case["Hg"], case["Wg"])]


def _tokens(grid):
    return grid[0] * grid[1] * grid[2]


def _dtype(name):
    return torch.float32 if name == "f32" else torch.bfloat16


def _esize(name):
    return 4 if name == "f32" else 2


def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * K + N * K + (N if case["bias"] else 0)) + _esize(case["out"]) * M * N,
                "flops": 2 * M * N * K}
    if kind == "block":
        L, H, K = _tokens(_grids(case)[0]), case["H"], case["K"]
        N = 3 * H * 128
        return {"bytes": 2 * (L * K + N * K + (N if case["bias"] else 0) + 2 * L * H * 128),
                "flops": 2 * L * N * K + 4 * H * L * L * 128}
    H, D = case["H"], case["D"]
    ei, eo = _esize(case["dtype"]), _esize(case["out"])
    if kind == "cross":
        keys = sum(_ints(case["text_len"])) + case["B"] * case["n_image"]
        rows = case["B"] * case["Lq"]
        return {"bytes": H * D * (rows * (ei + eo) + 2 * keys * ei), "flops": 4 * H * D * case["Lq"] * keys}
    B = case.get("B", 1)
    Ls = [_tokens(g) for g in _grids(case)]
    lse = 4 * B * H * sum(Ls) if case.get("lse") else 0
    return {"bytes": B * H * D * sum(Ls) * (3 * ei + eo) + lse, "flops": 4 * B * H * D * sum(L * L for L in Ls)}


def tolerance(case):
    # 16-bit results: one rounding to 8 significand bits is 1.7e-3 of the result.  fp32 results of attention: the
    # operands of both products carry 11 significand bits (4e-4 of the result).  fp32 results of a projection of
    # bf16 rows: only the order of an fp32 sum differs.
    if case["out"] == "bf16":
        return {"rel": 7e-3}
    if case["kind"] == "linear":
        return {"rel": 2e-6}
    return {"rel": 2e-3}


# ---- inputs ----

def _randn(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32).to(dtype)


def _rows(gen, shape, case):
    """Activations [..., tokens, H, D]; with a normalisation in the call, tokens differ in gain."""
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)
    if case["norm"] != "none":
        x *= torch.exp(0.3 * torch.randn(shape[:-2] + (1, 1), generator=gen, device=DEVICE, dtype=torch.float32))
    return x.to(_dtype(case["dtype"]))


def _norm_weights(gen, case):
    if case["norm"] == "none":
        return None
    n = case["H"] * case.get("D", 128)
    return tuple(1.0 + 0.25 * torch.randn(n, generator=gen, device=DEVICE, dtype=torch.float32) for _ in range(2))


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    kind = case["kind"]
    if kind in ("linear", "block"):
        M = case["M"] if kind == "linear" else _tokens(_grids(case)[0])
        N = case["N"] if kind == "linear" else 3 * case["H"] * 128
        K = case["K"]
        x = _randn(gen, (M, K), torch.bfloat16)
        w = (torch.randn((N, K), generator=gen, device=DEVICE, dtype=torch.float32) * K ** -0.5).to(torch.bfloat16)
        b = (0.1 * torch.randn(N, generator=gen, device=DEVICE, dtype=torch.float32)).to(torch.bfloat16)
        return dict(x=x, w=w, bias=b if case["bias"] else None,
                    gamma=_norm_weights(gen, case) if kind == "block" else None)
    H, D = case["H"], case["D"]
    if kind == "packed":
        n = sum(_tokens(g) for g in _grids(case))
        q, k, v = (_rows(gen, (n, H, D), case) for _ in range(3))
    elif kind == "self":
        B, L = case["B"], _tokens(_grids(case)[0])
        if case["layout"] == "qkv":  # the columns of one projection's output rows
            rows = _rows(gen, (B, L, 3 * H, D), case)
            q, k, v = rows[:, :, :H], rows[:, :, H:2 * H], rows[:, :, 2 * H:]
        else:
            q, k, v = (_rows(gen, (B, L, H, D), case) for _ in range(3))
            if case["layout"] == "bhld":  # head-major storage
                q, k, v = (t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    else:
        B, Lk = case["B"], case["n_text"] + case["n_image"]
        q = _rows(gen, (B, case["Lq"], H, D), case)
        k = _rows(gen, (B, Lk, H, D), case)
        v = _rows(gen, (B, Lk, H, D), case)
    return dict(q=q, k=k, v=v, gamma=_norm_weights(gen, case))


def _key_mask(case):
    mask = torch.zeros((case["B"], case["n_text"] + case["n_image"]), dtype=torch.uint8)
    for b, n in enumerate(_ints(case["text_len"])):
        mask[b, :n] = 1
        mask[b, case["n_text"]:] = 1
    return mask


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind = case["kind"]
    if kind == "linear":
        s["out"] = torch.empty((case["M"], case["N"]), dtype=_dtype(case["out"]), device=DEVICE)
        return s
    norm = None
    if case["norm"] != "none":
        norm = (case["norm"], EPS) + s["gamma"]
    s["norm"] = norm
    if kind == "block":
        L, H = _tokens(_grids(case)[0]), case["H"]
        s["q"] = torch.empty((1, L, H, 128), dtype=torch.bfloat16, device=DEVICE)
        s["out"] = torch.empty_like(s["q"])
        p = dit.self_attn_params(s["q"], s["q"], s["q"], s["out"], _grids(case)[0], SPLITS[128], norm=norm)
        s["ws"] = torch.empty(dit.dit_attn_workspace_bytes(p), dtype=torch.uint8, device=DEVICE)
        return s
    q, k, v = s["q"], s["k"], s["v"]
    s["out"] = torch.empty(q.shape, dtype=_dtype(case["out"]), device=DEVICE)
    split = SPLITS[case["D"]]
    if kind == "self":
        p = dit.self_attn_params(q, k, v, s["out"], _grids(case)[0], split, norm=norm)
        nbytes = dit.dit_attn_workspace_bytes(p)
        if case["lse"]:
            s["lse"] = torch.empty((case["B"], case["H"], q.shape[1]), dtype=torch.float32, device=DEVICE)
    elif kind == "packed":
        nbytes = dit.dit_attn_varlen_workspace_bytes(
            dit.varlen_attn_params(q, k, v, s["out"], _grids(case), split, norm=norm))
    else:
        s["split"] = case["n_text"] if case["two_softmax"] else 0
        nbytes = dit.dit_cross_attn_workspace_bytes(
            dit.cross_attn_params(q, k, v, s["out"], split=s["split"], norm=norm))
        if case["keys"] == "mask":
            s["mask"] = _key_mask(case).to(DEVICE)
        else:
            s["kv_len"] = torch.tensor([[n, case["n_image"]] for n in _ints(case["text_len"])], dtype=torch.int32,
                                       device=DEVICE)
    s["ws"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=DEVICE)
    if kind == "cross":
        s["flags"] = 0
        if case["resident"]:  # the first denoising step packs the conditioning keys, the later ones reuse them
            _cross(s)
            s["flags"] = dit.DIT_FLAG_KV_RESIDENT
    return s


# ---- one pass ----

def _cross(s):
    if s["case"]["keys"] == "mask":
        return dit.dit_cross_attn_forward(s["q"], s["k"], s["v"], s["mask"], out=s["out"], flags=s["flags"],
                                          workspace=s["ws"], split=s["split"], norm=s["norm"])
    return dit.dit_cross_attn_forward_lengths(s["q"], s["k"], s["v"], s["kv_len"], s["case"]["n_text"], out=s["out"],
                                              flags=s["flags"], workspace=s["ws"], split=s["split"], norm=s["norm"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linear":
        return dit.dit_linear_forward(s["x"], s["w"], s["bias"], out=s["out"])
    if kind == "cross":
        return _cross(s)
    if kind == "block":
        grid = _grids(case)[0]
        dit.dit_qkv_proj_forward(s["x"], s["w"], s["bias"], grid, SPLITS[128], case["H"], q_out=s["q"],
                                 workspace=s["ws"], norm=s["norm"])
        out = dit.dit_attn_forward(s["q"], None, None, grid, SPLITS[128], out=s["out"], workspace=s["ws"],
                                   flags=dit.DIT_FLAG_KV_RESIDENT, norm=s["norm"])
        return s["q"], out
    split = SPLITS[case["D"]]
    if kind == "packed":
        return dit.dit_attn_varlen_forward(s["q"], s["k"], s["v"], _grids(case), split, out=s["out"],
                                           workspace=s["ws"], norm=s["norm"])
    return dit.dit_attn_forward(s["q"], s["k"], s["v"], _grids(case)[0], split, out=s["out"], lse=s.get("lse"),
                                workspace=s["ws"], norm=s["norm"])


# ---- the same in 64 bits ----

def _angles(grid, D):
    """[tokens, D/2] rotation angles: pair i of an axis of d channels turns by position * base^(-2i/d)."""
    T, Hg, Wg = grid
    n = torch.arange(T * Hg * Wg, device=DEVICE)
    pos = (n // (Hg * Wg), n // Wg % Hg, n % Wg)
    parts = []
    for p, d in zip(pos, SPLITS[D]):
        freq = ROPE_BASE ** (-2.0 * torch.arange(d // 2, device=DEVICE, dtype=torch.float64) / d)
        parts.append(p.double()[:, None] * freq)
    return torch.cat(parts, dim=1)


def _rotate(x, ang):
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x[:, 0::2], x[:, 1::2]
    return torch.stack((a * c - b * s, a * s + b * c), dim=2).reshape(x.shape)


def _attend(q, k, v):
    """softmax(q k^T / sqrt(D)) v of one head, [Lq, D] and [Lk, D] in 64 bits; also the log-sum-exp."""
    out = torch.empty_like(q)
    lse = torch.empty(q.shape[0], dtype=torch.float64, device=q.device)
    kt = (k * q.shape[1] ** -0.5).t().contiguous()
    step = max(64, min(q.shape[0], (1 << 27) // k.shape[0]))
    for i in range(0, q.shape[0], step):
        p = q[i:i + step] @ kt
        m = p.amax(dim=1, keepdim=True)
        p.sub_(m).exp_()
        l = p.sum(dim=1, keepdim=True)
        out[i:i + step] = (p @ v) / l
        lse[i:i + step] = (m + torch.log(l))[:, 0]
    return out, lse


def _normed(x, mode, gamma):
    """RMS normalisation of [tokens, H, D] rows in 64 bits."""
    if mode == "none":
        return x
    dims = (2,) if mode == "head" else (1, 2)
    y = x / torch.sqrt((x * x).mean(dim=dims, keepdim=True) + EPS)
    return y * gamma.double().view(1, x.shape[1], x.shape[2])


def _exact_self(q, k, v, grid, mode, gamma):
    """[L, H, D] rows of one request."""
    q, k, v = q.double(), k.double(), v.double()
    gq, gk = gamma if gamma is not None else (None, None)
    q, k = _normed(q, mode, gq), _normed(k, mode, gk)
    ang = _angles(grid, q.shape[2])
    out = torch.empty_like(q)
    lse = torch.empty((q.shape[1], q.shape[0]), dtype=torch.float64, device=q.device)
    for h in range(q.shape[1]):
        out[:, h], lse[h] = _attend(_rotate(q[:, h], ang), _rotate(k[:, h], ang), v[:, h].contiguous())
    return out, lse


def _exact_cross(case, s):
    mask = _key_mask(case).bool().to(DEVICE)
    Lk, cut = mask.shape[1], case["n_text"]
    groups = ((0, cut), (cut, Lk)) if case["two_softmax"] else ((0, Lk),)
    out = torch.zeros(s["q"].shape, dtype=torch.float64, device=DEVICE)
    gq, gk = s["gamma"] if s["gamma"] is not None else (None, None)
    for b in range(case["B"]):
        q = _normed(s["q"][b].double(), case["norm"], gq)
        k = _normed(s["k"][b].double(), case["norm"], gk)
        v = s["v"][b].double()
        for lo, hi in groups:
            keep = torch.nonzero(mask[b, lo:hi])[:, 0] + lo
            for h in range(case["H"]):
                out[b, :, h] += _attend(q[:, h].contiguous(), k[keep, h], v[keep, h])[0]
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("linear", "block"):
        y = s["x"].double() @ s["w"].double().t().contiguous()
        if s["bias"] is not None:
            y += s["bias"].double()
        if kind == "linear":
            return y
        q, k, v = y.view(y.shape[0], 3, case["H"], 128).unbind(1)
        out, _ = _exact_self(q, k, v, _grids(case)[0], case["norm"], s["gamma"])
        return q[None], out[None]
    if kind == "cross":
        return _exact_cross(case, s)
    if kind == "packed":
        out, n = torch.empty(s["q"].shape, dtype=torch.float64, device=DEVICE), 0
        for g in _grids(case):
            m = n + _tokens(g)
            out[n:m], _ = _exact_self(s["q"][n:m], s["k"][n:m], s["v"][n:m], g, case["norm"], s["gamma"])
            n = m
        return out
    res = [_exact_self(s["q"][b], s["k"][b], s["v"][b], _grids(case)[0], case["norm"], s["gamma"])
           for b in range(case["B"])]
    out = torch.stack([r[0] for r in res])
    return (out, torch.stack([r[1] for r in res])) if case["lse"] else out
