"""Short sequences, which one launch computes (16 or 32 query rows a workgroup, one key tile a wavefront and further ones in
turn): edges of query blocks and key tiles, more tiles than wavefronts, both row counts, each normalisation, strides and
output type, against the oracle; the workspace it leaves; and the calls that are to give the same bits."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import compare, to_dev, to_f64

pytestmark = pytest.mark.gpu

SPLITS = {64: (22, 20, 22), 128: (44, 42, 42)}

CASES = [  # batch, grid, heads, head_dim, dtype of the inputs, normalisation, head-major storage
    (1, (1, 1, 1), 1, 64, "bf16", None, False),          # one key, one row
    (2, (1, 3, 5), 2, 128, "f32", "head", False),        # 15: less than a block of rows
    (1, (1, 1, 17), 3, 64, "f32", "token", True),        # 17
    (1, (3, 3, 7), 2, 128, "bf16", "token", False),      # 63
    (1, (1, 8, 8), 40, 64, "bf16", "head", False),       # 64
    (2, (1, 5, 13), 5, 128, "bf16", None, True),         # 65
    (1, (1, 1, 257), 2, 128, "f32", None, False),        # a long table: 22 + 21 + 257 * 21 entries are too many, general path
    (1, (3, 7, 11), 9, 128, "f32", "token", False),      # 231
    (1, (1, 7, 59), 12, 64, "bf16", "token", False),     # 413: 32 rows a workgroup
    (1, (8, 8, 8), 8, 64, "bf16", "head", False),        # 512: every wavefront one tile, the last size in one round
    (1, (1, 13, 45), 6, 64, "f32", "token", False),      # 585: ten tiles on eight wavefronts, the last one of 9 keys
    (1, (6, 8, 8), 10, 128, "bf16", None, False),        # 384: the longest at head_dim 128
    (1, (1, 7, 55), 3, 128, "f32", "head", False),       # 385: one more, general path
    (1, (4, 16, 16), 8, 64, "f32", "head", False),       # 1,024: two tiles each, 32 rows
    (1, (7, 11, 13), 4, 64, "bf16", None, True),         # 1,001
    (1, (1, 7, 59), 12, 64, "f32", None, True),          # 413: 32 fp32 rows a workgroup in one launch
    (1, (1, 3, 43), 4, 128, "f32", None, False),         # 129: three key tiles, the last one of a single key
]


def _rms(x, mode, gamma, H, D):
    if mode is None:
        return x
    axes = (3,) if mode == "head" else (2, 3)
    return x / np.sqrt((x * x).mean(axis=axes, keepdims=True) + 1e-6) * gamma.reshape(1, 1, H, D).astype(np.float64)


def _wide(a):
    return (a.astype(np.uint32) << 16).view(np.float32) if a.dtype == np.uint16 else a


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%s-H%d-D%d-%s-%s-%d" % (
    c[0], "x".join(map(str, c[1])), c[2], c[3], c[4], c[5], c[6]))
def test_short_sequence(case):
    import torch

    nb, grid, H, D, dtype, mode, head_major = case
    split, L = SPLITS[D], grid[0] * grid[1] * grid[2]
    cfg = dict(B=nb, grid=grid, H=H, D=D, split=split, dtype=dtype, seed=17)
    qn, kn, vn = wl.self_attn_inputs(cfg)
    q, k, v = to_dev(qn), to_dev(kn), to_dev(vn)
    if head_major:
        q, k, v = (t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    rng = np.random.default_rng(5)
    gq, gk = ((1 + 0.25 * rng.standard_normal(H * D)).astype(np.float32) for _ in range(2))
    norm = None if mode is None else (mode, 1e-6, to_dev(gq), to_dev(gk))
    out = torch.full((nb, L, H, D), float("nan"), device="cuda")
    lse = torch.full((nb, H, L), float("nan"), device="cuda")
    need = B.dit_attn_workspace_bytes(B.self_attn_params(q, k, v, out, grid, split, norm=norm))
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    B.dit_attn_forward(q, k, v, grid, split, out=out, lse=lse, workspace=ws, norm=norm)

    # the oracle takes rows that are normalised already, in fp32
    f32 = [np.ascontiguousarray(_rms(_wide(x).astype(np.float64), mode, g, H, D).astype(np.float32)) for x, g in ((qn, gq), (kn, gk))]
    ref = oracle.self_attn(f32[0], f32[1], np.ascontiguousarray(_wide(vn)), grid, split)
    # The bar of 16-bit operands.  (q' and k' are off by 2^-12 of their value each, so a score of 64 to 128 products of unit
    # size by up to 2^-11 * 128 * 0.64 / sqrt(128) = 3.5e-3 and typically a tenth of that; so much of its probability times
    # |v| up to 4.5 is what a result is off by, 1e-2 of the RMS where a row of normalised heads sits on few keys.)
    compare(to_f64(out), ref, what="short %s" % (case,))

    # the same rows rounded
    out16 = B.dit_attn_forward(q, k, v, grid, split, out_dtype=torch.bfloat16, workspace=ws, norm=norm)
    assert torch.equal(out16, out.to(torch.bfloat16))
    # tiles that are resident: the same operands
    kept = ws.clone()
    again, lse2 = B.dit_attn_forward(q, None, None, grid, split, out_dtype=torch.float32, workspace=ws, norm=norm, want_lse=True,
                                     flags=B.DIT_FLAG_KV_RESIDENT)
    assert torch.equal(again, out) and torch.equal(lse2, lse) and torch.equal(ws, kept)
    # one packed request
    if nb == 1:
        packed = B.dit_attn_varlen_forward(q[0], k[0], v[0], [grid], split, out_dtype=torch.float32, norm=norm)
        assert torch.equal(packed, out[0])
    # the general path: the same results but for rounding, and the same workspace: rotation table and tile images
    ws_g = torch.zeros(need, dtype=torch.uint8, device="cuda")
    out_g, lse_g = B.dit_attn_forward(q, k, v, grid, split, out_dtype=torch.float32, want_lse=True, workspace=ws_g, norm=norm,
                                      flags=B.DIT_FLAG_SMALL_WORKGROUP)
    # (both are off by the same roundings of the operands; those of the probabilities differ with the reference maximum,
    # independently, and are the smaller part: the error as a whole may not be larger by more than a few per cent)
    err, err_g = (float(np.sqrt(np.mean((to_f64(o) - ref) ** 2))) for o in (out, out_g))
    assert err <= 1.1 * err_g + 1e-7, (err, err_g)
    assert (lse - lse_g).abs().max().item() < 1e-3
    table = 8 * (grid[0] * split[0] + grid[1] * split[1] + grid[2] * split[2]) // 2
    assert torch.equal(ws[:table], ws_g[:table])
    n = (table + 255) // 256 * 256 + nb * H * ((L + 63) // 64) * 2 * (18 if D == 128 else 10) * 1024
    assert torch.equal(ws[:n], ws_g[:n])


def test_output_over_the_keys():
    """Rows of out in the place of k's: the keys are packed before the first row is written."""
    import torch

    grid, H, D = (2, 8, 8), 4, 64
    qn, kn, vn = wl.self_attn_inputs(dict(B=1, grid=grid, H=H, D=D, split=SPLITS[D], dtype="f32", seed=3))
    q, k, v = to_dev(qn), to_dev(kn), to_dev(vn)
    ref = oracle.self_attn(qn, kn, vn, grid, SPLITS[D])
    B.dit_attn_forward(q, k, v, grid, SPLITS[D], out=k)
    compare(to_f64(k), ref, what="out over k")


@pytest.mark.parametrize("place", ["q columns", "k", "v", "lse over k", "lse over the weights"])
@pytest.mark.parametrize("grid,H,D,dtype,mode", [
    ((2, 8, 8), 4, 64, "f32", None), ((1, 7, 59), 12, 64, "bf16", "token"), ((4, 9, 16), 6, 64, "f32", "head"),
    ((3, 7, 9), 4, 128, "f32", "head"), ((6, 8, 8), 10, 128, "bf16", "head"), ((1, 5, 13), 2, 128, "bf16", None),
])
def test_place_of_the_results_does_not_change_them(grid, H, D, dtype, mode, place):
    """out or lse where the key rows or their weights are, or between them (the columns of one q/k/v buffer): the keys are
    packed before the first row is written, and every bit of out, lse and the workspace is that of the call beside them."""
    import torch

    split, L = SPLITS[D], grid[0] * grid[1] * grid[2]
    if place == "lse over the weights" and mode is None:
        pytest.skip("no weights")
    cfg = dict(B=1, grid=grid, H=H, D=D, split=split, dtype=dtype, seed=23)
    rng = np.random.default_rng(6)
    gq, gk = ((1 + 0.25 * rng.standard_normal(H * D)).astype(np.float32) for _ in range(2))
    rows = [to_dev(x) for x in wl.self_attn_inputs(cfg)]
    need = B.dit_attn_workspace_bytes(B.self_attn_params(*rows, rows[0], grid, split, norm=(mode, 1e-6, None, None) if mode else None))

    def call(where):
        buf = torch.stack(rows, dim=2)  # [1, L, 3, H, D]
        q, k, v = (buf[:, :, i] for i in range(3)) if where == "q columns" else (x.clone() for x in rows)
        gamma_k = torch.zeros(max(H * D, H * L), device="cuda")
        gamma_k[:H * D] = to_dev(gk)
        norm = None if mode is None else (mode, 1e-6, to_dev(gq), gamma_k[:H * D])
        out = {"q columns": q, "k": k, "v": v}.get(where, torch.full_like(rows[0], float("nan")))
        lse = torch.full((1, H, L), float("nan"), device="cuda")
        if where == "lse over k":
            lse = k.view(-1).view(torch.float32)[:H * L].view(1, H, L)
        if where == "lse over the weights":
            lse = gamma_k[:H * L].view(1, H, L)
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        B.dit_attn_forward(q, k, v, grid, split, out=out, lse=lse, workspace=ws, norm=norm)
        return out.contiguous(), lse.clone(), ws

    for got, beside in zip(call(place), call("beside")):
        assert torch.equal(got, beside)


@pytest.mark.parametrize("grid,H", [((3, 7, 11), 4), ((6, 8, 8), 10)])
def test_projection_then_attention_in_place(grid, H):
    """What the fused projection promises of its tiles, with out over the q columns of the rows of the separate route."""
    import torch

    D, K, L = 128, 128, grid[0] * grid[1] * grid[2]
    rng = np.random.default_rng(9)
    x, w = (to_dev(wl.f32_to_bf16_bits((rng.standard_normal(s) * K ** -0.25).astype(np.float32))) for s in ((L, K), (3 * H * D, K)))
    q, ws = B.dit_qkv_proj_forward(x, w, None, grid, SPLITS[D], H)
    fused = B.dit_attn_forward(q, None, None, grid, SPLITS[D], flags=B.DIT_FLAG_KV_RESIDENT, workspace=ws)
    q, k, v = (B.dit_linear_forward(x, w).view(1, L, 3, H, D)[:, :, i] for i in range(3))
    B.dit_attn_forward(q, k, v, grid, SPLITS[D], out=q)
    assert torch.equal(fused, q)
