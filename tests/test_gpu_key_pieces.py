"""Self-attention whose query tiles are computed in pieces along the keys and put together afterwards: shapes in which
every tile is (fewer tiles than compute units) and in which only those of the last round are, ragged on both sides
(last key tile, last query tile), both head dimensions, both output types; against the oracle, and against the
whole-tile form that a workspace without room for the pieces gets."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import compare, to_dev, to_f64

pytestmark = pytest.mark.gpu

SHAPES = [  # batch, grid, heads, head_dim, dtype of the inputs, flags
    (1, (1, 45, 77), 3, 128, "bf16", 0),                      # all tiles, 55 key tiles, last one of 9 keys
    (2, (3, 31, 33), 12, 128, "f32", 0),                      # 256 of 288 tiles whole
    (1, (1, 45, 77), 3, 64, "bf16", B.DIT_FLAG_BIG_WORKGROUP),
    (1, (2, 40, 40), 2, 128, "bf16", B.DIT_FLAG_QK_BF16 | B.DIT_FLAG_PV_BF16),
]


@pytest.mark.parametrize("case", SHAPES, ids=lambda c: "%dx%s-H%d-D%d-%s-%d" % (c[0], "x".join(map(str, c[1])), c[2], c[3], c[4], c[5]))
def test_pieces_against_oracle_and_whole_tiles(case):
    import torch

    nb, grid, H, D, dtype, flags = case
    split = (44, 42, 42) if D == 128 else (22, 20, 22)
    L = grid[0] * grid[1] * grid[2]
    cfg = dict(B=nb, grid=grid, H=H, D=D, split=split, dtype=dtype, seed=91)
    qn, kn, vn = wl.self_attn_inputs(cfg)
    q, k, v = to_dev(qn), to_dev(kn), to_dev(vn)
    out = torch.empty((nb, L, H, D), dtype=torch.float32, device="cuda")
    lse = torch.empty((nb, H, L), dtype=torch.float32, device="cuda")
    need = B.dit_attn_workspace_bytes(B.self_attn_params(q, k, v, out, grid, split, flags=flags))
    up = lambda x: (x + 255) // 256 * 256
    table = 8 * (grid[0] * split[0] + grid[1] * split[1] + grid[2] * split[2]) // 2
    whole = up(table) + nb * H * ((L + 63) // 64) * 2 * (18 if D == 128 else 10) * 1024
    assert need > whole, "this shape is meant to be computed in pieces"
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    ws.view(torch.float32).fill_(float("nan"))  # every piece that is read must have been written
    B.dit_attn_forward(q, k, v, grid, split, out=out, lse=lse, flags=flags, workspace=ws)
    got, got_lse = to_f64(out), to_f64(lse)
    # 16-bit output of the same call is the same numbers rounded
    out16 = B.dit_attn_forward(q, k, v, grid, split, out_dtype=torch.bfloat16, flags=flags, workspace=ws)
    assert torch.equal(out16, out.to(torch.bfloat16))
    # whole tiles: the same scores and probabilities, summed in fewer parts; what differs is the reference maximum of
    # a row's probabilities, which changes their rounding to 11 (bf16 operands: 8) significant bits
    out_w, lse_w = B.dit_attn_forward(q, k, v, grid, split, out_dtype=torch.float32, want_lse=True, flags=flags,
                                      workspace=ws[:whole].clone())
    rms = float(np.sqrt(np.mean(got ** 2)))
    bf16_ops = bool(flags & B.DIT_FLAG_PV_BF16)
    assert np.abs(to_f64(out_w) - got).max() <= (4e-2 if bf16_ops else 1e-2) * rms
    assert np.abs(to_f64(lse_w) - got_lse).max() < (1e-2 if bf16_ops else 1e-3)

    compare(got, oracle.self_attn(qn, kn, vn, grid, split), tol=4e-2 if bf16_ops else 2e-2, what="pieces %s" % (case,))


@pytest.mark.parametrize("grids,H,D", [(((2, 9, 17), (1, 45, 77), (1, 40, 60)), 3, 128), (((1, 50, 61), (1, 1, 5)), 5, 64),
                                       (((1, 45, 77),), 3, 128)], ids=["three", "long-and-short-d64", "one"])
def test_packed_requests_in_pieces(grids, H, D):
    import torch

    split = (44, 42, 42) if D == 128 else (22, 20, 22)
    cfg = dict(grids=grids, H=H, D=D, split=split, dtype="bf16", seed=92)
    qn, kn, vn = wl.varlen_attn_inputs(cfg)
    q, k, v = to_dev(qn), to_dev(kn), to_dev(vn)
    n = q.shape[0]
    out = torch.empty((n, H, D), dtype=torch.float32, device="cuda")
    lse = torch.empty((H, n), dtype=torch.float32, device="cuda")
    need = B.dit_attn_varlen_workspace_bytes(B.varlen_attn_params(q, k, v, out, grids, split))
    whole = B.dit_attn_varlen_workspace_bytes(
        B.varlen_attn_params(q, k, v, out, grids, split, flags=B.DIT_FLAG_SMALL_WORKGROUP))
    assert need > whole, "this batch is meant to be computed in pieces"
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    ws.view(torch.float32).fill_(float("nan"))
    B.dit_attn_varlen_forward(q, k, v, grids, split, out=out, lse=lse, workspace=ws)
    out_w, lse_w = B.dit_attn_varlen_forward(q, k, v, grids, split, out_dtype=torch.float32, want_lse=True,
                                             workspace=ws[:whole].clone())
    assert (lse_w - lse).abs().max().item() < 1e-3
    first = 0
    for g in grids:
        rows = slice(first, first + g[0] * g[1] * g[2])
        first = rows.stop
        ref = oracle.self_attn(qn[None, rows], kn[None, rows], vn[None, rows], g, split)[0]
        compare(to_f64(out[rows]), ref, what="request %s in pieces" % (g,))
        compare(to_f64(out_w[rows]), ref, what="request %s whole" % (g,))


@pytest.mark.parametrize("packed", [False, True], ids=["one-sequence", "packed"])
def test_bf16_scores_that_overflow_in_some_tiles(packed):
    """bf16 score operands can make a score -inf in fp32: such a key has no weight, and its row's result is that of the
    other keys, also where a piece of the keys starts with a tile of nothing else (whichever tiles the pieces start at:
    row i overflows in tile i only, rows 43 to 86 in one or several thirds of the sequence, which then hold whole
    pieces).  The latent grid has one frame, so the channels of the first rotary section are not rotated."""
    import torch

    grid, H, D, split = (1, 45, 77), 3, 128, (44, 42, 42)
    L = grid[1] * grid[2]
    n_tiles = (L + 63) // 64
    flags = B.DIT_FLAG_QK_BF16
    cfg = dict(B=1, grid=grid, H=H, D=D, split=split, dtype="f32", seed=93)
    q, k, v = wl.self_attn_inputs(cfg)
    q[..., :44] = 0.0
    k[..., :44] = 0.0
    for t in range(1, 43):  # (tile 0 stays ordinary: every row has a finite score in the first tile)
        q[:, t, :, t] = 1e30
        k[:, 64 * t:64 * (t + 1), :, t] = -1e30
    k[:, 64 * 18:64 * 37, :, 43] = -1e30
    q[:, 43:65, :, 43] = 1e30
    k[:, 64 * 37:, :, 0] = -1e30
    q[:, 65:87, :, 0] = 1e30
    q[:, 76:87, :, 43] = 1e30
    qn, kn, vn = (wl.f32_to_bf16_bits(a) for a in (q, k, v))
    ref, ref_lse = oracle.self_attn(qn, kn, vn, grid, split, rows=np.arange(128), want_lse=True)
    qd, kd, vd = to_dev(qn), to_dev(kn), to_dev(vn)
    if packed:
        short = (1, 3, 7)  # (a second request makes it a packed call; its rows repeat the first ones)
        n = L + 21
        qd, kd, vd = (torch.cat([t[0], t[0, :21]]) for t in (qd, kd, vd))
        p = B.varlen_attn_params(qd, kd, vd, qd, [grid, short], split, flags=flags)
        need = B.dit_attn_varlen_workspace_bytes(p)
        p.flags |= B.DIT_FLAG_SMALL_WORKGROUP
        assert need > B.dit_attn_varlen_workspace_bytes(p), "this batch is meant to be computed in pieces"
        out, lse = B.dit_attn_varlen_forward(qd, kd, vd, [grid, short], split, out_dtype=torch.float32, want_lse=True,
                                             flags=flags)
        out, lse = out[None, :L], lse[None, :, :L]
    else:
        assert n_tiles == 55
        p = B.self_attn_params(qd, kd, vd, qd, grid, split, flags=flags)
        need = B.dit_attn_workspace_bytes(p)
        p.flags |= B.DIT_FLAG_SMALL_WORKGROUP
        assert need > B.dit_attn_workspace_bytes(p), "this shape is meant to be computed in pieces"
        out, lse = B.dit_attn_forward(qd, kd, vd, grid, split, out_dtype=torch.float32, want_lse=True, flags=flags)
    compare(to_f64(out[:, :128]), ref, tol=4e-2, what="rows whose scores overflow")  # (8-bit score operands)
    assert np.abs(to_f64(lse[..., :128]) - ref_lse).max() < 1e-1


def test_small_workgroups_make_rows_independent_of_the_rest_of_the_call():
    """What the header promises for SMALL_WORKGROUP, in a shape that is cut into pieces without it: a sequence's rows keep
    their bits next to another batch entry, with fewer heads, among packed requests and in a larger workspace."""
    import torch

    grid, other, H, D, split = (1, 45, 77), (2, 9, 17), 3, 128, (44, 42, 42)
    L = grid[1] * grid[2]
    q, k, v = (to_dev(a) for a in wl.self_attn_inputs(dict(B=2, grid=grid, H=H, D=D, split=split, dtype="bf16", seed=94)))
    flags = B.DIT_FLAG_SMALL_WORKGROUP
    both = B.dit_attn_forward(q, k, v, grid, split, flags=flags)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    one = B.dit_attn_forward(q[1:], k[1:], v[1:], grid, split, flags=flags, workspace=ws)
    assert torch.equal(one[0], both[1])
    two = B.dit_attn_forward(q[1:, :, 1:], k[1:, :, 1:], v[1:, :, 1:], grid, split, flags=flags)
    assert torch.equal(two[0], both[1, :, 1:])
    n = other[0] * other[1] * other[2]
    packed = [torch.cat([t[0, :n], t[1]]) for t in (q, k, v)]
    assert torch.equal(B.dit_attn_varlen_forward(*packed, [other, grid], split, flags=flags)[n:], both[1])
