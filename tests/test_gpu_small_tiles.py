"""Attention in whole tiles of few query rows: 16 rows a wavefront, in workgroups of 4 (64 rows) or 8 (128 rows), which
take the place of 4 wavefronts of 32 where all workgroups of a call fit one round.  Tile and sequence edges, both sides of the
two limits, each operand type, against the oracle; a head's rows keep their bits on either side of the limits."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import compare, to_dev, to_f64

pytestmark = pytest.mark.gpu

SMALL = B.DIT_FLAG_SMALL_WORKGROUP
SPLITS = {64: (22, 20, 22), 128: (44, 42, 42)}


@pytest.mark.parametrize("grid,H,D,dtype,flags", [
    ((1, 1, 1), 1, 128, "bf16", SMALL),                                  # one row, one key
    ((1, 1, 63), 2, 64, "f32", SMALL),
    ((1, 5, 13), 3, 128, "bf16", SMALL),                                 # 65: a second tile of one row, two key tiles
    ((1, 3, 43), 2, 64, "bf16", SMALL | B.DIT_FLAG_QK_BF16 | B.DIT_FLAG_PV_BF16),  # 129: three key tiles
    ((1, 8, 32), 64, 64, "bf16", SMALL),                                 # 256 tiles of 64 rows: the last call in those
    ((1, 8, 32), 65, 64, "bf16", SMALL),                                 # 130 tiles of 128 rows by 8 wavefronts
    ((3, 11, 13), 50, 128, "bf16", 0),                                   # 429 rows, 200 tiles
    ((1, 1, 321), 85, 128, "bf16", SMALL | B.DIT_FLAG_PV_BF16),          # 255
    ((1, 1, 321), 86, 128, "bf16", SMALL | B.DIT_FLAG_QK_BF16),          # 258: 4 wavefronts of 32 rows
], ids=lambda x: str(x).replace(" ", ""))
def test_small_tiles(grid, H, D, dtype, flags):
    import torch

    L, split = grid[0] * grid[1] * grid[2], SPLITS[D]
    qn, kn, vn = wl.self_attn_inputs(dict(B=1, grid=grid, H=H, D=D, split=split, dtype=dtype, seed=29))
    q, k, v = to_dev(qn), to_dev(kn), to_dev(vn)
    out, lse = B.dit_attn_forward(q, k, v, grid, split, flags=flags, out_dtype=torch.float32, want_lse=True)
    few = min(H, 3)
    head = lambda x: np.ascontiguousarray(x[:, :, :few])
    bf16_ops = bool(flags & (B.DIT_FLAG_QK_BF16 | B.DIT_FLAG_PV_BF16))  # (8 significant bits instead of 11)
    compare(to_f64(out[:, :, :few]), oracle.self_attn(head(qn), head(kn), head(vn), grid, split), tol=4e-2 if bf16_ops else 2e-2,
            what="small tiles")
    # the first heads alone, and eight copies of all of them: other workgroup shapes, the same bits
    fl = flags | SMALL
    ref, lref = B.dit_attn_forward(q, k, v, grid, split, flags=fl, out_dtype=torch.float32, want_lse=True)
    a, la = B.dit_attn_forward(q[:, :, :few], k[:, :, :few], v[:, :, :few], grid, split, flags=fl, out_dtype=torch.float32, want_lse=True)
    assert torch.equal(a, ref[:, :, :few]) and torch.equal(la, lref[:, :few])
    n = 1 + 520 // (H * ((L + 127) // 128))
    many = [t.repeat(1, 1, n, 1) for t in (q, k, v)]
    m, lm = B.dit_attn_forward(*many, grid, split, flags=fl, out_dtype=torch.float32, want_lse=True)
    assert torch.equal(m, ref.repeat(1, 1, n, 1)) and torch.equal(lm, lref.repeat(1, n, 1))
    # packed with another request, in a call of one round and in one of more
    other = tuple(torch.cat([t[0], t[0]]) for t in (q, k, v))
    p = B.dit_attn_varlen_forward(*other, [grid, grid], split, flags=fl, out_dtype=torch.float32)
    assert torch.equal(p, torch.cat([ref[0], ref[0]]))


@pytest.mark.parametrize("nb,Lq,H,D,keys,out,norm", [
    (1, 1, 1, 128, (1, 0), "f32", None),           # one query, one key
    (2, 63, 3, 64, (64, 65), "bf16", "head"),      # one and two key tiles
    (3, 65, 2, 128, (130, 1, 257), "bf16", None),  # 64-row tiles, the second of one row; three, one and five key tiles
    (1, 200, 64, 64, (200,), "f32", "token"),      # 256 tiles of 64 rows
    (1, 200, 65, 128, (77,), "bf16", "head"),      # 130 tiles of 128 rows by 8 wavefronts
    (1, 129, 129, 64, (300,), "bf16", None),       # 258 tiles of 128 rows: the general layout
], ids=lambda x: str(x).replace(" ", ""))
def test_small_tiles_of_cross_attention(nb, Lq, H, D, keys, out, norm):
    """The chained kernel with one query tile a workgroup: against the oracle, and bit for bit against 8 wavefronts of 32 rows."""
    import torch

    Lk = max(keys) + 3
    rng = np.random.default_rng(11)
    f = lambda n: (rng.standard_normal((nb, n, H, D)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    qn, kn, vn = f(Lq), f(Lk), f(Lk)
    q, k, v = to_dev(qn), to_dev(kn), to_dev(vn)
    n_keys = (list(keys) * nb)[:nb]
    kv_len = torch.tensor([[n, 0] for n in n_keys], dtype=torch.int32, device="cuda")
    valid = np.zeros((nb, Lk), np.uint8)
    for b, n in enumerate(n_keys):
        valid[b, :n] = 1
    nm = None if norm is None else (norm, 1e-6, None, None)
    dt = torch.float32 if out == "f32" else torch.bfloat16
    run = lambda flags: B.dit_cross_attn_forward_lengths(q, k, v, kv_len, Lk, out_dtype=dt, norm=nm, flags=flags)
    got = run(0)
    assert torch.equal(got, run(B.DIT_FLAG_BIG_WORKGROUP)) and torch.equal(got, run(SMALL))
    wide = lambda x: (x.astype(np.uint32) << 16).view(np.float32)

    def rows(x):
        x = wide(x).astype(np.float64)
        if norm is not None:
            axes = (3,) if norm == "head" else (2, 3)
            x = x / np.sqrt((x * x).mean(axis=axes, keepdims=True) + 1e-6)
        return np.ascontiguousarray(x.astype(np.float32))

    ref = oracle.cross_attn(rows(qn), rows(kn), wide(vn), valid)
    ref[np.asarray(n_keys) == 0] = 0.0
    compare(to_f64(got), ref, bf16_out=out == "bf16", what="cross, small tiles")
