"""Self-attention in whole tiles of few query rows: 16 rows a wavefront, in workgroups of 4 (64 rows) or 8 (128 rows), which
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
