"""GPU parity of dit_attn_forward (through the C ABI) against the CPU fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import TOL, compare, to_dev, to_f64

pytestmark = pytest.mark.gpu

VARIANTS = {
    "default_f16_f16": 0,
    "qk_f16_pv_bf16": B.DIT_FLAG_QK_F16 | B.DIT_FLAG_PV_BF16,
}


def run_self(cfg, q, k, v, flags=0, out_dtype=None, origin=(0, 0, 0), want_lse=False, scale=0.0, base=10000.0):
    import torch

    qd, kd, vd = to_dev(q), to_dev(k), to_dev(v)
    res = B.dit_attn_forward(qd, kd, vd, cfg["grid"], cfg["split"], origin=origin, flags=flags,
                             out_dtype=out_dtype, want_lse=want_lse, scale=scale, rope_base=base)
    torch.cuda.synchronize()
    return res


def test_tiny_config_fp32_inputs_all_rows():
    import torch

    cfg = wl.CONFIGS["tiny"]
    q, k, v = wl.self_attn_inputs(cfg)
    ref, ref_lse = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"], want_lse=True)
    out, lse = run_self(cfg, q, k, v, out_dtype=torch.float32, want_lse=True)
    compare(to_f64(out), ref, what="tiny f32->f32")
    assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3
    out = run_self(cfg, q, k, v, flags=B.DIT_FLAG_WIDE_QTILE, out_dtype=torch.float32)
    compare(to_f64(out), ref, what="tiny f32->f32 wide")
    # same config with inputs pre-rounded to bf16 (comparable with the bf16 configs)
    qb, kb, vb = wl.self_attn_inputs(cfg, dtype="bf16")
    refb = oracle.self_attn(qb, kb, vb, cfg["grid"], cfg["split"])
    outb = run_self(cfg, qb, kb, vb, out_dtype=torch.float32)
    compare(to_f64(outb), refb, what="tiny bf16->f32")
    outb = run_self(cfg, qb, kb, vb)
    compare(to_f64(outb), refb, bf16_out=True, what="tiny bf16->bf16")


SHAPES = {
    "auto": 0,
    "qb1_4w": B.DIT_FLAG_SMALL_WORKGROUP,
    "qb2_4w": B.DIT_FLAG_WIDE_QTILE,
    "qb1_8w": B.DIT_FLAG_BIG_WORKGROUP,
    # the same pipeline on 32x32x16 matrix instructions (the default runs on 16x16x32)
    "m32_4w": B.DIT_FLAG_MFMA_32X32 | B.DIT_FLAG_SMALL_WORKGROUP,
    "m32_8w": B.DIT_FLAG_MFMA_32X32 | B.DIT_FLAG_BIG_WORKGROUP,
    "simple_qb1": B.DIT_FLAG_SIMPLE_SCHEDULE,
    "simple_qb2": B.DIT_FLAG_SIMPLE_SCHEDULE | B.DIT_FLAG_WIDE_QTILE,
}


@pytest.mark.parametrize("name", sorted(VARIANTS))
@pytest.mark.parametrize("wide", sorted(SHAPES))
def test_mid_config_all_rows(name, wide):
    """6,240 tokens x 4 heads: 98 key tiles (ragged tail of 32), all rows compared, for every
    operand-type variant and every kernel shape (query rows per wavefront, wavefronts per
    workgroup, pipelined or plain schedule)."""
    import torch

    cfg = wl.CONFIGS["mid"]
    q, k, v = wl.self_attn_inputs(cfg)
    ref = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"])
    flags = VARIANTS[name] | SHAPES[wide]
    out = run_self(cfg, q, k, v, flags=flags, out_dtype=torch.float32)
    compare(to_f64(out), ref, what="mid %s wide=%s f32 out" % (name, wide))
    out = run_self(cfg, q, k, v, flags=flags)
    compare(to_f64(out), ref, bf16_out=True, what="mid %s wide=%s bf16 out" % (name, wide))


@pytest.mark.parametrize("pv", [B.DIT_FLAG_PV_BF16, B.DIT_FLAG_PV_F16])
def test_mid_config_bf16_score_operands_reported(pv):
    """q', k' re-rounded to bf16 (8 significant bits) after the rotation put max|err| at about
    2.5e-2 x RMS over 3.2M outputs -- past the 2e-2 bar, which is why fp16 score operands are the
    default.  The variant is selectable; its error is printed and held to a looser 4e-2."""
    import torch

    cfg = wl.CONFIGS["mid"]
    q, k, v = wl.self_attn_inputs(cfg)
    ref = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"])
    out = run_self(cfg, q, k, v, flags=B.DIT_FLAG_QK_BF16 | pv, out_dtype=torch.float32)
    compare(to_f64(out), ref, tol=4e-2, what="mid bf16 score operands, pv flag %d, f32 out" % pv)


@pytest.mark.parametrize("wide", [False, True])
def test_fused_rope_on_load(wide):
    import torch

    cfg = wl.CONFIGS["mid"]
    q, k, v = wl.self_attn_inputs(cfg)
    ref, ref_lse = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"], want_lse=True)
    flags = B.DIT_FLAG_KV_FUSED | B.DIT_FLAG_PV_BF16 | (B.DIT_FLAG_WIDE_QTILE if wide else 0)
    out, lse = run_self(cfg, q, k, v, flags=flags, out_dtype=torch.float32, want_lse=True)
    compare(to_f64(out), ref, what="mid fused wide=%s" % wide)
    assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3


@pytest.mark.parametrize("grid", [(1, 1, 1), (1, 1, 2), (1, 3, 21), (1, 1, 64), (1, 5, 13), (2, 8, 8), (1, 3, 43),
                                  (3, 7, 19)])
@pytest.mark.parametrize("D", [64, 128])
def test_ragged_sizes(grid, D):
    """Token counts 1, 2, 63, 64, 65, 128, 129, 399: below, at and just past tile boundaries."""
    import torch

    split = (22, 20, 22) if D == 64 else (44, 42, 42)
    cfg = dict(B=2, grid=grid, H=3, D=D, split=split, dtype="bf16", seed=99 + D + grid[2])
    q, k, v = wl.self_attn_inputs(cfg)
    ref, ref_lse = oracle.self_attn(q, k, v, grid, split, want_lse=True)
    for flags in tuple(SHAPES.values()) + ((B.DIT_FLAG_KV_FUSED | B.DIT_FLAG_PV_BF16,) if D == 128 else ()):
        out, lse = run_self(cfg, q, k, v, flags=flags, out_dtype=torch.float32, want_lse=True)
        compare(to_f64(out), ref, what="ragged %s D=%d flags=%d" % (grid, D, flags))
        assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3


@pytest.mark.parametrize("D,dtype,flags", [(128, "bf16", 0), (128, "bf16", B.DIT_FLAG_QK_BF16 | B.DIT_FLAG_PV_BF16), (64, "f32", 0),
                                           (64, "bf16", B.DIT_FLAG_PV_BF16)])
def test_four_wavefronts_of_32_rows_steady_state(D, dtype, flags):
    """More than 256 tiles of 128 rows, so that SMALL stays 4 x 32 rows (fewer are reshaped to 16 rows a wavefront): its key
    loop over 49 tiles, the last one of 48 keys, rows across every head's first and last query tiles against the oracle."""
    import torch

    grid, H = (4, 26, 30), 11
    L = grid[0] * grid[1] * grid[2]
    assert (L + 127) // 128 * H > 256
    cfg = dict(B=1, grid=grid, H=H, D=D, split=(44, 42, 42) if D == 128 else (22, 20, 22), dtype=dtype, seed=77 + D)
    q, k, v = wl.self_attn_inputs(cfg)
    rows = np.concatenate([np.arange(256), np.arange(1400, 1500), np.arange(L - 200, L)])
    ref, ref_lse = oracle.self_attn(q, k, v, grid, cfg["split"], rows=rows, want_lse=True)
    out, lse = run_self(cfg, q, k, v, flags=flags | B.DIT_FLAG_SMALL_WORKGROUP, out_dtype=torch.float32, want_lse=True)
    compare(to_f64(out)[:, rows], ref, tol=2 * TOL if flags & B.DIT_FLAG_QK_BF16 else TOL, what="4 x 32 rows, D=%d %s %d" % (D, dtype, flags))
    # (a score of unit size on bf16 operands is off by 2^-8 sqrt(2 / 3) = 3e-3 typically, and the sum over 3,120 keys averages)
    assert np.max(np.abs(to_f64(lse)[:, :, rows] - ref_lse)) < (1e-2 if flags & B.DIT_FLAG_QK_BF16 else 5e-3)


@pytest.mark.parametrize("name", ["qb1_8w", "qb1_4w", "m32_8w", "m32_4w", "qb2_4w", "simple_qb1"])
def test_head_dim_64_steady_state_all_rows(name):
    """head_dim 64 over 68 key tiles and 17 (8-wavefront) or 34 query tiles per head: the key loop of each form
    in steady state (the ragged cases above end after seven tiles), every row against the oracle, fp32 inputs
    as in the tiny reference shape and bf16 inputs."""
    import torch

    for dtype, seed in (("bf16", 6401), ("f32", 6402)):
        cfg = dict(B=1, grid=(4, 32, 34), H=2, D=64, split=(22, 20, 22), dtype=dtype, seed=seed)
        q, k, v = wl.self_attn_inputs(cfg)
        ref, ref_lse = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"], want_lse=True)
        out, lse = run_self(cfg, q, k, v, flags=SHAPES[name], out_dtype=torch.float32, want_lse=True)
        compare(to_f64(out), ref, what="d64, 4,352 tokens, %s, %s in" % (name, dtype))
        assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3


def test_peaky_softmax_origin_scale_base():
    """q, k scaled x2 with scale 0.11: scores ~ N(0, 5^2), the softmax concentrates on a few keys
    and the running maximum keeps moving; non-zero origin, explicit scale and base.  (Larger
    scores push the rounding of the 16-bit score operands themselves past the bar: the absolute
    score error grows with |score| while the bar is fixed.)"""
    import torch

    cfg = dict(B=1, grid=(3, 9, 17), H=2, D=128, split=(44, 42, 42), dtype="bf16", seed=4242)
    q, k, v = wl.self_attn_inputs(cfg, gain=2.0)
    ref = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"], origin=(5, -3, 11), scale=0.11, base=500.0)
    for flags in tuple(SHAPES.values()) + (B.DIT_FLAG_KV_FUSED | B.DIT_FLAG_PV_BF16,):
        out = run_self(cfg, q, k, v, flags=flags, out_dtype=torch.float32, origin=(5, -3, 11), scale=0.11, base=500.0)
        compare(to_f64(out), ref, what="peaky flags=%d" % flags)


def test_head_major_layout_and_determinism():
    """[B, H, L, D] storage through strides; two runs are bitwise identical."""
    import torch

    cfg = dict(B=2, grid=(2, 6, 11), H=3, D=128, split=(44, 42, 42), dtype="bf16", seed=777)
    q, k, v = wl.self_attn_inputs(cfg)
    ref = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"])
    qd, kd, vd = (to_dev(a).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for a in (q, k, v))
    assert qd.stride(2) > qd.stride(1)
    out = torch.empty((2, 3, 132, 128), dtype=torch.float32, device="cuda").permute(0, 2, 1, 3)
    B.dit_attn_forward(qd, kd, vd, cfg["grid"], cfg["split"], out=out)
    torch.cuda.synchronize()
    compare(to_f64(out), ref, what="head-major layout")
    out2 = torch.empty_like(out)
    B.dit_attn_forward(qd, kd, vd, cfg["grid"], cfg["split"], out=out2)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)


FULL = {
    "dit_1p3b": dict(edge=64, n_random=128),
    "dit_14b": dict(edge=64, n_random=128),
    "dit_14b_hires": dict(edge=64, n_random=32),
}


@pytest.mark.parametrize("name", sorted(FULL))
def test_full_size_sampled_rows(name):
    """The reference shapes at full size, default flags (the configuration the benchmark times);
    rows {0..63}, {L-64..L-1} and seeded random rows of every head are checked."""
    import torch

    cfg = wl.CONFIGS[name]
    q, k, v = wl.self_attn_inputs(cfg)
    L = q.shape[1]
    rows = wl.sample_rows(L, cfg["seed"], **FULL[name])
    ref = oracle.self_attn(q, k, v, cfg["grid"], cfg["split"], rows=rows)
    out = run_self(cfg, q, k, v, out_dtype=torch.float32)
    compare(to_f64(out[:, torch.from_numpy(rows).cuda()]), ref, what="%s f32 out" % name)
    del out
    out = run_self(cfg, q, k, v)
    compare(to_f64(out[:, torch.from_numpy(rows).cuda()]), ref, bf16_out=True, what="%s bf16 out" % name)


@pytest.mark.parametrize("base,origin", [(10000.0, 0), (10000.0, 1 << 20), (1e-10, 3), (3e38, 1 << 20)])
def test_rotation_table_against_extended_precision(base, origin):
    """The table sits at the start of the workspace: fp32 (cos, sin) of fp64 angles.  An entry may be off by its own
    rounding (2^-25 at most) and by the fp64 error of the angle: the power and the product with the position, an ulp
    each and a half for good measure.  (The exponent -2i/d is taken as the double that it rounds to.)"""
    import torch

    grid, split = (5, 3, 4), (44, 42, 42)
    q = torch.zeros((1, 60, 1, 128), dtype=torch.bfloat16, device="cuda")
    p = B.self_attn_params(q, q, q, q, grid, split)
    ws = torch.empty(B.dit_attn_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    B.dit_attn_forward(q, q, q, grid, split, origin=(origin,) * 3, rope_base=base, workspace=ws)
    n = sum(g * d // 2 for g, d in zip(grid, split))
    tab = ws[:8 * n].view(torch.float32).cpu().numpy().reshape(n, 2)
    ext = np.longdouble
    base = ext(np.float32(base))
    phi = np.concatenate([(np.arange(g) + origin).astype(ext)[:, None] * np.power(base, (-(np.arange(d // 2) / np.float64(d // 2))).astype(ext))
                          for g, d in zip(grid, split)], axis=None)
    allow = 2.0 ** -25 + np.abs(phi) * ext(2.5 * 2.0 ** -53)
    for got, want in ((tab[:, 0], np.cos(phi)), (tab[:, 1], np.sin(phi))):
        err = np.abs(got.astype(ext) - want)
        assert np.all(err <= allow), "entry %d: off by %g, allowed %g" % (int(np.argmax(err / allow)), err.max(), allow[np.argmax(err / allow)])


@pytest.mark.parametrize("split", [(44, 42, 42), (2, 2, 124), (126, 2, 0), (2, 0, 126), (62, 0, 66), (0, 30, 98), (64, 32, 32)])
def test_axes_that_end_behind_odd_numbers_of_pairs(split):
    """The prologue fetches rotation entries two pairs at a time; the second is of the next axis where one ends behind an
    odd number of pairs (first, second, both, neighbouring ends, empty axes).  Last positions of every axis included."""
    import torch

    cfg = dict(B=1, grid=(3, 5, 19), H=2, D=128, split=split, dtype="bf16", seed=sum(split[:2]))
    q, k, v = wl.self_attn_inputs(cfg)
    ref = oracle.self_attn(q, k, v, cfg["grid"], split)
    for flags in (0, B.DIT_FLAG_SMALL_WORKGROUP):
        out = B.dit_attn_forward(to_dev(q), to_dev(k), to_dev(v), cfg["grid"], split, flags=flags,
                                 out_dtype=torch.float32)
        torch.cuda.synchronize()
        compare(to_f64(out), ref, what="split %s flags %d" % (split, flags))


@pytest.mark.parametrize("out_f32", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L", [1, 31, 33, 255, 257, 304])
def test_staged_output_rows_at_tile_edges(L, D, out_f32):
    """8 wavefronts stage their output rows: sequences that end one row either side of a wavefront's 32 rows and of a
    query tile, in rows that stand apart (nothing between them may change), with the log-sum-exp."""
    import torch

    split = (22, 20, 22) if D == 64 else (44, 42, 42)
    cfg = dict(B=2, grid=(1, 1, L), H=3, D=D, split=split, dtype="bf16", seed=L + D)
    q, k, v = wl.self_attn_inputs(cfg)
    ref, ref_lse = oracle.self_attn(q, k, v, cfg["grid"], split, want_lse=True)
    rows = torch.full((2, L, 3, D + 8), 7.0, dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
    lse = torch.full((2, 3, L), 7.0, dtype=torch.float32, device="cuda")
    B.dit_attn_forward(to_dev(q), to_dev(k), to_dev(v), cfg["grid"], split, flags=B.DIT_FLAG_BIG_WORKGROUP,
                       out=rows[..., :D], lse=lse)
    torch.cuda.synchronize()
    assert bool((rows[..., D:] == 7.0).all())
    compare(to_f64(rows[..., :D]), ref, bf16_out=not out_f32, what="L=%d D=%d" % (L, D))
    assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3


@pytest.mark.parametrize("flags", [B.DIT_FLAG_BIG_WORKGROUP, B.DIT_FLAG_SMALL_WORKGROUP, 0])  # (0: the kernel for short sequences)
@pytest.mark.parametrize("side", ["q", "k"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
def test_rotated_pairs_are_rounded_as_stated(D, dtype, side, flags):
    """A rotated pair is (fma(x0, cos, -(x1 sin)), fma(x1, cos, x0 sin)) in fp32, in q as in k: pairs are drawn until
    there are some at every place in the row whose fp16 operand is another one if the other product is rounded by itself.
    Sequences of one token whose rows hold such a pair and zeros: the log-sum-exp is the score itself.  Its error beside
    the operands': a sum of two exact products and a product with ln 2, rounded or truncated to fp32, and ln 2 in
    fp32, 2^-23 of the terms' magnitudes each."""
    import torch

    ext = np.longdouble
    split, origin = ((22, 20, 22) if D == 64 else (44, 42, 42)), (3, 17, 29)
    z = torch.zeros((1, 1, 1, D), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.dit_attn_workspace_bytes(B.self_attn_params(z, z, z, z, (1, 1, 1), split, origin=origin)),
                     dtype=torch.uint8, device="cuda")
    B.dit_attn_forward(z, z, z, (1, 1, 1), split, origin=origin, workspace=ws)  # the table stands at the start of it
    tab = ws[:4 * D].view(torch.float32).cpu().numpy().reshape(D // 2, 2).astype(ext)
    qscale = ext(np.float32(np.float32(1.0) / np.sqrt(np.float32(D))) * np.float32(1.4426950408889634))

    def f32(x):
        return x.astype(np.float32).astype(ext)

    def operands(x0, x1, i, scale, other):
        """fp16 operands of the pairs (x0, x1) at place i; other: the other products rounded by themselves."""
        c, s = tab[i, 0], tab[i, 1]
        y0 = f32(f32(x0 * c) - x1 * s) if other else f32(x0 * c - f32(x1 * s))
        y1 = f32(f32(x1 * c) + x0 * s) if other else f32(x1 * c + f32(x0 * s))
        return np.stack([f32(y * scale).astype(np.float16).astype(np.float64) for y in (y0, y1)], axis=-1)

    rng = np.random.default_rng(D)
    bits = 16 if dtype == "bf16" else 0  # low bits of an fp32 number that are zero
    rows, want, allow = [], [], []
    for i in range(D // 2):
        x = rng.uniform(0.5, 2.0, (2, 1 << 16)).astype(np.float32) * np.float32(1 - 2 * (i & 1))
        x = (x.view(np.uint32) >> bits << bits).view(np.float32).astype(ext)
        scale = qscale if side == "q" else ext(1)
        a, b = (operands(x[0], x[1], i, scale, other) for other in (False, True))
        y = rng.uniform(0.5, 2.0, 2).astype(np.float32)
        y = (y.view(np.uint32) >> bits << bits).view(np.float32).astype(ext)
        o = operands(y[0], y[1], i, qscale if side == "k" else ext(1), False)
        terms = a * o * np.log(2.0)
        room = 3 * 2.0 ** -23 * np.abs(terms).sum(-1)
        for n in np.nonzero(np.abs(((a - b) * o).sum(-1)) * np.log(2.0) > 4 * room)[0][:4]:
            pair = np.zeros((2, D), dtype=np.float32)
            pair[0, 2 * i:2 * i + 2], pair[1, 2 * i:2 * i + 2] = x[:, n], y
            rows.append(pair if side == "q" else pair[::-1])
            want.append(terms[n].sum())
            allow.append(room[n])
    assert D // 2 <= len(rows) <= 256  # (one round of workgroups)
    rows = torch.from_numpy(np.stack(rows, axis=1)).to("cuda", torch.float32 if dtype == "f32" else torch.bfloat16)
    q, k = (r[:, None, None, :].contiguous() for r in rows)
    _, lse = B.dit_attn_forward(q, k, k, (1, 1, 1), split, origin=origin, flags=flags, want_lse=True)
    torch.cuda.synchronize()
    off = np.abs(to_f64(lse)[:, 0, 0] - np.array(want)) > np.array(allow)
    assert not off.any(), "%d of %d scores are not of the operands stated" % (off.sum(), off.size)
