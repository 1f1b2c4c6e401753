"""What happens at the edge of the fp16 range.  The default MFMA operands are fp16, whose largest finite
value is 65504, while bf16 inputs can hold far larger magnitudes.  The documented behaviour: fp16 operands
saturate at +-65504 (the result is the definition applied to the clamped operands, finite and deterministic),
and DIT_FLAG_QK_BF16 | DIT_FLAG_PV_BF16 is the opt-out that keeps the whole bf16 range.

The expected values come from the oracle alone: for the saturating case it is given the same inputs with the
out-of-range entries clamped (as float32, since 65504 has no bf16 bit pattern)."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import compare, to_dev, to_f64

pytestmark = pytest.mark.gpu

BIG = 7.0e4  # finite in bf16 (rounds to 70144), beyond fp16
F16_MAX = 65504.0
BF16_ALL = B.DIT_FLAG_QK_BF16 | B.DIT_FLAG_PV_BF16


def plant(bits, rng, n, value):
    """Overwrite n random entries of a bf16 tensor with +-value; returns the positions."""
    x = wl.bf16_bits_to_f32(bits).copy()
    flat = x.reshape(-1)
    idx = rng.choice(flat.size, size=n, replace=False)
    flat[idx] = value * rng.choice([-1.0, 1.0], size=n)
    return wl.f32_to_bf16_bits(x), idx


def test_self_attention_values_beyond_fp16():
    """|v| = 7e4 in a few hundred entries: default flags give the clamped-v result, bf16 operands the exact one."""
    import torch

    cfg = dict(B=1, grid=(2, 9, 17), H=2, D=128, split=(44, 42, 42), dtype="bf16", seed=77)
    q, k, v = wl.self_attn_inputs(cfg)
    v_big, _ = plant(v, np.random.default_rng(5), 300, BIG)
    widen = wl.bf16_bits_to_f32
    v_clamped = np.clip(widen(v_big), -F16_MAX, F16_MAX)
    assert np.abs(widen(v_big)).max() > 7e4 and np.abs(v_clamped).max() == F16_MAX
    ref_clamped = oracle.self_attn(widen(q), widen(k), v_clamped, cfg["grid"], cfg["split"])
    ref_exact = oracle.self_attn(q, k, v_big, cfg["grid"], cfg["split"])
    assert np.abs(ref_clamped - ref_exact).max() > 0.05 * np.sqrt(np.mean(ref_exact ** 2))  # the clamp is visible

    qd, kd, vd = to_dev(q), to_dev(k), to_dev(v_big)
    for name, flags in (("default", 0), ("plain schedule", B.DIT_FLAG_SIMPLE_SCHEDULE)):
        out = B.dit_attn_forward(qd, kd, vd, cfg["grid"], cfg["split"], out_dtype=torch.float32, flags=flags)
        torch.cuda.synchronize()
        compare(to_f64(out), ref_clamped, what="v beyond fp16, %s: saturated operands" % name)
    # bf16 operands: no saturation, the exact definition.  The outputs that a huge value feeds are thousands of
    # times the others, so the bar is taken per element: the documented 4e-2 x RMS of bf16 score operands on the
    # scale of the ORDINARY outputs (those of the unplanted v) plus 2 % of the element's magnitude (bf16 P: 2^-9 per
    # probability, bf16 scores: a per cent or two of a probability) -- a third of the 6.6 % by which a clamp at
    # 65504 would lower the planted contributions, so the two behaviours stay distinguishable.
    out = B.dit_attn_forward(qd, kd, vd, cfg["grid"], cfg["split"], out_dtype=torch.float32, flags=BF16_ALL)
    torch.cuda.synchronize()
    rms_plain = np.sqrt(np.mean(oracle.self_attn(q, k, v, cfg["grid"], cfg["split"]) ** 2))
    # "the element itself" without cancellation between planted values of opposite sign: sum_j p_j |v_j|
    magnitude = oracle.self_attn(q, k, v_big & np.uint16(0x7FFF), cfg["grid"], cfg["split"])
    allow = 4e-2 * rms_plain + 2e-2 * magnitude
    got = to_f64(out)
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - ref_exact) <= allow), "bf16 operands: max err/allowed %.3f" % np.max(
        np.abs(got - ref_exact) / allow)
    assert np.any(np.abs(ref_clamped - ref_exact) > 2.0 * allow)  # a saturating path would fail the line above


def test_cross_attention_keys_beyond_fp16():
    """|k| = 7e4 in one channel of four keys per (request, head); q is zero except for +-2^-10 in that channel,
    so the four keys score +-6.0 exactly (+-5.6 once clamped to 65504) against ~0 for all others: large enough
    to tell the clamped result from the exact one, small enough that operand rounding cannot flip anything.
    An unclamped fp16 conversion would make these keys infinite and the output NaN."""
    import torch

    cfg = dict(B=2, Lq=150, n_text=100, n_image=57, H=2, D=128, dtype="bf16", min_text=20, seed=78)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    rng = np.random.default_rng(6)
    c0 = 37
    widen = wl.bf16_bits_to_f32
    qf = np.zeros(q.shape, dtype=np.float32)
    qf[..., c0] = 2.0 ** -10 * rng.choice([-1.0, 1.0], size=q.shape[:-1])
    kf = widen(k).copy()
    for b in range(cfg["B"]):
        keys_ok = np.flatnonzero(valid[b])
        for h in range(cfg["H"]):
            pick = rng.choice(keys_ok, size=4, replace=False)
            kf[b, pick[:2], h, c0] = BIG
            kf[b, pick[2:], h, c0] = -BIG
    q_bits, k_bits = wl.f32_to_bf16_bits(qf), wl.f32_to_bf16_bits(kf)
    assert np.array_equal(widen(q_bits), qf)
    ref_clamped = oracle.cross_attn(qf, np.clip(widen(k_bits), -F16_MAX, F16_MAX), widen(v), valid)
    ref_exact = oracle.cross_attn(q_bits, k_bits, v, valid)
    rms = np.sqrt(np.mean(ref_exact ** 2))
    assert np.abs(ref_clamped - ref_exact).max() > 3e-2 * rms  # the two behaviours can be told apart

    qd, kd, vd, md = to_dev(q_bits), to_dev(k_bits), to_dev(v), torch.from_numpy(valid).cuda()
    for name, flags in (("default", 0), ("pipelined", B.DIT_FLAG_PIPELINED_SCHEDULE)):
        out = B.dit_cross_attn_forward(qd, kd, vd, md, out_dtype=torch.float32, flags=flags)
        torch.cuda.synchronize()
        compare(to_f64(out), ref_clamped, what="k beyond fp16, %s: saturated operands" % name)
    out = B.dit_cross_attn_forward(qd, kd, vd, md, out_dtype=torch.float32, flags=BF16_ALL)
    torch.cuda.synchronize()
    compare(to_f64(out), ref_exact, what="k beyond fp16, bf16 operands: full range")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_infinities_saturate_and_nan_stays(dtype):
    """v holds +-infinity and values past the range in either half of a pair of neighbouring channels: they count as
    +-65504, and the other channel of the pair is untouched.  A NaN in v makes its channel NaN and no other."""
    import torch

    cfg = dict(B=1, grid=(2, 5, 9), H=1, D=64, split=(22, 20, 22), dtype=dtype, seed=79)
    q, k, v = wl.self_attn_inputs(cfg)
    widen = wl.bf16_bits_to_f32 if dtype == "bf16" else np.asarray
    vf = widen(v).copy()
    vf[0, 3, 0, 6], vf[0, 11, 0, 9], vf[0, 40, 0, 20], vf[0, 41, 0, 21] = np.inf, -np.inf, BIG, -BIG
    ref = oracle.self_attn(widen(q), widen(k), np.clip(vf, -F16_MAX, F16_MAX), cfg["grid"], cfg["split"])
    vf[0, 17, 0, 33] = np.nan
    v_in = wl.f32_to_bf16_bits(vf) if dtype == "bf16" else vf
    out = B.dit_attn_forward(to_dev(q), to_dev(k), to_dev(v_in), cfg["grid"], cfg["split"], out_dtype=torch.float32)
    got = to_f64(out)
    assert np.all(np.isnan(got[..., 33]))
    keep = [c for c in range(64) if c != 33]
    compare(got[..., keep], ref[..., keep], what="infinities in v (%s)" % dtype)


@pytest.mark.parametrize("flags", [0, B.DIT_FLAG_QK_BF16, BF16_ALL, B.DIT_FLAG_BIG_WORKGROUP])
def test_scores_that_rise_by_millions_from_tile_to_tile(flags):
    """Scores far beyond fp16 itself, whose running maximum rises (for some rows falls) by up to 6e7 with every key tile:
    a row's softmax has then one key, whatever the tile or piece of the keys it is found in, and rows beside it keep theirs.
    Self-attention in pieces (the latent grid has one frame, so the first rotary section is not rotated) and chained
    cross-attention."""
    import torch

    grid, H, D, split = (1, 45, 77), 3, 128, (44, 42, 42)
    L = grid[1] * grid[2]
    cfg = dict(B=1, grid=grid, H=H, D=D, split=split, dtype="f32", seed=81)
    q, k, v = wl.self_attn_inputs(cfg)
    q[..., :2] = 0.0
    k[..., :2] = 0.0
    for t in range(L // 64):
        k[:, 64 * t + 5 + t % 7, :, 0] = 1000.0 * (t + 1)
    q[:, ::3, :, 0] = np.resize(np.float32([1.0, 30.0, -30.0, 3e4, -3e4, 5e5]), L // 3)[None, :, None]
    qn, kn, vn = (wl.f32_to_bf16_bits(a) for a in (q, k, v))
    picks = np.arange(0, 600)
    ref, ref_lse = oracle.self_attn(qn, kn, vn, grid, split, rows=picks, want_lse=True)
    qd, kd, vd = to_dev(qn), to_dev(kn), to_dev(vn)
    p = B.self_attn_params(qd, kd, vd, qd, grid, split, flags=flags)
    need = B.dit_attn_workspace_bytes(p)
    p.flags = (flags & ~B.DIT_FLAG_BIG_WORKGROUP) | B.DIT_FLAG_SMALL_WORKGROUP
    assert need > B.dit_attn_workspace_bytes(p), "this shape is meant to be computed in pieces"
    out, lse = B.dit_attn_forward(qd, kd, vd, grid, split, out_dtype=torch.float32, want_lse=True, flags=flags)
    tol = 4e-2 if flags & B.DIT_FLAG_QK_BF16 else 2e-2
    compare(to_f64(out[:, :600]), ref, tol=tol, what="rising scores, self, flags=%d" % flags)
    # (a score's operand rounding: 2^-12 of it in fp16, 2^-9 in bf16, on either side)
    rel = 2.0 ** -8 if flags & B.DIT_FLAG_QK_BF16 else 2.0 ** -11
    assert np.all(np.abs(to_f64(lse[..., :600]) - ref_lse) <= 0.1 + rel * np.abs(ref_lse))
    valid = np.ones((1, L), dtype=np.uint8)
    cref = oracle.cross_attn(qn[:, :600], kn, vn, valid)
    cout = B.dit_cross_attn_forward(qd[:, :600], kd, vd, None, out_dtype=torch.float32, flags=flags)
    compare(to_f64(cout), cref, tol=tol, what="rising scores, cross, flags=%d" % flags)
