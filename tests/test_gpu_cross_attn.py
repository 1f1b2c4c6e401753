"""GPU parity of dit_cross_attn_forward (through the C ABI) against the CPU fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import compare, to_dev, to_f64

pytestmark = pytest.mark.gpu


def run_cross(q, k, v, valid, **kw):
    import torch

    vd = torch.from_numpy(valid).cuda() if valid is not None else None
    res = B.dit_cross_attn_forward(to_dev(q), to_dev(k), to_dev(v), vd, **kw)
    torch.cuda.synchronize()
    return res


SHAPES = {
    "auto": 0,
    "pipe_qb1_4w": B.DIT_FLAG_PIPELINED_SCHEDULE | B.DIT_FLAG_SMALL_WORKGROUP,
    "pipe_qb1_8w": B.DIT_FLAG_PIPELINED_SCHEDULE | B.DIT_FLAG_BIG_WORKGROUP,
    "pipe_qb2_4w": B.DIT_FLAG_PIPELINED_SCHEDULE | B.DIT_FLAG_WIDE_QTILE,
    "chain_4w": B.DIT_FLAG_SMALL_WORKGROUP,
    "chain_8w": B.DIT_FLAG_BIG_WORKGROUP,
    "simple_qb1": B.DIT_FLAG_SIMPLE_SCHEDULE,
    "simple_qb2": B.DIT_FLAG_SIMPLE_SCHEDULE | B.DIT_FLAG_WIDE_QTILE,
}


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("wide", sorted(SHAPES))
def test_small_cross_with_masks(D, wide):
    import torch

    cfg = dict(B=3, Lq=333, n_text=512, n_image=257, H=2, D=D, dtype="bf16", min_text=16, seed=31 + D)
    q, k, v, valid, text_len = wl.cross_attn_inputs(cfg)
    valid[2, :] = 0
    valid[2, 700] = 1  # a request with a single valid key: output = that value row
    ref, ref_lse = oracle.cross_attn(q, k, v, valid, want_lse=True)
    flags = SHAPES[wide]
    out, lse = run_cross(q, k, v, valid, flags=flags, out_dtype=torch.float32, want_lse=True)
    compare(to_f64(out), ref, what="cross D=%d wide=%s" % (D, wide))
    assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3
    out = run_cross(q, k, v, valid, flags=flags)
    compare(to_f64(out), ref, bf16_out=True, what="cross D=%d wide=%s bf16 out" % (D, wide))
    # no mask at all
    ref2 = oracle.cross_attn(q, k, v, None)
    out2 = run_cross(q, k, v, None, flags=flags, out_dtype=torch.float32)
    compare(to_f64(out2), ref2, what="cross no mask")


def test_fully_masked_request_and_garbage_under_mask():
    import torch

    cfg = dict(B=2, Lq=70, n_text=100, n_image=29, H=2, D=128, dtype="bf16", min_text=5, seed=5)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    valid[1, :] = 0
    # huge finite garbage under the mask must not leak into request 0
    kb = wl.bf16_bits_to_f32(k).copy(); vb = wl.bf16_bits_to_f32(v).copy()
    kb[0, valid[0] == 0] = 3.0e4; vb[0, valid[0] == 0] = -3.0e4
    k2, v2 = wl.f32_to_bf16_bits(kb), wl.f32_to_bf16_bits(vb)
    ref, ref_lse = oracle.cross_attn(q, k2, v2, valid, want_lse=True)
    assert np.all(np.isneginf(ref_lse[1]))
    for name, flags in sorted(SHAPES.items()):
        out, lse = run_cross(q, k2, v2, valid, out_dtype=torch.float32, want_lse=True, flags=flags)
        o = to_f64(out)
        compare(o[0], ref[0], what="garbage under mask, %s" % name)
        assert np.all(o[1] == 0.0)
        assert np.all(np.isneginf(to_f64(lse)[1]))


def test_full_size_cross_sampled_rows():
    """4 requests x 32,760 queries x 769 keys x 40 heads, default flags; sampled rows of every head."""
    import torch

    cfg = wl.CONFIGS["cross_14b"]
    q, k, v, valid, text_len = wl.cross_attn_inputs(cfg)
    rows = wl.sample_rows(cfg["Lq"], cfg["seed"], edge=64, n_random=128)
    ref = oracle.cross_attn(q, k, v, valid, rows=rows)
    out = run_cross(q, k, v, valid)
    compare(to_f64(out[:, torch.from_numpy(rows).cuda()]), ref, bf16_out=True, what="cross_14b bf16 out")
    del out
    out = run_cross(q, k, v, valid, out_dtype=torch.float32)
    compare(to_f64(out[:, torch.from_numpy(rows).cuda()]), ref, what="cross_14b f32 out")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_text,n_image", [(200, 57), (128, 64), (7, 300), (512, 257)])
def test_decoupled_cross_attention(D, n_text, n_image):
    """Two softmaxes (text keys, image keys) added: splits on and off tile boundaries, padded text,
    one request whose text is fully masked, one whose image part is fully masked."""
    import torch

    cfg = dict(B=4, Lq=300, n_text=n_text, n_image=n_image, H=2, D=D, dtype="bf16", min_text=1, seed=900 + D + n_text)
    q, k, v, valid, text_len = wl.cross_attn_inputs(cfg)
    valid[2, :n_text] = 0          # request 2: only the image sequence attends
    valid[3, n_text:] = 0          # request 3: only the text sequence attends
    ref = oracle.cross_attn_decoupled(q, k, v, n_text, valid)
    for flags in (0, B.DIT_FLAG_QK_F16 | B.DIT_FLAG_PV_BF16):
        out = run_cross(q, k, v, valid, out_dtype=torch.float32, split=n_text, flags=flags)
        compare(to_f64(out), ref, what="decoupled D=%d split=%d flags=%d" % (D, n_text, flags))
    out = run_cross(q, k, v, valid, split=n_text)
    compare(to_f64(out), ref, bf16_out=True, what="decoupled D=%d split=%d bf16 out" % (D, n_text))
    # no mask at all, and a split at the end (= joint softmax)
    ref2 = oracle.cross_attn_decoupled(q, k, v, n_text, None)
    compare(to_f64(run_cross(q, k, v, None, out_dtype=torch.float32, split=n_text)), ref2, what="decoupled no mask")
    ref3 = oracle.cross_attn(q, k, v, valid)
    compare(to_f64(run_cross(q, k, v, valid, out_dtype=torch.float32, split=n_text + n_image)), ref3,
            what="split at Lk is the joint softmax")


def test_decoupled_rejects_lse():
    import torch

    cfg = dict(B=1, Lq=64, n_text=64, n_image=64, H=1, D=128, dtype="bf16", min_text=1, seed=5)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    with pytest.raises(B.DitError) as e:
        run_cross(q, k, v, valid, split=64, want_lse=True)
    assert e.value.status == B.DIT_ERR_UNSUPPORTED


def test_full_size_decoupled_cross_sampled_rows():
    """cross_14b shape with the text / image keys as two softmaxes (split at 512)."""
    import torch

    cfg = wl.CONFIGS["cross_14b"]
    q, k, v, valid, text_len = wl.cross_attn_inputs(cfg)
    rows = wl.sample_rows(cfg["Lq"], cfg["seed"], edge=64, n_random=128)
    ref = oracle.cross_attn_decoupled(q, k, v, cfg["n_text"], valid, rows=rows)
    out = run_cross(q, k, v, valid, out_dtype=torch.float32, split=cfg["n_text"])
    compare(to_f64(out[:, torch.from_numpy(rows).cuda()]), ref, what="cross_14b decoupled f32 out")
    del out
    out = run_cross(q, k, v, valid, split=cfg["n_text"])
    compare(to_f64(out[:, torch.from_numpy(rows).cuda()]), ref, bf16_out=True, what="cross_14b decoupled bf16 out")


@pytest.mark.parametrize("split", [0, 300])
@pytest.mark.parametrize("shape", [0, B.DIT_FLAG_PIPELINED_SCHEDULE])
def test_scattered_key_masks_are_compacted(split, shape):
    """Validity scattered over the keys instead of a padded tail: every third key, a request with
    two isolated keys in different tiles, a request with one whole tile valid in the middle, and a
    request with every key valid.  The library packs the valid keys densely into tiles (the order of
    keys does not matter to attention); output and log-sum-exp against the oracle on all rows, and a
    second call on the resident tiles with the mask pointer gone."""
    import torch

    if split and shape:
        pytest.skip("the decoupled form has no pipelined kernel")
    cfg = dict(B=4, Lq=150, n_text=300, n_image=215, H=2, D=128, dtype="bf16", min_text=16, seed=401)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    Lk = k.shape[1]
    valid[:] = 0
    valid[0, ::3] = 1
    valid[1, 70] = valid[1, 400] = 1
    valid[2, 320:384] = 1
    valid[3, :] = 1
    if split:  # every key group of every request keeps at least one key
        valid[1, 10] = 1
        valid[2, 5] = 1
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    want_lse = split == 0
    res = run_cross(q, k, v, valid, flags=shape, split=split, workspace=ws, out_dtype=torch.float32, want_lse=want_lse)
    if split:
        ref = oracle.cross_attn_decoupled(q, k, v, split, valid)
        compare(to_f64(res), ref, what="scattered masks, decoupled")
    else:
        ref, ref_lse = oracle.cross_attn(q, k, v, valid, want_lse=True)
        out, lse = res
        compare(to_f64(out), ref, what="scattered masks, joint, flags %d" % shape)
        assert np.max(np.abs(to_f64(lse) - ref_lse)) < 5e-3
    q2 = wl.cross_attn_inputs(cfg, seed=402)[0]
    nan = torch.full((cfg["B"], Lk, cfg["H"], cfg["D"]), float("nan"), dtype=torch.bfloat16, device="cuda")
    out2 = B.dit_cross_attn_forward(to_dev(q2), nan, nan, None, flags=shape | B.DIT_FLAG_KV_RESIDENT, split=split,
                                    workspace=ws, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref2 = oracle.cross_attn_decoupled(q2, k, v, split, valid) if split else oracle.cross_attn(q2, k, v, valid)
    compare(to_f64(out2), ref2, what="scattered masks, resident call")


@pytest.mark.parametrize("D,shape", [(64, "chain_4w"), (128, "chain_4w"), (128, "chain_8w")])
def test_chained_query_tiles_all_rows(D, shape):
    """Enough query tiles that the default kernel's workgroups take two or three in a row (about five
    workgroups per compute unit), with requests of 0, 1, 2 and 3 key tiles -- odd and even numbers of steps,
    so that the wrap-around of the key-tile stream starts the next query tile in either K' buffer -- and a
    ragged last query tile.  Every row of every request against the oracle, output and log-sum-exp."""
    import torch

    # 202 query tiles x 4 requests x 6 heads over 256 compute units: chains of three (the last one shorter);
    # 151 x 4 x 6: chains of two
    Lq = 128 * 201 + 37 if shape == "chain_4w" else 256 * 150 + 37
    H = 6
    cfg = dict(B=4, Lq=Lq, n_text=150, n_image=42, H=H, D=D, dtype="bf16", min_text=5, seed=77 + D)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    valid[:] = 0
    valid[1, 3:43] = 1                   # 40 keys: one tile
    valid[2, 0:150:2] = 1                # 75 scattered keys + 25 below: two tiles
    valid[2, 150:175] = 1
    valid[3, :] = 1                      # 192 keys: three full tiles
    ref, ref_lse = oracle.cross_attn(q, k, v, valid, want_lse=True)
    out, lse = run_cross(q, k, v, valid, out_dtype=torch.float32, want_lse=True, flags=SHAPES[shape])
    o, l = to_f64(out), to_f64(lse)
    assert np.all(o[0] == 0.0) and np.all(np.isneginf(l[0]))
    for b in (1, 2, 3):
        compare(o[b], ref[b], what="chained, request %d, %s" % (b, shape))
        assert np.allclose(l[b], ref_lse[b], rtol=0, atol=2e-3)


def _mask_from_lengths(kv_len, second_start, Lk):
    valid = np.zeros((kv_len.shape[0], Lk), dtype=np.uint8)
    for b, (l0, l1) in enumerate(kv_len):
        valid[b, :l0] = 1
        valid[b, second_start:second_start + l1] = 1
    return valid


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", ["auto", "chain_8w", "pipe_qb1_4w", "simple_qb1"])
def test_key_counts_instead_of_mask(D, shape):
    """dit_cross_attn_forward_lengths: two counts per request instead of a byte mask.  Against the oracle on the
    mask the counts stand for, and bit for bit against the mask form of the library (same keys, same order)."""
    import torch

    n_text, n_image = 200, 77
    cfg = dict(B=5, Lq=300, n_text=n_text, n_image=n_image, H=3, D=D, dtype="bf16", min_text=5, seed=31 + D)
    q, k, v, _, _ = wl.cross_attn_inputs(cfg)
    kv_len = np.array([[200, 77], [1, 0], [0, 0], [64, 64], [130, 5]], dtype=np.int32)
    valid = _mask_from_lengths(kv_len, n_text, n_text + n_image)
    ref, ref_lse = oracle.cross_attn(q, k, v, valid, want_lse=True)
    flags = SHAPES[shape]
    dq, dk, dv = to_dev(q), to_dev(k), to_dev(v)
    out, lse = B.dit_cross_attn_forward_lengths(dq, dk, dv, torch.from_numpy(kv_len).cuda(), n_text, flags=flags,
                                                out_dtype=torch.float32, want_lse=True)
    torch.cuda.synchronize()
    o, l = to_f64(out), to_f64(lse)
    for b in range(5):
        if kv_len[b].sum() == 0:
            assert np.all(o[b] == 0.0) and np.all(np.isneginf(l[b]))
        else:
            compare(o[b], ref[b], what="key counts, request %d, %s" % (b, shape))
            assert np.allclose(l[b], ref_lse[b], rtol=0, atol=2e-3)
    out_m = run_cross(q, k, v, valid, flags=flags, out_dtype=torch.float32)
    assert torch.equal(out, out_m)
    # counts outside their range are clamped, never read out of bounds
    wild = torch.tensor([[10 ** 6, 10 ** 6], [-5, 3], [0, 0], [64, 64], [130, 5]], dtype=torch.int32).cuda()
    out_w = B.dit_cross_attn_forward_lengths(dq, dk, dv, wild, n_text, flags=flags, out_dtype=torch.float32)
    torch.cuda.synchronize()
    clamped = _mask_from_lengths(np.array([[200, 77], [0, 3], [0, 0], [64, 64], [130, 5]]), n_text, n_text + n_image)
    compare(to_f64(out_w)[1], oracle.cross_attn(q, k, v, clamped)[1], what="clamped counts")
    assert torch.equal(out_w[0], out[0])


@pytest.mark.parametrize("D", [64, 128])
def test_key_counts_decoupled_and_resident(D):
    """The decoupled form (a softmax per sequence) from counts, then new queries against the tiles that call left."""
    import torch

    n_text, n_image = 150, 70
    cfg = dict(B=3, Lq=200, n_text=n_text, n_image=n_image, H=2, D=D, dtype="bf16", min_text=5, seed=5 + D)
    q, k, v, _, _ = wl.cross_attn_inputs(cfg)
    kv_len = np.array([[150, 70], [33, 0], [0, 65]], dtype=np.int32)
    valid = _mask_from_lengths(kv_len, n_text, n_text + n_image)
    ref = oracle.cross_attn_decoupled(q, k, v, n_text, valid)
    dlen = torch.from_numpy(kv_len).cuda()
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    out = B.dit_cross_attn_forward_lengths(to_dev(q), to_dev(k), to_dev(v), dlen, n_text, split=n_text,
                                           out_dtype=torch.float32, workspace=ws)
    torch.cuda.synchronize()
    compare(to_f64(out), ref, what="decoupled from key counts")
    with pytest.raises(B.DitError):  # the second range of the decoupled form starts at the split
        B.dit_cross_attn_forward_lengths(to_dev(q), to_dev(k), to_dev(v), dlen, n_text - 1, split=n_text, workspace=ws)
    q2 = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(q)[:, ::-1].copy())
    nan = torch.full_like(to_dev(k), float("nan"))
    out2 = B.dit_cross_attn_forward_lengths(to_dev(q2), nan, nan, None, n_text, split=n_text, workspace=ws,
                                            flags=B.DIT_FLAG_KV_RESIDENT, out_dtype=torch.float32)
    torch.cuda.synchronize()
    compare(to_f64(out2), oracle.cross_attn_decoupled(q2, k, v, n_text, valid), what="resident tiles from key counts")


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("Lk", [63, 65, 1000, 4096, 4097, 4500])
def test_scattered_masks_short_and_long(Lk, split):
    """Valid keys anywhere: masks that the pre-pack sorts out by itself (up to 4,096 keys) and longer ones that are listed
    beforehand; all, none, one and about half of the keys valid; huge values under the mask."""
    import torch

    cut = (Lk // 3) if split else 0
    cfg = dict(B=4, Lq=65, n_text=Lk - 1, n_image=1, H=2, D=64, dtype="bf16", min_text=1, seed=500 + Lk)
    q, k, v, _, _ = wl.cross_attn_inputs(cfg)
    valid = (np.random.default_rng(Lk).random((4, Lk)) < 0.5).astype(np.uint8)
    valid[1], valid[2] = 1, 0
    valid[3] = 0
    valid[3, Lk - 1] = 1
    v = v.copy()
    v[valid == 0] = wl.f32_to_bf16_bits(np.float32(3.0e38))
    ref = oracle.cross_attn_decoupled(q, k, v, cut, valid) if split else oracle.cross_attn(q, k, v, valid)
    out = B.dit_cross_attn_forward(to_dev(q), to_dev(k), to_dev(v), torch.from_numpy(valid).cuda(),
                                   out_dtype=torch.float32, split=cut)
    got = to_f64(out)
    assert np.all(got[2] == 0.0)
    compare(got, ref, what="scattered mask Lk=%d split=%d" % (Lk, cut))


@pytest.mark.parametrize("split", [0, 700])
def test_many_heads_with_listed_masks_of_moderate_length(split):
    """Masks of fewer than 4,096 keys that are listed ahead of the pre-pack because many heads would read them: the same
    bits as the first heads alone, whose tiles find their keys by themselves, and the oracle's numbers."""
    import torch

    Lk, H, few = 3300, 200, 2
    cfg = dict(B=1, Lq=33, n_text=Lk - 1, n_image=1, H=few, D=64, dtype="bf16", min_text=1, seed=611)
    q, k, v, _, _ = wl.cross_attn_inputs(cfg)
    valid = (np.random.default_rng(611).random((1, Lk)) < 0.4).astype(np.uint8)
    ref = oracle.cross_attn_decoupled(q, k, v, split, valid) if split else oracle.cross_attn(q, k, v, valid)
    qd, kd, vd, vald = to_dev(q), to_dev(k), to_dev(v), torch.from_numpy(valid).cuda()
    alone = B.dit_cross_attn_forward(qd, kd, vd, vald, out_dtype=torch.float32, split=split)
    compare(to_f64(alone), ref, what="two heads, split=%d" % split)
    many = [t.repeat(1, 1, H // few, 1) for t in (qd, kd, vd)]
    out = B.dit_cross_attn_forward(*many, vald, out_dtype=torch.float32, split=split)
    assert torch.equal(out, alone.repeat(1, 1, H // few, 1))


# requests, heads, query tiles a head (the last one of 11 rows), keys of either range: of the next two tests, whose chains are
# to cross from head to head in the middle of a chain (a host test holds them to that)
CHAINS_ONE, CHAINS_TWO = (4, 24, 7, (320,)), (7, 20, 4, (270, 320))


@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_chains_run_on_into_the_next_heads(D, big):
    """More query tiles than compute units and few of them a head, so that a workgroup's chain goes from one head to the
    next, with requests of 1, 2, 4 and 5 key tiles (every way through the step loop) whose last tiles hold one key, some
    and all; normalised rows (their weights differ from head to head).  Every row against the oracle."""
    import torch

    nw = 8 if big else 4
    nb, H, tiles, (Lk,) = CHAINS_ONE
    Lq = 32 * nw * (tiles - 1) + 11
    cfg = dict(B=nb, Lq=Lq, n_text=Lk, n_image=0, H=H, D=D, dtype="bf16", min_text=5, seed=91 + D)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    keys = (1, 128, 255, 257)
    valid[:] = 0
    for b, n in enumerate(keys):
        valid[b, :n] = 1
    rng = np.random.default_rng(5)
    gq, gk = (1.0 + 0.25 * rng.standard_normal(H * D).astype(np.float32) for _ in range(2))
    qn, kn = (oracle.qk_rmsnorm(x, g.reshape(H, D), 1e-6, "head") for x, g in ((q, gq), (k, gk)))
    ref, ref_lse = oracle.cross_attn(qn, kn, oracle.as_f64(v), valid, want_lse=True)
    flags = B.DIT_FLAG_BIG_WORKGROUP if big else B.DIT_FLAG_SMALL_WORKGROUP
    norm = ("head", 1e-6, torch.from_numpy(gq).cuda(), torch.from_numpy(gk).cuda())
    out, lse = run_cross(q, k, v, valid, flags=flags, norm=norm, out_dtype=torch.float32, want_lse=True)
    o = to_f64(out)
    for b in range(4):
        compare(o[b], ref[b], what="%d keys, %d wavefronts" % (keys[b], nw))
    assert np.allclose(to_f64(lse), ref_lse, rtol=0, atol=2e-3)


@pytest.mark.parametrize("out_f32", [False, True])
@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_chains_with_two_softmaxes(D, big, out_f32):
    """Two passes per query tile in chains over several heads (bf16 rows of head_dim 128; the others run on the plain
    kernel): requests with nothing in one range or in both, with one tile in either, and with 1 to 5 tiles whose last ones
    hold one key, some and all; a ragged last query tile, output rows that stand apart (the first pass's result
    waits in them: nothing between them may change).  Every row against the oracle; per-token normalised rows."""
    import torch

    nw = 8 if big else 4
    nb, H, tiles, (n_text, n_image) = CHAINS_TWO
    Lq = 32 * nw * (tiles - 1) + 11
    counts = [(0, 65), (128, 0), (1, 1), (65, 130), (0, 0), (192, 64), (257, 320)]
    cfg = dict(B=nb, Lq=Lq, n_text=n_text, n_image=n_image, H=H, D=D, dtype="bf16", min_text=5, seed=17 + D)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    valid[:] = 0
    for b, (n, m) in enumerate(counts):
        valid[b, :n] = 1
        valid[b, n_text:n_text + m] = 1
    rng = np.random.default_rng(6)
    gq, gk = (1.0 + 0.25 * rng.standard_normal(H * D).astype(np.float32) for _ in range(2))
    qn, kn = (oracle.qk_rmsnorm(x, g.reshape(H, D), 1e-6, "token") for x, g in ((q, gq), (k, gk)))
    ref = oracle.cross_attn_decoupled(qn, kn, oracle.as_f64(v), n_text, valid)
    flags = B.DIT_FLAG_BIG_WORKGROUP if big else B.DIT_FLAG_SMALL_WORKGROUP
    norm = ("token", 1e-6, torch.from_numpy(gq).cuda(), torch.from_numpy(gk).cuda())
    rows = torch.full((len(counts), Lq, H, D + 8), 7.0, dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
    B.dit_cross_attn_forward(to_dev(q), to_dev(k), to_dev(v), torch.from_numpy(valid).cuda(), flags=flags, norm=norm,
                             split=n_text, out=rows[..., :D])
    torch.cuda.synchronize()
    assert bool((rows[..., D:] == 7.0).all())
    o = to_f64(rows[..., :D])
    for b, c in enumerate(counts):
        compare(o[b], ref[b], bf16_out=not out_f32, what="%d + %d keys, %d wavefronts" % (c + (nw,)))


@pytest.mark.parametrize("out_f32", [False, True])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_rows_do_not_depend_on_the_rest_of_the_call(D, two, out_f32):
    """A request has the same bits alone as with more query rows behind its own, in a batch, with more heads, and with keys
    padded to a larger capacity: calls of 16 to 2,000 query tiles of 256 rows, either side of every line by which
    calls are laid over the chip."""
    import torch

    H, Lq, n_text, n_image = 8, 300, 100, 65
    cfg = dict(B=1, Lq=Lq, n_text=n_text, n_image=n_image, H=H, D=D, dtype="bf16", min_text=16, seed=3 * D)
    q, k, v, valid, _ = wl.cross_attn_inputs(cfg)
    valid[:] = 1
    valid[:, 83:n_text] = 0
    qd, kd, vd = (to_dev(x) for x in (q, k, v))
    md = torch.from_numpy(valid).cuda()
    dt = torch.float32 if out_f32 else torch.bfloat16

    def run(q, k, v, m, n=n_text):
        return B.dit_cross_attn_forward(q, k, v, m, split=n if two else 0, out_dtype=dt)[:1, :Lq, :H]

    alone = run(qd, kd, vd, md)
    others = [x.flip(1).expand(5, -1, -1, -1) for x in (qd, kd, vd)]  # five requests with rows of their own
    for n_q in (Lq, 2000, 17000):
        many = torch.cat([qd] + [qd.flip(1)] * (n_q // Lq), dim=1)[:, :n_q].contiguous()
        assert torch.equal(run(many, kd, vd, md), alone), "%d query rows" % n_q
        batch = torch.cat([many, many.flip(1).expand(5, -1, -1, -1)])
        assert torch.equal(run(batch, *(torch.cat([x, o]) for x, o in zip((kd, vd), others[1:])), md.expand(6, -1).contiguous()),
                           alone), "%d query rows in a batch of 6" % n_q
        heads = [torch.cat([x] + [x.flip(2)] * 4, dim=2) for x in (many, kd, vd)]
        assert torch.equal(run(*heads, md), alone), "%d query rows, %d heads" % (n_q, 5 * H)
        pad = lambda x: torch.cat([x[:, :n_text], x[:, :1].expand(-1, 412, *x.shape[2:]), x[:, n_text:]], dim=1).contiguous()
        wide = pad(md)
        wide[:, n_text:512] = 0
        assert torch.equal(run(many, pad(kd), pad(vd), wide, 512), alone), "%d query rows, room for 512 keys" % n_q


@pytest.mark.parametrize("split", [0, 64])
def test_rows_past_the_caches_have_the_same_bits(split):
    """More output rows than the caches hold are stored past them, in whole 64-byte sectors only; the same call into rows
    that start 16 bytes off stores through them."""
    import torch

    nb, Lq, H, D, Lk = 2, 26300, 40, 128, 130
    g = torch.Generator(device="cuda").manual_seed(11)
    q, k, v = (torch.randn(nb, n, H, D, generator=g, device="cuda").to(torch.bfloat16) for n in (Lq, Lk, Lk))
    assert 2 * q.numel() > 512 << 20
    aligned = torch.empty_like(q)
    shifted = torch.empty(q.numel() + 8, dtype=q.dtype, device="cuda")[8:].view(q.shape)
    assert aligned.data_ptr() % 64 == 0 and shifted.data_ptr() % 64 == 16
    for out in (aligned, shifted):
        B.dit_cross_attn_forward(q, k, v, out=out, split=split, flags=B.DIT_FLAG_BIG_WORKGROUP)
    assert torch.equal(aligned.view(torch.int16), shifted.view(torch.int16))
    ref = torch.zeros(64, H, D, dtype=torch.float64)  # the last rows of the last request
    for a, b in ((0, split), (split, Lk)):
        if b > a:
            qf, kf, vf = (t.double().cpu().transpose(0, 1) for t in (q[-1, -64:], k[-1, a:b], v[-1, a:b]))
            ref += (torch.softmax(qf @ kf.transpose(1, 2) * D ** -0.5, dim=-1) @ vf).transpose(0, 1)
    compare(to_f64(aligned[-1, -64:]), ref.numpy(), bf16_out=True, what="rows past the caches, split %d" % split)
