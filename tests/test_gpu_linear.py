"""GPU parity of the dense projection y = x w^T + bias (dit_linear_forward) against the CPU fp64
oracle.  Tolerance: the 16-bit inputs are exact on both sides and every product is exact in fp32, so
the only error is the fp32 accumulation of K terms (at most K * 2^-24 relative to sum |x_k w_k|, in
practice a random walk) and, for bf16 output, the final rounding (half a unit in the last place).
With unit-variance outputs sum |x w| is about 0.64 * sqrt(K) * RMS(y); the bound used is
2^-22 * sqrt(K) * RMS(y) (4.3e-5 * RMS at K = 5,120), far below the 2e-2 of the attention contract."""
import numpy as np
import pytest

import oracle
from paper_2601_20655_amd import binding as B
from paper_2601_20655_amd import workloads as wl
from gpu_util import compare, to_dev, to_f64

pytestmark = pytest.mark.gpu


def tol(K):
    return 2.0 ** -22 * K ** 0.5


@pytest.mark.parametrize("out", ["f32", "bf16"])
@pytest.mark.parametrize("with_bias", [True, False])
def test_small_projection_all_elements(out, with_bias):
    import torch

    cfg = wl.CONFIGS["proj_small"]
    x, w, b = wl.linear_inputs(cfg)
    y = B.dit_linear_forward(to_dev(x), to_dev(w), to_dev(b) if with_bias else None,
                             out_dtype=torch.float32 if out == "f32" else torch.bfloat16)
    torch.cuda.synchronize()
    ref = oracle.linear(x, w, b if with_bias else None)
    compare(to_f64(y), ref, bf16_out=out == "bf16", tol=tol(cfg["K"]), what="proj_small %s" % out)


@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (31, 264, 64), (257, 8, 128), (256, 256, 64), (513, 1000, 320)])
def test_edge_shapes(M, N, K):
    """One row, one feature quad pair, exact tile multiples, one row past a tile."""
    import torch

    cfg = dict(M=M, N=N, K=K, seed=31 + M)
    x, w, b = wl.linear_inputs(cfg)
    y = B.dit_linear_forward(to_dev(x), to_dev(w), to_dev(b), out_dtype=torch.float32)
    torch.cuda.synchronize()
    compare(to_f64(y), oracle.linear(x, w, b), tol=tol(K), what="M=%d N=%d K=%d" % (M, N, K))


def test_row_strides_and_untouched_padding():
    """x, w and y are column slices of wider buffers; the columns of y's buffer outside the slice keep
    their contents."""
    import torch

    cfg = dict(M=300, N=72, K=128, seed=5)
    x, w, b = wl.linear_inputs(cfg)
    xb = torch.zeros((300, 128 + 64), dtype=torch.bfloat16, device="cuda")
    wb = torch.zeros((72, 128 + 8), dtype=torch.bfloat16, device="cuda")
    yb = torch.full((300, 72 + 24), 7.0, dtype=torch.float32, device="cuda")
    xb[:, 64:] = to_dev(x)
    wb[:, :128] = to_dev(w)
    B.dit_linear_forward(xb[:, 64:], wb[:, :128], to_dev(b), out=yb[:, 8:80])
    torch.cuda.synchronize()
    compare(to_f64(yb[:, 8:80]), oracle.linear(x, w, b), tol=tol(128), what="strided")
    assert torch.all(yb[:, :8] == 7.0) and torch.all(yb[:, 80:] == 7.0)


def test_exact_small_integers():
    """Integer-valued inputs whose sums fit 24 bits: every output is exact, whatever the order."""
    import torch

    rng = np.random.default_rng(11)
    x = rng.integers(-8, 9, size=(260, 192)).astype(np.float32)
    w = rng.integers(-8, 9, size=(264, 192)).astype(np.float32)
    bias = rng.integers(-64, 65, size=264).astype(np.float32)
    xb, wb, bb = (wl.f32_to_bf16_bits(a) for a in (x, w, bias))
    y = B.dit_linear_forward(to_dev(xb), to_dev(wb), to_dev(bb), out_dtype=torch.float32)
    torch.cuda.synchronize()
    assert np.array_equal(to_f64(y), oracle.linear(xb, wb, bb))


@pytest.mark.parametrize("name", ["out_proj_14b", "qkv_proj_14b"])
def test_full_size_sampled_rows(name):
    """The benchmark's shapes and launch: 192 sampled token rows (first, last, seeded in between),
    every feature, against the oracle; bf16 output as the benchmark writes it."""
    import torch

    cfg = wl.CONFIGS[name]
    x, w, b = wl.linear_inputs(cfg)
    y = B.dit_linear_forward(to_dev(x), to_dev(w), to_dev(b))
    torch.cuda.synchronize()
    rows = wl.sample_rows(cfg["M"], cfg["seed"], edge=40, n_random=112)
    got = to_f64(y[torch.from_numpy(rows).cuda()])
    ref = oracle.linear(x[rows], w, b)
    compare(got, ref, bf16_out=True, tol=tol(cfg["K"]), what=name)


@pytest.mark.parametrize("M", [255, 256, 257, 511, 513])
@pytest.mark.parametrize("N", [248, 256, 264])
def test_tile_boundaries_exact(M, N):
    """Token and feature counts one short of, on and one past a tile boundary, with integer-valued
    inputs whose sums fit 24 bits: every output, bias included, must be exact (no tolerance), so a row
    or feature quad that lands in the wrong place, is dropped or is written twice cannot hide."""
    import torch

    K = 128
    rng = np.random.default_rng(1000 * M + N)
    x = rng.integers(-8, 9, size=(M, K)).astype(np.float32)
    w = rng.integers(-8, 9, size=(N, K)).astype(np.float32)
    bias = rng.integers(-64, 65, size=N).astype(np.float32)
    xb, wb, bb = (wl.f32_to_bf16_bits(a) for a in (x, w, bias))
    y = torch.full((M + 2, N + 8), -77.0, dtype=torch.float32, device="cuda")
    B.dit_linear_forward(to_dev(xb), to_dev(wb), to_dev(bb), out=y[1:M + 1, :N])
    torch.cuda.synchronize()
    assert np.array_equal(to_f64(y[1:M + 1, :N]), oracle.linear(xb, wb, bb))
    # the guard rows and columns around the output keep their contents
    assert torch.all(y[0] == -77.0) and torch.all(y[M + 1] == -77.0) and torch.all(y[:, N:] == -77.0)


@pytest.mark.parametrize("K", [64, 128, 192])
@pytest.mark.parametrize("out", ["f32", "bf16"])
def test_several_tiles_per_workgroup_exact(K, out):
    """More tiles than the device has compute units, with one to three steps per tile: a workgroup walks
    two or three tiles as one stream, and the loads run a whole tile or two ahead of the MFMAs.  Ragged in
    both directions; integer-valued inputs whose sums fit 24 bits (and, for bf16 output, results of at
    most 8 significant bits), so every output must be exact."""
    import torch

    M, N = 6000, 6152
    rng = np.random.default_rng(7 * K + (out == "f32"))
    hi = 9 if out == "f32" else 2
    x = rng.integers(-hi + 1, hi, size=(M, K)).astype(np.float32)
    w = rng.integers(-hi + 1, hi, size=(N, K)).astype(np.float32)
    bias = rng.integers(-8, 9, size=N).astype(np.float32)
    xb, wb, bb = (wl.f32_to_bf16_bits(a) for a in (x, w, bias))
    ref = oracle.linear(xb, wb, bb)
    if out == "bf16":
        assert np.max(np.abs(ref)) <= 256  # |sum| <= K + 8 <= 200: exactly representable
    y = torch.full((M + 1, N + 8), -77.0, dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda")
    B.dit_linear_forward(to_dev(xb), to_dev(wb), to_dev(bb), out=y[:M, :N])
    torch.cuda.synchronize()
    assert np.array_equal(to_f64(y[:M, :N]), ref)
    assert torch.all(y[M] == -77.0) and torch.all(y[:, N:] == -77.0)


@pytest.mark.parametrize("M,N,K", [
    (33, 72, 64),        # 32 x 64 tiles, one step, fewer steps than stages
    (1, 4104, 448),      # the same: one row, ragged features
    (2783, 144, 64),     # 64 x 64
    (130, 3664, 704),    # the same, more steps than stages
    (1031, 3592, 64),    # 64 x 128
    (1031, 3592, 256),   # the same, more steps than stages
    (1025, 3080, 320),   # 128 x 128
    (1250, 4104, 256),   # 96 x 256 (half a chunk of loads per wavefront)
    (3502, 1560, 64),    # 128 x 256
    (2500, 3336, 576),   # 160 x 256 (half a chunk)
])
@pytest.mark.parametrize("out", ["f32", "bf16"])
def test_small_tiles(M, N, K, out):
    """Shapes at which tiles smaller than 256 x 256 are taken, ragged on both sides, from one step on (more steps
    than twice the LDS stages: test_small_tiles_reuse_their_stages); all elements."""
    import torch

    cfg = dict(M=M, N=N, K=K, seed=61 + M)
    x, w, b = wl.linear_inputs(cfg)
    y = torch.full((M, N + 8), 7.0, dtype=torch.float32 if out == "f32" else torch.bfloat16, device="cuda")
    B.dit_linear_forward(to_dev(x), to_dev(w), to_dev(b), out=y[:, :N])
    compare(to_f64(y[:, :N]), oracle.linear(x, w, b), bf16_out=out == "bf16", tol=tol(K), what="M=%d N=%d K=%d" % (M, N, K))
    assert torch.all(y[:, N:] == 7.0)


# every small tile with at least twice as many steps as LDS stages, plus one: each stage is refilled and read again
# (tile as choose_linear_form names it, stages, M, N, K; test_layout_host.py checks that the shapes run on these tiles)
STAGE_REUSE = [(11, 6, 2, 760, 832), (21, 5, 130, 3664, 704), (22, 3, 897, 4136, 448), (42, 5, 513, 3624, 704),
               (34, 3, 3603, 1048, 448), (44, 3, 3468, 1544, 448), (54, 3, 2500, 3336, 576)]


@pytest.mark.parametrize("form,stages,M,N,K", STAGE_REUSE)
def test_small_tiles_reuse_their_stages(form, stages, M, N, K):
    """Integer-valued inputs whose sums fit 24 bits: a fragment read before its stage has arrived, or after the next step
    has been written over it, cannot hide in a tolerance."""
    import torch

    rng = np.random.default_rng(K + M)
    x = rng.integers(-8, 9, size=(M, K)).astype(np.float32)
    w = rng.integers(-8, 9, size=(N, K)).astype(np.float32)
    bias = rng.integers(-64, 65, size=N).astype(np.float32)
    xb, wb, bb = (wl.f32_to_bf16_bits(a) for a in (x, w, bias))
    y = torch.full((M + 1, N), -77.0, dtype=torch.float32, device="cuda")
    B.dit_linear_forward(to_dev(xb), to_dev(wb), to_dev(bb), out=y[:M])
    assert np.array_equal(to_f64(y[:M]), oracle.linear(xb, wb, bb))
    assert torch.all(y[M] == -77.0)
