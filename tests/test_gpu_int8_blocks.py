"""GPU parity of the int8-code path on blocked operands ("int8 blocks"): the same codes, integer sums and outputs as the
qvggt_*_i8 entry points, whose parity against the oracle is tests/test_gpu_int8_path.py; accumulators also directly against the
oracle's integer product."""
import numpy as np
import pytest
import torch

import oracle
import synth
from synth import f32_to_bf16_bits
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _blocks(codes_np):
    lib = G.gpu_layout_int8(codes_np, 1)
    rows, K = codes_np.shape
    out = torch.full((G.q.qvggt_i8b_bytes(rows, K),), 0x5A, dtype=torch.uint8, device=G.DEV).view(torch.int8)
    G.q.qvggt_int8_to_blocks(lib, rows, K, out)
    return lib, out


def test_int8_to_blocks_layout():
    rows, K = 300, 256
    codes = np.random.default_rng(0).integers(-128, 128, (rows, K)).astype(np.int8)
    lib, out = _blocks(codes)
    L, B = lib.cpu().numpy(), out.cpu().numpy()
    r = np.arange(rows)
    for kt in range(K // 64):
        for ch in range(4):
            slot = ch ^ ((r % 16) >> 2)
            start = ((r // 128) * (K // 64) + kt) * 8192 + (r % 128) * 64 + slot * 16
            got = B[start[:, None] + np.arange(16)[None, :]]
            assert np.array_equal(got, L[:, kt * 64 + ch * 16: kt * 64 + ch * 16 + 16])


@pytest.mark.parametrize("M,N,K", [(64, 128, 128), (1, 16, 128), (300, 384, 256), (1374, 3072, 1024), (257, 1024, 4096), (33, 48, 8192),
                                   (500, 1040, 768)])
def test_i8b_gemm_bit_exact(M, N, K):
    rng = np.random.default_rng(M + N + K)
    qx = rng.integers(-128, 128, (M, K)).astype(np.int8)
    qw = rng.integers(-128, 128, (N, K)).astype(np.int8)
    dx = np.exp(rng.uniform(-3, 1, M)).astype(np.float32)
    dw = np.exp(rng.uniform(-8, -4, N)).astype(np.float32)
    bias_bits = f32_to_bf16_bits((rng.standard_normal(N) * 0.02).astype(np.float32))
    (Xl, Xb), (Wl, Wb) = _blocks(qx), _blocks(qw)
    Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    acc = torch.full((M, N), 12345, dtype=torch.int32, device=G.DEV)
    G.q.qvggt_i8b_gemm(Xb, G.to_dev(dx), Wb, G.to_dev(dw), G.to_dev(bias_bits), M, N, K, Y, acc)
    assert np.array_equal(acc.cpu().numpy(), oracle.int_gemm(qx, qw))
    Y8 = torch.empty_like(Y)
    G.q.qvggt_i8_gemm(Xl, G.to_dev(dx), Wl, G.to_dev(dw), G.to_dev(bias_bits), M, N, K, Y8, None)
    assert torch.equal(Y, Y8)


# tests/test_gemm_plan.py holds the plan to what this table says of each problem (K = 1024: in tiles with the dump only)
BOTH_TILE_SHAPES = [(66000, 512, 256, "small"), (33000, 1024, 512, "small"), (17000, 4096, 1024, "big+deep"), (8400, 2000, 4096, "big+deep")]


@pytest.mark.parametrize("M,N,K", [p[:3] for p in BOTH_TILE_SHAPES])
def test_i8b_gemm_both_tile_shapes(M, N, K):
    """Whole rounds of big tiles plus a remainder in 128 x 128 tiles, in one launch or, for the accumulator dump, in two (at small K all rows
    in one launch of small tiles): every row equals the row-major kernel's."""
    gen = torch.Generator(device="cpu").manual_seed(M)
    qx = torch.randint(-128, 128, (M, K), generator=gen, dtype=torch.int8).numpy()
    qw = torch.randint(-128, 128, (N, K), generator=gen, dtype=torch.int8).numpy()
    rng = np.random.default_rng(M)
    dx = np.exp(rng.uniform(-3, 1, M)).astype(np.float32)
    dw = np.exp(rng.uniform(-8, -4, N)).astype(np.float32)
    (Xl, Xb), (Wl, Wb) = _blocks(qx), _blocks(qw)
    Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    G.q.qvggt_i8b_gemm(Xb, G.to_dev(dx), Wb, G.to_dev(dw), None, M, N, K, Y, None)
    Y8 = torch.empty_like(Y)
    G.q.qvggt_i8_gemm(Xl, G.to_dev(dx), Wl, G.to_dev(dw), None, M, N, K, Y8, None)
    assert torch.equal(Y, Y8)
    tiles_n = (N + 255) // 256
    seam = ((M + 255) // 256 * tiles_n // 256 * 256 // tiles_n) * 256          # where the rest begins, if there is one
    rows = np.unique(np.concatenate([np.arange(0, 8), np.arange(seam - 8, min(seam + 8, M)), np.arange(M - 200, M), rng.choice(M, 200, replace=False)]))
    acc = torch.full((M, N), 12345, dtype=torch.int32, device=G.DEV)
    G.q.qvggt_i8b_gemm(Xb, G.to_dev(dx), Wb, G.to_dev(dw), None, M, N, K, Y, acc)
    assert np.array_equal(acc[torch.from_numpy(rows).to(G.DEV)].cpu().numpy(), oracle.int_gemm(qx[rows], qw))


# 256-row tiles, several per block, last ones of a few rows and channels, alone and with a rest; K of both bodies that blocks have (tests/test_gemm_plan.py holds
# them to the plan)
BIG_TILES = [(39527, 528, 128, "big"), (39654, 528, 512, "big"), (39410, 528, 768, "big"), (39282, 528, 1280, "big"), (35194, 3728, 256, "big+deep"),
             (32775, 912, 768, "big+deep"), (32782, 784, 4096, "big+deep")]


def _device_blocks(codes):
    out = torch.full((G.q.qvggt_i8b_bytes(*codes.shape),), 0x5A, dtype=torch.int8, device=G.DEV)
    G.q.qvggt_int8_to_blocks(codes, *codes.shape, out)
    return out


@pytest.mark.parametrize("M,N,K", [p[:3] for p in BIG_TILES])
@pytest.mark.parametrize("with_bias", [True, False])
def test_i8b_gemm_several_big_tiles_per_block(M, N, K, with_bias):
    """Every row equals the row-major kernel's."""
    g = torch.Generator(device=G.DEV).manual_seed(M + K)
    Xl = torch.randint(-128, 128, (M, K), generator=g, device=G.DEV, dtype=torch.int8)
    Wl = torch.randint(-128, 128, (N, K), generator=g, device=G.DEV, dtype=torch.int8)
    dx, dw = torch.rand(M, device=G.DEV, generator=g) + 0.1, torch.rand(N, device=G.DEV, generator=g) * 1e-3
    bias = torch.randn(N, device=G.DEV, generator=g).to(torch.bfloat16) if with_bias else None
    Y = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=G.DEV)
    want = Y.clone()
    G.q.qvggt_i8b_gemm(_device_blocks(Xl), dx, _device_blocks(Wl), dw, bias, M, N, K, Y, None)
    G.q.qvggt_i8_gemm(Xl, dx, Wl, dw, bias, M, N, K, want, None)
    assert torch.equal(Y, want)              # the row behind the last one is not written


# The kernel with the weights in registers (tests/test_gemm_plan.py holds these to the rule): last steps of 1 to 31 tokens, ranges of unequal length, last
# waves of 16 and 48 channels and waves without any, more groups of channels than compute units, Y past the caches and through them (3056)
RESIDENT = [(2017, 4112), (10993, 3056), (8223, 3120), (20995, 1040), (300, 66064)]


@pytest.mark.parametrize("M,N", RESIDENT)
@pytest.mark.parametrize("with_bias", [True, False])
def test_i8b_gemm_with_resident_weights(M, N, with_bias):
    """Every row equals the row-major kernel's, all 256 codes and sums beyond 2^24 among them."""
    K = 1024
    g = torch.Generator(device=G.DEV).manual_seed(M + N)
    Xl = torch.randint(-128, 128, (M, K), generator=g, device=G.DEV, dtype=torch.int8)
    Wl = torch.randint(-128, 128, (N, K), generator=g, device=G.DEV, dtype=torch.int8)
    Xl[:: 37] = -128
    Wl[:: 19] = -128
    Xb, Wb = (torch.full((G.q.qvggt_i8b_bytes(c.shape[0], K),), 0x5A, dtype=torch.int8, device=G.DEV) for c in (Xl, Wl))
    G.q.qvggt_int8_to_blocks(Xl, M, K, Xb)
    G.q.qvggt_int8_to_blocks(Wl, N, K, Wb)
    dx, dw = torch.rand(M, device=G.DEV, generator=g) + 0.1, torch.rand(N, device=G.DEV, generator=g) * 1e-3
    bias = torch.randn(N, device=G.DEV, generator=g).to(torch.bfloat16) if with_bias else None
    Y = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=G.DEV)
    want = Y.clone()
    G.q.qvggt_i8b_gemm(Xb, dx, Wb, dw, bias, M, N, K, Y, None)
    G.q.qvggt_i8_gemm(Xl, dx, Wl, dw, bias, M, N, K, want, None)
    assert torch.equal(Y, want)              # the row behind the last one is not written


@pytest.mark.parametrize("K,rows", [(1024, 1031), (2048, 300), (4096, 203)])
@pytest.mark.parametrize("bits", [8, 6])
def test_rotate_quant_i8b_equals_the_row_major_kernel(K, rows, bits):
    rng = np.random.default_rng(K + bits)
    x = rng.standard_t(3, (rows, K)).astype(np.float32)
    x[:, rng.choice(K, K // 100, replace=False)] *= 50
    X = f32_to_bf16_bits(x)
    signs = (rng.integers(0, 2, K) * 2 - 1).astype(np.int8)
    inv = (1.0 / (np.sqrt(K) * np.exp(rng.uniform(-1, 1, K)))).astype(np.float32)
    Xd, sd, invd = G.to_dev(X), G.to_dev(signs), G.to_dev(inv)
    Xq, sx = G.gpu_rsq_i8(Xd, sd, invd, bits)
    want = torch.full((G.q.qvggt_i8b_bytes(rows, K),), 0x5A, dtype=torch.uint8, device=G.DEV).view(torch.int8)
    G.q.qvggt_int8_to_blocks(Xq, rows, K, want)
    got = torch.full_like(want, 0x5A)
    sxb = torch.empty_like(sx)
    G.q.qvggt_rotate_smooth_quant_i8b(Xd, sd, invd, bits, got, sxb)
    assert torch.equal(sx, sxb) and torch.equal(got, want)


@pytest.mark.parametrize("rows", [1, 3, 127, 129, 385, 4097])
def test_rows_of_2048_leave_as_int8_blocks(rows):
    """Two rows a tile, four 16-byte chunks a row: with an odd last row, on both sides of a 128-row block and with several tiles per wave, the codes are the
    row-major kernel's, and rows behind them are not written."""
    K = 2048
    g = torch.Generator(device=G.DEV).manual_seed(rows)
    X = torch.randn(rows, K, device=G.DEV, generator=g).to(torch.bfloat16)
    inv = torch.rand(K, device=G.DEV, generator=g) + 0.5
    Xq, sx = G.gpu_rsq_i8(X, None, inv, 8)
    want = torch.full((G.q.qvggt_i8b_bytes(rows, K),), 0x5A, dtype=torch.uint8, device=G.DEV).view(torch.int8)
    G.q.qvggt_int8_to_blocks(Xq, rows, K, want)
    got, sxb = torch.full_like(want, 0x5A), torch.empty_like(sx)
    G.q.qvggt_rotate_smooth_quant_i8b(X, None, inv, 8, got, sxb)
    blocks = [b.view(-1, K // 64, 128, 64) for b in (got, want)]
    r = torch.arange(rows, device=G.DEV)
    assert torch.equal(sx, sxb) and torch.equal(*[b[r // 128, :, r % 128] for b in blocks])
    if rows % 128: assert (blocks[0][rows // 128, :, rows % 128:] == 0x5A).all().item()


@pytest.mark.parametrize("name,M,bits", [("fc1", 3000, 8), ("fc2", 700, 8), ("fc1", 130, 6)])
def test_linear_i8b(name, M, bits):
    s = synth.layer_spec(5, name)
    K, N = s.K, s.N
    rng = np.random.default_rng(M)
    x = rng.standard_t(3, (M, K)).astype(np.float32)
    X = f32_to_bf16_bits(x)
    W, bias, signs = synth.make_weights(s), synth.make_bias(s), synth.make_signs(s)
    pg = G.gpu_prep_i8(W, X[:512], signs, bits)
    Wb = torch.empty(G.q.qvggt_i8b_bytes(N, K), dtype=torch.int8, device=G.DEV)
    G.q.qvggt_int8_to_blocks(pg["Wq"], N, K, Wb)
    Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    ws = torch.empty(G.q.qvggt_workspace_bytes_i8b(M, N, K), dtype=torch.uint8, device=G.DEV)
    G.q.qvggt_linear_i8b(G.to_dev(X), pg["signs"], pg["inv"], bits, Wb, pg["sw"], G.to_dev(bias), Y, ws)
    assert torch.equal(Y, G.gpu_linear_i8(G.to_dev(X), pg, G.to_dev(bias)))
    po = oracle.prepare_weights(W, oracle.rotated_col_absmax(X[:512], pre_signs=signs), pre_signs=signs, bits=bits)
    want = oracle.linear(X, po, bias=bias, pre_signs=signs, bits=bits)
    assert G.rel_fro(G.bf16_bits(Y), want.Y) <= G.Y_REL_FRO


@pytest.mark.parametrize("name,n_random", [("fc1", 600), ("fc2", 300)])
def test_linear_i8b_full_size(name, n_random):
    """The benchmark's shapes (137400 tokens) in the launch configuration bench.py times: every element of Y equals the row-major
    path's, and a seeded sample of rows is within the output bound of the oracle's."""
    s = synth.layer_spec(5, name)
    rng = np.random.default_rng(len(name) + 8)
    rows = np.unique(np.concatenate([np.arange(synth.SPECIAL_TOKENS), np.arange(s.M - 64, s.M), rng.choice(s.M, n_random, replace=False)]))
    signs = synth.make_signs(s)
    W, Xc, bias = synth.make_weights(s), synth.make_calibration(s), synth.make_bias(s)
    po = oracle.prepare_weights(W, oracle.rotated_col_absmax(Xc, pre_signs=signs), pre_signs=signs, alpha=0.5, bits=8)
    pg = G.gpu_prep_i8(W, Xc, signs, 8)
    X = synth.make_activation_frames(s)
    Xd = G.to_dev(X)
    want = oracle.linear(X[rows], po, bias=bias, pre_signs=signs, bits=8)
    del X
    Wb = torch.empty(G.q.qvggt_i8b_bytes(s.N, s.K), dtype=torch.int8, device=G.DEV)
    G.q.qvggt_int8_to_blocks(pg["Wq"], s.N, s.K, Wb)
    Y = torch.full((s.M, s.N), float("nan"), dtype=torch.bfloat16, device=G.DEV)
    ws = torch.empty(G.q.qvggt_workspace_bytes_i8b(s.M, s.N, s.K), dtype=torch.uint8, device=G.DEV)
    G.q.qvggt_linear_i8b(Xd, pg["signs"], pg["inv"], 8, Wb, pg["sw"], G.to_dev(bias), Y, ws)
    idx = torch.from_numpy(rows).to(G.DEV)
    err = G.rel_fro(G.bf16_bits(Y[idx]), want.Y)
    assert err <= G.Y_REL_FRO, err
    assert torch.equal(Y, G.gpu_linear_i8(Xd, pg, G.to_dev(bias)))
