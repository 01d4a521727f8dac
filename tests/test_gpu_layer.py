"""DsfqLinear's fused making of a layer (bf16 rows, K = 1024, 2048, 4096) against the entry points it stands for: the same outputs, bit for bit."""
import pytest
import torch

from tests import gpu_util as G

pytestmark = pytest.mark.gpu
q = G.q


def _rows(n, k, seed, scale=1.0):
    g = torch.Generator(device=G.DEV).manual_seed(seed)
    x = torch.randn(n, k, device=G.DEV, generator=g) * scale
    x[:, torch.randint(0, k, (7,), device=G.DEV, generator=g)] *= 50
    return x.to(torch.bfloat16)


# one calibration row and the fewest channels; rows that end inside a tile, a wave's share and a block; more than two blocks per compute unit
@pytest.mark.parametrize("K", [1024, 2048, 4096])
@pytest.mark.parametrize("M,N", [(1, 16), (5, 144), (97, 128), (1374, 1024), (5496, 4096), (20000, 48)])
@pytest.mark.parametrize("bits,act_bits", [(4, 4), (8, 8), (4, 8), (6, 6)])
def test_layer_is_made_of_the_same_bits(K, M, N, bits, act_bits):
    W, X = _rows(N, K, N + K, 0.02), _rows(M, K, M + K)
    W[N // 2] = 0
    signs = (torch.randint(0, 2, (K,), device=G.DEV, dtype=torch.int8) * 2 - 1).contiguous() if M % 2 else None
    layer = q.DsfqLinear(W, None, signs, X, alpha=0.4, bits=bits, act_bits=act_bits)
    a, sw, inv = torch.empty(K, device=G.DEV), torch.empty(N, device=G.DEV), torch.empty(K, device=G.DEV)
    q.qvggt_rotated_col_absmax(X, signs, a)
    if (bits, act_bits) == (4, 4):
        Wq, lost = torch.empty(N, K // 2, dtype=torch.uint8, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV)
        q.qvggt_prep_weights(W, a, signs, 0.4, Wq, sw, inv)
        blocks, got = torch.zeros_like(layer.Wf), layer.Wf
        q.qvggt_codes_to_e2m3(Wq, N, K, blocks, lost)
        # padding rows of the last block are written by neither; a code 0 may carry a sign in one of the two
        assert (G.decode_e2m3_rows(got.cpu().numpy(), N, K) == G.decode_e2m3_rows(blocks.cpu().numpy(), N, K)).all()
    else:
        Wq = torch.empty(N, K, dtype=torch.int8, device=G.DEV)
        q.qvggt_prep_weights_i8(W, a, signs, 0.4, bits, Wq, sw, inv)
        blocks, got = torch.zeros_like(layer.Wb), layer.Wb
        q.qvggt_int8_to_blocks(Wq, N, K, blocks)
        rows = torch.arange(N, device=G.DEV)
        tiles = [b.view(-1, K // 64, 128, 64)[rows // 128, :, rows % 128] for b in (got, blocks)]
        assert torch.equal(*tiles)
    assert torch.equal(layer.Wq, Wq) and torch.equal(layer.w_scale, sw) and torch.equal(layer.inv_smooth, inv)


def test_a_weight_that_is_no_number_is_refused():
    W = _rows(64, 1024, 3, 0.02)
    W[3, 5] = float("nan")
    with pytest.raises(RuntimeError, match="no E2M3 value"):
        q.DsfqLinear(W, None, None, _rows(40, 1024, 4))


OTHER_K = [128, 256, 512, 768, 1280, 1536, 1792, 2560, 3072, 3584, 5120, 6144, 8192]


# rows that end inside a group of four and a 128-row block; above 4096 rows, where four waves share one, groups instead of single rows leave together
@pytest.mark.parametrize("K", OTHER_K)
@pytest.mark.parametrize("N", [16, 144, 4112])
@pytest.mark.parametrize("dtype,calibrated", [(torch.bfloat16, True), (torch.float32, False)])
def test_layers_of_other_sizes_keep_the_same_codes_in_both_forms(K, N, dtype, calibrated):
    W, X = _rows(N, K, N + K, 0.02).to(dtype), _rows(33, K, K).to(dtype)
    W[N // 2], W[1, 3], W[5, 7], W[5, 8] = 0, float("nan"), float("inf"), float("-inf")
    signs = (torch.randint(0, 2, (K,), device=G.DEV, dtype=torch.int8) * 2 - 1).contiguous() if calibrated else None
    layer = q.DsfqLinear(W, None, signs, X if calibrated else None, alpha=0.4)
    a, sw, inv = torch.empty(K, device=G.DEV), torch.empty(N, device=G.DEV), torch.empty(K, device=G.DEV)
    q.qvggt_rotated_col_absmax(X, signs, a)
    Wq, lost = torch.empty(N, K // 2, dtype=torch.uint8, device=G.DEV), torch.zeros(1, dtype=torch.int32, device=G.DEV)
    q.qvggt_prep_weights(W, a if calibrated else None, signs, 0.4, Wq, sw, inv)
    blocks = torch.zeros_like(layer.Wf)
    q.qvggt_codes_to_e2m3(Wq, N, K, blocks, lost)
    assert int(lost.item()) == 0                        # also with weights that are no numbers
    assert torch.equal(layer.Wq, Wq) and torch.equal(layer.w_scale, sw) and torch.equal(layer.inv_smooth, inv)
    rows = torch.arange(N, device=G.DEV)
    assert torch.equal(*[b.view(-1, K // 64, 128, 48)[rows // 128, :, rows % 128] for b in (layer.Wf, blocks)])


@pytest.mark.parametrize("K", [128, 768])
def test_a_layer_of_another_size_is_made_and_applied_inside_a_capture(K):
    W, X = _rows(64, K, 1, 0.02), _rows(40, K, 2)
    want = q.DsfqLinear(W, None, None, X)(X)
    other = _rows(40, K, 3)
    want_other = q.DsfqLinear(W, None, None, other)(other)
    graph, fed = torch.cuda.CUDAGraph(), X.clone()
    with torch.cuda.graph(graph):
        Y = q.DsfqLinear(W, None, None, fed)(fed)
    for x, y in ((X, want), (other, want_other), (X, want)):
        fed.copy_(x)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y.view(torch.int16), y.view(torch.int16))
