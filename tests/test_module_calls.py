"""DsfqLinear's choice of an entry point, and what it refuses before any, without a GPU."""
import copy
import pickle

import pytest
import torch

from paper_2509_21302_amd import binding as B
from paper_2509_21302_amd.module import DsfqLinear


@pytest.fixture
def taken(monkeypatch):
    """kinds of the calls that reach the library, which does not run"""
    kinds = []

    def native_linear(kind, X, *a):
        kinds.append(kind)
        return torch.empty(X.shape[0], 16, dtype=torch.bfloat16)
    monkeypatch.setattr(B, "native_linear", native_linear)
    return kinds


def _layer(K, N=16, bits=4, pre_gelu=False, wide=None):
    layer = DsfqLinear.__new__(DsfqLinear)
    layer.__dict__.update(N=N, K=K, bits=bits, act_bits=bits, bias=None, signs=None, packed=bits == 4, pre_gelu=pre_gelu, gelu_table=None,
                          w_scale=None, inv_smooth=None, Wq=torch.empty(0), _ws=(-1, None))
    blocks = torch.empty(0) if bits == 4 or K in (1024, 2048, 4096) else None
    layer.__dict__["Wf" if bits == 4 else "Wb"] = blocks
    return layer


@pytest.mark.parametrize("bits,pre_gelu", [(4, False), (4, True), (8, False)])
@pytest.mark.parametrize("K,other", [(1024, 512), (1024, 2048), (4096, 1024), (512, 1024), (768, 512)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_rows_of_another_length_are_refused(taken, bits, pre_gelu, K, other, dtype):
    if pre_gelu and (K not in (1024, 4096) or dtype != torch.bfloat16):
        pytest.skip("no such layer or input")
    layer = _layer(K, bits=bits, pre_gelu=pre_gelu)
    with pytest.raises(B.QvggtError, match="QVGGT_ERR_SHAPE"):
        layer(torch.zeros(3, other, dtype=dtype))
    assert not taken
    layer(torch.zeros(3, K, dtype=dtype))
    assert len(taken) == 1


def test_a_layer_of_an_earlier_build_is_called_as_before(taken):
    """A layer that was copied or saved with the attributes it has always had (here without anything newer)."""
    layer = _layer(1024)
    assert set(layer.__dict__) == {"N", "K", "bits", "act_bits", "bias", "signs", "packed", "pre_gelu", "gelu_table", "w_scale", "inv_smooth", "Wq", "Wf", "_ws"}
    layer(torch.zeros(5000, 1024, dtype=torch.bfloat16))
    old = _layer(768)
    old.Wf = None                           # sizes that had no second form of the codes
    old(torch.zeros(5000, 768, dtype=torch.bfloat16))
    assert taken == [B.E2M3, B.PACKED]


@pytest.mark.parametrize("rows,cols,dtype", [(2, 48, torch.bfloat16), (3, 64, torch.bfloat16), (3, 48, torch.uint8), (0, 48, torch.bfloat16)])
def test_an_output_that_a_call_does_not_fit_is_refused(taken, rows, cols, dtype):
    layer, X = _layer(1024, N=48), torch.zeros(3, 1024, dtype=torch.bfloat16)
    with pytest.raises(B.QvggtError, match="QVGGT_ERR_SHAPE"):
        layer(X, out=torch.empty(rows, cols, dtype=dtype))
    assert not taken
    for fits in (torch.empty(3, 48, dtype=torch.bfloat16), torch.empty(5, 16, dtype=torch.bfloat16), torch.empty(3, 48)):
        layer(X, out=fits)
    assert len(taken) == 3


@pytest.mark.parametrize("K", [128, 768, 5120, 8192])
@pytest.mark.parametrize("calibrated", [True, False])
def test_a_layer_of_other_sizes_is_made_without_waiting(monkeypatch, K, calibrated):
    """Sizes that have no fused making: one call writes both forms of the codes, and nothing is read back from the device."""
    calls = []
    for name in B.EXPORTS:
        if hasattr(B, name) and "bytes" not in name:
            monkeypatch.setattr(B, name, lambda *a, name=name: calls.append(name))
    monkeypatch.setattr(torch.Tensor, "item", lambda self: pytest.fail("the host waits for the device"))
    W = torch.zeros(32, K)
    layer = DsfqLinear(W, calibration=W if calibrated else None)
    assert calls == ["qvggt_rotated_col_absmax"] * calibrated + ["qvggt_prep_weights_e2m3"]
    assert layer.Wf.numel() == B.qvggt_e2m3_bytes(32, K) and layer.Wq.shape == (32, K // 2)


@pytest.fixture
def made(monkeypatch, taken):
    """Layers of the constructor, whose kernels do not run."""
    for name in B.EXPORTS:
        if hasattr(B, name) and "bytes" not in name:
            monkeypatch.setattr(B, name, lambda *a: None)
    monkeypatch.setattr(torch.Tensor, "item", lambda self: 0)
    return lambda K, N=32: DsfqLinear(torch.zeros(N, K), calibration=torch.zeros(4, K))


@pytest.mark.parametrize("K,N,dtype,rows,kind", [(768, 128, torch.bfloat16, 4097, B.E2M3), (8192, 320, torch.bfloat16, 4097, B.E2M3), (768, 112, torch.bfloat16, 4097, B.PACKED),
                                                 (768, 112, torch.bfloat16, 4096, B.E2M3), (768, 432, torch.float32, 4097, B.PACKED), (1792, 432, torch.bfloat16, 4097, B.PACKED),
                                                 (1792, 448, torch.bfloat16, 4097, B.E2M3), (256, 4096, torch.bfloat16, 4097, B.PACKED), (4096, 320, torch.float32, 4097, B.PACKED)])
def test_many_rows_take_the_form_that_was_measured_faster(taken, made, K, N, dtype, rows, kind):
    made(K, N)(torch.zeros(rows, K, dtype=dtype))
    assert taken == [kind]


def _assign(layer):
    layer.Wq = layer.Wq.clone()


@pytest.mark.parametrize("K", [128, 768, 1024, 8192])
@pytest.mark.parametrize("write", [_assign, lambda l: l.Wq.fill_(1), lambda l: l.Wq[3:5].copy_(l.Wq[:2]), lambda l: B._written(l.Wq)])
@pytest.mark.parametrize("inference", [False, True])
def test_other_packed_codes_are_the_ones_that_count(taken, made, K, write, inference):
    """f32 rows, and bf16 rows of other sizes, as long as there was one form of the codes: what is in Wq is what they are multiplied with."""
    X = torch.zeros(3, K)
    with torch.inference_mode(inference):
        layer = made(K)
        layer(X)
        write(layer)
        layer(X)
        for again in (copy.copy(layer), copy.deepcopy(layer), pickle.loads(pickle.dumps(layer))):
            again(X)
    assert taken == [B.E2M3] + [B.PACKED] * 4


@pytest.mark.parametrize("K", [128, 768, 1024])
@pytest.mark.parametrize("again", [copy.copy, copy.deepcopy, lambda l: pickle.loads(pickle.dumps(l)), lambda l: copy.deepcopy(copy.deepcopy(l))])
def test_copies_of_a_layer_keep_both_forms(taken, made, K, again):
    """Whatever versions the copy's tensors count, and those of the layer it is a copy of."""
    X, layer = torch.zeros(3, K), made(K)
    B._written(layer.Wq)
    layer._blocks_of = (layer.Wq, layer.Wq._version)               # as where the codes were made by a call that counts
    twin = again(layer)
    twin(X)
    twin.Wq.zero_()
    twin(X)
    assert taken == [B.E2M3, B.PACKED]
