"""A small convenience object around the C ABI: one quantized linear layer, prepared once, applied many times.

It only allocates device tensors with torch and calls the entry points of the same names; no arithmetic of the
method happens here.  `bits` = 4 uses the packed 4-bit path, 5..8 the int8-code path (Sec. 4.1 settings, appendix);
`act_bits` different from `bits` is a mixed-precision layer (e.g. 4-bit weights, 8-bit activations) on the int8-code path.
"""
from __future__ import annotations

import contextlib
from typing import Optional

import torch

from . import binding as q


_MATRIX_CORE_ROWS = (768, 1536, 3072, 6144, 2560, 5120, 8192)      # beside 1024, 2048 and 4096: sizes whose bf16 rows kernel 1 takes through the matrix cores


class DsfqLinear:
    """Y = X W^T + b with W and X quantized as in Sec. 3.2 (rotation, smoothing, per-channel / per-token codes).

    weight: [N, K] bf16 or f32 device tensor; bias: [N] bf16 device tensor or None; signs: int8 [K] of +-1 or None;
    calibration: [M_cal, K] activations for the smoothing statistic, or None for rotation only (c = 1).

    The weight codes are kept in two forms (1.25 bytes a weight in the 4-bit setting): Wq, and the blocks Wf or Wb that bf16 rows of K = 1024, 2048 and
    4096 are multiplied with.  Other rows of a 4-bit layer take Wf only while Wq is the tensor, and as it was, when Wf was made of it; other codes
    assigned to Wq or written into it are the ones that count.  A layer keeps one workspace, into which a call's first kernel
    writes what its second reads: calls of one layer follow each other on one stream, from one thread at a time; several streams or threads
    take a layer each.
    """

    def __init__(self, weight: torch.Tensor, bias: Optional[torch.Tensor] = None, signs: Optional[torch.Tensor] = None,
                 calibration: Optional[torch.Tensor] = None, alpha: float = 0.5, bits: int = 4,
                 act_bits: Optional[int] = None, pre_gelu: bool = False):
        act_bits = bits if act_bits is None else act_bits
        if not 4 <= bits <= 8 or not 4 <= act_bits <= 8:
            raise ValueError("bits and act_bits must be in 4..8")
        self.N, self.K = weight.shape
        # pre_gelu: the layer computes GELU(X) W^T + b, the activation applied as X is read (fc2 of an MLP block fed with fc1's output)
        if pre_gelu and not (bits == 4 and act_bits == 4 and self.K in (1024, 2048, 4096)):
            raise ValueError("pre_gelu needs the 4-bit setting and K = 1024, 2048 or 4096")
        self.pre_gelu = pre_gelu
        self.gelu_table = None
        if pre_gelu:         # the activation as a table of correctly rounded bf16 results, built on the device once
            self.gelu_table = torch.empty(q.qvggt_gelu_table_bytes(), dtype=torch.uint8, device=weight.device)
            q.qvggt_gelu_table(self.gelu_table)
        self.bits, self.act_bits, self.bias, self.signs = bits, act_bits, bias, signs
        self.packed = bits == 4 and act_bits == 4            # both 4-bit: two codes per byte; otherwise int8 codes
        dev = weight.device
        # the codes are kept in a second form, the blocks that the fast GEMMs read: E2M3 numbers, and int8 blocks for the sizes whose kernel 1
        # writes them.  bf16 rows of those sizes with a calibration batch are made in three launches, the others one entry point at a time
        blocks = self.K in (1024, 2048, 4096)
        fused = (blocks and calibration is not None and weight.dtype == calibration.dtype == torch.bfloat16 and calibration.dim() == 2
                 and calibration.shape[0] > 0 and calibration.shape[1] == self.K)
        absmax = None
        if fused:
            rows = calibration.shape[0]
            scratch = torch.empty(q.qvggt_layer_workspace_bytes(rows, self.N, self.K), dtype=torch.uint8, device=dev)
            q.qvggt_layer_statistics(weight, calibration, signs, scratch)
        elif calibration is not None:
            absmax = torch.empty(self.K, dtype=torch.float32, device=dev)
            q.qvggt_rotated_col_absmax(calibration, signs, absmax)
        self.w_scale = torch.empty(self.N, dtype=torch.float32, device=dev)
        self.inv_smooth = torch.empty(self.K, dtype=torch.float32, device=dev)
        if self.packed:
            with torch.inference_mode(False) if torch.is_inference_mode_enabled() else contextlib.nullcontext():       # versions are counted
                self.Wq = torch.empty(self.N, self.K // 2, dtype=torch.uint8, device=dev)
            self.Wf = torch.empty(q.qvggt_e2m3_bytes(self.N, self.K), dtype=torch.uint8, device=dev)
            if not blocks:                   # nothing to count there, and nothing to wait for
                q.qvggt_prep_weights_e2m3(weight, absmax, signs, alpha, self.Wq, self.Wf, self.w_scale, self.inv_smooth)
            else:
                lost = torch.empty(1, dtype=torch.int32, device=dev) if fused else torch.zeros(1, dtype=torch.int32, device=dev)
                if fused:
                    q.qvggt_layer_codes(weight, rows, signs, alpha, bits, False, self.Wq, self.Wf, self.w_scale, self.inv_smooth, lost, scratch)
                else:
                    q.qvggt_prep_weights(weight, absmax, signs, alpha, self.Wq, self.w_scale, self.inv_smooth)
                    q.qvggt_codes_to_e2m3(self.Wq, self.N, self.K, self.Wf, lost)
                n = int(lost.item())
                if n != 0:                   # cannot happen with absmax steps of numbers (codes lie in [-7, 7])
                    raise RuntimeError(f"{n} weight codes -8 have no E2M3 value")
        else:
            self.Wq = torch.empty(self.N, self.K, dtype=torch.int8, device=dev)
            self.Wb = torch.empty(q.qvggt_i8b_bytes(self.N, self.K), dtype=torch.int8, device=dev) if blocks else None
            if fused:
                q.qvggt_layer_codes(weight, rows, signs, alpha, bits, True, self.Wq, self.Wb, self.w_scale, self.inv_smooth, None, scratch)
            else:
                q.qvggt_prep_weights_i8(weight, absmax, signs, alpha, bits, self.Wq, self.w_scale, self.inv_smooth)
                if blocks:
                    q.qvggt_int8_to_blocks(self.Wq, self.N, self.K, self.Wb)
        if self.packed:
            self._blocks_of = (self.Wq, self.Wq._version)
        self._ws = (-1, None)       # rows the workspace is large enough for, the workspace

    _blocks_of = None               # the packed codes that Wf was made of, and their version (layers of earlier builds: not known)

    def _blocks_hold(self) -> bool:
        made = self._blocks_of
        return made is not None and made[0] is self.Wq and made[1] == self.Wq._version

    def __getstate__(self):         # a copy's tensors count their versions anew
        state = dict(self.__dict__)
        if "_blocks_of" in state:
            state["_blocks_of"] = self._blocks_hold()
        return state

    def __setstate__(self, state):
        self.__dict__.update(state)
        if "_blocks_of" in state:
            self._blocks_of = (self.Wq, self.Wq._version) if state["_blocks_of"] else None

    def _workspace(self, M: int, dev) -> torch.Tensor:
        rows, ws = self._ws         # read and replaced as a pair: a thread that comes at a bad moment is given one that is large enough
        if M <= rows and ws.device == dev:       # what M rows need grows with M
            return ws
        need = q.qvggt_workspace_bytes(M, self.N, self.K) if self.packed else q.qvggt_workspace_bytes_i8(M, self.N, self.K)
        if self.packed and self.Wf is not None:
            need = max(need, q.qvggt_workspace_bytes_e2m3(M, self.N, self.K))
        if not self.packed and self.Wb is not None:
            need = max(need, q.qvggt_workspace_bytes_i8b(M, self.N, self.K))
        if ws is None or ws.numel() < need or ws.device != dev:
            ws = torch.empty(need, dtype=torch.uint8, device=dev)
        self._ws = (M, ws)
        return ws

    def __call__(self, X: torch.Tensor, out: Optional[torch.Tensor] = None) -> torch.Tensor:
        """X: [M, K] bf16 or f32 on the GPU; returns bf16 [M, N] (written into `out` when given)."""
        M, K = X.shape
        if K != self.K:                                  # the entry points take K from X, and E2M3 blocks of another K would be read as this one's
            raise q.QvggtError(q.ERR_SHAPE, "DsfqLinear")
        if out is not None and out.dim() == 2 and (out.shape[1] > self.N or out.numel() * out.element_size() < 2 * M * out.shape[1]):
            raise q.QvggtError(q.ERR_SHAPE, "DsfqLinear: out")     # written, or weights read, past their end
        bf16 = X.dtype == torch.bfloat16
        if self.pre_gelu:
            if not bf16:
                raise ValueError("pre_gelu needs bf16 input")
            kind, W, bits = q.GELU, self.Wf, 4
        elif self.packed and self.Wf is not None and (bf16 and self.K in (1024, 2048, 4096) or
                                                      (M <= 4096 or self.K >= 512 and self.N >= (128 if bf16 and self.K in _MATRIX_CORE_ROWS else 448)) and self._blocks_hold()):
            # (many rows of few channels or features are kernel 1 and the stores of Y; kernel 1 writes nibbles faster, by up to 15 % where it is not on
            # the matrix cores.  us of both kernels, nibbles / E2M3 blocks: f32 41505 x 768 -> 128 43.6 / 48.0, 20000 x 4096 -> 320 133 / 146, bf16 105364 x 256 -> 48
            # 41.4 / 55.6, 99022 x 1792 -> 320 240 / 242; 41505 x 768 -> 128 36.8 / 34.1, 20000 x 8192 -> 320 187 / 186, 24000 x 6144 -> 128 120 / 127; 10992 x 768 ->
            # 3072 44.2 / 32.5, f32 64 x 128 -> 128 5.2 / 3.4.  Over 3000 random sizes of more than 4096 rows the rule is 1.3 % above the better of the two;
            # most of that is K = 128 and 256 with many channels, which stay with nibbles: 7662 x 256 -> 3632 35.7 / 24.4)
            kind, W, bits = q.E2M3, self.Wf, 4
        elif self.packed:                                # the same Y, bit for bit
            kind, W, bits = q.PACKED, self.Wq, 4
        elif bf16 and self.Wb is not None:
            kind, W, bits = q.INT8_BLOCKS, self.Wb, self.act_bits
        else:                                            # the same Y
            kind, W, bits = q.INT8, self.Wq, self.act_bits
        rows, ws = self._ws         # as _workspace does
        if M > rows or ws.get_device() != X.get_device():
            ws = self._workspace(M, X.device)
        Y = q.native_linear(kind, X, self.signs, self.inv_smooth, self.gelu_table, W, self.w_scale, self.bias, out, ws, self.N, bits)
        if Y is not None:
            return Y
        Y = out if out is not None else torch.empty(M, self.N, dtype=torch.bfloat16, device=X.device)
        call = getattr(q, q.LINEAR_KINDS[kind])
        if kind == q.GELU:
            call(X, self.signs, self.inv_smooth, self.gelu_table, W, self.w_scale, self.bias, Y, ws)
        elif kind in (q.INT8, q.INT8_BLOCKS):
            call(X, self.signs, self.inv_smooth, bits, W, self.w_scale, self.bias, Y, ws)
        else:
            call(X, self.signs, self.inv_smooth, W, self.w_scale, self.bias, Y, ws)
        return Y
