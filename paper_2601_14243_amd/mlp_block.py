"""Composition of the library's entry points into the MLP block of a decoder layer with
FP8-saved activations (Jet-RL Sec. 4.1: the tensors saved for the backward GEMMs are the FP8 ones
the forward GEMMs consumed; gradients between operators stay bf16; Sec. 4.2: one fused row +
column quantization per gradient, column re-quantization of the saved FP8 activations).

Every arithmetic step is one call into libjet.so; this module only orders the calls and keeps
the saved tensors.  Layout: the gate and up projections are one weight [2 I, H] (gate rows first),
so their output is one [M, 2 I] tensor and their backward is one DGrad and one WGrad.

    forward :  x --row quant--> (qx)  --FProp W_gu-->  gu  --SiLU*mul, row quant--> (qh)  --FProp W_d-->  y
    saved   :  qx (FP8 + scales), gu (bf16, input of the element-wise operator), qh (FP8 + scales)
    backward:  dy --row+col quant--> DGrad W_d^T --> dh ;  WGrad(dy^T, qh^T) --> dW_d
               (gu, dh) --SiLU*mul backward, row+col quant--> dgu, qdgu --> DGrad W_gu^T --> dx ;
               WGrad(dgu^T, qx^T) --> dW_gu
"""
from __future__ import annotations

from . import binding as jet

# The gate/up gradient is quantized where it is formed from 1024 tiles of 128x128 on: one pass over memory less, but half as many
# workgroups with three times the work.  Two calls / one, us on 256 CUs, captured and (called one by one), by tiles:
#   96    512x3072   13.4 / 18.8  (15.4 / 23.3)     640   2048x5120   45.1 / 43.5  (40.9 / 43.0)    1536   8192x3072   90.8 / 86.1  (85.1 / 81.0)
#   192   1024x3072  19.3 / 20.4  (20.7 / 23.3)     768   4096x3072   51.6 / 47.1  (47.5 / 45.8)    1728   1024x27648  105 / 95.7   (98.4 / 89.3)
#   320   1024x5120  27.9 / 29.7  (26.7 / 30.0)     864   512x27648   57.4 / 56.3  (52.3 / 55.2)    1792   2048x14336  107 / 97.6   (101 / 89.9)
#   384   2048x3072  31.0 / 31.3  (29.4 / 31.4)     896   1024x14336  59.5 / 57.2  (54.3 / 55.1)    3584   4096x14336  220 / 190    (219 / 161)
#   448   512x14336  33.9 / 32.4  (32.4 / 31.7)    1024   2048x8192   67.6 / 61.1  (59.3 / 59.5)   14336  16384x14336  880 / 726    (840 / 627)
#   512   1024x8192  36.9 / 34.1  (35.0 / 33.6)    1024   16384x1024  66.7 / 60.8  (60.1 / 56.9)
# Below 400 tiles one call loses (captured 512x8192, 256 tiles, 23.4 / 21.7 apart); from there to the line it is 2 to 9 % faster
# in a captured block and 5 % faster to 6 % slower in one that is not, where the second call's launch hides behind the first; from
# the line on neither loses.
QUANT_IN_BWD_FROM = 1024 * 128 * 128


class MlpWeights:
    """FP8 copies of the two master weights: (q, s, qT, sT) each, as jet_quant_weight writes them."""

    def __init__(self, w_gu, w_d):
        self.inter, self.hidden = w_gu.shape[0] // 2, w_gu.shape[1]
        if tuple(w_d.shape) != (self.hidden, self.inter):
            raise ValueError("w_d must be [hidden, inter] for w_gu [2 inter, hidden]")
        self.gu = jet.quant_weight(w_gu, transposed=True)
        self.d = jet.quant_weight(w_d, transposed=True)

    def requantize(self, w_gu, w_d):
        """After an optimizer step on the bf16 masters: the same buffers are overwritten."""
        jet.quant_weight(w_gu, transposed=True, out=self.gu)
        jet.quant_weight(w_d, transposed=True, out=self.d)


def forward(x, w: MlpWeights):
    """x bf16 [M, H] -> (y bf16 [M, H], saved)."""
    I = w.inter
    qx = jet.quant_act(x)
    gu = jet.fp8_linear_fwd(qx["q_row"], qx["s_row"], w.gu[0], w.gu[1])
    qh = jet.silu_mul_quant(gu[:, :I], gu[:, I:])
    y = jet.fp8_linear_fwd(qh["q_row"], qh["s_row"], w.d[0], w.d[1])
    return y, {"qx": qx, "gu": gu, "qh": qh}


def backward(saved, dy, w: MlpWeights):
    """dy bf16 [M, H] -> dict(dx [M, H], dw_gu [2 I, H], dw_d [H, I]) in bf16, plus the
    intermediate tensors (for tests)."""
    I = w.inter
    qx, gu, qh = saved["qx"], saved["gu"], saved["qh"]
    qdy = jet.quant_act(dy, row=True, col=True)
    dh = jet.fp8_linear_dgrad(qdy["q_row"], qdy["s_row"], w.d[2], w.d[3])
    qhT = jet.quant_act(qh["q_row"], qh["s_row"], row=False, col=True)
    dw_d = jet.fp8_linear_wgrad(qdy["q_colT"], qdy["s_colT"], qhT["q_colT"], qhT["s_colT"])
    if dh.numel() >= QUANT_IN_BWD_FROM:
        dgu, qdgu = jet.silu_mul_bwd_quant(gu[:, :I], gu[:, I:], dh)
    else:
        dgu = jet.silu_mul_bwd(gu[:, :I], gu[:, I:], dh)
        qdgu = jet.quant_act(dgu, row=True, col=True)
    dx = jet.fp8_linear_dgrad(qdgu["q_row"], qdgu["s_row"], w.gu[2], w.gu[3])
    qxT = jet.quant_act(qx["q_row"], qx["s_row"], row=False, col=True)
    dw_gu = jet.fp8_linear_wgrad(qdgu["q_colT"], qdgu["s_colT"], qxT["q_colT"], qxT["s_colT"])
    return {"dx": dx, "dw_gu": dw_gu, "dw_d": dw_d, "qdy": qdy, "dh": dh, "qhT": qhT, "dgu": dgu,
            "qdgu": qdgu, "qxT": qxT}


def saved_bytes(M: int, hidden: int, inter: int) -> dict:
    """Bytes kept between forward and backward per block, against saving the same tensors in bf16."""
    fp8 = lambda rows, cols: rows * cols + 4 * rows * (cols // 128)
    ours = fp8(M, hidden) + 2 * M * 2 * inter + fp8(M, inter)
    bf16 = 2 * M * hidden + 2 * M * 2 * inter + 2 * M * inter
    return {"fp8_saved": ours, "bf16_saved": bf16, "ratio": ours / bf16}
