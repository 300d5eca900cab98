"""Tiled kernel, short K-slices: fewer k tiles than the DMA ring has stages, one period of it, one tile more, for every
height, width and format of the kernel, whole or split once.  Against the oracle."""
import numpy as np
import pytest
import torch

import paper_2312_08583_amd as P
from oracle import fp6_oracle as O
from paper_2312_08583_amd import binding as B
from paper_2312_08583_amd import inputs

from gpu_util import assert_y_close, to_np16

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _plans():
    for fmt in ("fp6", "fp5", "v2", "bf16", "fgq"):
        for bm in (32, 64) if fmt == "fgq" else (32, 64, 128):
            for width in (4, 8):
                yield fmt, bm, width, 0
    yield "fp6", 128, 4, 1


@pytest.mark.parametrize("fmt,bm,width,kw", list(_plans()))
def test_short_slices(fmt, bm, width, kw):
    N, M = (width + 1) * 64, bm + 3
    variant = B.FP6_VARIANT_GEMM | B.FP6_HINT_BLOCK_M(bm) | B.FP6_HINT_WIDTH(width) | (B.FP6_HINT_KWAYS(2) if kw else 0)
    quantize, linear, oracle = {
        "fp6": (P.fp6_quantize_pack, P.fp6_linear_variant, O.linear), "fp5": (P.fp5_quantize_pack, P.fp5_linear, O.linear5),
        "v2": (P.fp6_quantize_pack_v2, P.fp6_linear_v2, O.linear),
        "bf16": (P.fp6_quantize_pack_v2, P.fp6_linear_v2_bf16, O.linear_bf16), "fgq": (None, None, None)}[fmt]
    ws = P.new_workspace(64 << 20, DEV)
    for ktiles, split in [(1, 1), (2, 1), (3, 1), (4, 1), (5, 1), (6, 1), (7, 1), (9, 1), (6, 2), (10, 2), (24, 2)]:
        if kw and (ktiles // split) % 2:
            continue
        K, block = ktiles * 64, 64 if ktiles % 2 else 128
        W = inputs.weight(N, K, seed=6100 + ktiles, sigma=0.02, outlier_frac=0.001, device=DEV)
        X = (inputs.activation_bf16 if fmt == "bf16" else inputs.activation)(M, K, seed=6200 + ktiles, device=DEV)
        xb = X.cpu().view(torch.int16).numpy().view(np.uint16)
        if fmt == "fgq":
            codes, scales = O.quantize_fgq(to_np16(W), block)
            Y = P.fp6_linear_fgq(X, *P.fp6_quantize_pack_fgq(W, block), N, K, block, variant, split, workspace=ws)
            Yref = O.linear_fgq(xb, codes, scales, block)
        else:
            codes, scales = (O.quantize5 if fmt == "fp5" else O.quantize)(to_np16(W))
            Y = linear(X, *quantize(W), N, K, variant, split, workspace=ws)
            Yref = oracle(xb, codes, scales)
        torch.cuda.synchronize()
        if fmt == "bf16":
            y = Y.cpu().double().numpy()     # half a unit in the last of 8 significant bits, and the fp32 sums
            assert (np.abs(y - Yref) <= 2.0 ** -8 * np.abs(Yref) + 1e-4 * (np.abs(Yref) + np.sqrt(np.mean(Yref ** 2)))).all()
        else:
            assert_y_close(Y, Yref, (fmt, bm, width, ktiles, split))
