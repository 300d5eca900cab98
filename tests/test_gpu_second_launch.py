"""Tiled plans whose K-slices are added by a second launch: row counts that are no multiple of 4 or 16, a last workgroup
with missing channel blocks, slice counts around the eight that are loaded at a time, every format.  Against the oracle; a
second call on the same workspace gives the same bits.  Two cases stay below the lines and are added by the last workgroup
to arrive: little per block of Y; three slices of 64 KB where all blocks together have much."""
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


def _variant(bm, width):
    return B.FP6_VARIANT_GEMM | B.FP6_HINT_BLOCK_M(bm) | B.FP6_HINT_WIDTH(width)


FORMATS = {"fp6": B.FP6_FORMAT_E3M2, "fgq": B.FP6_FORMAT_E3M2, "fp5": B.FP6_FORMAT_E3M1, "v2": B.FP6_FORMAT_E3M2_V2,
           "bf16": B.FP6_FORMAT_E3M2_V2_BF16}


@pytest.mark.parametrize("fmt,M,bm,width,split,meeting", [("fp6", 97, 128, 4, 3, 3), ("fp6", 130, 128, 8, 9, 3), ("fp6", 33, 64, 4, 8, 3),
                                                          ("fp6", 31, 32, 8, 24, 3), ("fp5", 101, 64, 4, 6, 3), ("v2", 66, 64, 8, 4, 3),
                                                          ("bf16", 259, 128, 4, 3, 3), ("fgq", 62, 64, 8, 12, 3),
                                                          ("fp6", 201, 32, 4, 4, 1), ("fp6", 1000, 64, 4, 3, 1),
                                                          ("fp6", 513, 64, 4, 3, 3), ("fp6", 208, 64, 4, 4, 3)])
def test_slices_added_by_a_second_launch(fmt, M, bm, width, split, meeting):
    N, K, block = 9 * 64, 72 * 64, 512
    plan = P.fp6_linear_plan(M, N, K, format=FORMATS[fmt], block=block if fmt == "fgq" else 0, variant=_variant(bm, width), split_k=split)
    assert plan["meeting"] == meeting, plan
    W = inputs.weight(N, K, seed=5200 + M, sigma=0.02, outlier_frac=0.001, device=DEV)
    act = inputs.activation_bf16 if fmt == "bf16" else inputs.activation
    X = act(M, K, seed=5300 + M, device=DEV)
    wb = to_np16(W)
    if fmt == "fgq":
        planes, (codes, scales) = P.fp6_quantize_pack_fgq(W, block), O.quantize_fgq(wb, block)
    elif fmt == "fp5":
        planes, (codes, scales) = P.fp5_quantize_pack(W), O.quantize5(wb)
    else:
        planes = P.fp6_quantize_pack(W) if fmt == "fp6" else P.fp6_quantize_pack_v2(W)
        codes, scales = O.quantize(wb)
    xb = X.cpu().view(torch.int16).numpy().view(np.uint16)
    Yref = {"fgq": lambda: O.linear_fgq(xb, codes, scales, block), "fp5": lambda: O.linear5(xb, codes, scales),
            "bf16": lambda: O.linear_bf16(xb, codes, scales)}.get(fmt, lambda: O.linear(xb, codes, scales))()
    fn = {"fp6": P.fp6_linear_variant, "fp5": P.fp5_linear, "v2": P.fp6_linear_v2, "bf16": P.fp6_linear_v2_bf16}.get(fmt)
    v = _variant(bm, width)
    ws = P.new_workspace(256 << 20, DEV)
    if fmt == "fgq":
        call = lambda: P.fp6_linear_fgq(X, *planes, N, K, block, v, split, workspace=ws)
    else:
        call = lambda: fn(X, *planes, N, K, v, split, workspace=ws)
    Y, Y2 = call(), call()
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2)
    assert not ws[:B.FP6_WORKSPACE_ZERO_BYTES].any()
    if fmt == "bf16":
        y = Y.cpu().double().numpy()         # half a unit in the last of 8 significant bits, and the fp32 sums
        assert (np.abs(y - Yref) <= 2.0 ** -8 * np.abs(Yref) + 1e-4 * (np.abs(Yref) + np.sqrt(np.mean(Yref ** 2)))).all()
    else:
        assert_y_close(Y, Yref, (fmt, M, split))
