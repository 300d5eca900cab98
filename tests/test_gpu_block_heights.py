"""Tiled kernel, block heights between the powers of two: the rows of X are dealt evenly to the blocks along M, so that a plan of
64 or 128 rows runs with 48, 80, 96 or 112.  Every height, width, format and kind of K-split, at ragged heights and channel counts:
bit for bit what the forced plan of 64 or 128 rows gives (the same products in the same order), and against the oracle."""
import shutil

import numpy as np
import pytest
import torch

import paper_2312_08583_amd as P
from oracle import fp6_oracle as O
from paper_2312_08583_amd import binding as B
from paper_2312_08583_amd import inputs

from gpu_util import assert_y_close, to_np16
from test_codegen_guard import _scratch_sizes

DEV = "cuda"
FORMATS = {"fp6": 6, "fp5": 5, "v2": 7, "bf16": 8, "fgq": 6}
# (format, M, N, K, plan); K of fewer k tiles than the ring has stages, of one more, and odd ones
CASES = [
    ("fp6", 69, 21056, 64, "gemm 48x256 split1"), ("fp6", 33, 16640, 1536, "gemm 48x256 split3 counter"),
    ("fp6", 133, 27840, 320, "gemm 80x256 split1"), ("fp6", 65, 20672, 3072, "gemm 80x256 k2 split3 second-launch"),
    ("fp6", 257, 12544, 192, "gemm 96x256 split1"), ("fp6", 269, 6272, 3072, "gemm 96x256 k2 split3 second-launch"),
    ("fp6", 281, 24896, 320, "gemm 96x512 split1"), ("fp6", 195, 16832, 448, "gemm 112x256 split1"),
    ("fp6", 203, 9344, 3072, "gemm 112x256 k2 split3 second-launch"), ("fp6", 324, 22528, 576, "gemm 112x512 split1"),
    ("fp5", 72, 21312, 128, "gemm 48x256 split1"), ("fp5", 131, 27136, 256, "gemm 80x256 split1"),
    ("fp5", 161, 20736, 320, "gemm 96x256 split1"), ("fp5", 286, 24896, 320, "gemm 96x512 split1"),
    ("fp5", 521, 6272, 192, "gemm 112x256 split1"), ("fp5", 321, 23168, 64, "gemm 112x512 split1"),
    ("v2", 65, 20992, 320, "gemm 48x256 split1"), ("v2", 130, 25024, 64, "gemm 80x256 split1"),
    ("v2", 164, 20736, 256, "gemm 96x256 split1"), ("v2", 263, 24768, 576, "gemm 96x512 split1"),
    ("v2", 386, 8448, 448, "gemm 112x256 split1"), ("v2", 323, 21888, 192, "gemm 112x512 split1"),
    ("bf16", 33, 16448, 2048, "gemm 48x256 split2 counter"), ("bf16", 68, 20544, 3072, "gemm 80x256 split3 second-launch"),
    ("bf16", 257, 12352, 320, "gemm 96x256 split1"), ("bf16", 282, 24704, 128, "gemm 96x512 split1"),
    ("bf16", 533, 6272, 448, "gemm 112x256 split1"), ("bf16", 322, 21696, 576, "gemm 112x512 split1"),
    ("fgq", 71, 20672, 320, "gemm 48x256 split1"), ("fgq", 33, 17344, 1536, "gemm 48x256 split3 counter"),
    ("fgq", 131, 25024, 192, "gemm 48x512 split1"),
]


def _plan(fmt, M, N, K, block, **kw):
    return P.fp6_linear_plan(M, N, K, format=FORMATS[fmt], block=block, **kw)


def _block(fmt, K):
    return (64 if K % 128 else 128) if fmt == "fgq" else 0


@pytest.mark.parametrize("fmt,M,N,K,text", CASES)
def test_the_rows_are_dealt_evenly(fmt, M, N, K, text):
    plan = _plan(fmt, M, N, K, _block(fmt, K))
    assert P.plan_text(plan).rsplit(" wg", 1)[0] == text
    blocks = -(-M // plan["block_m"])
    assert plan["block_m"] == -(-M // (16 * blocks)) * 16


def test_forced_heights_stay_as_they_are():
    for bm in (32, 64, 128):
        assert P.fp6_linear_plan(70, 4096, 4096, variant=B.FP6_VARIANT_GEMM | B.FP6_HINT_BLOCK_M(bm))["block_m"] == bm
    for bm in (48, 80, 96, 112):
        with pytest.raises(P.Fp6Error):
            P.fp6_linear_plan(70, 4096, 4096, variant=B.FP6_VARIANT_GEMM | B.FP6_HINT_BLOCK_M(bm))
    for dequant in (1, 2):             # the ablations exist for 32, 64 and 128 rows
        assert P.fp6_linear_plan(100, 8192, 8192, variant=B.FP6_HINT_DEQUANT(dequant))["block_m"] in (32, 64, 128)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source,kernels", [("fp6_gemm_heights.hip", 11), ("fp6_gemm_heights_v2.hip", 16),
                                            ("fp6_gemm_heights_fp5_fgq.hip", 10)])
def test_these_kernels_do_not_spill(source, kernels):
    sizes = {k: v for k, v in _scratch_sizes(source).items() if "gemm_kernel" in k}
    assert len(sizes) == kernels and all(v == 0 for v in sizes.values()), sizes


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,N,K,text", CASES)
def test_block_heights(fmt, M, N, K, text):
    block = _block(fmt, K)
    plan = _plan(fmt, M, N, K, block)
    W = inputs.weight(N, K, seed=8100 + M, sigma=0.02, outlier_frac=0.001, device=DEV)
    X = (inputs.activation_bf16 if fmt == "bf16" else inputs.activation)(M, K, seed=8200 + M, device=DEV)
    planes = (P.fp6_quantize_pack_fgq(W, block) if fmt == "fgq" else
              {"fp6": P.fp6_quantize_pack, "fp5": P.fp5_quantize_pack}.get(fmt, P.fp6_quantize_pack_v2)(W))
    fn = {"fp6": P.fp6_linear_variant, "fp5": P.fp5_linear, "v2": P.fp6_linear_v2, "bf16": P.fp6_linear_v2_bf16,
          "fgq": P.fp6_linear_fgq}[fmt]
    forced = (B.FP6_VARIANT_GEMM | B.FP6_HINT_BLOCK_M(128 if plan["block_m"] > 64 else 64) | B.FP6_HINT_WIDTH(plan["width"]) |
              (B.FP6_HINT_KWAYS(2) if plan["waves"] > plan["width"] else 0))
    wide = _plan(fmt, M, N, K, block, variant=forced, split_k=plan["split_k"])
    ws = P.new_workspace(max(plan["workspace_bytes"], wide["workspace_bytes"], 16), DEV)
    tail = (block,) if block else ()
    Y = [fn(X, *planes, N, K, *tail, workspace=ws), fn(X, *planes, N, K, *tail, workspace=ws),
         fn(X, *planes, N, K, *tail, forced, plan["split_k"], workspace=ws)]
    torch.cuda.synchronize()
    for y in Y[1:]:
        assert torch.equal(Y[0].view(torch.int16), y.view(torch.int16))
    if plan["split_k"] > 1:
        assert not ws[:B.FP6_WORKSPACE_ZERO_BYTES].any()
    # the oracle, on the first and last channels and some between
    pick = torch.cat([torch.arange(96), torch.arange(N - 96, N), torch.arange(100, N - 100, N // 200)])
    wb, xb = to_np16(W[pick.to(DEV)].contiguous()), X.cpu().view(torch.int16).numpy().view(np.uint16)
    y = Y[0].cpu()[:, pick]
    if fmt == "fgq":
        Yref = O.linear_fgq(xb, *O.quantize_fgq(wb, block), block)
    else:
        Yref = {"fp5": O.linear5, "bf16": O.linear_bf16}.get(fmt, O.linear)(xb, *(O.quantize5 if fmt == "fp5" else O.quantize)(wb))
    if fmt == "bf16":
        yd = y.double().numpy()               # half a unit in the last of 8 significant bits, and the fp32 sums
        assert (np.abs(yd - Yref) <= 2.0 ** -8 * np.abs(Yref) + 1e-4 * (np.abs(Yref) + np.sqrt(np.mean(Yref ** 2)))).all()
    else:
        assert_y_close(y, Yref, (fmt, M, N, K))
