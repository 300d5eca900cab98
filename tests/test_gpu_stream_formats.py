"""Streaming kernel at 17 to 32 rows for FP5 and plane layout 2: where the planner takes it, and the results against the oracle."""
import numpy as np
import pytest
import torch

import paper_2312_08583_amd as P
from oracle import fp6_oracle as O
from paper_2312_08583_amd import binding as B
from paper_2312_08583_amd import inputs

from gpu_util import assert_y_close, to_np16

DEV = "cuda"
FORMATS = {"fp5": 5, "v2": 7, "bf16": 8}


def _check(fmt, M, N, K):
    W = inputs.weight(N, K, seed=9600 + M, sigma=0.02, outlier_frac=0.001, device=DEV)
    X = (inputs.activation_bf16 if fmt == "bf16" else inputs.activation)(M, K, seed=9700 + M, device=DEV)
    planes = (P.fp5_quantize_pack if fmt == "fp5" else P.fp6_quantize_pack_v2)(W)
    fn = {"fp5": P.fp5_linear, "v2": P.fp6_linear_v2, "bf16": P.fp6_linear_v2_bf16}[fmt]
    Y = [fn(X, *planes, N, K), fn(X, *planes, N, K)]
    assert torch.equal(Y[0].view(torch.int16), Y[1].view(torch.int16))
    pick = torch.arange(N) if N <= 1100 else torch.cat([torch.arange(96), torch.arange(N - 96, N), torch.arange(100, N - 100, N // 200)])
    wb, xb = to_np16(W[pick.to(DEV)].contiguous()), X.cpu().view(torch.int16).numpy().view(np.uint16)
    Yref = {"fp5": O.linear5, "v2": O.linear, "bf16": O.linear_bf16}[fmt](xb, *(O.quantize5 if fmt == "fp5" else O.quantize)(wb))
    y = Y[0].cpu()[:, pick]
    if fmt == "bf16":
        yd = y.double().numpy()               # half a unit in the last of 8 significant bits, and the fp32 sums
        assert (np.abs(yd - Yref) <= 2.0 ** -8 * np.abs(Yref) + 1e-4 * (np.abs(Yref) + np.sqrt(np.mean(Yref ** 2)))).all()
    else:
        assert_y_close(y, Yref, (fmt, M, N, K))


@pytest.mark.parametrize("fmt", list(FORMATS))
def test_where_the_planner_takes_it(fmt):
    plan = lambda M, nblocks, ktiles, **kw: P.fp6_linear_plan(M, nblocks * 64, ktiles * 64, format=FORMATS[fmt], **kw)
    for M, nblocks, ktiles in [(17, 16, 16), (32, 112, 64), (24, 128, 56), (20, 160, 134), (32, 256, 84), (17, 400, 16)]:
        p = plan(M, nblocks, ktiles)
        assert (p["variant"], p["block_m"]) == (B.FP6_VARIANT_DECODE, 32)
    for M, nblocks, ktiles in [(33, 16, 16), (32, 112, 65), (24, 159, 134), (24, 257, 84), (32, 256, 85)]:
        assert plan(M, nblocks, ktiles)["variant"] == B.FP6_VARIANT_GEMM
    # more channel blocks than run the straight-code form of the stream, with up to six k tiles: 1.09 of the tiled kernel's time
    for M, nblocks, ktiles, takes in [(24, 256, 2, True), (24, 257, 6, False), (24, 257, 7, True), (24, 422, 4, False), (31, 448, 7, True)]:
        assert (plan(M, nblocks, ktiles)["variant"] == B.FP6_VARIANT_DECODE) == takes, (M, nblocks, ktiles)
    assert plan(24, 64, 64, split_k=2)["variant"] == B.FP6_VARIANT_GEMM            # forced splits stay with the tiled kernel
    with pytest.raises(P.Fp6Error):                                                # and forcing the kernel is refused as before
        plan(24, 64, 64, variant=B.FP6_VARIANT_DECODE)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,N,K", [(17, 192, 64), (32, 1088, 832), (25, 1024, 4096), (31, 10304, 1152), (18, 16448, 704), (24, 2752, 9344),
                                   (24, 5504, 5184)])          # (258 workgroups of 27 k tiles)
def test_two_blocks_of_rows(fmt, M, N, K):
    assert P.fp6_linear_plan(M, N, K, format=FORMATS[fmt])["variant"] == B.FP6_VARIANT_DECODE
    _check(fmt, M, N, K)


# k tiles of an unsplit layer: the short form up to 15 (every number of tiles to a wavefront), straight code above (every number of last tiles);
# with 257 workgroups always the short form, its steady state included (27: seven tiles and six)
@pytest.mark.gpu
@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("nblocks,ktiles", [(160, k) for k in (5, 12, 13, 15, 16, 17, 18, 23, 28, 33, 38, 43)] + [(257, 13), (257, 23), (257, 27)])
def test_every_number_of_tiles(fmt, nblocks, ktiles):
    M, N, K = 17 + ktiles % 16, nblocks * 64, ktiles * 64
    plan = P.fp6_linear_plan(M, N, K, format=FORMATS[fmt])
    assert (plan["variant"], plan["split_k"], plan["workgroups"]) == (B.FP6_VARIANT_DECODE, 1, nblocks)
    _check(fmt, M, N, K)
