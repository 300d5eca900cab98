"""K-slices of different lengths: K/64 that the planner's split does not divide, in both kernel families and every format.
On the GPU against the oracle, with the planner's workspace and with one that only the even split fits; in groups and on
the static scratch."""
import numpy as np
import pytest
import torch

import paper_2312_08583_amd as P
from oracle import fp6_oracle as O
from paper_2312_08583_amd import binding as B
from paper_2312_08583_amd import inputs

from gpu_util import assert_y_close, oracle_reference, to_np16

DEV = "cuda"
FORMATS = {"fp6": 6, "fp5": 5, "v2": 7, "bf16": 8, "fgq": 6}
# (format, M, N, K); the last five of this list: streaming kernel
SHAPES = [("fp6", 79, 2752, 9344), ("fp6", 130, 1152, 73 * 64), ("fp6", 333, 1024, 202 * 64), ("fp5", 70, 1152, 67 * 64),
          ("v2", 200, 1152, 79 * 64), ("bf16", 333, 1152, 94 * 64), ("fgq", 66, 1152, 106 * 64),
          ("fp6", 1, 1088, 101 * 64), ("fp6", 16, 1088, 131 * 64), ("fp6", 40, 1088, 131 * 64), ("fp5", 3, 1088, 101 * 64),
          ("fgq", 5, 1088, 202 * 64)]
# here the even slices need more workspace than the uneven ones (in the others less, or none)
EVEN_NEEDS_MORE = [("fp6", 66, 2112, 2112), ("fp6", 17, 1024, 10816)]
SHAPES += EVEN_NEEDS_MORE


def _plan(fmt, M, N, K, **kw):
    return P.fp6_linear_plan(M, N, K, format=FORMATS[fmt], block=128 if fmt == "fgq" else 0, **kw)


@pytest.mark.parametrize("fmt,M,N,K", SHAPES)
def test_the_planner_splits_these_unevenly(fmt, M, N, K):
    plan = _plan(fmt, M, N, K)
    assert (K // 64) % plan["split_k"] != 0, P.plan_text(plan)
    with pytest.raises(P.Fp6Error):               # a forced split still has to divide K/64
        _plan(fmt, M, N, K, split_k=plan["split_k"])


# uneven slices would save little or nothing here (measured, even / uneven: 8.2 / 11.4 us, 9.9 / 13.5, 10.8 / 14.4, 18.2 / 24.3,
# 10.2 / 11.2; streaming kernel 5.7 / 6.3, 4.8 / 5.0, 7.2 / 7.8, 13.4 / 15.2, 13.2 / 14.5, 6.7 / 7.4)
@pytest.mark.parametrize("fmt,M,N,K", [("bf16", 483, 576, 1088), ("v2", 64, 4672, 1728), ("fp6", 269, 1024, 1728),
                                       ("fp5", 244, 3136, 3712), ("fp6", 324, 576, 1088), ("fp6", 2, 2496, 3904),
                                       ("fp6", 1, 1088, 2944), ("fp6", 20, 4352, 1984), ("fp6", 1, 8320, 9344),
                                       ("fp6", 3, 8768, 8384), ("fp5", 1, 4608, 5056)])
def test_the_planner_leaves_these_even(fmt, M, N, K):
    assert (K // 64) % _plan(fmt, M, N, K)["split_k"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,N,K", SHAPES)
def test_uneven_slices(fmt, M, N, K):
    block = 128
    W = inputs.weight(N, K, seed=7100 + M, sigma=0.02, outlier_frac=0.001, device=DEV)
    X = (inputs.activation_bf16 if fmt == "bf16" else inputs.activation)(M, K, seed=7200 + M, device=DEV)
    xb, wb = X.cpu().view(torch.int16).numpy().view(np.uint16), to_np16(W)
    if fmt == "fgq":
        codes, scales = O.quantize_fgq(wb, block)
        planes, Yref = P.fp6_quantize_pack_fgq(W, block), O.linear_fgq(xb, codes, scales, block)
        call = lambda ws: P.fp6_linear_fgq(X, *planes, N, K, block, workspace=ws)
    else:
        codes, scales = (O.quantize5 if fmt == "fp5" else O.quantize)(wb)
        planes = {"fp6": P.fp6_quantize_pack, "fp5": P.fp5_quantize_pack}.get(fmt, P.fp6_quantize_pack_v2)(W)
        Yref = {"fp5": O.linear5, "bf16": O.linear_bf16}.get(fmt, O.linear)(xb, codes, scales)
        fn = {"fp6": P.fp6_linear, "fp5": P.fp5_linear, "v2": P.fp6_linear_v2, "bf16": P.fp6_linear_v2_bf16}[fmt]
        call = lambda ws: fn(X, *planes, N, K, workspace=ws)
    need = _plan(fmt, M, N, K)["workspace_bytes"]
    ws, short = P.new_workspace(need, DEV), P.new_workspace(need - 16, DEV)
    Y = [call(ws), call(ws)]
    assert not ws[:B.FP6_WORKSPACE_ZERO_BYTES].any()
    if (fmt, M, N, K) in EVEN_NEEDS_MORE:
        with pytest.raises(P.Fp6Error, match="workspace missing or too small"):
            call(short)
    else:
        Y.append(call(short))                     # the even split
    torch.cuda.synchronize()
    assert torch.equal(Y[0], Y[1])
    for y in Y:
        if fmt == "bf16":
            yd = y.cpu().double().numpy()         # half a unit in the last of 8 significant bits, and the fp32 sums
            assert (np.abs(yd - Yref) <= 2.0 ** -8 * np.abs(Yref) + 1e-4 * (np.abs(Yref) + np.sqrt(np.mean(Yref ** 2)))).all()
        else:
            assert_y_close(y, Yref, (fmt, M, N, K))


def _fp6_layers(M, shapes, seed):
    made = []
    for i, (N, K) in enumerate(shapes):
        W = inputs.weight(N, K, seed=seed + i, sigma=0.02, outlier_frac=0.001, device=DEV)
        X = inputs.activation(M, K, seed=seed + 50 + i, device=DEV)
        made.append(((X,) + tuple(P.fp6_quantize_pack(W)) + (N, K), oracle_reference(W, X)[2]))
    return [layer for layer, _ in made], [Yref for _, Yref in made]


# groups: one launch over the summed N; in sequence at more than 16 rows (even slices need more workspace than the
# uneven ones there); in sequence with different K
GROUPS = [(2, [(576, 101 * 64), (512, 101 * 64)]), (17, [(1024, 10816), (1024, 10816)]), (2, [(1088, 101 * 64), (1088, 131 * 64)])]


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", GROUPS)
def test_groups_of_uneven_layers(M, shapes):
    shared = M <= 16 and len({K for _, K in shapes}) == 1
    for N, K in [(sum(N for N, _ in shapes), shapes[0][1])] if shared else shapes:
        assert (K // 64) % P.fp6_linear_plan(M, N, K)["split_k"] != 0
    layers, Yrefs = _fp6_layers(M, shapes, seed=7300 + M)
    need = P.fp6_linear_group_workspace_bytes(M, shapes)
    ws = P.new_workspace(need, DEV)
    for _ in range(2):
        ys = P.fp6_linear_group(layers, workspace=ws)
        for Y, Yref in zip(ys, Yrefs):
            assert_y_close(Y, Yref, (M, shapes))
        assert not ws[:B.FP6_WORKSPACE_ZERO_BYTES].any()
    for Y, Z in zip(ys, P.fp6_linear_group(layers)):           # the wrapper allocates what the query reports
        assert torch.equal(Y, Z)
    if not shared:
        for layer, Y in zip(layers, ys):
            assert torch.equal(Y, P.fp6_linear(*layer))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(17, 1024, 10816), (2, 1088, 101 * 64)])
def test_uneven_slices_on_the_static_scratch(M, N, K):
    assert (K // 64) % P.fp6_linear_plan(M, N, K)["split_k"] != 0
    (layer,), (Yref,) = _fp6_layers(M, [(N, K)], seed=7400 + M)
    for _ in range(2):
        Y = P.fp6_linear_static(*layer)
        assert_y_close(Y, Yref, (M, N, K))
    assert torch.equal(Y, P.fp6_linear(*layer))


@pytest.mark.gpu
def test_equal_slices_where_uneven_ones_exceed_the_static_scratch():
    M, N, K = 2020, 2176, 6464
    assert P.fp6_linear_workspace_bytes(M, N, K) > P.FP6_STATIC_SCRATCH_BYTES
    assert (K // 64) % P.fp6_linear_plan(M, N, K)["split_k"] != 0
    W = inputs.weight(N, K, seed=7500, sigma=0.02, outlier_frac=0.001, device=DEV)
    X = inputs.activation(M, K, seed=7501, device=DEV)
    planes = P.fp6_quantize_pack(W)
    Y = P.fp6_linear_static(X, *planes, N, K)
    assert torch.equal(Y, P.fp6_linear(X, *planes, N, K, workspace=P.new_workspace(P.FP6_STATIC_SCRATCH_BYTES, DEV)))
    rows = [0, 127, 128, 1000, M - 1]          # a row of Y depends on its row of X only
    _, _, Yref = oracle_reference(W, X[rows])
    assert_y_close(Y[rows], Yref, (M, N, K))
    assert_y_close(P.fp6_linear(X, *planes, N, K)[rows], Yref, (M, N, K))


@pytest.mark.gpu
@pytest.mark.parametrize("dequant", [1, 2])
@pytest.mark.parametrize("M,N,K", [(8, 1088, 101 * 64), (130, 1152, 73 * 64)])
def test_ablations_on_uneven_slices(M, N, K, dequant):
    variant = B.FP6_HINT_DEQUANT(dequant)
    assert (K // 64) % P.fp6_linear_plan(M, N, K, variant=variant)["split_k"] != 0
    (layer,), (Yref,) = _fp6_layers(M, [(N, K)], seed=7600 + M)
    X, hi, lo, sc, N, K = layer
    assert_y_close(P.fp6_linear_variant(X, hi, lo, sc, N, K, variant), Yref, (M, N, K, dequant))
