"""Streaming kernel: the two forms of its stream (straight code for the last tiles, or one branch to each), on both sides of the lines
between them - slices of 12 k tiles and more (15 with two blocks of rows), 512 workgroups (256 with several blocks of rows) and more - and every number of last
tiles that a wavefront can be left with.  Against the oracle."""
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
# k tiles of a slice: four wavefronts with 3 tiles each (the short form) and with 3 to 11, so that each number of last tiles comes up
KTILES = [12, 13, 18, 23, 28, 33, 38, 43]


def _check(fmt, M, N, K, variant=B.FP6_VARIANT_DECODE, split=1):
    block = 64 if fmt == "fgq" else 0
    W = inputs.weight(N, K, seed=9100 + K, sigma=0.02, outlier_frac=0.001, device=DEV)
    X = (inputs.activation_bf16 if fmt == "bf16" else inputs.activation)(M, K, seed=9200 + M, device=DEV)
    planes = (P.fp6_quantize_pack_fgq(W, block) if fmt == "fgq" else
              {"fp6": P.fp6_quantize_pack, "fp5": P.fp5_quantize_pack}.get(fmt, P.fp6_quantize_pack_v2)(W))
    fn = {"fp6": P.fp6_linear_variant, "fp5": P.fp5_linear, "v2": P.fp6_linear_v2, "bf16": P.fp6_linear_v2_bf16,
          "fgq": P.fp6_linear_fgq}[fmt]
    Y = fn(X, *planes, N, K, *((block,) if block else ()), variant, split)
    pick = torch.arange(N) if N <= 1024 else torch.cat([torch.arange(96), torch.arange(N - 96, N), torch.arange(100, N - 100, N // 100)])
    wb, xb = to_np16(W[pick.to(DEV)].contiguous()), X.cpu().view(torch.int16).numpy().view(np.uint16)
    y = Y.cpu()[:, pick]
    if fmt == "fgq":
        Yref = O.linear_fgq(xb, *O.quantize_fgq(wb, block), block)
    else:
        Yref = {"fp5": O.linear5, "bf16": O.linear_bf16}.get(fmt, O.linear)(xb, *(O.quantize5 if fmt == "fp5" else O.quantize)(wb))
    if fmt == "bf16":
        yd = y.double().numpy()               # half a unit in the last of 8 significant bits, and the fp32 sums
        assert (np.abs(yd - Yref) <= 2.0 ** -8 * np.abs(Yref) + 1e-4 * (np.abs(Yref) + np.sqrt(np.mean(Yref ** 2)))).all()
    else:
        assert_y_close(y, Yref, (fmt, M, N, K, split))


@pytest.mark.parametrize("fmt,M", [("fp6", 1), ("fp6", 16), ("fp6", 17), ("fp6", 32), ("fp6", 33), ("fp6", 64), ("fp5", 3), ("fp5", 9),
                                   ("v2", 2), ("bf16", 16), ("fgq", 7)])
@pytest.mark.parametrize("ktiles", KTILES)
def test_every_number_of_last_tiles(fmt, M, ktiles):
    _check(fmt, M, 192, ktiles * 64)


@pytest.mark.parametrize("fmt,M,N", [("fp6", 5, 512 * 64), ("fp6", 5, 513 * 64), ("bf16", 4, 513 * 64), ("fgq", 9, 513 * 64),
                                     ("fp5", 16, 513 * 64), ("fp6", 24, 256 * 64), ("fp6", 24, 257 * 64), ("fp6", 50, 257 * 64)])
def test_as_many_workgroups_as_fit_and_one_more(fmt, M, N):
    _check(fmt, M, N, 13 * 64)


@pytest.mark.parametrize("nblocks,ktiles", [(3, 15), (3, 16), (3, 17), (256, 16), (257, 16)])
def test_two_blocks_of_rows_on_both_sides_of_their_lines(nblocks, ktiles):
    _check("fp6", 25, nblocks * 64, ktiles * 64)


@pytest.mark.parametrize("dequant", [1, 2])
@pytest.mark.parametrize("ktiles", KTILES)
def test_the_ablations_run_the_forms_of_the_method(dequant, ktiles):
    """The same products times powers of two in the same order: bit for bit the method's results."""
    M, N, K = 8, 192, ktiles * 64
    W, X = inputs.weight(N, K, seed=9100 + K, sigma=0.02, outlier_frac=0.001, device=DEV), inputs.activation(M, K, seed=9200 + M, device=DEV)
    planes = P.fp6_quantize_pack(W)
    Y = [P.fp6_linear_variant(X, *planes, N, K, B.FP6_VARIANT_DECODE | hint, 1) for hint in (0, B.FP6_HINT_DEQUANT(dequant))]
    assert torch.equal(*Y)


@pytest.mark.parametrize("ktiles,split", [(12, 2), (26, 2), (52, 4), (39, 3)])
def test_slices(ktiles, split):
    _check("fp6", 12, 320, ktiles * 64, split=split)
    _check("fp6", 30, 320, ktiles * 64, split=split)


@pytest.mark.parametrize("half", [1, 2])
@pytest.mark.parametrize("ktiles", KTILES)
def test_half_tiles(half, ktiles):
    for fmt in ("fp6", "fp5"):
        _check(fmt, 4, 192, ktiles * 64, B.FP6_VARIANT_DECODE | B.FP6_HINT_HALF(half))


@pytest.mark.parametrize("Ns,ktiles", [((128, 64, 192), 12), ((128, 64, 192), 13), ((256 * 64, 257 * 64), 13)])
def test_group(Ns, ktiles):
    M, K = 6, ktiles * 64
    layers, refs = [], []
    for i, N in enumerate(Ns):
        W = inputs.weight(N, K, seed=9300 + i, sigma=0.02, outlier_frac=0.001, device=DEV)
        X = inputs.activation(M, K, seed=9400 + i, device=DEV)
        layers.append((X, *P.fp6_quantize_pack(W), N, K))
        refs.append(O.linear(to_np16(X), *O.quantize(to_np16(W[:192].contiguous()))))
    for Y, ref in zip(P.fp6_linear_group(layers), refs):
        assert_y_close(Y.cpu()[:, :192], ref, (Ns, ktiles))
