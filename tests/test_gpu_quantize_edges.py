"""The offline step at the sizes where its kernels change: rows that just fit and just miss the rounds a workgroup keeps
in registers, more work items than workgroups, channel blocks that do not fill the dies, short scale blocks whose last
chunk of tiles is ragged.  Bit-exact against the oracle and the numpy statement of the layouts."""
import numpy as np
import pytest
import torch

import paper_2312_08583_amd as P
from oracle import fp6_oracle as O
from paper_2312_08583_amd import inputs

from gpu_util import from_np16, to_np16
from layout_ref import pack_planes, pack_planes5, pack_planes_v2

pytestmark = pytest.mark.gpu
DEV = "cuda"

FORMATS = {"fp6": (P.fp6_quantize_pack, O.quantize, pack_planes),
           "fp5": (P.fp5_quantize_pack, O.quantize5, pack_planes5),
           "v2": (P.fp6_quantize_pack_v2, O.quantize, pack_planes_v2)}


def _check(fmt, W):
    pack, quantize, planes = FORMATS[fmt]
    hi, lo, sc = pack(W)
    codes, scales = quantize(to_np16(W))
    hi_o, lo_o = planes(codes)
    assert np.array_equal(to_np16(sc), scales)
    assert np.array_equal(hi.cpu().numpy(), hi_o) and np.array_equal(lo.cpu().numpy(), lo_o)


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("N,K", [(64, 64), (64, 128), (128, 192), (64, 256), (64, 1024), (576, 1088), (64, 2048), (64, 2112),
                                 (64, 4096), (128, 4160), (64, 5632), (64, 5696), (64, 8192), (64, 8256), (64, 9216),
                                 (64, 9280), (64, 16384), (64, 16448), (64, 28672)])
def test_row_scales_at_the_edges_of_the_register_rounds(fmt, N, K):
    _check(fmt, inputs.weight(N, K, seed=7100 + K, sigma=0.02, outlier_frac=0.001, device=DEV))


@pytest.mark.parametrize("N,K", [(2112, 9280), (4160, 4160), (8256, 192)])
def test_more_work_items_than_workgroups(N, K):
    _check("fp6", inputs.weight(N, K, seed=7200 + K, sigma=0.02, outlier_frac=0.001, device=DEV))


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("N,K", [(64, 7168), (64, 7232), (1024, 7232), (1088, 7232), (1024, 28672), (1088, 8256), (1088, 9216),
                                 (1088, 9280), (1088, 16384), (1088, 16448), (64, 131136)])
def test_few_long_rows_and_just_too_many_of_them(fmt, N, K):
    # up to 16 channel blocks of more than 7168 columns: maxima and codes in two launches
    _check(fmt, inputs.weight(N, K, seed=7150 + N + K, sigma=0.02, outlier_frac=0.001, device=DEV))


@pytest.mark.parametrize("N,K,block", [(128, 32768, 8192), (192, 65536, 8192), (64, 65536, 65536)])
def test_few_long_fine_grained_blocks(N, K, block):
    W = inputs.weight(N, K, seed=7350 + N, sigma=0.02, outlier_frac=0.001, device=DEV)
    hi, lo, sc = P.fp6_quantize_pack_fgq(W, block)
    codes, scales = O.quantize_fgq(to_np16(W), block)
    hi_o, lo_o = pack_planes(codes)
    assert np.array_equal(to_np16(sc), scales.T)
    assert np.array_equal(hi.cpu().numpy(), hi_o) and np.array_equal(lo.cpu().numpy(), lo_o)


@pytest.mark.parametrize("block,K", [(64, 64), (64, 1088), (128, 2176), (256, 1280), (512, 1536), (1024, 3072), (2048, 4096)])
def test_fine_grained_blocks_and_ragged_chunks(block, K):
    N = 192
    W = inputs.weight(N, K, seed=7300 + K, sigma=0.02, outlier_frac=0.001, device=DEV)
    hi, lo, sc = P.fp6_quantize_pack_fgq(W, block)
    codes, scales = O.quantize_fgq(to_np16(W), block)
    hi_o, lo_o = pack_planes(codes)
    assert np.array_equal(to_np16(sc), scales.T)
    assert np.array_equal(hi.cpu().numpy(), hi_o) and np.array_equal(lo.cpu().numpy(), lo_o)


@pytest.mark.parametrize("fmt", sorted(FORMATS))
@pytest.mark.parametrize("amax_bits", [0x0001, 0x001B, 0x0029, 0x0280, 0x1234, 0x3555, 0x3C00, 0x7BFF])
def test_every_magnitude_up_to_amax(fmt, amax_bits):
    # both signs of every fp16 magnitude up to the row maximum (the smallest scales are fp16 subnormals of a few bits,
    # whose quotients saturate; scale 0 for the first): every rounding decision, ties included
    vals = np.arange(0, amax_bits + 1, dtype=np.uint16)
    K = 64 * ((2 * vals.size + 63) // 64)
    row = np.full(K, amax_bits, np.uint16)
    row[:vals.size] = vals
    row[vals.size:2 * vals.size] = vals | 0x8000
    _check(fmt, from_np16(np.tile(row, (64, 1))))
