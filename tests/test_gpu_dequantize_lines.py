"""Dequantize: every code at every place of a tile, numbers of tiles that fill no workgroup, every format: bit for bit S * value(code),
whose only rounding is the conversion to fp16."""
import pytest
import torch

import paper_2312_08583_amd as P
from paper_2312_08583_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("fmt", ["fp6", "fp5", "v2", "fgq"])
@pytest.mark.parametrize("N,K", [(64, 64), (64, 192), (320, 64), (192, 1088), (128, 2048)])
def test_dequantize(fmt, N, K):
    g = torch.Generator(device=DEV).manual_seed(N + K)
    hi = torch.randint(0, 256, (N * K // 2,), dtype=torch.uint8, device=DEV, generator=g)
    lo = torch.randint(0, 256, (N * K // (8 if fmt == "fp5" else 4),), dtype=torch.uint8, device=DEV, generator=g)
    block = 64 if fmt == "fgq" else K
    scales = (torch.rand(K // block, N, device=DEV, generator=g) * 0.1).half()
    scales[0, 0], scales[0, -1] = 65504.0, 6e-8                        # results that overflow fp16, and that fall below it
    sc = scales if fmt == "fgq" else scales[0].contiguous()
    codes = {"fp5": B.fp5_unpack_codes, "v2": B.fp6_unpack_codes_v2}.get(fmt, B.fp6_unpack_codes)(hi, lo, N, K).long()
    W = (B.fp6_dequantize_fgq(hi, lo, sc, N, K, block) if fmt == "fgq" else
         {"fp6": B.fp6_dequantize, "fp5": B.fp5_dequantize, "v2": B.fp6_dequantize_v2}[fmt](hi, lo, sc, N, K))
    mb = 1 if fmt == "fp5" else 2
    ex, m = (codes >> mb) & 7, (codes & ((1 << mb) - 1)).double() / (1 << mb)
    value = torch.where(ex > 0, (1 + m) * torch.pow(2.0, ex.double() - 3), m * 0.25)
    value = torch.where((codes >> (3 + mb)) > 0, -value, value)
    ref = (scales.double().repeat_interleave(block, 0).t() * value).float().half()      # (exact in fp32)
    assert torch.equal(W.view(torch.int16), ref.view(torch.int16))
