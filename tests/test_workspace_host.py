"""What a call accepts as workspace, on the host (CPU only).

The C ABI is linked with launchers that launch nothing and keep the plan they were given, so every decision up to the
launch is the library's own and no pointer is ever used.  For single layers and for groups: the size that the query
reports is accepted, also where that plan's slices are uneven and the even ones would need more; so is what the even
slices need; less than both is refused before anything is launched; and the plan that would run fits what was given."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_2312_08583_amd import binding as B
from paper_2312_08583_amd import build as hip_build

STUBS = r"""
#include "fp6_internal.hpp"
namespace fp6 {
static long launches, used;          // since the last take_*: launches, and the largest workspace of their plans
static hipError_t keep(const LinearPlan& p)
{
    const long need = p.split_k > 1 ? (long)(kZeroBytes + p.partial_bytes) : 0;
    launches++;
    used = need > used ? need : used;
    return hipSuccess;
}
hipError_t launch_quantize_pack(int, const uint16_t*, int64_t, int64_t, int64_t, void*, void*, uint16_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_unpack_codes(int, const void*, const void*, int64_t, int64_t, uint8_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_dequantize(int, const void*, const void*, const uint16_t*, int64_t, int64_t, int64_t, uint16_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_decode_group(const LinearPlan& p, int, const GroupLayer*, int64_t, int64_t, void*, hipStream_t) { return keep(p); }
hipError_t launch_decode(const LinearPlan& p, const uint16_t*, int64_t, const void*, const void*, const uint16_t*, int64_t, int64_t,
                         uint16_t*, void*, hipStream_t) { return keep(p); }
hipError_t launch_gemm(const LinearPlan& p, const uint16_t*, int64_t, const void*, const void*, const uint16_t*, int64_t, int64_t,
                       uint16_t*, void*, hipStream_t) { return keep(p); }
}  // namespace fp6
extern "C" long take_launches(void) { const long n = fp6::launches; fp6::launches = 0; return n; }
extern "C" long take_used(void) { const long n = fp6::used; fp6::used = 0; return n; }
// workspace of the automatic plan, even slices only
extern "C" long even_need(int format, int64_t M, int64_t N, int64_t K, int64_t block)
{
    fp6::LinearPlan p;
    if (!fp6::make_plan(format, M, N, K, block, 0, 0, &p, true)) return -1;
    return p.split_k > 1 ? (long)(fp6::kZeroBytes + p.partial_bytes) : 0;
}
"""


@pytest.fixture(scope="module")
def abi(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    tmp = tmp_path_factory.mktemp("abi")
    stubs, lib = str(tmp / "stubs.hip"), str(tmp / "libabi_stubs.so")
    with open(stubs, "w") as f:
        f.write(STUBS)
    subprocess.run(["hipcc", *hip_build.FLAGS, "-I", hip_build.CSRC, "-shared", "-o", lib,
                    os.path.join(hip_build.CSRC, "fp6_abi.hip"), stubs], check=True, capture_output=True)
    L = ctypes.CDLL(lib)
    for name in ("fp6_linear", "fp5_linear", "fp6_linear_v2", "fp6_linear_fgq", "fp6_linear_workspace_bytes",
                 "fp5_linear_workspace_bytes", "fp6_linear_v2_workspace_bytes", "fp6_linear_fgq_workspace_bytes",
                 "fp6_linear_group", "fp6_linear_group_workspace_bytes"):
        getattr(L, name).restype, getattr(L, name).argtypes = getattr(B.lib(), name).restype, getattr(B.lib(), name).argtypes
    L.take_launches.restype = L.take_used.restype = L.even_need.restype = ctypes.c_long
    L.even_need.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 4
    L.take_launches(), L.take_used()
    return L


A = 16          # an aligned address that nothing uses


def _group(L, M, shapes, nbytes):
    arr = (B.LinearProblem * len(shapes))(*[B.LinearProblem(A, A, A, A, N, K, A) for N, K in shapes])
    return L.fp6_linear_group(M, arr, len(shapes), A if nbytes else None, nbytes, None)


def _check(L, call, need, even, least, launches, what):
    """call(bytes) -> status: accepted from `least` on, and the plan that runs fits what was given."""
    assert L.take_launches() == 0
    for nbytes in {need, even, least, need + 16, even + 16}:
        assert call(nbytes) == 0, (what, nbytes, need, even)
        assert L.take_launches() == launches and L.take_used() <= nbytes, (what, nbytes, need, even)
    for nbytes in {0, B.FP6_WORKSPACE_ZERO_BYTES, least - 1} if least else {}:
        if nbytes < least:
            assert call(nbytes) == -4 and L.take_launches() == 0, (what, nbytes, need, even)


def _layer(rng, lo=1024):
    N = 64 * rng.randint(lo // 64, 28672 // 64)
    return N, 64 * rng.randint(lo // 64, min(28672, 28672 * 8192 // N) // 64)


def test_single_layers(abi):
    rng = random.Random(1)
    uneven_larger = uneven_smaller = 0
    for _ in range(3000):
        fmt = rng.choice(["fp6", "fp5", "v2", "fgq"])
        M = int(2 ** rng.uniform(0, 11))
        N, K = _layer(rng, 256)
        block = 0
        if fmt == "fgq":
            block, K = 128, max(128, K // 128 * 128)
        need = {"fp6": lambda: abi.fp6_linear_workspace_bytes(M, N, K), "fp5": lambda: abi.fp5_linear_workspace_bytes(M, N, K, 0, 0),
                "v2": lambda: abi.fp6_linear_v2_workspace_bytes(M, N, K, 0, 0),
                "fgq": lambda: abi.fp6_linear_fgq_workspace_bytes(M, N, K, block, 0, 0)}[fmt]()
        even = abi.even_need({"fp5": 5, "v2": 7}.get(fmt, 6), M, N, K, block)
        call = {"fp6": lambda b: abi.fp6_linear(A, M, A, A, A, N, K, A, A if b else None, b, None),
                "fp5": lambda b: abi.fp5_linear(A, M, A, A, A, N, K, A, A if b else None, b, None, 0, 0),
                "v2": lambda b: abi.fp6_linear_v2(A, M, A, A, A, N, K, A, A if b else None, b, None, 0, 0),
                "fgq": lambda b: abi.fp6_linear_fgq(A, M, A, A, A, N, K, block, A, A if b else None, b, None, 0, 0)}[fmt]
        _check(abi, call, need, even, min(need, even), 1, (fmt, M, N, K))
        uneven_larger += need > even
        uneven_smaller += need < even
    assert uneven_larger > 20 and uneven_smaller > 20, (uneven_larger, uneven_smaller)


def test_groups(abi):
    rng = random.Random(2)
    known = [(40, [(5184, 5184)] * 3), (66, [(2112, 2112)] * 3), (97, [(10112, 4480)] * 2), (176, [(8704, 4032)] * 2),
             (17, [(1024, 10816)] * 2)]
    drawn = []
    for _ in range(3000):
        N, K = _layer(rng)
        same = rng.random() < 0.7
        drawn.append((int(2 ** rng.uniform(0, 11)), [(N if rng.random() < 0.5 else 64 * rng.randint(16, 200),
                                                      K if same else 64 * rng.randint(16, 200)) for _ in range(rng.randint(1, 4))]))
    larger = smaller = 0
    for M, shapes in known + drawn:
        arr = (B.LinearProblem * len(shapes))(*[B.LinearProblem(A, A, A, A, N, K, A) for N, K in shapes])
        need = abi.fp6_linear_group_workspace_bytes(M, arr, len(shapes))
        shared = len(shapes) > 1 and M <= 16 and len({K for _, K in shapes}) == 1
        singles = [(sum(N for N, _ in shapes), shapes[0][1])] if shared else shapes
        even = max(abi.even_need(6, M, N, K, 0) for N, K in singles)
        # in sequence, each layer takes whichever of its two plans fits
        fits = max(min(abi.even_need(6, M, N, K, 0), abi.fp6_linear_workspace_bytes(M, N, K)) for N, K in singles)
        _check(abi, lambda b: _group(abi, M, shapes, b), need, even, fits, 1 if shared else len(shapes), (M, shapes))
        larger += need > even
        smaller += need < even
    assert larger > 20 and smaller > 20, (larger, smaller)
