// Tiled kernel: dispatch, and the instantiations of the method itself (FP6, bias-shift unpack, row scales).
#include "fp6_gemm_kernel.hpp"

namespace fp6 {

hipError_t launch_gemm(const LinearPlan& p, const uint16_t* X, int64_t M, const void* hi, const void* lo,
                       const uint16_t* scales, int64_t N, int64_t K, uint16_t* Y, void* workspace,
                       hipStream_t stream)
{
    if (p.block_m & (p.block_m - 1)) return launch_gemm_heights(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    if (p.format != kE3M2 || p.gshift >= 0 || p.dequant != kBiasShift)
        return launch_gemm_variant(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    if (p.gbn == 4 && p.kw == 2)
        return launch_gemm_t<128, kBiasShift, false, kE3M2, 4, 2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    if (p.gbn == 4) {
        switch (p.block_m) {
            case 32: return launch_gemm_t<32, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 64: return launch_gemm_t<64, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            default: return launch_gemm_t<128, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        }
    }
    switch (p.block_m) {
        case 32: return launch_gemm_t<32>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        case 64: return launch_gemm_t<64>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        default: return launch_gemm_t<128>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    }
}

}  // namespace fp6
