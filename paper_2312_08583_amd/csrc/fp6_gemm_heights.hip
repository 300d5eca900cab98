// Tiled kernel: the block heights between the powers of two (48, 80, 96 and 112 rows), FP6 in plane layout 1.
#include "fp6_gemm_kernel.hpp"

namespace fp6 {

hipError_t launch_gemm_heights(const LinearPlan& p, const uint16_t* X, int64_t M, const void* hi, const void* lo,
                               const uint16_t* scales, int64_t N, int64_t K, uint16_t* Y, void* workspace, hipStream_t stream)
{
    if (layout2(p.format)) return launch_gemm_heights_v2(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    if (p.format == kE3M1 || p.gshift >= 0) return launch_gemm_heights_fp5_fgq(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    // Rings of three stages up to 80 KB where two workgroups share a compute unit (against two stages 2 to 7 % faster at 80 to 112
    // rows; a fourth at 48 rows is 1 % slower), of three stages with eight wavefronts and of two with two K-ways (one more: no gain).
    if (p.kw == 2) {
        switch (p.block_m) {
            case 80: return launch_gemm_t<80, 2, kBiasShift, false, kE3M2, 4, 2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 96: return launch_gemm_t<96, 2, kBiasShift, false, kE3M2, 4, 2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            default: return launch_gemm_t<112, 2, kBiasShift, false, kE3M2, 4, 2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        }
    }
    if (p.gbn == 4) {
        switch (p.block_m) {
            case 48: return launch_gemm_t<48, 3, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 80: return launch_gemm_t<80, 3, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 96: return launch_gemm_t<96, 3, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            default: return launch_gemm_t<112, 3, kBiasShift, false, kE3M2, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        }
    }
    switch (p.block_m) {
        case 48: return launch_gemm_t<48, 4, kBiasShift, false, kE3M2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        case 80: return launch_gemm_t<80, 3, kBiasShift, false, kE3M2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        case 96: return launch_gemm_t<96, 3, kBiasShift, false, kE3M2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        default: return launch_gemm_t<112, 3, kBiasShift, false, kE3M2>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    }
}

}  // namespace fp6
