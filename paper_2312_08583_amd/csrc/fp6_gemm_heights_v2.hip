// Tiled kernel: the block heights between the powers of two (48, 80, 96 and 112 rows), plane layout 2 against fp16 and bf16 activations.
#include "fp6_gemm_kernel.hpp"

namespace fp6 {

hipError_t launch_gemm_heights_v2(const LinearPlan& p, const uint16_t* X, int64_t M, const void* hi, const void* lo,
                               const uint16_t* scales, int64_t N, int64_t K, uint16_t* Y, void* workspace, hipStream_t stream)
{
    if (p.format == kE3M2B && p.gbn == 4) {
        switch (p.block_m) {
            case 48: return launch_gemm_t<48, kBiasShift, false, kE3M2B, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 80: return launch_gemm_t<80, kBiasShift, false, kE3M2B, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 96: return launch_gemm_t<96, kBiasShift, false, kE3M2B, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            default: return launch_gemm_t<112, kBiasShift, false, kE3M2B, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        }
    }
    if (p.format == kE3M2B) {
        switch (p.block_m) {
            case 48: return launch_gemm_t<48, kBiasShift, false, kE3M2B>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 80: return launch_gemm_t<80, kBiasShift, false, kE3M2B>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 96: return launch_gemm_t<96, kBiasShift, false, kE3M2B>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            default: return launch_gemm_t<112, kBiasShift, false, kE3M2B>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        }
    }
    if (p.gbn == 4) {
        switch (p.block_m) {
            case 48: return launch_gemm_t<48, kBiasShift, false, kE3M2H, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 80: return launch_gemm_t<80, kBiasShift, false, kE3M2H, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            case 96: return launch_gemm_t<96, kBiasShift, false, kE3M2H, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
            default: return launch_gemm_t<112, kBiasShift, false, kE3M2H, 4>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        }
    }
    switch (p.block_m) {
        case 48: return launch_gemm_t<48, kBiasShift, false, kE3M2H>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        case 80: return launch_gemm_t<80, kBiasShift, false, kE3M2H>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        case 96: return launch_gemm_t<96, kBiasShift, false, kE3M2H>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
        default: return launch_gemm_t<112, kBiasShift, false, kE3M2H>(p, X, M, hi, lo, scales, N, K, Y, workspace, stream);
    }
}

}  // namespace fp6
