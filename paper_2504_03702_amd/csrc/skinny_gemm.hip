// The per-request side maps of calls of at most 16 requests as launches of their own (see skinny_gemm.h).
#include "skinny_gemm.h"

namespace {

const int kSkinnyWaves = 8;

template <int EPI, bool GATHER, int G>
__global__ __launch_bounds__(kSkinnyWaves * 64) void skinny_gemm_kernel(SkinnyArgs p) {
    __shared__ __align__(16) unsigned char smem[kSkinnyLds];
    skinny_block<EPI, kSkinnyWaves, GATHER, G>(p, blockIdx.x, smem);
}

}  // namespace

// Requirements: at most 16 rows in use (A holds at least 16 rows, the unused ones finite), N % 64 == 0,
// K % 64 == 0 (both hold for every per-request map of a bf16 model: K is its hidden or feed-forward width).
// EPI_RESIDUAL_MAPPED takes A as [16][2K] (hi | lo) and leaves no pieces (res.pstats is null); EPI_GELU_SPLIT and
// EPI_Q_MAPPED read the stream rows of the requests' first tokens.
void launch_skinny_gemm_bf16(GemmEpilogue epi, const SkinnyArgs& p, hipStream_t s) {
    const dim3 grid((unsigned)(p.N / kSkinnyCols)), block(kSkinnyWaves * 64);
    switch (epi) {
        case EPI_GELU_SPLIT: hipLaunchKernelGGL((skinny_gemm_kernel<EPI_GELU_SPLIT, true, 2>), dim3((unsigned)(p.N / 32)), block, 0, s, p); break;
        case EPI_RESIDUAL_MAPPED:
            // No pieces of 64 columns to leave (the last layer), so 16 columns a block: what a unit can have on its way from
            // memory bounds this, and 48 units ask for more than 12 (one prompt, hidden 768: second feed-forward map 14.8 ->
            // 6.5 us, output projection 6.4 -> 4.2; the first feed-forward map, 96 blocks of 32, is no faster with 192).
            hipLaunchKernelGGL((skinny_gemm_kernel<EPI_RESIDUAL_MAPPED, false, 1>), dim3((unsigned)(p.N / 16)), block, 0, s, p);
            break;
        case EPI_Q_MAPPED: hipLaunchKernelGGL((skinny_gemm_kernel<EPI_Q_MAPPED, true, 4>), grid, block, 0, s, p); break;
        default: break;                                  // the other epilogues have no per-request form
    }
}
