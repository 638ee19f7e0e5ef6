// bf16 maps of calls with few activation rows, and the per-request maps of calls with many requests.
//
// Such a map has too few 128 x 128 or 256 x 256 tiles to fill the chip, and a tile's time is the latency of its
// slices one after the other: at 1200 rows of hidden 768 the 128 x 128 kernel took 0.75 us a 64-deep slice, 36 us for
// the second feed-forward map.  Here a workgroup (four wavefronts, 2 x 2) owns one tile of 64 x 64 to 128 x 128 and keeps
// STAGES - 1 slices on their way to LDS (global_load_lds), so a slice costs its share of the unit's LDS and L2 rate and
// not a trip to memory; a wavefront reads the fragments of the next slice while its MFMAs of the current one run.  The
// accumulation order over k is that of the larger tiles and the epilogues are the same expressions, so the results are
// equal to theirs to the last bit and the choice between the kernels is free.  (Of hi | lo rows, below, both form the two
// parts' sums apart and add them; one chain over 2K would differ in the last digits.)
//
// Per-request maps of 64 requests (hidden 768 / 3072, hi | lo rows): 76 us a launch on the 128 x 128 tiles, 10.7 here.
//
// A launch can carry the layer's per-request side map (skinny_gemm.h) in further workgroups, and makes the row
// statistics of its operand from the 64-column pieces in its prologue: with few rows a layer's time is made of
// launches, and this leaves five of ten.
#include "skinny_gemm.h"
#include "small_gemm.h"

namespace {

constexpr int kNoSide = -1;
constexpr int kSideGroups = kSkinnyCols / 16;

// G: groups of 16 columns of a block of the side map
template <int EPI, int TM, int TN, int STAGES, int SIDE, int G>
__global__ __launch_bounds__(256, TM == 2 && TN == 1 ? 2 : 1) void small_gemm_kernel(SmallGemm p, SkinnyArgs side, int side_blocks) {
    constexpr int kBytes = STAGES * 64 * (TM + TN) * 128;
    static_assert(SIDE == kNoSide || kBytes >= kSkinnyLds, "LDS regions");
    __shared__ __align__(1024) unsigned char smem[kBytes];
    __shared__ float2 s_st[64 * TM];
    if (SIDE != kNoSide) {
        if ((int)blockIdx.x < side_blocks) {
            if ((int)blockIdx.x * 16 * G < side.N)
                skinny_block<SIDE, 4, SIDE != EPI_RESIDUAL_MAPPED, G>(side, blockIdx.x, smem);
            return;
        }
    }
    small_tile<EPI, TM, TN, STAGES>(p, blockIdx.x - side_blocks, smem, s_st);
}

template <int EPI, int SIDE>
void launch(const SmallGemm& p, const SkinnyArgs* side, hipStream_t s) {
    const SkinnyArgs sd = SIDE != kNoSide ? *side : SkinnyArgs{};
    constexpr int kParts = EPI == EPI_GELU_SPLIT || EPI == EPI_RESIDUAL_MAPPED ? 2 : 1;   // rows of the tile per row of the result
    auto tiles_of = [&](int64_t rows, int bm, int bn) { return (rows * kParts + bm - 1) / bm * (p.N / bn); };
    auto tiles = [&](int bm, int bn) { return tiles_of(p.likely_rows ? p.likely_rows : p.max_rows, bm, bn); };
    const int64_t usual = p.usual_rows ? p.usual_rows : p.max_rows;
    auto blocks = [&](int groups) { return SIDE != kNoSide ? (int)align_up((size_t)(sd.N / (16 * groups)), 8) : 0; };
    auto grid = [&](int bm, int bn, int groups) {
        return dim3((unsigned)(blocks(groups) + (tiles_of(p.max_rows, bm, bn) + 7) / 8 * 8));
    };
#define PS_SMALL(TM, TN, STAGES, G) \
    hipLaunchKernelGGL((small_gemm_kernel<EPI, TM, TN, STAGES, SIDE, G>), grid(64 * TM, 64 * TN, G), dim3(256), 0, s, p, sd, blocks(G))
    // Blocks of 32 columns for the first feed-forward map's side map: half the loads a block, where the launch waits for
    // those blocks, that is while they and the tiles have places at the same time (one prompt of hidden 768, 192 + 48
    // places of 512, 342 -> 326 us a call, 5 of 432 + 48 410 -> 396; 6 of 480 + 48 take 421, with 32 columns 435; 3 padded to 512, half of 528 + 48, 765 -> 744).
    constexpr int kFine = SIDE == EPI_GELU_SPLIT ? 2 : kSideGroups;
    // At most one 64 x 64 tile per compute unit: a unit to itself, seven slices on their way.  Beyond that what the unit
    // reads from LDS and L2 per product counts: 128 x 64 tiles, two to a unit (1536 rows of hidden 768, the query-key-value
    // map, 468 tiles for 512 places, 18.5 -> 16.0 us, the second feed-forward map 31.7 -> 26.0; where the tiles just pass the
    // places, 540 at 1782 rows, the second wave shows: 22 us).  The maps back to the hidden width have few columns
    // and a long contraction: 128 x 128 with three slices on their way once that still gives every other unit a tile
    // (1922 rows of hidden 1024: 54.5 -> 44.5 us).
    constexpr bool kResid = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_RESIDUAL_MAPPED;
    if (tiles(64, 64) <= 256) {
        PS_SMALL(1, 1, 8, kFine);
        return;
    }
    if constexpr (kResid) {
        if (tiles(128, 128) >= 128) {
            PS_SMALL(2, 2, 4, kSideGroups);
            return;
        }
    }
    if constexpr (kFine != kSideGroups) {
        if (tiles_of(usual, 128, 64) + blocks(kSideGroups) <= 512) {
            PS_SMALL(2, 1, 3, kFine);
            return;
        }
    }
    PS_SMALL(2, 1, 3, kSideGroups);
#undef PS_SMALL
}

}  // namespace

// Requirements: N % 64 == 0, K % 128 == 0; every buffer holds max_rows rows with max_rows % 64 == 0 (whole tiles are
// in bounds).  EPI_GELU_SPLIT and EPI_RESIDUAL_MAPPED take A as [rows][2K] (hi | lo).  Three maps come with a side map:
// EPI_BIAS_RESIDUAL with EPI_RESIDUAL_MAPPED, EPI_BIAS_GELU with EPI_GELU_SPLIT, EPI_KV with EPI_Q_MAPPED; the others with
// none.
void launch_small_gemm_bf16(GemmEpilogue epi, const SmallGemm& p, const SkinnyArgs* side, hipStream_t s) {
    switch (epi) {
        case EPI_QKV: launch<EPI_QKV, kNoSide>(p, nullptr, s); break;
        case EPI_BIAS_RESIDUAL: launch<EPI_BIAS_RESIDUAL, EPI_RESIDUAL_MAPPED>(p, side, s); break;
        case EPI_BIAS_GELU: launch<EPI_BIAS_GELU, EPI_GELU_SPLIT>(p, side, s); break;
        case EPI_KV: launch<EPI_KV, EPI_Q_MAPPED>(p, side, s); break;
        case EPI_GELU_SPLIT: launch<EPI_GELU_SPLIT, kNoSide>(p, nullptr, s); break;
        case EPI_RESIDUAL_MAPPED: launch<EPI_RESIDUAL_MAPPED, kNoSide>(p, nullptr, s); break;
        case EPI_Q_MAPPED: launch<EPI_Q_MAPPED, kNoSide>(p, nullptr, s); break;
        default: break;
    }
}
