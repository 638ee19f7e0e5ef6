// bf16 maps of calls with few activation rows, and the per-request maps of calls with many requests.
//
// Such a map has too few 128 x 128 or 256 x 256 tiles to fill the chip, and a tile's time is the latency of its
// slices one after the other: at 1200 rows of hidden 768 the 128 x 128 kernel took 0.75 us a 64-deep slice, 36 us for
// the second feed-forward map.  Here a workgroup (four wavefronts, 2 x 2) owns one 64 x 64 tile and keeps STAGES - 1
// slices on their way to LDS (global_load_lds, 16 KB a slice), so a slice costs its share of the unit's LDS and L2
// rate and not a trip to memory; a wavefront reads the fragments of the next slice while its MFMAs of the current one
// run.  The accumulation order over k is that of the larger tiles and the epilogues are the same expressions, so the
// results are equal to theirs to the last bit and the choice between the kernels is free.
//
// Per-request maps of 64 requests (hidden 768 / 3072, hi | lo rows): 76 us a launch on the 128 x 128 tiles, 23 here.
//
// A launch can carry the layer's per-request side map (skinny_gemm.h) in further workgroups, and makes the row
// statistics of its operand from the 64-column pieces in its prologue: with few rows a layer's time is made of
// launches, and this leaves five of ten.
#include "skinny_gemm.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define GLOBAL_AS __attribute__((address_space(1)))
#define LDS_AS __attribute__((address_space(3)))

constexpr int kStage = 2 * 64 * 128;          // a 64-deep slice: 64 rows of A, then 64 rows of W, 128 bytes each
constexpr int kOutLd = 72;                    // floats per row of the staged tile (spreads the half-waves' writes)
constexpr int kNoSide = -1;

template <int N>
__device__ __forceinline__ void wait_vm() {
    if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if constexpr (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else if constexpr (N == 24) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
    else static_assert(N < 0, "wait count");
}

// Workgroup barrier for data in LDS.  __syncthreads() would also wait for every slice still on its way.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int EPI, int STAGES, int SIDE>
__global__ __launch_bounds__(256) void small_gemm_kernel(SmallGemm p, SkinnyArgs side, int side_blocks) {
    static_assert(STAGES * kStage >= 64 * kOutLd * 4 && STAGES * kStage >= kSkinnyLds, "LDS regions");
    __shared__ __align__(1024) unsigned char smem[STAGES * kStage];
    __shared__ float2 s_st[64];
    if (SIDE != kNoSide) {
        if ((int)blockIdx.x < side_blocks) {
            if ((int)blockIdx.x * kSkinnyCols < side.N) skinny_block<SIDE, 4, SIDE != EPI_RESIDUAL_MAPPED>(side, blockIdx.x, smem);
            return;
        }
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = p.N, K = p.K;
    const ResidualSrc& res = p.res;

    // ---- tile: XCD x (workgroups x, x + 8, ...) takes a contiguous run, row tiles fastest: a column of W is read
    // by one or two XCDs, the few rows of A by all of them
    const int rows = *p.rows;
    const int m_tiles = (rows + 63) >> 6, tiles = m_tiles * (N >> 6);
    const int b = blockIdx.x - side_blocks, per_xcd = (tiles + 7) >> 3, slot = b >> 3;
    const int tile = (b & 7) * per_xcd + slot;
    if (slot >= per_xcd || tile >= tiles) return;
    const int tn = tile / m_tiles, tm = tile - tn * m_tiles;
    const int m0 = tm * 64, n0 = tn * 64;

    // ---- slices: DMA j of wavefront w brings rows 8 (4 j + w) .. + 7 of the 128 (A's, then W's) ----------------
    const unsigned lane_off = (unsigned)((lane >> 3) * K + (((lane & 7) ^ (lane >> 3) ^ (wave & 1)) * 8)) * 2u;
    const unsigned char *src[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 8 * (4 * (j & 1) + wave);
        src[j] = (const unsigned char*)(j < 2 ? p.A + (int64_t)(m0 + r) * K : p.W + (int64_t)(n0 + r) * K);
    }
    auto dma = [&](int kt) {
        unsigned char* at = smem + (kt & (STAGES - 1)) * kStage;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(src[j] + (int64_t)kt * 128 + lane_off),
                                             (LDS_AS void*)(at + (4 * j + wave) * 1024), 16, 0, 0);
    };
    const int nk = K / 64;

    // ---- what the epilogue needs from memory is requested before the slices; item it of a thread is columns
    // 8 cg .. 8 cg + 7 of row r0 + 32 it -----------------------------------------------------------------------
    constexpr bool RESID = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_RESIDUAL_MAPPED;
    constexpr bool MAPPED = EPI == EPI_RESIDUAL_MAPPED || EPI == EPI_Q_MAPPED;
    constexpr bool FOLD = EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_Q_MAPPED || EPI == EPI_BIAS_GELU;
    constexpr bool PIECES = FOLD && !MAPPED;             // may make the statistics itself
    const int cg = threadIdx.x & 7, r0 = threadIdx.x >> 3, col = n0 + 8 * cg;
    int64_t row[2];                                      // the row in the stream or the output
    bool live[2];
    float2 st[2], pv[2][4];                              // pv: pieces cg, cg + 8, cg + 16, cg + 24 (at most 32 a row)
    uint4 yh[2], yl[2];
    const int pieces = K >> 6;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int r = m0 + r0 + 32 * it;
        row[it] = r;
        live[it] = EPI == EPI_BIAS_RESIDUAL ? r < rows : true;
        st[it] = make_float2(0.f, 0.f);
        if (MAPPED) {
            live[it] = r < rows && res.seq_len[r] > 0;
            row[it] = live[it] ? res.row_map[r] : 0;
        }
        if (PIECES && p.pstats_in) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                pv[it][c] = cg + 8 * c < pieces ? p.pstats_in[(int64_t)r * pieces + cg + 8 * c] : make_float2(0.f, 0.f);
        } else if (FOLD || RESID) {
            st[it] = res.stats[row[it]];
        }
        if (RESID) {
            yh[it] = *(const uint4*)(res.y_hi + row[it] * N + col);
            yl[it] = *(const uint4*)(res.y_lo + row[it] * N + col);
        }
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < nk) dma(s);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int r = m0 + r0 + 32 * it;
        if (PIECES && p.pstats_in) {
            // the pairing of the statistics kernel's 16 lanes: lane l adds pieces l, l + 16; lanes 0-7, lanes 8-15
            const float sum = row8_sum(pv[it][0].x + pv[it][2].x) + row8_sum(pv[it][1].x + pv[it][3].x);
            const float sq = row8_sum(pv[it][0].y + pv[it][2].y) + row8_sum(pv[it][1].y + pv[it][3].y);
            if (r < *p.live_rows) {
                st[it] = ln_moments(sum, sq, p.inv_n, p.eps);
                if (tn == 0 && cg == 0 && p.stats_out) p.stats_out[r] = st[it];
            }
        }
        if (EPI == EPI_BIAS_RESIDUAL && SIDE != kNoSide) {
            for (int q = 0; q < p.n_side; ++q)           // a request's first row is the side map's
                if (p.row_start[q] == r && p.seq_len[q] > 0) live[it] = false;
        }
        if ((EPI == EPI_QKV || EPI == EPI_KV) && cg == 0) s_st[r0 + 32 * it] = st[it];   // (read after the loop's barriers)
    }

    // ---- contraction ----------------------------------------------------------------------------------------
    const int wm = wave >> 1, wn = wave & 1, frow = lane & 31, fhalf = lane >> 5;
    const unsigned char* sa = smem + (wm * 32 + frow) * 128;
    const unsigned char* sb = smem + 64 * 128 + (wn * 32 + frow) * 128;
    int koff[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) koff[ks] = ((2 * ks + fhalf) ^ lds_swz(frow)) * 16;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    bf16x8 fa[2][4], fb[2][4];
    // slice kt has landed (everything older than the STAGES - 2 newest slices has), then every wavefront is past its
    // reads of slice kt - 1, whose stage the next DMA overwrites
    auto next_slice = [&](int kt, bf16x8* a, bf16x8* w) {
        if (kt + STAGES - 2 < nk) wait_vm<4 * (STAGES - 2)>();
        else wait_vm<0>();
        lds_barrier();
        if (kt + STAGES - 1 < nk) dma(kt + STAGES - 1);
        const int at = (kt & (STAGES - 1)) * kStage;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            a[ks] = *(const bf16x8*)(sa + at + koff[ks]);
            w[ks] = *(const bf16x8*)(sb + at + koff[ks]);
        }
    };
    auto multiply = [&](const bf16x8* a, const bf16x8* w) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], w[ks], acc, 0, 0, 0);
    };
    next_slice(0, fa[0], fb[0]);
    for (int kt = 0; kt < nk; kt += 2) {                 // (K is a multiple of 256: nk is even)
        next_slice(kt + 1, fa[1], fb[1]);
        multiply(fa[0], fb[0]);
        if (kt + 2 < nk) next_slice(kt + 2, fa[0], fb[0]);
        multiply(fa[1], fb[1]);
    }

    // ---- epilogue: the tile goes through LDS, then 8 consecutive columns (or rows of a value column) per thread -------
    __syncthreads();                                     // the last slices have been read
    float* out = (float*)smem;
#pragma unroll
    for (int e = 0; e < 16; ++e)
        out[(32 * wm + 8 * (e >> 2) + 4 * fhalf + (e & 3)) * kOutLd + 32 * wn + frow] = acc[e];
    __syncthreads();

    const int v_col0 = EPI == EPI_KV ? p.hidden : 2 * p.hidden;
    if ((EPI == EPI_QKV || EPI == EPI_KV) && n0 >= v_col0) {
        // value columns, transposed: feature c, 8 consecutive rows per thread
        const int c = threadIdx.x & 63;
        const float cc = res.colsum[n0 + c], dd = p.bias[n0 + c];
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int rg = (threadIdx.x >> 6) + 4 * it;
            float v[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float2 sv = s_st[8 * rg + r];
                v[r] = fmaf(out[(8 * rg + r) * kOutLd + c], sv.y, fmaf(-sv.x * sv.y, cc, dd));
            }
            *(uint4*)(p.vt + (int64_t)(n0 - v_col0 + c) * p.max_rows + m0 + 8 * rg) =
                make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
        }
        return;
    }

    auto load8 = [](const float* q, float* v) {
        const float4 a = *(const float4*)q, c = *(const float4*)(q + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
    };
    float bv[8], g8[8], b8[8];
    load8(p.bias + col, bv);
    if (RESID) { load8(res.gamma + col, g8); load8(res.beta + col, b8); }
    if (FOLD) load8(res.colsum + col, g8);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        float a[8], v[8];
        load8(out + (r0 + 32 * it) * kOutLd + 8 * cg, a);
        if (RESID) {
            const uint32_t hw[4] = {yh[it].x, yh[it].y, yh[it].z, yh[it].w}, lw[4] = {yl[it].x, yl[it].y, yl[it].z, yl[it].w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float y0 = __uint_as_float(hw[t] << 16) + __uint_as_float(lw[t] << 16);
                const float y1 = __uint_as_float(hw[t] & 0xffff0000u) + __uint_as_float(lw[t] & 0xffff0000u);
                v[2 * t] = a[2 * t] + bv[2 * t] + ((y0 - st[it].x) * st[it].y * g8[2 * t] + b8[2 * t]);
                v[2 * t + 1] = a[2 * t + 1] + bv[2 * t + 1] + ((y1 - st[it].x) * st[it].y * g8[2 * t + 1] + b8[2 * t + 1]);
            }
            float sm = 0.f, sq = 0.f;
            if (res.pstats) {
                sm = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
                sq = (fmaf(v[0], v[0], v[1] * v[1]) + fmaf(v[2], v[2], v[3] * v[3])) +
                     (fmaf(v[4], v[4], v[5] * v[5]) + fmaf(v[6], v[6], v[7] * v[7]));
                sm = row8_sum(sm);
                sq = row8_sum(sq);
            }
            if (live[it]) {
                uint32_t ho[4], lo[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    ho[t] = cvt_pk_bf16(v[2 * t], v[2 * t + 1]);
                    lo[t] = cvt_pk_bf16(v[2 * t] - __uint_as_float(ho[t] << 16), v[2 * t + 1] - __uint_as_float(ho[t] & 0xffff0000u));
                }
                *(uint4*)(res.x_out + row[it] * N + col) = make_uint4(ho[0], ho[1], ho[2], ho[3]);
                *(uint4*)((bf16_t*)p.C + row[it] * N + col) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                if (res.pstats && cg == 0) res.pstats[row[it] * (N >> 6) + tn] = make_float2(sm, sq);
            }
            continue;
        }
#pragma unroll
        for (int t = 0; t < 8; ++t)
            v[t] = FOLD ? fmaf(a[t], st[it].y, fmaf(-st[it].x * st[it].y, g8[t], bv[t])) : a[t] + bv[t];
        if (EPI == EPI_BIAS_GELU || EPI == EPI_GELU_SPLIT) {
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = gelu_erf(v[t]);
        }
        if (!live[it]) continue;
        const uint4 o = make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
        const int64_t ldc = (EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_Q_MAPPED) ? 2 * (int64_t)p.hidden
                            : EPI == EPI_GELU_SPLIT ? 2 * (int64_t)N : (int64_t)N;
        bf16_t* c = (bf16_t*)p.C + row[it] * ldc + col + (EPI == EPI_KV ? p.hidden : 0);   // keys sit after the queries
        *(uint4*)c = o;
        if (EPI == EPI_GELU_SPLIT) {
            // second half of the row: what the first rounding lost, as bf16 again
            const uint32_t h[4] = {o.x, o.y, o.z, o.w};
            uint32_t l[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                l[t] = cvt_pk_bf16(v[2 * t] - __uint_as_float(h[t] << 16), v[2 * t + 1] - __uint_as_float(h[t] & 0xffff0000u));
            *(uint4*)(c + N) = make_uint4(l[0], l[1], l[2], l[3]);
        }
    }
}

template <int EPI, int SIDE>
void launch(const SmallGemm& p, const SkinnyArgs* side, hipStream_t s) {
    const int side_blocks = side ? (int)align_up((size_t)(side->N / kSkinnyCols), 8) : 0;
    const int64_t tiles = (p.max_rows + 63) / 64 * (p.N / 64);
    const dim3 grid((unsigned)(side_blocks + (tiles + 7) / 8 * 8));
    const SkinnyArgs sd = side ? *side : SkinnyArgs{};
    // one tile per compute unit at most: a unit to itself, seven slices on their way; otherwise two share it
    if (tiles <= 256) hipLaunchKernelGGL((small_gemm_kernel<EPI, 8, SIDE>), grid, dim3(256), 0, s, p, sd, side_blocks);
    else hipLaunchKernelGGL((small_gemm_kernel<EPI, 4, SIDE>), grid, dim3(256), 0, s, p, sd, side_blocks);
}

}  // namespace

// Requirements: N % 64 == 0, K % 128 == 0; every buffer holds max_rows rows with max_rows % 64 == 0 (whole tiles are
// in bounds).  The side map, where there is one: EPI_RESIDUAL_MAPPED beside EPI_BIAS_RESIDUAL, EPI_GELU_SPLIT beside
// EPI_BIAS_GELU, EPI_Q_MAPPED beside EPI_KV.
void launch_small_gemm_bf16(GemmEpilogue epi, const SmallGemm& p, const SkinnyArgs* side, hipStream_t s) {
    switch (epi) {
        case EPI_QKV: launch<EPI_QKV, kNoSide>(p, nullptr, s); break;
        case EPI_BIAS_RESIDUAL:
            if (side) launch<EPI_BIAS_RESIDUAL, EPI_RESIDUAL_MAPPED>(p, side, s);
            else launch<EPI_BIAS_RESIDUAL, kNoSide>(p, nullptr, s);
            break;
        case EPI_BIAS_GELU:
            if (side) launch<EPI_BIAS_GELU, EPI_GELU_SPLIT>(p, side, s);
            else launch<EPI_BIAS_GELU, kNoSide>(p, nullptr, s);
            break;
        case EPI_KV:
            if (side) launch<EPI_KV, EPI_Q_MAPPED>(p, side, s);
            else launch<EPI_KV, kNoSide>(p, nullptr, s);
            break;
        case EPI_GELU_SPLIT: launch<EPI_GELU_SPLIT, kNoSide>(p, nullptr, s); break;
        case EPI_RESIDUAL_MAPPED: launch<EPI_RESIDUAL_MAPPED, kNoSide>(p, nullptr, s); break;
        case EPI_Q_MAPPED: launch<EPI_Q_MAPPED, kNoSide>(p, nullptr, s); break;
        default: break;
    }
}
