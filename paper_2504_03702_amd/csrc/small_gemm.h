// Device code of one tile of the small bf16 maps (see small_gemm.hip for what they are and what they measured).
#pragma once

#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define GLOBAL_AS __attribute__((address_space(1)))
#define LDS_AS __attribute__((address_space(3)))

template <int N>
__device__ __forceinline__ void wait_vm() {
    if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if constexpr (N == 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    else if constexpr (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else if constexpr (N == 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else if constexpr (N == 24) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
    else static_assert(N < 0, "wait count");
}

// Workgroup barrier for data in LDS.  __syncthreads() would also wait for every slice still on its way.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// TM, TN: 32 x 32 blocks of a wavefront; the four wavefronts' tile is 64 TM x 64 TN.  The per-request maps whose operand
// carries each value as hi + lo (columns [0, K) and [K, 2K) of a row) put a request's hi part in the tile's upper half
// and its lo part in the lower: one slice of W serves both and the two results are added in the epilogue: half as many
// steps as a contraction over 2K (64 requests of hidden 768: 23 -> 10.7 us a launch).
// b: number of the tile's workgroup; smem: STAGES slices; s_st: BM row statistics (EPI_QKV and EPI_KV only).
template <int EPI, int TM, int TN, int STAGES>
__device__ __forceinline__ void small_tile(const SmallGemm& p, int b, unsigned char* smem, float2* s_st) {
    constexpr bool DUAL = EPI == EPI_GELU_SPLIT || EPI == EPI_RESIDUAL_MAPPED;
    constexpr int BM = 64 * TM, BN = 64 * TN, ROWS = DUAL ? BM / 2 : BM, NIT = ROWS / 32;   // ROWS: of the result
    constexpr int kStage = (BM + BN) * 128;   // a 64-deep slice: the rows of A, then those of W, 128 bytes each
    constexpr int kOutLd = BN + 8;            // floats per row of the staged tile (spreads the half-waves' writes)
    constexpr int NDMA = 2 * (TM + TN);       // DMAs of a wavefront per slice
    constexpr bool EARLY = TM * TN == 1;      // the previous sums are requested before the contraction (registers allow it)
    static_assert(STAGES * kStage >= BM * (kOutLd + 1) * 4, "LDS regions");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = p.N, K = p.K;
    const ResidualSrc& res = p.res;

    // ---- tile: XCD x (workgroups x, x + 8, ...) takes a contiguous run, row tiles fastest: a column of W is read
    // by one or two XCDs, the few rows of A by all of them
    const int rows = *p.rows;
    const int m_tiles = (rows + ROWS - 1) / ROWS, tiles = m_tiles * (N / BN);
    const int per_xcd = (tiles + 7) >> 3, slot = b >> 3;
    const int tile = (b & 7) * per_xcd + slot;
    if (slot >= per_xcd || tile >= tiles) return;
    const int tn = tile / m_tiles, tm = tile - tn * m_tiles;
    const int m0 = tm * ROWS, n0 = tn * BN;

    // ---- slices: DMA j of wavefront w brings rows 8 (4 j + w) .. + 7 of the slice's (A's, then W's) ------------
    const int lda = DUAL ? 2 * K : K;
    const unsigned chunk = (unsigned)((lane & 7) ^ (lane >> 3) ^ (wave & 1)) * 16u;
    const unsigned a_off = (unsigned)((lane >> 3) * lda) * 2u + chunk, w_off = (unsigned)((lane >> 3) * K) * 2u + chunk;
    const unsigned char* src[NDMA];
#pragma unroll
    for (int j = 0; j < NDMA; ++j) {
        const int r = 8 * (4 * (j < 2 * TM ? j : j - 2 * TM) + wave);
        const bool lo = DUAL && r >= ROWS;
        src[j] = (const unsigned char*)(j < 2 * TM ? p.A + (int64_t)(m0 + r - (lo ? ROWS : 0)) * lda + (lo ? K : 0)
                                                   : p.W + (int64_t)(n0 + r) * K);
    }
    int wr = 0;                                          // stage of the next slice to bring
    auto dma = [&](int j, int kt, unsigned char* at) {
        __builtin_amdgcn_global_load_lds((const GLOBAL_AS void*)(src[j] + (int64_t)kt * 128 + (j < 2 * TM ? a_off : w_off)),
                                         (LDS_AS void*)(at + (4 * j + wave) * 1024), 16, 0, 0);
    };
    const int nk = K / 64;

    // ---- what the epilogue needs from memory is requested before the slices; item it of a thread is columns
    // 8 cg .. 8 cg + 7 (of every 64) of row r0 + 32 it -----------------------------------------------------------------------
    constexpr bool RESID = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_RESIDUAL_MAPPED;
    constexpr bool MAPPED = EPI == EPI_RESIDUAL_MAPPED || EPI == EPI_Q_MAPPED;
    constexpr bool FOLD = EPI == EPI_QKV || EPI == EPI_KV || EPI == EPI_Q_MAPPED || EPI == EPI_BIAS_GELU;
    constexpr bool PIECES = FOLD && !MAPPED;             // may make the statistics itself
    const int cg = threadIdx.x & 7, r0 = threadIdx.x >> 3, col0 = n0 + 8 * cg;
    int64_t row[NIT];                                    // the row in the stream or the output
    bool live[NIT];
    float2 st[NIT], pv[NIT][4];                          // pv: pieces cg, cg + 8, cg + 16, cg + 24 (at most 32 a row)
    uint4 yh[TN][NIT], yl[TN][NIT];
    auto load_previous = [&]() {
#pragma unroll
        for (int it = 0; it < NIT; ++it)
#pragma unroll
            for (int c = 0; c < TN; ++c) {
                yh[c][it] = *(const uint4*)(res.y_hi + row[it] * N + col0 + 64 * c);
                yl[c][it] = *(const uint4*)(res.y_lo + row[it] * N + col0 + 64 * c);
            }
    };
    const int pieces = K >> 6;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int r = m0 + r0 + 32 * it;
        row[it] = r;
        live[it] = true;
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
    }
    if (RESID && EARLY) load_previous();
    int side_len = 0, side_first = 0;                    // lane q: of request q, whose first row is the side map's
    if (EPI == EPI_BIAS_RESIDUAL) {
        side_len = p.seq_len[min(lane, p.n_side - 1)];
        side_first = p.row_start[min(lane, p.n_side - 1)];
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) {
        if (s >= nk) continue;
#pragma unroll
        for (int j = 0; j < NDMA; ++j) dma(j, s, smem + wr * kStage);
        wr = wr + 1 == STAGES ? 0 : wr + 1;
    }
    asm volatile("" ::: "memory");
    // ---- the rows' statistics ---------------------------------------------------------------------------------
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
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
        if ((EPI == EPI_QKV || EPI == EPI_KV) && cg == 0) s_st[r0 + 32 * it] = st[it];   // (read after the loop's barriers)
    }

    // ---- contraction ----------------------------------------------------------------------------------------
    const int wm = wave >> 1, wn = wave & 1, frow = lane & 31, fhalf = lane >> 5;
    const unsigned char* sa = smem + (wm * 32 * TM + frow) * 128;
    const unsigned char* sb = smem + BM * 128 + (wn * 32 * TN + frow) * 128;
    int koff[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) koff[ks] = ((2 * ks + fhalf) ^ lds_swz(frow)) * 16;
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    struct Frags { bf16x8 a[4][TM], w[4][TN]; };
    Frags f0, f1;
    int rd = 0;                                          // stage of the next slice to read
    // slice kt has landed (everything older than the STAGES - 2 newest slices has), and every wavefront is past its
    // reads of slice kt - 1, whose stage the next DMA overwrites
    auto land = [&](int kt) {
        if (kt + STAGES - 2 < nk) wait_vm<NDMA * (STAGES - 2)>();
        else wait_vm<0>();
        lds_barrier();
    };
    constexpr int NREAD = 4 * (TM + TN), NMFMA = 4 * TM * TN;
    auto read = [&](int q, Frags& f, int at) {           // fragment q of the slice in stage `at`
        const int ks = q / (TM + TN), i = q % (TM + TN);
        if (i < TM) f.a[ks][i] = *(const bf16x8*)(sa + at + i * 4096 + koff[ks]);
        else f.w[ks][i - TM] = *(const bf16x8*)(sb + at + (i - TM) * 4096 + koff[ks]);
    };
    auto multiply = [&](int m, const Frags& f) {
        const int ks = m / (TM * TN), i = m / TN % TM, j = m % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[ks][i], f.w[ks][j], acc[i][j], 0, 0, 0);
    };
    auto next_stage = [&](int& st) {
        const int at = st * kStage;
        st = st + 1 == STAGES ? 0 : st + 1;
        return at;
    };
    // The products of slice kt - 1 with the reads of slice kt and the DMAs of slice kt + STAGES - 1 spread among them.  In
    // one queue behind the other, as the compiler leaves them, a 128 x 64 tile's slice cost the sum of what its DMAs, its reads
    // and its products take: 1357 rows of hidden 768, second feed-forward map 25.7 -> 23.6 us, first 21.7 -> 20.5,
    // query-key-value map 16.1 -> 15.5.  (64 x 64 tiles, alone in their units: no change.)
    auto slice = [&](int kt, const Frags& cur, Frags& nxt) {
        land(kt);
        const bool more = kt + STAGES - 1 < nk;
        unsigned char* to = smem + wr * kStage;
        const int at = next_stage(rd);
#pragma unroll
        for (int m = 0; m < NMFMA; ++m) {
            multiply(m, cur);
            if (more) {
#pragma unroll
                for (int j = m * NDMA / NMFMA; j < (m + 1) * NDMA / NMFMA; ++j) dma(j, kt + STAGES - 1, to);
            }
#pragma unroll
            for (int q = m * NREAD / NMFMA; q < (m + 1) * NREAD / NMFMA; ++q) read(q, nxt, at);
            __builtin_amdgcn_sched_barrier(0);
        }
        wr = wr + 1 == STAGES ? 0 : wr + 1;
    };
    land(0);
    if (STAGES - 1 < nk) {
        unsigned char* to = smem + next_stage(wr);
#pragma unroll
        for (int j = 0; j < NDMA; ++j) dma(j, STAGES - 1, to);
    }
    const int at0 = next_stage(rd);
#pragma unroll
    for (int q = 0; q < NREAD; ++q) read(q, f0, at0);
    for (int kt = 0; kt < nk - 2; kt += 2) {             // (K is a multiple of 256: nk is even)
        slice(kt + 1, f0, f1);
        slice(kt + 2, f1, f0);
    }
    slice(nk - 1, f0, f1);
#pragma unroll
    for (int m = 0; m < NMFMA; ++m) multiply(m, f1);

    if (EPI == EPI_BIAS_RESIDUAL) {
        // (behind the contraction: ahead of it the loads would be waited for, with every slice on its way; a loop of scalar
        // loads, as it was, took a trip to memory a request: 8 requests, output projection 12.2 -> 10.2 us, second feed-forward map 23.3 -> 21.2)
        const int side_row = side_len > 0 ? side_first : -1;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            live[it] = row[it] < rows;
            for (int q = 0; q < p.n_side; ++q)
                if (__builtin_amdgcn_readlane(side_row, q) == (int)row[it]) live[it] = false;
        }
    }

    // ---- epilogue: the tile goes through LDS, then 8 consecutive columns (or rows of a value column) per thread -------
    if (RESID && !EARLY) load_previous();
    __syncthreads();                                     // the last slices have been read
    float* out = (float*)smem;
    // value columns are read back by rows: another row length keeps those reads off each other's banks
    const int v_col0 = EPI == EPI_KV ? p.hidden : 2 * p.hidden;
    const bool values = (EPI == EPI_QKV || EPI == EPI_KV) && n0 >= v_col0;
    const int out_ld = values ? kOutLd + 1 : kOutLd;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                out[(32 * (TM * wm + i) + 8 * (e >> 2) + 4 * fhalf + (e & 3)) * out_ld + 32 * (TN * wn + j) + frow] = acc[i][j][e];
    __syncthreads();

    if (values) {
        // transposed: 8 consecutive rows of a feature per thread, whole lines of Vt (64 rows) by 8 neighbouring threads (16
        // bytes of 64 features an access: query-key-value map of 1357 rows 15.5 us, 13.9 so)
#pragma unroll
        for (int it = 0; it < BM * BN / 2048; ++it) {
            const int at = threadIdx.x + 256 * it, c = (at >> 3) % BN, r0 = 64 * ((at >> 3) / BN) + 8 * (at & 7);
            const float cc = res.colsum[n0 + c], dd = p.bias[n0 + c];
            float v[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float2 sv = s_st[r0 + r];
                v[r] = fmaf(out[(r0 + r) * out_ld + c], sv.y, fmaf(-sv.x * sv.y, cc, dd));
            }
            *(uint4*)(p.vt + (int64_t)(n0 - v_col0 + c) * p.max_rows + m0 + r0) =
                make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7]));
        }
        return;
    }

    auto load8 = [](const float* q, float* v) {
        const float4 a = *(const float4*)q, c = *(const float4*)(q + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
    };
#pragma unroll
    for (int pc = 0; pc < TN; ++pc) {
        float bv[8], g8[8], b8[8];
        const int col = col0 + 64 * pc;
        load8(p.bias + col, bv);
        if (RESID) { load8(res.gamma + col, g8); load8(res.beta + col, b8); }
        if (FOLD) load8(res.colsum + col, g8);
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            float a[8], v[8];
            load8(out + (r0 + 32 * it) * kOutLd + 64 * pc + 8 * cg, a);
            if (DUAL) {
                load8(out + (ROWS + r0 + 32 * it) * kOutLd + 64 * pc + 8 * cg, v);
#pragma unroll
                for (int t = 0; t < 8; ++t) a[t] += v[t];
            }
            if (RESID) {
                const uint32_t hw[4] = {yh[pc][it].x, yh[pc][it].y, yh[pc][it].z, yh[pc][it].w}, lw[4] = {yl[pc][it].x, yl[pc][it].y, yl[pc][it].z, yl[pc][it].w};
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float2 y = stream_join2(hw[t], lw[t]);
                    v[2 * t] = residual_sum(a[2 * t], y.x, st[it], g8[2 * t], b8[2 * t] + bv[2 * t]);
                    v[2 * t + 1] = residual_sum(a[2 * t + 1], y.y, st[it], g8[2 * t + 1], b8[2 * t + 1] + bv[2 * t + 1]);
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
                    for (int t = 0; t < 4; ++t) stream_split2(v[2 * t], v[2 * t + 1], ho[t], lo[t]);
                    *(uint4*)(res.x_out + row[it] * N + col) = make_uint4(ho[0], ho[1], ho[2], ho[3]);
                    *(uint4*)((bf16_t*)p.C + row[it] * N + col) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                    if (res.pstats && cg == 0) res.pstats[row[it] * (N >> 6) + (n0 >> 6) + pc] = make_float2(sm, sq);
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
}

}  // namespace
