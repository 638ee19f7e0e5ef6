// Device code of the per-request side maps (one row per request: the error-compensated output projection and
// feed-forward block of each request's first row, and the last layer's queries) for calls of at most 16 requests.
//
//   C[r, n] = sum_k A[r, k] * W[n, k]  for r < 16, then the same epilogues as the tiled GEMM's per-request forms.
//
// With so few rows the map is a stream over W: a tiled kernel would put one tile on a handful of compute units and
// walk the whole contraction there, slice after slice, each waiting out a trip to memory.  Here a workgroup owns 64, 32
// or 16 output columns (16 G) and the contraction is split in 8 shares, dealt to its wavefronts: each issues
// v_mfma_f32_16x16x32_bf16 on fragments loaded straight from global memory (A: request r = lane % 16, sixteen
// consecutive k per lane and 64-deep round; W the same with its row = output column), several rounds' loads
// requested before the first is used.  Where A carries each value as hi + lo, a W fragment serves both parts.  The
// shares' partial 16 x 16 G results are added through LDS in a fixed order; one wavefront applies the epilogue.  The
// result does not depend on the number of wavefronts (8 in the kernel of its own, 4 where the block shares a launch
// with the map of all rows), but it differs from the tiled kernels' in the last bits (another order of additions),
// so a request's prediction in a call of at most 16 requests need not be bit-equal to the same request's in a larger
// call.
#pragma once

#include "device_util.h"
#include "internal.h"

namespace {

typedef __bf16 sk_bf16x8 __attribute__((ext_vector_type(8)));
typedef float sk_f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSkinnyShares = 8;     // parts of the contraction, added in this order
constexpr int kSkinnyCols = 64;      // most output columns per workgroup: one piece of the rows' partial statistics
constexpr int kSkinnyLds = kSkinnyShares * 4 * 64 * 16 + 4 * 64 * 16 + 16 * 8;

// sum over the 16 lanes that share lane / 16, every one of them gets it; fixed order
__device__ __forceinline__ float sum16(float v) {
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 8, 64);
    return v;
}

// Row statistics of request frow's first row from the 64-column pieces (at most 32), by the four lanes that hold that
// row: lane group fq adds pieces 4 fq .. 4 fq + 3 (mod 16), so the additions pair up exactly as in the statistics kernel.
struct SkinnyPieces {
    float2 v[8];
    __device__ __forceinline__ void load(const float2* __restrict__ ps, int pieces, int fq) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int at = 4 * fq + (c & 3) + 16 * (c >> 2);
            v[c] = ps[min(at, pieces - 1)];
            if (at >= pieces) v[c] = make_float2(0.f, 0.f);
        }
    }
    __device__ __forceinline__ float2 stats(float inv_n, float eps) const {
        float a = ((v[0].x + v[4].x) + (v[1].x + v[5].x)) + ((v[2].x + v[6].x) + (v[3].x + v[7].x));
        float b = ((v[0].y + v[4].y) + (v[1].y + v[5].y)) + ((v[2].y + v[6].y) + (v[3].y + v[7].y));
        a += __shfl_xor(a, 16, 64); b += __shfl_xor(b, 16, 64);
        a += __shfl_xor(a, 32, 64); b += __shfl_xor(b, 32, 64);
        return ln_moments(a, b, inv_n, eps);
    }
};

// One block of 16 G output columns by NW wavefronts; smem: kSkinnyLds bytes.  EPI_GELU_SPLIT and EPI_RESIDUAL_MAPPED
// take hi | lo rows (each W fragment serves two MFMAs).  GATHER: the rows of A are taken from the stream itself, at
// each request's first row: for EPI_Q_MAPPED the hi parts, for EPI_GELU_SPLIT the LayerNorm of the sums (both parts
// joined), as hi | lo.
// G: groups of 16 columns of a block; 4 where it leaves pieces of 64 columns.
template <int EPI, int NW, bool GATHER, int G = kSkinnyCols / 16>
__device__ void skinny_block(const SkinnyArgs& p, int block, unsigned char* smem) {
    constexpr bool DUAL = EPI != EPI_Q_MAPPED;
    constexpr bool NORM = GATHER && EPI == EPI_GELU_SPLIT;
    constexpr int SH = kSkinnyShares / NW;
    const ResidualSrc& res = p.res;
    const int N = p.N, K = p.K;
    sk_f32x4(*s_part)[4][64] = (sk_f32x4(*)[4][64])smem;    // [share][column group][lane]: 16 rows x 16 columns each
    sk_f32x4(*s_sum)[64] = (sk_f32x4(*)[64])(smem + kSkinnyShares * 4 * 64 * 16);
    float2* s_st = (float2*)(smem + (kSkinnyShares + 1) * 4 * 64 * 16);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 15, fq = lane >> 4;
    const int n0 = block * 16 * G;
    const int n_req = p.n_req;
    // The stream row of request frow.  (Absent requests take the last one's, faulty ones have a row start inside the
    // buffers too; the results of both are not stored.)
    int64_t arow = frow;
    float2 ast = make_float2(0.f, 0.f);
    bool a_live = false;
    SkinnyPieces pieces;
    if (GATHER) {
        arow = res.row_map[min(frow, n_req - 1)];
        a_live = frow < n_req && res.seq_len[min(frow, n_req - 1)] > 0;
        if (p.stats_from == SKINNY_STATS_PIECES) {
            pieces.load(p.pstats_in + arow * (K >> 6), K >> 6, fq);
        } else if (NORM && p.stats_from == SKINNY_STATS_ROWS) {   // two passes over the rows themselves, a wavefront each
            for (int r = wave; r < min(16, n_req); r += NW) {
                const int64_t at = (int64_t)res.row_map[r] * K;
                const float2 v = row_moments(res.y_hi + at, res.y_lo + at, K, p.eps, lane);
                if (lane == 0) s_st[r] = v;
            }
            __syncthreads();
            ast = s_st[min(frow, n_req - 1)];
        } else {
            ast = res.stats[arow];
        }
    }

    // ---- what the epilogue will need from memory (wavefront 0), requested behind the first round's operands ------
    // Element e of column group g in a lane is C[4 * fq + e, n0 + 16 g + frow].
    bool live[4] = {false, false, false, false};
    int64_t srow[4] = {0, 0, 0, 0};                     // first row of request 4 fq + e in the stream
    float2 st[4];
    float yprev[4][4];                                  // previous sums of the stream at (request e, column group g)
    float bv[4], cs[4] = {0.f, 0.f, 0.f, 0.f}, gm[4] = {0.f, 0.f, 0.f, 0.f}, bt[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI != EPI_GELU_SPLIT && wave == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = min(4 * fq + e, n_req - 1);   // the request; uniform over the 16 lanes that share fq
            srow[e] = res.row_map[r];
            live[e] = 4 * fq + e < n_req && res.seq_len[r] > 0;
        }
    }
    auto epilogue_loads = [&]() {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int c = n0 + 16 * g + frow;
            bv[g] = p.bias[c];
            if (EPI == EPI_Q_MAPPED) cs[g] = res.colsum[c];
            if (EPI == EPI_RESIDUAL_MAPPED) { gm[g] = res.gamma[c]; bt[g] = res.beta[c]; }
        }
        if (EPI == EPI_RESIDUAL_MAPPED) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                st[e] = res.stats[srow[e]];
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int64_t at = srow[e] * N + n0 + 16 * g + frow;
                    yprev[e][g] = stream_join(res.y_hi[at], res.y_lo[at]);
                }
            }
        }
    };

    // ---- contraction: a share of k, 64 deep per round (two MFMA steps): a lane reads 32 consecutive bytes of its
    // row, the four lanes of a row one whole 128-byte line ----------------------------------------------------
    const int total_rounds = K / 64;                    // dealt to the shares as evenly as whole rounds allow
    const int lda = DUAL && !NORM ? 2 * K : K;
    const int64_t wg = (int64_t)16 * K;                 // next column group: 16 rows of W further
    const bool on = frow < n_req;
    // A wavefront's shares are neighbours in k: it goes through their rounds in one run, so the loads in flight together
    // may belong to two shares.  A share of no rounds (K below 512) leaves zeros.  Two rounds at a time, in a loop that is
    // not unrolled: what a unit's address path takes for lanes that read a row each (not the trip to memory) and, in code
    // that runs once, the fetching of instructions are what this costs.  One prompt, hidden 768 / 3072, us a launch, before
    // (three rounds at a time, share by share, absent ones loaded too) / one / two / three rounds: output projection
    // 9.4 / 6.9 / 6.9 / 7.3, first feed-forward map 12.7 / 12.4 / 12.4 / 12.4, second 15.7 / 16.0 / 16.1 / 16.4.  Reading 64
    // bytes of a row per quad of lanes and exchanging the chunks among them costs more than it saves (10.5, 16.7, 24.8).
    constexpr int U = 2;                                // rounds whose loads are in flight together
    const int first = wave * SH;
    const int r0 = first * total_rounds / kSkinnyShares, r1 = (first + SH) * total_rounds / kSkinnyShares;
    sk_f32x4 acc[G];
    int share = first, share_end = (first + 1) * total_rounds / kSkinnyShares;
    auto clear = [&]() {
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = sk_f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto close_shares = [&](int t) {                    // round t belongs to a later share
        while (share < first + SH && t >= share_end) {
#pragma unroll
            for (int g = 0; g < G; ++g) s_part[share][g][lane] = acc[g];
            clear();
            ++share;
            share_end = (share + 1) * total_rounds / kSkinnyShares;
        }
    };
    clear();
    const bf16_t* ap = (NORM ? res.y_hi : p.A) + arow * lda + 16 * fq;
    const bf16_t* lp = NORM ? res.y_lo + arow * lda + 16 * fq : ap + K;
    const bf16_t* wp = p.W + (int64_t)(n0 + frow) * K + 16 * fq;
    const float *gp = NORM ? res.gamma + 16 * fq : nullptr, *bp = NORM ? res.beta + 16 * fq : nullptr;
#pragma unroll 1
    for (int t0 = r0; t0 == r0 || t0 < r1; t0 += U) {
        sk_bf16x8 fa[U][2] = {}, fl[DUAL ? U : 1][2] = {}, fw[U][G][2];
        float4 gv[NORM ? U : 1][4], bb[NORM ? U : 1][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u;
            if (t >= r1) continue;                      // uniform
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (on) {                               // (the other lanes' rows are nobody's)
                    fa[u][h] = *(const sk_bf16x8*)(ap + 64 * t + 8 * h);
                    if (DUAL) fl[u][h] = *(const sk_bf16x8*)(lp + 64 * t + 8 * h);
                }
#pragma unroll
                for (int g = 0; g < G; ++g) fw[u][g][h] = *(const sk_bf16x8*)(wp + g * wg + 64 * t + 8 * h);
            }
            if (NORM) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    gv[u][q] = *(const float4*)(gp + 64 * t + 4 * q);
                    bb[u][q] = *(const float4*)(bp + 64 * t + 4 * q);
                }
            }
        }
        if (t0 == r0) {
            asm volatile("" ::: "memory");              // the operands first
            if (wave == 0) epilogue_loads();
            if (GATHER && p.stats_from == SKINNY_STATS_PIECES) ast = pieces.stats(p.inv_n, p.eps);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t0 + u >= r1) continue;
            close_shares(t0 + u);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (NORM) {
                    union { sk_bf16x8 v; uint32_t w[4]; } yh, yl;
                    yh.v = fa[u][h];
                    yl.v = fl[u][h];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float4 ga = gv[u][2 * h + (t >> 1)], be = bb[u][2 * h + (t >> 1)];
                        const float2 y = stream_join2(yh.w[t], yl.w[t]);
                        const float x0 = ln_apply(y.x, ast, (t & 1) ? ga.z : ga.x, (t & 1) ? be.z : be.x);
                        const float x1 = ln_apply(y.y, ast, (t & 1) ? ga.w : ga.y, (t & 1) ? be.w : be.y);
                        const uint32_t o = pack_bf16x2(x0, x1);
                        yh.w[t] = o;
                        yl.w[t] = pack_bf16x2(x0 - __uint_as_float(o << 16), x1 - __uint_as_float(o & 0xffff0000u));
                    }
                    fa[u][h] = yh.v;
                    fl[u][h] = yl.v;
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[u][h], fw[u][g][h], acc[g], 0, 0, 0);
                    if (DUAL) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl[u][h], fw[u][g][h], acc[g], 0, 0, 0);
                }
            }
        }
    }
    close_shares(total_rounds);
    __syncthreads();
    if (wave < G) {                                     // column group `wave`: the eight partial results in order
        sk_f32x4 t = s_part[0][wave][lane];
#pragma unroll
        for (int w = 1; w < kSkinnyShares; ++w) {
            const sk_f32x4 q = s_part[w][wave][lane];
            t[0] += q[0]; t[1] += q[1]; t[2] += q[2]; t[3] += q[3];
        }
        s_sum[wave][lane] = t;
    }
    __syncthreads();
    if (wave != 0) return;
    if (GATHER && p.stats_out && block == 0 && fq == 0 && a_live) p.stats_out[arow] = ast;
    if (GATHER && EPI == EPI_Q_MAPPED) {
#pragma unroll
        for (int e = 0; e < 4; ++e) st[e] = make_float2(__shfl(ast.x, 4 * fq + e, 64), __shfl(ast.y, 4 * fq + e, 64));
    }
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = s_sum[g][lane];
    if (EPI == EPI_GELU_SPLIT) {
        bf16_t* C = (bf16_t*)p.C;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t r = 4 * fq + e;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int c = n0 + 16 * g + frow;
                const float v = gelu_erf(acc[g][e] + bv[g]);
                const bf16_t hi = f32_to_bf16(v);
                C[r * 2 * N + c] = hi;
                C[r * 2 * N + N + c] = f32_to_bf16(v - bf16_to_f32(hi));
            }
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t row = srow[e];
        if (EPI == EPI_Q_MAPPED) {
            bf16_t* C = (bf16_t*)p.C;
            const float nm = -st[e].x * st[e].y;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float v = fmaf(acc[g][e], st[e].y, fmaf(nm, cs[g], bv[g]));
                if (live[e]) C[row * 2 * p.hidden + n0 + 16 * g + frow] = f32_to_bf16(v);
            }
        } else {
            bf16_t* Cl = (bf16_t*)p.C;
            float sm = 0.f, sq = 0.f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int c = n0 + 16 * g + frow;
                const float o = residual_sum(acc[g][e], yprev[e][g], st[e], gm[g], bt[g] + bv[g]);
                sm += o;
                sq = fmaf(o, o, sq);
                if (live[e]) {
                    const uint32_t w = __float_as_uint(o) + 0x8000u;          // see stream_split2
                    res.x_out[row * N + c] = (bf16_t)(w >> 16);
                    Cl[row * N + c] = (bf16_t)w;
                }
            }
            if (G == kSkinnyCols / 16 && res.pstats) {
                sm = sum16(sm);
                sq = sum16(sq);
                if (live[e] && frow == 0) res.pstats[row * (N >> 6) + (n0 >> 6)] = make_float2(sm, sq);
            }
        }
    }
}

}  // namespace
