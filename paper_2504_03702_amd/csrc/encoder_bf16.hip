// bf16 encoder path: the per-layer sequence of MFMA GEMMs and attention launches.  There is no
// LayerNorm kernel: a residual epilogue writes the new sums of the residual stream in two 16-bit
// halves hi and lo (hi, the sum rounded to bf16, is the next map's operand) and leaves per-row partial sums; a small kernel turns those into (mean, 1/std),
// and the next map, which carries the LayerNorm's scale and shift in its weights, finishes the
// normalisation in its own epilogue.
#include "device_util.h"
#include "internal.h"

namespace {

// The sum of 16 consecutive lanes, in every one of them; fixed order.
__device__ __forceinline__ float lanes16_sum(float v) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 16);
    return v;
}

// Statistics of one row from the partial sums the residual epilogues leave, by 16 lanes: lane p takes the pieces p,
// p + 16, ...; the 16 partial results are added in a fixed order.  Biased variance as E[v^2] - mean^2 (the rows are
// residual-stream sums, whose mean is small against their spread).
__device__ __forceinline__ float2 piece_stats(const float2* __restrict__ row, int pieces, int p, float inv_n, float eps) {
    float sm = 0.f, sq = 0.f;
    for (int c = p; c < pieces; c += 16) {
        const float2 v = row[c];
        sm += v.x;
        sq += v.y;
    }
    sm = lanes16_sum(sm);
    sq = lanes16_sum(sq);
    return ln_moments(sm, sq, inv_n, eps);
}

// Two things the maps after a residual one need, in one launch (they depend on the same sums, and in small calls a
// launch is what they cost: 5 + 7 us apart).  The first gather_blocks workgroups, a wavefront per request, make the
// operand of the per-request feed-forward map: row r is the fp32 LayerNorm of request r's first row of the stream, split
// into two bf16 values per element (x ~ hi + lo, |x - hi - lo| <= 2^-17 |x|), hi in columns [0, H), lo in [H, 2H); zeros
// for faulty requests and padding rows.  The others, 16 lanes per row, make the row statistics of the stream.
// TWO_PASS (the last layer, where the epilogues leave no pieces): a first row's statistics from the row itself, and they
// are left in stats.
template <bool TWO_PASS>
__global__ __launch_bounds__(256) void ln_stats_gather_kernel(const float2* __restrict__ pstats, float2* __restrict__ stats,
                                                              int H, float inv_n, float eps,
                                                              const int32_t* __restrict__ total_rows, int gather_blocks,
                                                              const bf16_t* __restrict__ y_hi, const bf16_t* __restrict__ y_lo,
                                                              const float* __restrict__ gamma, const float* __restrict__ beta,
                                                              int n_req, const int32_t* __restrict__ seq_len,
                                                              const int32_t* __restrict__ row_start, bf16_t* __restrict__ out) {
    const int pieces = H >> 6, lane = threadIdx.x & 63;
    if ((int)blockIdx.x >= gather_blocks) {
        const int64_t row = (int64_t)(blockIdx.x - gather_blocks) * 16 + (threadIdx.x >> 4);
        if (row >= *total_rows) return;                 // whole 16-lane groups leave together
        const float2 st = piece_stats(pstats + row * pieces, pieces, lane & 15, inv_n, eps);
        if ((lane & 15) == 0) stats[row] = st;
        return;
    }
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    uint2* oh = (uint2*)(out + (int64_t)r * 2 * H);
    uint2* ol = oh + H / 4;
    if (r >= n_req || seq_len[r] <= 0) {
        for (int i = lane; i < H / 4; i += 64) oh[i] = ol[i] = make_uint2(0u, 0u);
        return;
    }
    const int64_t row = row_start[r];
    float2 st;
    if (TWO_PASS) {
        st = row_moments(y_hi + row * H, y_lo + row * H, H, eps, lane);
        if (lane == 0) stats[row] = st;
    } else {
        st = piece_stats(pstats + row * pieces, pieces, lane & 15, inv_n, eps);
    }
    const uint2 *yh = (const uint2*)(y_hi + row * H), *yl = (const uint2*)(y_lo + row * H);
    for (int i = lane; i < H / 4; i += 64) {
        const uint2 h = yh[i], l = yl[i];
        const float4 g = ((const float4*)gamma)[i], b = ((const float4*)beta)[i];
        const float2 ya = stream_join2(h.x, l.x), yb = stream_join2(h.y, l.y);
        const float x0 = ln_apply(ya.x, st, g.x, b.x), x1 = ln_apply(ya.y, st, g.y, b.y);
        const float x2 = ln_apply(yb.x, st, g.z, b.z), x3 = ln_apply(yb.y, st, g.w, b.w);
        const uint2 o = make_uint2(pack_bf16x2(x0, x1), pack_bf16x2(x2, x3));
        oh[i] = o;
        ol[i] = make_uint2(pack_bf16x2(x0 - __uint_as_float(o.x << 16), x1 - __uint_as_float(o.x & 0xffff0000u)),
                           pack_bf16x2(x2 - __uint_as_float(o.y << 16), x3 - __uint_as_float(o.y & 0xffff0000u)));
    }
}

}  // namespace

// The first feed-forward map of the per-request pass: the small tiles read W once for both halves of the operand but
// take two passes' worth of places; beyond 1024 of their 128 x 64 tiles (two waves of the chip's 512 places) the large
// kernel's 128 x 128 tiles are faster, with the same bits.  Small against large: hidden 768 (ffn 3072) 1280 requests, 960
// tiles, 24.6 / 24.8 us, 1536 30.4 / 28.1, 4096 90 / 57, 20000 409 / 234; hidden 1024 (ffn 4096) 1024 requests, 1024
// tiles, 29.3 / 30.7, 1280 36.0 / 35.6, 4096 150 / 81.
#define PS_SPLIT_TILES 1024

void run_encoder_bf16(const ps_model* m, int32_t n_req, const Workspace& ws, hipStream_t s) {
    const ps_model_info& f = m->info;
    const int H = f.hidden, F = f.ffn;
    bf16_t *x = (bf16_t*)ws.x, *qk = (bf16_t*)ws.qkv, *vt = (bf16_t*)ws.vt, *att = (bf16_t*)ws.att,
           *x1 = (bf16_t*)ws.x1, *g = (bf16_t*)ws.g;
    const int32_t* rows = &ws.meta->total_rows;        // the rows that belong to requests
    const int32_t* qkv_rows = &ws.meta->qkv_rows;     // QKV projection: those plus the slack the key tiles read
    const ResidualSrc none = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    const int32_t* n_req_dev = &ws.meta->n_req;
    int64_t* clk = m->profiling ? m->clk_slot : nullptr;   // clock probe of the large GEMMs
    // the stream entering layer 0 is the embedding LayerNorm of the sums the embed kernel left in (x, la)
    const float *sg = m->lne_g, *sbeta = m->lne_b;
    // row statistics of the stream (`rows_too`), and the per-request feed-forward operand (`res`, if not null)
    auto ln_stats = [&](float2* stats, bool rows_too, const ResidualSrc* res) {
        const unsigned gather = res ? (unsigned)(ws.cls_rows / 4) : 0, blocks = gather + (rows_too ? (unsigned)(ws.max_rows / 16) : 0);
        const ResidualSrc q = res ? *res : none;
        if (rows_too)
            hipLaunchKernelGGL(ln_stats_gather_kernel<false>, dim3(blocks), dim3(256), 0, s, ws.ps, stats, H, 1.0f / (float)H,
                               m->ln_eps, rows, (int)gather, q.y_hi, q.y_lo, q.gamma, q.beta, n_req, ws.seq_len, ws.row_start,
                               (bf16_t*)ws.cls_a);
        else
            hipLaunchKernelGGL(ln_stats_gather_kernel<true>, dim3(blocks), dim3(256), 0, s, ws.ps, stats, H, 1.0f / (float)H,
                               m->ln_eps, rows, (int)gather, q.y_hi, q.y_lo, q.gamma, q.beta, n_req, ws.seq_len, ws.row_start,
                               (bf16_t*)ws.cls_a);
    };
#define PS_TIMED(FAM, CALL) do { ProfScope p_(m, FAM, s); CALL; } while (0)
    // the per-request side maps of calls of more than 16 requests
    auto side_args = [&](const void* A, const void* W, const float* bias, const ResidualSrc& r, void* C, int N, int K) {
        SmallGemm p = {};
        p.A = (const bf16_t*)A; p.W = (const bf16_t*)W; p.bias = bias; p.res = r; p.C = C;
        p.max_rows = ws.cls_rows; p.N = N; p.K = K; p.hidden = H; p.rows = n_req_dev;
        return p;
    };
    auto side_gemm = [&](GemmEpilogue epi, const bf16_t* A, const void* W, const float* bias, const ResidualSrc& r, void* C,
                         int N, int K) {
        launch_small_gemm_bf16(epi, side_args(A, W, bias, r, C, N, K), nullptr, s);
    };
    const bool skinny = n_req <= PS_SKINNY_ROWS;
    auto skinny_args = [&](const void* A, const void* W, const float* bias, const ResidualSrc& r, void* C, int N, int K,
                           int stats_from, float2* stats_out) {
        return SkinnyArgs{(const bf16_t*)A, (const bf16_t*)W, bias, r, C, N, K, H, n_req,
                          stats_from, ws.ps, stats_out, 1.0f / (float)H, m->ln_eps};
    };
    // Calls of a few requests over few rows: a layer is five launches, each map's launch doing the per-request map
    // beside it and making the row statistics it needs from the previous launch's pieces.
    const bool fused = small_maps(ws, n_req, H);
    // With more of either, up to PS_CARRIED_REQUESTS, the launches of the maps of all rows carry the per-request ones.
    const bool carried = carries_side_maps(ws, n_req, H);
    for (int l = 0; l < f.layers; ++l) {
        const LayerWeights& w = m->layers[(size_t)l];
        // After the last layer only the first row of every request goes on (to the head), and within
        // that layer a row's output projection and feed-forward block depend on no other row: there the
        // all-row GEMMs and LayerNorms are skipped, attention computes the first rows only, and the
        // per-request side pass below, which every layer runs for accuracy, is all that is left.
        const bool last = l + 1 == f.layers;
        // the sums entering the layer are (x, la), those after the attention sublayer (x1, lb); the per-row
        // partial statistics are only needed where a map with a folded LayerNorm follows
        float2* ps = last ? nullptr : ws.ps;
        const ResidualSrc in = {x, ws.la, ws.sa, sg, sbeta, nullptr, nullptr, x1, ps, nullptr};
        const ResidualSrc mid = {x1, ws.lb, ws.sb, w.ln1_g, w.ln1_b, nullptr, nullptr, x, ps, nullptr};
        const ResidualSrc mid_cls = {x1, ws.lb, ws.sb, w.ln1_g, w.ln1_b, ws.row_start, ws.seq_len, x, ps, nullptr};
        // operands of the maps with a folded LayerNorm: row statistics and column sums
        const ResidualSrc fold_qkv = {nullptr, nullptr, ws.sa, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, w.c_qkv};
        const ResidualSrc fold_1 = {nullptr, nullptr, ws.sb, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, w.c_1};
        const float2* stats_in = l > 0 ? ws.ps : nullptr;   // (fused) pieces of the sums entering the layer; the embedding leaves statistics
        auto small = [&](const bf16_t* A, const void* W, const float* bias, const ResidualSrc& r, void* C, int N, int K,
                         const int32_t* n_rows, const float2* pieces, float2* stats_out) {
            return SmallGemm{A, (const bf16_t*)W, bias, r, C, vt, ws.max_rows, ws.likely_rows,
                             ws.likely_rows / (ws.padded ? 2 : 1), N, K, H, n_rows, rows, pieces, stats_out, 1.0f / (float)H, m->ln_eps, n_req, ws.row_start, ws.seq_len};
        };
        if (!last) {
            if (fused)
                PS_TIMED(PS_FAM_GEMM, launch_small_gemm_bf16(EPI_QKV, small(x, w.w_qkv, w.b_qkv, fold_qkv, qk, 3 * H, H, qkv_rows,
                                                                            stats_in, ws.sa), nullptr, s));
            else
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_QKV, x, (const bf16_t*)w.w_qkv, w.b_qkv, fold_qkv, qk, vt,
                                                       ws.max_rows, 3 * H, H, H, qkv_rows, &ws.meta->plan[PS_PLAN_QKV], clk, s));
        } else {
            // keys and values of all rows; queries of the requests' first rows only, by a side GEMM on
            // those rows gathered into the (not yet used) first-row buffer
            const ResidualSrc first_rows = {x, ws.la, ws.sa, nullptr, nullptr, ws.row_start, ws.seq_len, nullptr, nullptr, w.c_qkv};
            const ResidualSrc fold_kv = {nullptr, nullptr, ws.sa, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, w.c_qkv + H};
            if (fused) {
                const SkinnyArgs q = skinny_args(x, w.w_qkv, w.b_qkv, first_rows, qk, H, H, stats_in ? SKINNY_STATS_PIECES : SKINNY_STATS_GIVEN, nullptr);
                PS_TIMED(PS_FAM_GEMM, launch_small_gemm_bf16(EPI_KV, small(x, (const bf16_t*)w.w_qkv + (size_t)H * H, w.b_qkv + H, fold_kv, qk,
                                                                           2 * H, H, qkv_rows, stats_in, ws.sa), &q, s));
            } else {
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_KV, x, (const bf16_t*)w.w_qkv + (size_t)H * H, w.b_qkv + H, fold_kv,
                                                       qk, vt, ws.max_rows, 2 * H, H, H, qkv_rows, &ws.meta->plan[PS_PLAN_KV], clk, s));
                if (skinny) {
                    PS_TIMED(PS_FAM_REFINE, launch_skinny_gemm_bf16(EPI_Q_MAPPED, skinny_args(x, w.w_qkv, w.b_qkv, first_rows, qk, H, H,
                                                                                              SKINNY_STATS_GIVEN, nullptr), s));
                } else {
                    PS_TIMED(PS_FAM_REFINE, launch_cls_rows(m, n_req, ws, x, (bf16_t*)ws.cls_a, s));
                    PS_TIMED(PS_FAM_REFINE, side_gemm(EPI_Q_MAPPED, (const bf16_t*)ws.cls_a, w.w_qkv, w.b_qkv, first_rows, qk, H, H));
                }
            }
        }
        PS_TIMED(PS_FAM_ATTENTION, launch_attention_bf16(m, ws, last, s));
        // Output projection of all rows, and again for each request's first row from the hi | lo pairs the attention
        // kernel left in cls_a.  The feed-forward block again for those rows, the ones the head reads, with its input and
        // its GELU output carried as two bf16 values per element: bf16
        // rounding of these two tensors is the dominant error of the prediction and acts row by row, so the pass
        // removes it where it matters at < 1 % of the block's cost.
        const ResidualSrc in_cls = {x, ws.la, ws.sa, sg, sbeta, ws.row_start, ws.seq_len, x1, ps, nullptr};
        const ResidualSrc ffn_cls = {x1, ws.lb, ws.sb, w.ln1_g, w.ln1_b, ws.row_start, ws.seq_len, nullptr, nullptr, nullptr};
        if (skinny) {
            const SkinnyArgs so = skinny_args(ws.cls_a, w.w_od, w.b_o, in_cls, ws.lb, H, H, 0, nullptr);
            const SkinnyArgs s1 = skinny_args(nullptr, w.w_1d, w.b_1, ffn_cls, ws.cls_g, F, H,
                                              last ? SKINNY_STATS_ROWS : fused ? SKINNY_STATS_PIECES : SKINNY_STATS_GIVEN,
                                              last ? ws.sb : nullptr);
            const SkinnyArgs s2 = skinny_args(ws.cls_g, w.w_2d, w.b_2, mid_cls, ws.la, H, F, 0, nullptr);
            if (fused && !last) {
                PS_TIMED(PS_FAM_GEMM, launch_small_gemm_bf16(EPI_BIAS_RESIDUAL, small(att, w.w_o, w.b_o, in, ws.lb, H, H, rows, nullptr, nullptr), &so, s));
                PS_TIMED(PS_FAM_GEMM, launch_small_gemm_bf16(EPI_BIAS_GELU, small(x1, w.w_1, w.d_1, fold_1, g, F, H, rows, ws.ps, ws.sb), &s1, s));
                PS_TIMED(PS_FAM_GEMM, launch_small_gemm_bf16(EPI_BIAS_RESIDUAL, small(g, w.w_2, w.b_2, mid, ws.la, H, F, rows, nullptr, nullptr), &s2, s));
            } else if (!last) {
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_RESIDUAL, att, (const bf16_t*)w.w_o, w.b_o, in, ws.lb, nullptr, ws.max_rows,
                                                       H, H, H, rows, &ws.meta->plan[PS_PLAN_H], clk, s, ws.first_row, nullptr, &so));
                PS_TIMED(PS_FAM_LAYERNORM, ln_stats(ws.sb, true, nullptr));
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_GELU, x1, (const bf16_t*)w.w_1, w.d_1, fold_1, g, nullptr, ws.max_rows,
                                                       F, H, H, rows, &ws.meta->plan[PS_PLAN_F], clk, s, nullptr, nullptr, &s1));
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_RESIDUAL, g, (const bf16_t*)w.w_2, w.b_2, mid, ws.la, nullptr, ws.max_rows,
                                                       H, F, H, rows, &ws.meta->plan[PS_PLAN_H], clk, s, ws.first_row, nullptr, &s2));
            } else {
                PS_TIMED(PS_FAM_REFINE, launch_skinny_gemm_bf16(EPI_RESIDUAL_MAPPED, so, s));
                PS_TIMED(PS_FAM_REFINE, launch_skinny_gemm_bf16(EPI_GELU_SPLIT, s1, s));
                PS_TIMED(PS_FAM_REFINE, launch_skinny_gemm_bf16(EPI_RESIDUAL_MAPPED, s2, s));
            }
        } else if (carried && !last) {
            SmallGemm so = side_args(ws.cls_a, w.w_od, w.b_o, in_cls, ws.lb, H, H);
            SmallGemm s1 = side_args(ws.cls_a, w.w_1d, w.b_1, none, ws.cls_g, F, H);
            SmallGemm s2 = side_args(ws.cls_g, w.w_2d, w.b_2, mid_cls, ws.la, H, F);
            so.max_rows = s1.max_rows = s2.max_rows = (int64_t)align_up((size_t)n_req, 64);
            PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_RESIDUAL, att, (const bf16_t*)w.w_o, w.b_o, in, ws.lb, nullptr, ws.max_rows,
                                                   H, H, H, rows, &ws.meta->plan[PS_PLAN_H], clk, s, ws.first_row, &so));
            PS_TIMED(PS_FAM_LAYERNORM, ln_stats(ws.sb, true, &ffn_cls));
            PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_GELU, x1, (const bf16_t*)w.w_1, w.d_1, fold_1, g, nullptr, ws.max_rows,
                                                   F, H, H, rows, &ws.meta->plan[PS_PLAN_F], clk, s, nullptr, &s1));
            PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_RESIDUAL, g, (const bf16_t*)w.w_2, w.b_2, mid, ws.la, nullptr, ws.max_rows,
                                                   H, F, H, rows, &ws.meta->plan[PS_PLAN_H], clk, s, ws.first_row, &s2));
        } else {
            if (!last)
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_RESIDUAL, att, (const bf16_t*)w.w_o, w.b_o, in, ws.lb,
                                                       nullptr, ws.max_rows, H, H, H, rows, &ws.meta->plan[PS_PLAN_H], clk, s));
            PS_TIMED(PS_FAM_REFINE, side_gemm(EPI_RESIDUAL_MAPPED, (const bf16_t*)ws.cls_a, w.w_od, w.b_o, in_cls, ws.lb, H, H));
            PS_TIMED(PS_FAM_LAYERNORM, ln_stats(ws.sb, !last, &ffn_cls));
            if (!last) {
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_GELU, x1, (const bf16_t*)w.w_1, w.d_1, fold_1, g, nullptr,
                                                       ws.max_rows, F, H, H, rows, &ws.meta->plan[PS_PLAN_F], clk, s));
                PS_TIMED(PS_FAM_GEMM, launch_gemm_bf16(EPI_BIAS_RESIDUAL, g, (const bf16_t*)w.w_2, w.b_2, mid, ws.la,
                                                       nullptr, ws.max_rows, H, F, H, rows, &ws.meta->plan[PS_PLAN_H], clk, s));
            }
            if (ws.cls_rows / 64 * (F / 64) > PS_SPLIT_TILES)
                PS_TIMED(PS_FAM_REFINE, launch_gemm_bf16(EPI_GELU_SPLIT, (const bf16_t*)ws.cls_a, (const bf16_t*)w.w_1d, w.b_1, none,
                                                         ws.cls_g, nullptr, ws.cls_rows, F, 2 * H, H, n_req_dev, nullptr, nullptr, s));
            else
                PS_TIMED(PS_FAM_REFINE, side_gemm(EPI_GELU_SPLIT, (const bf16_t*)ws.cls_a, w.w_1d, w.b_1, none, ws.cls_g, F, H));
            PS_TIMED(PS_FAM_REFINE, side_gemm(EPI_RESIDUAL_MAPPED, (const bf16_t*)ws.cls_g, w.w_2d, w.b_2, mid_cls, ws.la, H, F));
        }
        if (!last && !fused)                             // (the head makes the last LayerNorm's statistics itself)
            PS_TIMED(PS_FAM_LAYERNORM, ln_stats(ws.sa, true, nullptr));
        sg = w.ln2_g;
        sbeta = w.ln2_b;
    }
#undef PS_TIMED
}
