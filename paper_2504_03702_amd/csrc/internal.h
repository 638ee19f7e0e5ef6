// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "preserve.h"

typedef uint16_t bf16_t;   // raw bf16 bit pattern

#define PS_ROW_ALIGN   8     // every request starts at a multiple of this many activation rows
#define PS_ROW_TILE    256   // activation buffers are padded to a multiple of this many rows
#define PS_ATT_BQ      128   // query rows per attention workgroup (bf16 path)
#define PS_MAX_ROWS    ((int64_t)1 << 27)   // most activation rows one call may need (tokens + requests * (M + 8))
#define PS_KEY_SLACK   64    // the last key tile of a request reads up to this many rows past its end: they
                             // must hold finite numbers (their weights are exactly zero), so the embedding
                             // zero-fills and the GEMMs cover that many rows beyond the last request

// Device weights of one encoder layer.  bf16 models: matrices are bf16, stored [out][in]
// (the contraction index contiguous) for the MFMA kernels; fp32 models: float, [in][out].
struct LayerWeights {
    void *w_qkv, *w_o, *w_1, *w_2;
    void *w_od, *w_1d, *w_2d;    // bf16 models: the plain W_o, W_1, W_2 of the per-request pass (w_1 has a LayerNorm folded in)
    float *b_qkv, *b_o, *b_1, *b_2;
    // bf16 models: the LayerNorm in front of the QKV and the first feed-forward map is folded into them.
    // With x = (y - mean) * rstd * gamma + beta:  x W + b = rstd * (y (gamma W) - mean * c) + d,
    // c[n] = sum_k gamma[k] W[k][n], d[n] = b[n] + sum_k beta[k] W[k][n].  w_qkv and w_1 hold gamma W,
    // b_qkv holds d of the QKV map, d_1 that of W_1 (b_1 stays the plain bias: the first-row pass uses it
    // with the plain w_1d), c_qkv and c_1 the column sums taken over the rounded gamma W.
    float *c_qkv, *c_1, *d_1;
    float *ln1_g, *ln1_b, *ln2_g, *ln2_b;
};

struct ProfRecord {
    int family;
    hipEvent_t start, stop;
};

struct ps_model {
    // event records of ps_profile_enable(); mutable so launch code holding a const model can log
    mutable bool profiling = false;
    mutable std::vector<ProfRecord> prof;
    mutable std::vector<hipEvent_t> event_pool;
    ps_model_info info;
    float ln_eps;
    int device;
    int lds_max;                 // largest LDS allocation of one workgroup on this device
    int64_t* clk_slot;           // device: {core cycles, timer ticks} of the last profiled GEMM launch
    void* blob;                  // the one device allocation everything below points into
    size_t blob_bytes;
    void *e_tok, *e_pos, *e_soft;     // embedding tables in the model's dtype, [rows][hidden]
    float *lne_g, *lne_b;
    std::vector<LayerWeights> layers;
    float *w_h1t;                // [head_hidden][hidden]
    float *b_h1, *w_h2;
    float b_h2;
};

// How a map's rows are cut into tiles (gemm_bf16.hip): m_tiles tiles of 256 rows, then tiles of 32 (tm0 + tm1) rows.
struct GemmPlan {
    int32_t m_tiles, tm0, tm1;
};
enum { PS_PLAN_QKV = 0, PS_PLAN_KV = 1, PS_PLAN_H = 2, PS_PLAN_F = 3, PS_PLANS = 4 };

// Per-call bookkeeping the prep kernel writes at the start of the workspace.
struct BatchMeta {
    int32_t total_rows;          // activation rows in use (padded request starts included)
    int32_t total_qtiles;        // attention query tiles over all requests
    int32_t n_req;               // requests in this call (row count of the per-request side GEMMs)
    int32_t qkv_rows;            // total_rows + PS_KEY_SLACK: rows the QKV projection covers
    GemmPlan plan[PS_PLANS];     // tiles of the maps of all rows
};

// Carved-up workspace of one ps_predict_load call.
struct Workspace {
    BatchMeta* meta;
    int32_t *seq_len;            // [B]   rows of request r (text + learnable prompts), 0 if faulty
    int32_t *row_start;          // [B+1] first activation row of request r
    int32_t *qtile_start;        // [B]   first attention query tile of request r (longest requests first in calls of many)
    int4 *qtiles;                // bf16 path: [query tiles] {first row and rows of the tile's request, its first query, request}
    int32_t *bad_req;            // [B]   set when a request's text holds an invalid token id
    int32_t *head_done;          // [B]   workgroups of the head that have left their sum
    float *head_sum;             // [B][32] the sums of their rounds of 64 hidden units
    void *x, *qkv, *vt, *att, *y, *x1, *g;
    // bf16 path: the residual stream is kept as the pre-LayerNorm sums of the last two sublayers,
    // each sum a float in two 16-bit halves hi and lo (device_util.h, stream_join), plus each row's (mean, 1/std); its
    // LayerNorm is recomputed wherever it is needed.  The hi parts are x (sums entering a layer) and x1
    // (sums after the attention sublayer): exactly the operands of the maps the LayerNorms are folded into.
    bf16_t *la, *lb;             // lo parts belonging to x and x1
    float2 *sa, *sb;
    float2 *ps;                  // [rows][hidden / 64] per-row partial (sum, sum of squares) of the newest sums
    uint8_t* first_row;          // [rows] bf16 path: 1 for the first row of a request
    void *cls_a, *cls_g;         // per-request rows of the [CLS] refinement: [cls_rows][2H], [cls_rows][2F] bf16
    int64_t cls_rows;
    int64_t max_rows;            // rows every activation buffer holds (multiple of PS_ROW_TILE)
    int64_t likely_rows;         // rows in use if the caller's offsets do not overlap (for choices that change no result)
    bool padded;                 // the caller's layout: how many of the rows are in use is for the device to know
    int64_t max_qtiles;
    size_t bytes;
};

Workspace plan_workspace(const ps_model_info& info, int64_t n_tokens, int32_t n_req, void* base);

// ---- launchers (each enqueues on `s`; all pointers are device pointers) -------------------
void launch_prep(const ps_model* m, const int32_t* offsets, const int32_t* lengths, int32_t n_req, int64_t n_tokens,
                 const Workspace& ws, ps_status* st, hipStream_t s);
void launch_embed(const ps_model* m, const int32_t* token_ids, const int32_t* offsets, int32_t n_req,
                  const Workspace& ws, ps_status* st, hipStream_t s);
void launch_head(const ps_model* m, int32_t n_req, const Workspace& ws, float* pred_f, int32_t* pred_tokens,
                 ps_status* st, hipStream_t s);
void run_encoder_f32(const ps_model* m, int32_t n_req, const Workspace& ws, hipStream_t s);
#define PS_NARROW_WIDTH 256  // fp32 models up to this hidden size (a multiple of 32): LayerNorms in one order of sums everywhere
// Whether that leaves the last layer's sums, not their LayerNorm, in ws.x (calls of few rows through a narrow model).
bool f32_maps_take_norms(const ps_model_info& info, int64_t max_rows);
void run_encoder_bf16(const ps_model* m, int32_t n_req, const Workspace& ws, hipStream_t s);

// bf16 kernels
enum GemmEpilogue {
    EPI_BIAS_GELU = 1, EPI_BIAS_RESIDUAL = 2, EPI_QKV = 3,
    EPI_GELU_SPLIT = 4,          // GELU, then the fp32 value stored as two bf16 (value ~ hi + lo) in [rows][2N]
    EPI_RESIDUAL_MAPPED = 5,     // EPI_BIAS_RESIDUAL with GEMM row r living at stream row row_map[r]
    EPI_KV = 6,                  // EPI_QKV without the query columns: W holds the key and value rows only
    EPI_Q_MAPPED = 7             // query columns only, GEMM row r stored at row row_map[r] of the [rows][2H] buffer
};
// The residual stream entering a sublayer: LayerNorm(y) with the row statistics already known.
struct ResidualSrc {
    const bf16_t* y_hi;      // [rows][hidden] pre-LayerNorm sums, value = stream_join(hi, lo)
    const bf16_t* y_lo;
    const float2* stats;     // [rows] (mean, 1 / sqrt(var + eps))
    const float* gamma;
    const float* beta;
    const int32_t* row_map;  // EPI_RESIDUAL_MAPPED: stream row of GEMM row r (the request's first row)
    const int32_t* seq_len;  //                       rows with seq_len[r] <= 0 are not stored
    // residual epilogues: the hi parts of the new sums (the lo parts go to the C argument); hi is also
    // the next map's operand.  Every 64-column piece of a row leaves its (sum, sum of squares) in
    // pstats[row][N / 64] (may be null for the per-request maps)
    bf16_t* x_out;
    float2* pstats;
    // epilogues of the maps a LayerNorm is folded into (EPI_QKV, EPI_KV, EPI_Q_MAPPED, EPI_BIAS_GELU):
    // `stats` are the statistics of the operand's rows, colsum is c above and the bias argument is d
    const float* colsum;
};
// The per-request forms (EPI_GELU_SPLIT, EPI_RESIDUAL_MAPPED, EPI_Q_MAPPED) for calls of at most PS_SKINNY_ROWS
// requests: a stream over W with the contraction split among a workgroup's wavefronts.
#define PS_SKINNY_ROWS 16
// Calls of more than PS_SKINNY_ROWS and up to this many requests: the launches of the maps of all rows carry the per-request ones
// in further workgroups, which take the units that the launch's last round leaves idle (64 padded prompts of hidden 768: of 256
// units the maps back to it use 200 to 230), instead of three launches of 7 to 15 us that use a few units each.  Milliseconds,
// apart / carried: six-layer encoder 17 requests 0.839 / 0.732, 40 1.213 / 1.046, 128 2.99 / 2.87, 256 5.25 / 5.13, 512 9.77 / 9.66;
// padded twelve-layer 33 2.80 / 2.33, 64 4.37 / 4.11, 200 10.96 / 10.75; packed 17 2.07 / 1.71, 400 20.06 / 19.82, 1024 49.8 / 49.6,
// 2048 even; production 24 6.82 / 6.49, 100 22.6 / 22.1, 400 78.7 / 78.4.
// In models wider than 768 the per-request tiles outgrow the idle units sooner, most of all beside short prompts, whose maps of all
// rows are short (three layers, prompts of 4 to 12 tokens, apart / carried: hidden 1024 600 requests 0.954 / 0.919, 700 1.061 / 1.086;
// 1280 400 1.012 / 0.972, 500 1.132 / 1.151; 1536 400 1.278 / 1.227, 700 1.875 / 1.943; 2048 300 1.701 / 1.612, 400 1.897 / 1.922,
// 1000 3.97 / 4.25; of 10 to 60 tokens 1024 700 2.214 / 2.173, 1280 500 2.300 / 2.246, 1536 500 3.013 / 3.003, 1000 5.94 / 6.08, 2048
// 400 4.069 / 4.010, 700 6.92 / 7.00, 1000 9.51 / 9.77): there requests times hidden size have a line, with fewer rows a request a
// lower one.
#define PS_CARRIED_REQUESTS 1024
#define PS_CARRIED_WIDTHS (800 * 1024)
#define PS_CARRIED_WIDTHS_SHORT (600 * 1024)
enum SkinnyStats { SKINNY_STATS_GIVEN = 0, SKINNY_STATS_PIECES = 1, SKINNY_STATS_ROWS = 2 };
struct SkinnyArgs {
    const bf16_t *A, *W;         // A: EPI_RESIDUAL_MAPPED only (the other two read the stream rows of the first tokens)
    const float* bias;
    ResidualSrc res;
    void* C;
    int N, K, hidden, n_req;
    // EPI_GELU_SPLIT, EPI_Q_MAPPED: where the first rows' LayerNorm statistics come from: res.stats, the 64-column
    // pieces in pstats_in, or two passes over the rows; stats_out (may be null) gets them
    int stats_from;
    const float2* pstats_in;
    float2* stats_out;
    float inv_n, eps;
};
void launch_skinny_gemm_bf16(GemmEpilogue epi, const SkinnyArgs& p, hipStream_t s);
// The maps of calls with few activation rows (tiles of 64 x 64 to 128 x 128, one workgroup each).  `side`: for
// EPI_BIAS_RESIDUAL, EPI_BIAS_GELU and EPI_KV the per-request map of the same layer, done by further workgroups of the
// launch (null for the others); rows of the residual stream that it writes are left to it.  pstats_in, if not null: the statistics of the operand's rows are made from these pieces
// and left in stats_out (res.stats otherwise).
struct SmallGemm {
    const bf16_t *A, *W;
    const float* bias;
    ResidualSrc res;
    void* C;
    bf16_t* vt;
    int64_t max_rows;            // rows the buffers hold; also the row stride of vt
    int64_t likely_rows;         // rows by which the tiles are chosen (0: max_rows)
    int64_t usual_rows;          // of padded calls half of them (0: max_rows)
    int N, K, hidden;
    const int32_t* rows;         // rows to compute
    const int32_t* live_rows;    // rows that belong to requests (the others take statistics of zero)
    const float2* pstats_in;
    float2* stats_out;
    float inv_n, eps;
    int n_side;                  // requests whose first rows the side map writes (0 without one)
    const int32_t *row_start, *seq_len;
};
void launch_small_gemm_bf16(GemmEpilogue epi, const SmallGemm& p, const SkinnyArgs* side, hipStream_t s);
// Whether a call of a few requests takes the small tiles, whose launches carry both maps: up to 3584 rows (of the workspace), of
// wide models fewer.  What of a padded call's slots is filled the host cannot see: those go by a line of their own.  Against the
// large tiles with the side maps carried, small / large, us, four layers, the lengths equal: packed, hidden 768, 2816 rows 378 /
// 420, 437 / 432, 3072 431 / 430, 3328 452 / 452; 1024, 2048 rows 410 / 478, 2304 484 / 484; 2048, 1280 rows 788 / 877, 1536 855 /
// 890 and 920 / 923, 1792 966 / 924, 2048 1120 / 1003.  Padded to 512 and filled to a half / full: hidden 768, 4352 rows 385 /
// 414 and 546 / 491, 4864 400 / 432 and 600 / 510; 1024, 3840 rows 480 / 496 and 694 / 588, 4352 497 / 515 and 872 / 672; 2048,
// 3840 rows 1358 / 1123 and 2364 / 1445; 3328 rows, where a quarter is 837 / 897 and a half 1089 / 976, are left to the small tiles.
inline bool small_maps(const Workspace& ws, int32_t n_req, int hidden) {
    auto within = [](int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : v > hi ? hi : v; };
    const int64_t most = ws.padded ? within(3932160 / hidden, 3584, 4608) : within(2300000 / hidden, 1536, 3584);
    return n_req <= PS_SKINNY_ROWS && ws.max_rows <= most;
}
// Whether the large maps of a call carry its per-request ones (the others have launches of their own, or take the small tiles).
inline bool carries_side_maps(const Workspace& ws, int32_t n_req, int hidden) {
    const int64_t most = ws.max_rows < 32 * (int64_t)n_req ? PS_CARRIED_WIDTHS_SHORT : PS_CARRIED_WIDTHS;
    const bool fits = n_req <= PS_CARRIED_REQUESTS && (hidden <= 768 || (int64_t)n_req * hidden <= most);
    return fits && !small_maps(ws, n_req, hidden);
}
// Whether a map of `max_rows` rows takes 256 x 256 tiles.
inline bool large_tiles(int64_t max_rows, int N) { return (max_rows + 255) / 256 * (N / 256) >= 128; }
// C[rows, N] = A[rows, K] * W^T (+ epilogue); W is [N][K] (EPI_GELU_SPLIT: [N][K / 2], A is hi | lo); rows = *total_rows (device).
// The residual epilogues write the new sums as hi (residual.x_out) + lo (C) bf16 pairs; all epilogues write bf16.  clk (device,
// may be null): workgroup 0 leaves {core clock cycles, constant-rate timer ticks} of its run there.
// side, few: EPI_BIAS_RESIDUAL and EPI_BIAS_GELU can carry the per-request map of the same sublayer (EPI_RESIDUAL_MAPPED,
// EPI_GELU_SPLIT) in further workgroups, few for at most PS_SKINNY_ROWS requests; rows that first_row marks are then left to it.
void launch_gemm_bf16(GemmEpilogue epi, const bf16_t* A, const bf16_t* W, const float* bias,
                      ResidualSrc res, void* C, bf16_t* vt, int64_t max_rows, int N, int K,
                      int hidden, const int32_t* total_rows, const GemmPlan* plan, int64_t* clk, hipStream_t s,
                      const uint8_t* first_row = nullptr, const SmallGemm* side = nullptr, const SkinnyArgs* few = nullptr);
// out[r][0:hidden] = x[first row of request r] for every request (zeros for faulty ones and padding rows).
void launch_cls_rows(const ps_model* m, int32_t n_req, const Workspace& ws, const bf16_t* x, bf16_t* out, hipStream_t s);
// first_rows_only: compute (at least) the first query row of every request and nothing beyond its
// first 32 rows; the rest of the output buffer keeps its old contents.
void launch_attention_bf16(const ps_model* m, const Workspace& ws, bool first_rows_only, hipStream_t s);
// Brackets the launches made during its lifetime with two events when profiling is on.
struct ProfScope {
    const ps_model* m;
    hipStream_t s;
    ProfRecord rec;
    bool live;
    ProfScope(const ps_model* model, int family, hipStream_t stream) : m(model), s(stream), live(false) {
        if (!m->profiling) return;
        hipEvent_t ev[2];
        for (int i = 0; i < 2; ++i) {
            if (!m->event_pool.empty()) {
                ev[i] = m->event_pool.back();
                m->event_pool.pop_back();
            } else if (hipEventCreate(&ev[i]) != hipSuccess) {
                return;
            }
        }
        rec = {family, ev[0], ev[1]};
        live = hipEventRecord(rec.start, s) == hipSuccess;
    }
    ~ProfScope() {
        if (!live) return;
        (void)hipEventRecord(rec.stop, s);
        m->prof.push_back(rec);
    }
};

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
