// Per-call bookkeeping, embedding gather + LayerNorm, and the pooling + regression head.
// These kernels are shared by the fp32 and the bf16 encoder paths.
#include "device_util.h"
#include "internal.h"

namespace {

// How a map of `rows` rows and n tile columns is cut into tiles for 256 workgroups (the whole wavefront calls, every lane
// weighs one candidate): all rows in tiles of one height, or as many whole rounds of 256-row tiles as there are (or one
// fewer) and the rest in tiles of one height.  Costs in thousandths of a full round of 256-row tiles.  A full round of
// lower tiles costs more than its share of rows (measured on 250 k and 440 k rows, the maps of hidden 768 and 1024: 224 rows
// 1.00-1.05 per row, 1.02 on average, 192 1.02-1.10, 1.04, 160 1.05-1.18, 1.11, 128 1.10-1.28, 1.19); a last round that leaves units idle runs
// faster, the chip's power being shared by fewer, down to 0.68 of a full one (153 tiles of 256 rows, contraction 3072:
// 70 us against 103).  Where all tiles fit one round, the lowest that do are the fastest however many units that leaves
// idle: query-key-value map of hidden 768, 4600 rows, 256 to 192 rows 26.9 / 26.3 / 24.9 us; maps back to hidden 1024,
// 8050 rows, 256 to 128 65.1 / 62.2 / 60.3 / 58.0 / 55.5; hidden 768, 16700 rows, 256 and 224 68.9 / 64.5.
__device__ GemmPlan plan_gemm(int rows, int n) {
    const int lane = threadIdx.x & 63;
    const int heights[5] = {8, 7, 6, 5, 4}, costs[5] = {1000, 888, 780, 690, 600};   // heights in blocks of 32 rows
    const int tiles = (rows + 255) / 256 * n, pick = min(lane / 5, 2);
    int h = 8, c = 1000;
#pragma unroll
    for (int i = 1; i < 5; ++i)
        if (lane % 5 == i) { h = heights[i]; c = costs[i]; }
    const int rounds = max(pick == 0 ? 0 : tiles / 256 - (pick - 1), 0), m = rounds * 256 / n;
    const int left = max(rows - 256 * m, 0), rest = (left + 32 * h - 1) / (32 * h) * n;
    int64_t cost = (int64_t)rounds * 1000 + (int64_t)(rest / 256) * c + (rounds > 0 ? 50 : 0);
    if (rounds == 0 && rest <= 256) cost = c;
    else if (rest % 256) cost += (int64_t)c * max(680, (rest % 256) * 1000 / 256) / 1000;
    int64_t best = lane < 15 ? cost * 64 + lane : INT64_MAX;
    for (int o = 8; o > 0; o >>= 1) {
        const int64_t other = __shfl_xor(best, o, 16);
        best = other < best ? other : best;
    }
    const int at = (int)(__shfl(best, 0, 64) & 63);
    return GemmPlan{__shfl(m, at, 64), (__shfl(h, at, 64) + 1) / 2, __shfl(h, at, 64) / 2};
}

// ------------------------------------------------------------------------------------------
// prep: one workgroup turns (offsets, lengths) into the packed row layout of this call.
// Request r occupies activation rows [row_start[r], row_start[r] + seq_len[r]); row_start is a
// multiple of PS_ROW_ALIGN.  A request with an impossible length, or whose span leaves the
// token array, gets seq_len 0.  The workspace was sized by the host for n_tokens token slots;
// offsets that overlap can ask for more rows than that: requests from the first one that does
// not fit onwards are dropped the same way, so no later kernel indexes past `row_capacity`.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void prep_kernel(const int32_t* __restrict__ offsets,
                                                    const int32_t* __restrict__ lengths, int n_req,
                                                    int n_soft, int max_pos, long long n_tokens,
                                                    long long row_capacity, int4 plan_cols, int sort_tiles, BatchMeta* meta,
                                                    int32_t* seq_len, int32_t* row_start,
                                                    int32_t* qtile_start, int32_t* bad_req,
                                                    int32_t* head_done, ps_status* st) {
    __shared__ long long s_rows[16], s_tiles[16];     // totals of the wavefronts
    __shared__ long long s_cut_rows, s_cut_tiles;     // rows / query tiles in front of the first request that does not fit
    __shared__ int s_class[64];                       // query tiles of the requests of one length (in key tiles)
    const int tid = threadIdx.x;
    if (tid < 64) s_class[tid] = 0;
    const int per = (n_req + 1023) / 1024;
    const int r0 = min(tid * per, n_req);
    const int r1 = min(r0 + per, n_req);
    long long rows = 0, tiles = 0;
    for (int r = r0; r < r1; ++r) {
        const long long o0 = offsets[r], o1 = offsets[r + 1];
        const long long span = o1 - o0;
        const long long len = lengths ? (long long)lengths[r] : span;
        const bool bad = o0 < 0 || o1 > n_tokens || span < 0 || len < 1 || len > span || len > max_pos - n_soft;
        const int S = bad ? 0 : (int)len + n_soft;
        if (bad) report_fault(st, PS_ST_BAD_LENGTH, r);
        seq_len[r] = S;
        bad_req[r] = 0;
        head_done[r] = 0;
        rows += (S + PS_ROW_ALIGN - 1) / PS_ROW_ALIGN * PS_ROW_ALIGN;
        tiles += (S + PS_ATT_BQ - 1) / PS_ATT_BQ;
    }
    // exclusive prefix sums over the threads: within a wavefront, then the wavefronts in front of it
    long long row_incl = rows, tile_incl = tiles;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long a = __shfl_up(row_incl, o, 64), b = __shfl_up(tile_incl, o, 64);
        if ((tid & 63) >= o) { row_incl += a; tile_incl += b; }
    }
    if ((tid & 63) == 63) {
        s_rows[tid >> 6] = row_incl;
        s_tiles[tid >> 6] = tile_incl;
    }
    __syncthreads();
    long long row = row_incl - rows, tile = tile_incl - tiles, all_rows = 0, all_tiles = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < tid >> 6) { row += s_rows[w]; tile += s_tiles[w]; }
        all_rows += s_rows[w];
        all_tiles += s_tiles[w];
    }
    if (tid == 0) {
        s_cut_rows = all_rows;
        s_cut_tiles = all_tiles;
    }
    __syncthreads();
    // Row starts are non-decreasing, so the requests that do not fit the workspace are a suffix: the first of
    // them starts where the last fitting one ends.
    bool cut_here = false;
    long long my_cut_rows = 0, my_cut_tiles = 0;
    for (int r = r0; r < r1; ++r) {
        const int S = seq_len[r];
        const long long sz = (S + PS_ROW_ALIGN - 1) / PS_ROW_ALIGN * PS_ROW_ALIGN;
        if (row + sz > row_capacity) {
            if (!cut_here && row <= row_capacity) { cut_here = true; my_cut_rows = row; my_cut_tiles = tile; }
            if (S > 0) report_fault(st, PS_ST_BAD_LENGTH, r);
            seq_len[r] = 0;
            row_start[r] = -1;                       // set below, once the cut is known
        } else {
            row_start[r] = (int32_t)row;
            qtile_start[r] = (int32_t)tile;
        }
        row += sz;
        tile += (S + PS_ATT_BQ - 1) / PS_ATT_BQ;
    }
    // at most one thread holds the first request that does not fit with a start inside the capacity
    if (cut_here) {
        s_cut_rows = my_cut_rows;
        s_cut_tiles = my_cut_tiles;
    }
    __syncthreads();
    const long long cut_rows = min(s_cut_rows, row_capacity), cut_tiles = s_cut_tiles;
    for (int r = r0; r < r1; ++r) {
        if (row_start[r] < 0) {
            row_start[r] = (int32_t)cut_rows;
            qtile_start[r] = (int32_t)cut_tiles;
        }
    }
    if (sort_tiles) {
        // Query tiles of the longest requests first: a tile takes as long as its request has keys, and the last ones to
        // start are what the attention kernel ends with.  Requests of one length in any order (no result depends on it).
        auto length_class = [](int S) { return 63 - min((S + 63) / 64, 63); };
        for (int r = r0; r < r1; ++r)
            if (seq_len[r] > 0) atomicAdd(&s_class[length_class(seq_len[r])], (seq_len[r] + PS_ATT_BQ - 1) / PS_ATT_BQ);
        __syncthreads();
        if (tid < 64) {
            const int own = s_class[tid];
            int incl = own;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int a = __shfl_up(incl, o, 64);
                if (tid >= o) incl += a;
            }
            s_class[tid] = incl - own;
        }
        __syncthreads();
        for (int r = r0; r < r1; ++r)
            if (seq_len[r] > 0)
                qtile_start[r] = atomicAdd(&s_class[length_class(seq_len[r])], (seq_len[r] + PS_ATT_BQ - 1) / PS_ATT_BQ);
    }
    if (tid == 1023) {
        row_start[n_req] = (int32_t)cut_rows;
        meta->total_rows = (int32_t)cut_rows;
        meta->total_qtiles = (int32_t)cut_tiles;
        meta->n_req = n_req;
        meta->qkv_rows = (int32_t)cut_rows + PS_KEY_SLACK;
    }
    const int plan = tid >> 6;                       // a wavefront each; tile columns of the maps, none for fp32 models
    if (plan < PS_PLANS && plan_cols.x > 0) {
        const int n = plan == PS_PLAN_QKV ? plan_cols.x : plan == PS_PLAN_KV ? plan_cols.y : plan == PS_PLAN_H ? plan_cols.z : plan_cols.w;
        const GemmPlan p = plan_gemm((int)cut_rows + (plan == PS_PLAN_QKV || plan == PS_PLAN_KV ? PS_KEY_SLACK : 0), n);
        if ((tid & 63) == 0) meta->plan[plan] = p;
    }
}

template <typename T> __device__ inline float load_elem(const T* p, int64_t i);
template <> __device__ inline float load_elem<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ inline float load_elem<bf16_t>(const bf16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
template <typename T> __device__ inline void store_elem(T* p, int64_t i, float v);
template <> __device__ inline void store_elem<float>(float* p, int64_t i, float v) { p[i] = v; }
template <> __device__ inline void store_elem<bf16_t>(bf16_t* p, int64_t i, float v) { p[i] = f32_to_bf16(v); }

// ------------------------------------------------------------------------------------------
// embed: one wavefront per activation row.  Text rows gather a token embedding, the last n_soft
// rows of a request take the learnable prompt vectors; both add the position embedding of the
// row's index within its request and go through the embedding LayerNorm.  Rows that belong to
// no request (alignment gaps, the tail up to the next row tile) are zero-filled so that every
// row a later tile touches holds finite numbers.
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const int32_t* __restrict__ token_ids,
                                                    const int32_t* __restrict__ offsets, int n_req,
                                                    const T* __restrict__ e_tok, const T* __restrict__ e_pos,
                                                    const T* __restrict__ e_soft,
                                                    const float* __restrict__ gamma,
                                                    const float* __restrict__ beta, float eps, int H,
                                                    int vocab, int n_soft, const BatchMeta* meta,
                                                    const int32_t* __restrict__ seq_len,
                                                    const int32_t* __restrict__ row_start,
                                                    int32_t* bad_req, T* __restrict__ x,
                                                    bf16_t* __restrict__ lo_out, float2* __restrict__ stats_out,
                                                    const int32_t* __restrict__ qtile_start, int4* __restrict__ qtiles,
                                                    uint8_t* __restrict__ first_row, ps_status* st) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int total = meta->total_rows;
    // calls of at most 64 requests: what a lane's request has is one trip to memory, and a count of the starts up to the row
    // finds the row's own (by bisection and one after the other it was a trip each: 768 rows of 16 requests, hidden 128, 5.0 ->
    // 4.4 us)
    const int few = n_req <= 64 ? min(lane, n_req - 1) : -1;
    const int q_start = few >= 0 ? row_start[few] : 0, q_len = few >= 0 ? seq_len[few] : 0, q_first = few >= 0 ? offsets[few] : 0;
    const int64_t live = ((int64_t)total + PS_KEY_SLACK + PS_ROW_TILE - 1) / PS_ROW_TILE * PS_ROW_TILE;
    if (row >= live) return;
    T* out = x + row * H;
    bf16_t* yrow = lo_out ? lo_out + row * H : nullptr;  // bf16 path: lo parts of the sums, and row statistics
    int r = -1, p = 0, S = 0, first = 0;
    if (row < total && few >= 0) {
        r = __popcll(__ballot(lane < n_req && q_start <= row)) - 1;
        p = (int)(row - __builtin_amdgcn_readlane(q_start, r));
        S = __builtin_amdgcn_readlane(q_len, r);
        first = __builtin_amdgcn_readlane(q_first, r);
    } else if (row < total) {
        int lo = 0, hi = n_req - 1;          // largest r with row_start[r] <= row
        while (lo < hi) {
            int mid = (lo + hi + 1) >> 1;
            if (row_start[mid] <= row) lo = mid; else hi = mid - 1;
        }
        r = lo;
        p = (int)(row - row_start[r]);
        S = seq_len[r];
        first = offsets[r];
    }
    if (first_row && lane == 0) first_row[row] = r >= 0 && S > 0 && p == 0;
    if (r < 0 || p >= S) {
        for (int i = lane; i < H; i += 64) {
            store_elem<T>(out, i, 0.f);
            if (yrow) yrow[i] = (bf16_t)PS_STREAM_ZERO_LO;
        }
        if (yrow && lane == 0) stats_out[row] = make_float2(0.f, 0.f);
        return;
    }
    if (qtiles && lane == 0 && p % PS_ATT_BQ == 0)
        qtiles[qtile_start[r] + p / PS_ATT_BQ] = make_int4((int)row - p, S, p, r);
    const int n_text = S - n_soft;
    const T* src;
    if (p < n_text) {
        const int id = token_ids[first + p];
        if (id < 0 || id >= vocab) {
            // faulty request: flagged here, its row zeroed; the head reports NaN / -1 for it
            if (lane == 0) {
                report_fault(st, PS_ST_BAD_TOKEN, r);
                bad_req[r] = 1;
            }
            for (int i = lane; i < H; i += 64) {
                store_elem<T>(out, i, 0.f);
                if (yrow) yrow[i] = (bf16_t)PS_STREAM_ZERO_LO;
            }
            if (yrow && lane == 0) stats_out[row] = make_float2(0.f, 0.f);
            return;
        }
        src = e_tok + (int64_t)id * H;
    } else {
        src = e_soft + (int64_t)(p - n_text) * H;
    }
    const T* pos = e_pos + (int64_t)p * H;
    if (sizeof(T) == 2 && yrow) {
        // bf16 models (H a multiple of 256, at most 2048): the row stays in registers, lane l holding the
        // 4-element chunks l, l + 64, ...; 8-byte loads, one pass over the tables
        const int nch = H >> 8;
        float4 e[8];
        float sum = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (c < nch) {
                const uint2 a = ((const uint2*)src)[lane + 64 * c], b = ((const uint2*)pos)[lane + 64 * c];
                e[c].x = __uint_as_float(a.x << 16) + __uint_as_float(b.x << 16);
                e[c].y = __uint_as_float(a.x & 0xffff0000u) + __uint_as_float(b.x & 0xffff0000u);
                e[c].z = __uint_as_float(a.y << 16) + __uint_as_float(b.y << 16);
                e[c].w = __uint_as_float(a.y & 0xffff0000u) + __uint_as_float(b.y & 0xffff0000u);
                sum += (e[c].x + e[c].y) + (e[c].z + e[c].w);
            }
        }
        const float mean = wave_sum(sum) / (float)H;
        float sq = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (c < nch) {
                const float dx = e[c].x - mean, dy = e[c].y - mean, dz = e[c].z - mean, dw = e[c].w - mean;
                sq += (dx * dx + dy * dy) + (dz * dz + dw * dw);
            }
        }
        const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)H + eps);
        // the sums as hi and lo (stream_split2); hi, not normalised, is the operand of the first QKV map, which has the
        // embedding LayerNorm folded into its weights and finishes it from the row statistics
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (c < nch) {
                uint2 hi, lo;
                stream_split2(stream_ties_to_even(e[c].x), stream_ties_to_even(e[c].y), hi.x, lo.x);
                stream_split2(stream_ties_to_even(e[c].z), stream_ties_to_even(e[c].w), hi.y, lo.y);
                ((uint2*)out)[lane + 64 * c] = hi;
                ((uint2*)yrow)[lane + 64 * c] = lo;
            }
        }
        if (lane == 0) stats_out[row] = make_float2(mean, rstd);
        return;
    }
    float sum = 0.f;
    for (int i = lane; i < H; i += 64) sum += load_elem<T>(src, i) + load_elem<T>(pos, i);
    const float mean = wave_sum(sum) / (float)H;
    float sq = 0.f;
    for (int i = lane; i < H; i += 64) {
        const float dlt = load_elem<T>(src, i) + load_elem<T>(pos, i) - mean;
        sq += dlt * dlt;
    }
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)H + eps);
    for (int i = lane; i < H; i += 64) {
        const float e = load_elem<T>(src, i) + load_elem<T>(pos, i);
        store_elem<T>(out, i, (e - mean) * rstd * gamma[i] + beta[i]);
    }
    if (yrow && lane == 0) stats_out[row] = make_float2(mean, rstd);
}

// ------------------------------------------------------------------------------------------
// head: workgroups of 16 wavefronts, `parts` of them per request.  c = final state of the request's first row
// (bf16 path: the last LayerNorm in fp32 from the row's sums, statistics in two passes); of a part's hidden units
// wavefront w takes j = w, w + 16, ..., four of them at a time (their loads are all requested before the first is used,
// the first four units' before the row itself): 64-lane dot products of c with rows of W_h1^T reduced across the
// wavefront, ReLU, times w_h2[j]; the sixteen partial sums are added in a fixed order.  With few requests the kernel's
// time is one compute unit's rate on W_h1 (2.4 MB: 37 us), so several workgroups share a request: each leaves its rounds'
// sums in the workspace and the last to arrive (a counter per request, cleared by prep) adds them in order.
// pred_tokens = clamp(rint(y), 0, d_max) with rint rounding half to even.
// ------------------------------------------------------------------------------------------
const int kHeadWaves = 16;
const int kHeadUnits = 4 * kHeadWaves;    // units of one round
const int kHeadSlots = 32;                // rounds whose sums are kept apart, so also the most workgroups per request

__device__ __forceinline__ float head_block_sum(float v, float* s_red) {
    v = wave_sum(v);
    __syncthreads();                                     // s_red's previous use is over
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < kHeadWaves; ++w) t += s_red[w];
    return t;
}

template <typename T>
__global__ __launch_bounds__(kHeadWaves * 64) void head_kernel(const T* __restrict__ x, const int32_t* __restrict__ seq_len,
                                                   const int32_t* __restrict__ row_start,
                                                   const int32_t* __restrict__ bad_req,
                                                   const bf16_t* __restrict__ y_lo,
                                                   const float* __restrict__ ln_g, const float* __restrict__ ln_b, float eps,
                                                   int H, int Hh,
                                                   const float* __restrict__ w_h1t, const float* __restrict__ b_h1,
                                                   const float* __restrict__ w_h2, float b_h2, int d_max,
                                                   int parts, float* __restrict__ part_sum, int32_t* __restrict__ part_done,
                                                   float* __restrict__ pred_f, int32_t* __restrict__ pred_tokens,
                                                   ps_status* st) {
    extern __shared__ float s_c[];           // [H], kHeadWaves partial sums, [kHeadWaves][kHeadSlots] the rounds' sums
    const int r = blockIdx.x / parts, part = blockIdx.x - r * parts;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t crow = row_start[r];       // (with the two others: one trip)
    if (seq_len[r] <= 0 || bad_req[r]) {
        if (threadIdx.x == 0 && part == 0) {
            pred_f[r] = __builtin_nanf("");
            pred_tokens[r] = -1;
        }
        return;
    }
    const int rounds = (Hh + kHeadUnits - 1) / kHeadUnits;
    const int rd0 = rounds * part / parts, rd1 = rounds * (part + 1) / parts;
    const int u0 = rd0 * kHeadUnits;
    // every round's sum is kept apart (those from the last slot on together), so the result does not depend on `parts`
    float* s_round = s_c + H + kHeadWaves;
    const bool wide = (H & 255) == 0 && H <= 2048;       // rows of whole 16-byte pieces per lane (all bf16 models)
    const int nch = H >> 8;
    float4 wv[4][4];
    // lane l holds the 4-element pieces l, l + 64, ... of a row, four pieces (1024 elements) at a time
    auto load_w = [&](int j0, int c0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(j0 + u * kHeadWaves, Hh - 1);      // (a unit past the end re-reads the last row)
            const float4* w = (const float4*)(w_h1t + (int64_t)j * H);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                wv[u][c] = c0 + c < nch ? w[lane + 64 * (c0 + c)] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    if (wide) load_w(u0 + wave, 0);
    asm volatile("" ::: "memory");
    if (y_lo) {
        // bf16 models (H at most 2048: two elements a thread): x holds the hi parts of the last sums
        const bf16_t* hi = (const bf16_t*)x + crow * H;
        const bf16_t* lo = y_lo + crow * H;
        const int i0 = threadIdx.x, i1 = threadIdx.x + kHeadWaves * 64;
        const float v0 = i0 < H ? stream_join(hi[i0], lo[i0]) : 0.f;
        const float v1 = i1 < H ? stream_join(hi[i1], lo[i1]) : 0.f;
        const float mean = head_block_sum(v0 + v1, s_c + H) / (float)H;
        const float d0 = i0 < H ? v0 - mean : 0.f, d1 = i1 < H ? v1 - mean : 0.f;
        const float rstd = 1.0f / sqrtf(head_block_sum(fmaf(d0, d0, d1 * d1), s_c + H) / (float)H + eps);
        if (i0 < H) s_c[i0] = fmaf(d0 * rstd, ln_g[i0], ln_b[i0]);
        if (i1 < H) s_c[i1] = fmaf(d1 * rstd, ln_g[i1], ln_b[i1]);
    } else if (ln_g) {
        // fp32 models whose maps take the LayerNorms (hidden at most PS_NARROW_WIDTH): x holds the last sums
        const float* c = (const float*)x + crow * H;
        const int i = threadIdx.x;
        const float2 st = narrow_moments(c, H, eps, i & 7);      // (by every eight lanes)
        if (i < H) s_c[i] = fmaf((c[i] - st.x) * st.y, ln_g[i], ln_b[i]);
    } else {
        const T* c = x + crow * H;
        for (int i = threadIdx.x; i < H; i += kHeadWaves * 64) s_c[i] = load_elem<T>(c, i);
    }
    __syncthreads();
    // the loop counts a wavefront's units, not the rounds: the kernel's time with many requests, one workgroup of them on
    // a compute unit at a time, follows how early a round's loads are requested (4096 requests, H 768: 574 us counting
    // rounds, 526 us so; H 1024: 862 / 827)
    const int u1 = min(rd1 * kHeadUnits, Hh);
    int rd = rd0;
    for (int j0 = u0 + wave; j0 < u1; j0 += kHeadUnits, ++rd) {
        float acc = 0.f;
        float dot[4] = {0.f, 0.f, 0.f, 0.f};
        if (wide) {
            for (int c0 = 0; c0 < nch; c0 += 4) {
                if (rd != rd0 || c0) load_w(j0, c0);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c0 + c < nch) {
                        const float4 cv = ((const float4*)s_c)[lane + 64 * (c0 + c)];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            dot[u] = fmaf(cv.x, wv[u][c].x, fmaf(cv.y, wv[u][c].y, fmaf(cv.z, wv[u][c].z, fmaf(cv.w, wv[u][c].w, dot[u]))));
                    }
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + u * kHeadWaves;
                if (j < Hh) {
                    const float* w = w_h1t + (int64_t)j * H;
                    for (int i = lane; i < H; i += 64) dot[u] = fmaf(s_c[i], w[i], dot[u]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = j0 + u * kHeadWaves;
            if (j < Hh) {
                const float d = wave_sum(dot[u]) + b_h1[j];
                acc += (d < 0.f ? 0.f : d) * w_h2[j];   // ReLU that lets a NaN through to the check below
            }
        }
        float* slot = s_round + wave * kHeadSlots + min(rd, kHeadSlots - 1);
        if (lane == 0) *slot = rd < kHeadSlots ? acc : *slot + acc;
    }
    if (lane == 0 && rd < min(rd1, kHeadSlots)) s_round[wave * kHeadSlots + rd] = 0.f;   // no unit of the last round is ours
    __syncthreads();
    if (threadIdx.x == 0) {
        float y = 0.f;
        for (int i = min(rd0, kHeadSlots); i < min(rd1, kHeadSlots); ++i) {
            float t = 0.f;
            for (int w = 0; w < kHeadWaves; ++w) t += s_round[w * kHeadSlots + i];
            if (parts > 1) __hip_atomic_store(part_sum + (int64_t)r * kHeadSlots + i, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            y += t;
        }
        if (parts > 1) {
            if (__hip_atomic_fetch_add(part_done + r, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) != parts - 1) return;
            y = 0.f;
            for (int i = 0; i < rounds; ++i)
                y += __hip_atomic_load(part_sum + (int64_t)r * kHeadSlots + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        y += b_h2;
        pred_f[r] = y;
        if (y != y) {
            pred_tokens[r] = -1;
            report_fault(st, PS_ST_NAN, r);
        } else {
            const float t = fminf(fmaxf(rintf(y), 0.f), (float)d_max);
            pred_tokens[r] = (int32_t)t;
        }
    }
}

// The bf16 input rows of each request's first token, one per request, for the side GEMM that computes
// only those rows' queries (last layer).  Rows of faulty requests and padding rows are zero.
__global__ __launch_bounds__(256) void cls_rows_kernel(const bf16_t* __restrict__ x, int H, int n_req,
                                                       const int32_t* __restrict__ seq_len,
                                                       const int32_t* __restrict__ row_start, bf16_t* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    uint4* o = (uint4*)(out + (int64_t)r * H);
    const bool live = r < n_req && seq_len[r] > 0;
    const uint4* src = live ? (const uint4*)(x + (int64_t)row_start[r] * H) : nullptr;
    for (int i = lane; i < H / 8; i += 64) o[i] = live ? src[i] : make_uint4(0u, 0u, 0u, 0u);
}

}  // namespace

void launch_cls_rows(const ps_model* m, int32_t n_req, const Workspace& ws, const bf16_t* x, bf16_t* out, hipStream_t s) {
    hipLaunchKernelGGL(cls_rows_kernel, dim3((unsigned)(ws.cls_rows / 4)), dim3(256), 0, s, x, m->info.hidden, n_req,
                       ws.seq_len, ws.row_start, out);
}

void launch_prep(const ps_model* m, const int32_t* offsets, const int32_t* lengths, int32_t n_req, int64_t n_tokens,
                 const Workspace& ws, ps_status* st, hipStream_t s) {
    const int h = m->info.hidden / 256, f = m->info.ffn / 256;
    // (calls that take the small tiles only, run_encoder_bf16, need none; nor do fp32 models)
    const bool planned = m->info.dtype == 1 && !small_maps(ws, n_req, m->info.hidden);
    const int4 plan_cols = planned ? make_int4(3 * h, 2 * h, h, f) : make_int4(0, 0, 0, 0);
    hipLaunchKernelGGL(prep_kernel, dim3(1), dim3(1024), 0, s, offsets, lengths, n_req, m->info.n_soft, m->info.max_pos,
                       (long long)n_tokens, (long long)(ws.max_rows - PS_KEY_SLACK), plan_cols, planned ? 1 : 0, ws.meta, ws.seq_len,
                       ws.row_start, ws.qtile_start, ws.bad_req, ws.head_done, st);
}

void launch_embed(const ps_model* m, const int32_t* token_ids, const int32_t* offsets, int32_t n_req,
                  const Workspace& ws, ps_status* st, hipStream_t s) {
    const ps_model_info& f = m->info;
    const unsigned blocks = (unsigned)(ws.max_rows / 4);
    if (f.dtype == 1)
        hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, token_ids, offsets, n_req,
                           (const bf16_t*)m->e_tok, (const bf16_t*)m->e_pos, (const bf16_t*)m->e_soft,
                           m->lne_g, m->lne_b, m->ln_eps, f.hidden, f.vocab, f.n_soft, ws.meta, ws.seq_len,
                           ws.row_start, ws.bad_req, (bf16_t*)ws.x, ws.la, ws.sa, ws.qtile_start, ws.qtiles,
                           carries_side_maps(ws, n_req, f.hidden) ? ws.first_row : nullptr, st);
    else
        hipLaunchKernelGGL(embed_kernel<float>, dim3(blocks), dim3(256), 0, s, token_ids, offsets, n_req,
                           (const float*)m->e_tok, (const float*)m->e_pos, (const float*)m->e_soft,
                           m->lne_g, m->lne_b, m->ln_eps, f.hidden, f.vocab, f.n_soft, ws.meta, ws.seq_len,
                           ws.row_start, ws.bad_req, (float*)ws.x, (bf16_t*)nullptr, (float2*)nullptr, (const int32_t*)nullptr,
                           (int4*)nullptr, (uint8_t*)nullptr, st);
}

void launch_head(const ps_model* m, int32_t n_req, const Workspace& ws, float* pred_f, int32_t* pred_tokens,
                 ps_status* st, hipStream_t s) {
    const ps_model_info& f = m->info;
    const size_t lds = sizeof(float) * (size_t)(f.hidden + kHeadWaves + kHeadWaves * kHeadSlots);   // (hidden <= 8192: 35 KB)
    // enough workgroups to fill the chip, a round of 64 units each at the least
    const int rounds = (f.head_hidden + kHeadUnits - 1) / kHeadUnits;
    int parts = 256 / n_req < rounds ? 256 / n_req : rounds;
    if (parts < 1 || rounds > kHeadSlots) parts = 1;
    const dim3 grid((unsigned)n_req * (unsigned)parts);
    const bool sums = f.dtype != 1 && f32_maps_take_norms(f, ws.max_rows);
    if (f.dtype == 1)
        hipLaunchKernelGGL(head_kernel<bf16_t>, grid, dim3(kHeadWaves * 64), lds, s, (const bf16_t*)ws.x, ws.seq_len, ws.row_start,
                           ws.bad_req, (const bf16_t*)ws.la, (const float*)m->layers.back().ln2_g,
                           (const float*)m->layers.back().ln2_b, m->ln_eps, f.hidden, f.head_hidden, m->w_h1t, m->b_h1, m->w_h2,
                           m->b_h2, f.d_max, parts, ws.head_sum, ws.head_done, pred_f, pred_tokens, st);
    else
        hipLaunchKernelGGL(head_kernel<float>, grid, dim3(kHeadWaves * 64), lds, s, (const float*)ws.x, ws.seq_len, ws.row_start,
                           ws.bad_req, (const bf16_t*)nullptr, sums ? (const float*)m->layers.back().ln2_g : nullptr,
                           sums ? (const float*)m->layers.back().ln2_b : nullptr, m->ln_eps, f.hidden,
                           f.head_hidden, m->w_h1t, m->b_h1, m->w_h2, m->b_h2, f.d_max, parts, ws.head_sum, ws.head_done, pred_f,
                           pred_tokens, st);
}
