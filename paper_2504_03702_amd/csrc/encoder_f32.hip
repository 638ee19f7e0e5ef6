// fp32 encoder path (models stored in fp32): kernels in full single precision.
// It exists for small models whose results must track the fp64 definition to 1e-4; the bf16
// MFMA path in encoder_bf16.hip is the one built for throughput.
#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace {

enum { F32_NONE = 0, F32_GELU = 1, F32_RESIDUAL = 2 };

typedef float f32x16 __attribute__((ext_vector_type(16)));

// C[m, n] = sum_k A[m, k] W[k, n] + bias[n], then GELU or + residual[m, n].
//
// v_mfma_f32_32x32x2_f32 (fp32 products and sums) on fragments straight from global memory: the matrices are small and
// sit in L2, and what a staged 64 x 64 tile cost was a trip to memory per 16-deep slice (23 us for K = 128, 75 us for
// K = 512 at 600 rows).  A workgroup owns TM x 32 rows and 32 columns; its four wavefronts split the contraction and
// their sums are added through LDS in order.  In a group of eight k lane l holds four consecutive ones of its row of A
// (one 16-byte load; lanes 32.. the upper four) and the same four rows of its column of W, a whole 128-byte line per
// row; eight groups are requested before the first is used.  Where K is no multiple of 4 the 16-byte loads are aligned to
// 4 bytes only (rows of A begin anywhere), which global loads may be.  TAIL: K is no multiple of 8; only the last group is
// looked at element by element (testing all of them, and columns beyond N in the same way, cost 512 prompts of a model with
// hidden 1000 26.3 ms, 13.4 so).
struct __attribute__((packed, aligned(4))) Float4Any { float x, y, z, w; };

template <int EPI, int TM, bool TAIL>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                       const float* __restrict__ bias,
                                                       const float* __restrict__ residual, float* __restrict__ C,
                                                       int N, int K, int n_first, const BatchMeta* meta) {
    __shared__ float s_part[4][TM * 32][33];
    const int m0 = blockIdx.x * 32 * TM, n0 = n_first + blockIdx.y * 32;
    if (m0 >= meta->total_rows) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 31, half = lane >> 5, n = n0 + row;
    const int groups = (K + 7) / 8, g0 = groups * wave / 4, g1 = groups * (wave + 1) / 4;
    const int g1_whole = TAIL ? min(g1, K / 8) : g1;
    const float* ap = A + (int64_t)(m0 + row) * K + 4 * half;    // rows are always inside the padded buffer
    const float* wp = W + (int64_t)(4 * half) * N + min(n, N - 1);
    f32x16 acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    constexpr int U = 8 / TM;
    for (int g = g0; g < g1_whole; g += U) {
        float a[U][TM][4], w[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 8 * min(g + u, g1_whole - 1);         // (past the end: the last group again, not used)
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const Float4Any v = *(const Float4Any*)(ap + (int64_t)(32 * i) * K + k);
                a[u][i][0] = v.x; a[u][i][1] = v.y; a[u][i][2] = v.z; a[u][i][3] = v.w;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) w[u][t] = wp[(int64_t)(k + t) * N];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g + u < g1_whole) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][i][t], w[u][t], acc[i], 0, 0, 0);
            }
        }
    }
    if (TAIL && g1 > K / 8) {                                   // the last wavefront
        const int k = K / 8 * 8;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool in = k + 4 * half + t < K;
            const float w = in ? wp[(int64_t)(k + t) * N] : 0.f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? ap[(int64_t)(32 * i) * K + k + t] : 0.f, w, acc[i], 0, 0, 0);
        }
    }
    // element e of a lane is row 8 (e / 4) + 4 half + e % 4, column lane % 32
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) s_part[wave][32 * i + 8 * (e >> 2) + 4 * half + (e & 3)][row] = acc[i][e];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4 * TM; ++i) {
        const int r = 8 * i + (threadIdx.x >> 5), c = threadIdx.x & 31;
        if (n0 + c >= N) continue;
        const int64_t at = (int64_t)(m0 + r) * N + n0 + c;
        float v = ((s_part[0][r][c] + s_part[1][r][c]) + (s_part[2][r][c] + s_part[3][r][c])) + bias[n0 + c];
        if (EPI == F32_GELU) v = 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
        if (EPI == F32_RESIDUAL) v += residual[at];
        C[at] = v;
    }
}

// A wavefront takes Q neighbouring rows of a head: their scores against the request's keys go to LDS, then
// a max, an exponential pass and a weighted sum of the value rows, all in fp32.  A lane takes a whole key, 16 bytes of it
// a load (a row per lane occupies the address unit for all 64 lanes, however few bytes it reads), and meets all Q rows with
// it; value rows are requested eight at a time.  Sums run in the order of the features and of the keys whatever Q is.
// 16 prompts of up to 64 tokens, 2 heads of 64: 12.2 us a launch with a feature or a value row a load, 9.6 so.
template <int Q>
__global__ __launch_bounds__(256) void attention_f32_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                            int H, int d, int n_req, int max_pos,
                                                            const BatchMeta* meta, const int32_t* __restrict__ seq_len,
                                                            const int32_t* __restrict__ row_start) {
    extern __shared__ __align__(16) float lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row0 = (blockIdx.x * 4 + wave) * Q;  // (requests start at multiples of 8: all Q rows are of one)
    const int head = blockIdx.y;
    if (row0 >= meta->total_rows) return;         // whole wavefront leaves together
    int lo = 0, hi = n_req - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (row_start[mid] <= row0) lo = mid; else hi = mid - 1;
    }
    const int base = row_start[lo], S = seq_len[lo];
    if (row0 - base >= S) return;
    const int rows = min(Q, S - (row0 - base));
    using Q4 = std::conditional_t<Q == 1, Float4Any, float4>;    // (one row a wavefront: no room is spent on alignment)
    const int d4 = Q == 1 ? d : (d + 3) & ~3;
    const int pos4 = Q == 1 ? max_pos : (max_pos + 3) & ~3;
    float* q = lds + wave * Q * (pos4 + d4);      // [Q][d4]
    float* sc = q + Q * d4;                       // [Q][max_pos]
    const int64_t ld = 3 * (int64_t)H;
    const float scale = 1.0f / sqrtf((float)d);
#pragma unroll
    for (int r = 0; r < Q; ++r)                   // (rows past the request's end: the last one again, not stored)
        for (int i = lane; i < d; i += 64) q[r * d4 + i] = qkv[(row0 + min(r, rows - 1)) * ld + head * d + i];
    __builtin_amdgcn_wave_barrier();
    float mx[Q];
#pragma unroll
    for (int r = 0; r < Q; ++r) mx[r] = -INFINITY;
    for (int t = lane; t < S; t += 64) {
        const float* k = qkv + (base + t) * ld + H + head * d;
        float s[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) s[r] = 0.f;
        int i = 0;
        for (; i + 32 <= d; i += 32) {
            Float4Any v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *(const Float4Any*)(k + i + 4 * u);
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int r = 0; r < Q; ++r) {
                    const Q4 qi = *(const Q4*)(q + r * d4 + i + 4 * u);
                    s[r] = fmaf(qi.x, v[u].x, s[r]);
                    s[r] = fmaf(qi.y, v[u].y, s[r]);
                    s[r] = fmaf(qi.z, v[u].z, s[r]);
                    s[r] = fmaf(qi.w, v[u].w, s[r]);
                }
        }
        for (; i < d; ++i) {
            const float ki = k[i];
#pragma unroll
            for (int r = 0; r < Q; ++r) s[r] = fmaf(q[r * d4 + i], ki, s[r]);
        }
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            s[r] *= scale;
            sc[r * max_pos + t] = s[r];
            mx[r] = fmaxf(mx[r], s[r]);
        }
    }
    float sum[Q];
#pragma unroll
    for (int r = 0; r < Q; ++r) {
        mx[r] = wave_max(mx[r]);
        sum[r] = 0.f;
        for (int t = lane; t < S; t += 64) {
            const float e = expf(sc[r * max_pos + t] - mx[r]);
            sc[r * max_pos + t] = e;
            sum[r] += e;
        }
        sum[r] = wave_sum(sum[r]);
    }
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < d; i += 64) {
        const float* v = qkv + (int64_t)base * ld + 2 * H + head * d + i;
        float o[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) o[r] = 0.f;
        int t = 0;
        for (; t + 8 <= S; t += 8) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = v[(t + u) * ld];
#pragma unroll
            for (int r = 0; r < Q; ++r)
#pragma unroll
                for (int u = 0; u < 8; ++u) o[r] = fmaf(sc[r * max_pos + t + u], x[u], o[r]);
        }
        for (; t < S; ++t) {
            const float x = v[t * ld];
#pragma unroll
            for (int r = 0; r < Q; ++r) o[r] = fmaf(sc[r * max_pos + t], x, o[r]);
        }
#pragma unroll
        for (int r = 0; r < Q; ++r)
            if (r < rows) out[(int64_t)(row0 + r) * H + head * d + i] = o[r] / sum[r];
    }
}

// The same sums in the same order for heads of whole 16-byte groups, with the keys and values of 64 positions at a time in LDS:
// a workgroup's rows (of one request) share them, and they come in whole lines.  A row a lane, as above, occupies the
// address unit for all 64 lanes of every 16 bytes of a key, and the value rows were a trip to memory for every eight of them.
// The first 64 keys' values are requested with the keys: short requests wait for memory once.  16 prompts of up to 64 tokens,
// 2 heads of 64: 9.3 -> 7.9 us a launch.
template <int Q>
__global__ __launch_bounds__(256) void attention_f32_staged_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                                   int H, int d, int n_req, int max_pos,
                                                                   const BatchMeta* meta, const int32_t* __restrict__ seq_len,
                                                                   const int32_t* __restrict__ row_start) {
    extern __shared__ __align__(16) float lds[];
    static_assert(4 * Q <= PS_ROW_ALIGN, "a workgroup's rows are of one request");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int first = blockIdx.x * 4 * Q, head = blockIdx.y;
    int base, S;
    if (n_req <= 64) {                            // one trip to memory, and a count of the starts up to this row
        const int start = row_start[min(lane, n_req - 1)], len = seq_len[min(lane, n_req - 1)];
        if (first >= meta->total_rows) return;
        const int at = __popcll(__ballot(lane < n_req && start <= first)) - 1;
        base = __builtin_amdgcn_readlane(start, at);
        S = __builtin_amdgcn_readlane(len, at);
    } else {
        if (first >= meta->total_rows) return;
        int lo = 0, hi = n_req - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (row_start[mid] <= first) lo = mid; else hi = mid - 1;
        }
        base = row_start[lo];
        S = seq_len[lo];
    }
    if (first - base >= S) return;                // the whole workgroup
    const int row0 = first + wave * Q, rows = min(Q, S - (row0 - base));   // (rows < 1: the wavefront only moves tiles)
    const int kld = d + 4, pos4 = (max_pos + 3) & ~3;
    float *kt = lds, *vt = kt + 64 * kld, *q = vt + 64 * d + wave * Q * (d + pos4), *sc = q + Q * d;
    const int64_t ld = 3 * (int64_t)H;
    const float scale = 1.0f / sqrtf((float)d);
    // thread's first 16-byte piece of a tile, and how far on the next one is
    const int per_row = d / 4, key0 = threadIdx.x / per_row, col0 = threadIdx.x - key0 * per_row;
    const int key_step = 256 / per_row, col_step = 256 - key_step * per_row;
    auto stage = [&](float* to, int to_ld, int t0, int part) {               // part: 1 keys, 2 values
        const int n = min(64, S - t0);
        const float* from = qkv + (int64_t)(base + t0) * ld + (int64_t)part * H + head * d;
        for (int key = key0, c = col0; key < n;) {
            *(float4*)(to + key * to_ld + 4 * c) = *(const float4*)(from + key * ld + 4 * c);
            key += key_step;
            c += col_step;
            if (c >= per_row) { c -= per_row; ++key; }
        }
    };
    stage(kt, kld, 0, 1);
    stage(vt, d, 0, 2);
#pragma unroll
    for (int r = 0; r < Q; ++r)                   // (rows past the request's end: the last one again, not stored)
        for (int i = lane; i < d; i += 64) q[r * d + i] = qkv[(base + min(row0 - base + r, S - 1)) * ld + head * d + i];
    float mx[Q];
#pragma unroll
    for (int r = 0; r < Q; ++r) mx[r] = -INFINITY;
    for (int t0 = 0; t0 < S; t0 += 64) {
        if (t0 > 0) {
            __syncthreads();
            stage(kt, kld, t0, 1);
        }
        __syncthreads();
        const int t = t0 + lane;
        if (t >= S || rows < 1) continue;
        float s[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) s[r] = 0.f;
#pragma unroll 4
        for (int i = 0; i < d; i += 4) {
            const float4 k = *(const float4*)(kt + lane * kld + i);
#pragma unroll
            for (int r = 0; r < Q; ++r) {
                const float4 qi = *(const float4*)(q + r * d + i);
                s[r] = fmaf(qi.x, k.x, s[r]);
                s[r] = fmaf(qi.y, k.y, s[r]);
                s[r] = fmaf(qi.z, k.z, s[r]);
                s[r] = fmaf(qi.w, k.w, s[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < Q; ++r) {
            s[r] *= scale;
            sc[r * pos4 + t] = s[r];
            mx[r] = fmaxf(mx[r], s[r]);
        }
    }
    float sum[Q];
#pragma unroll
    for (int r = 0; r < Q; ++r) {
        mx[r] = wave_max(mx[r]);
        sum[r] = 0.f;
        for (int t = lane; t < S && rows >= 1; t += 64) {
            const float e = expf(sc[r * pos4 + t] - mx[r]);
            sc[r * pos4 + t] = e;
            sum[r] += e;
        }
        sum[r] = wave_sum(sum[r]);
    }
    __builtin_amdgcn_wave_barrier();
    // 64 features at a time; the values of the first 64 positions are there the first time round
    for (int i0 = 0; i0 < d; i0 += 64) {
        const int i = i0 + lane;
        float o[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) o[r] = 0.f;
        for (int t0 = 0; t0 < S; t0 += 64) {
            if (S > 64 && (t0 > 0 || i0 > 0)) {
                __syncthreads();
                stage(vt, d, t0, 2);
                __syncthreads();
            }
            if (i >= d || rows < 1) continue;
            const int n = min(64, S - t0);
#pragma unroll 8
            for (int t = 0; t < n; ++t) {
                const float x = vt[t * d + i];
#pragma unroll
                for (int r = 0; r < Q; ++r) o[r] = fmaf(sc[r * pos4 + t0 + t], x, o[r]);
            }
        }
        if (i < d)
#pragma unroll
            for (int r = 0; r < Q; ++r)
                if (r < rows) out[(int64_t)(row0 + r) * H + head * d + i] = o[r] / sum[r];
    }
}

// The same maps in calls of few rows, where a launch costs as much as its work: a stream of sums whose LayerNorm is taken by
// whoever reads it instead of by a launch of its own.  NORM_A: A holds sums; a workgroup has its 32 rows' elements in
// registers, so their statistics are two sums over the lanes and wavefronts that hold a row (two passes, as the LayerNorm kernel
// makes them) while the weights are on their way; the first column of workgroups leaves them for the map that adds the stream
// again.  NORM_RES: residual holds sums, with those statistics.  K a multiple of 32 and at most 256 with NORM_A.
// 16 prompts, hidden 128, 2 layers: thirteen launches instead of seventeen, 88 -> 83 us; 25 prompts 93.6 -> 84.5, 40 107 -> 102.
// The sums are made in the order of layernorm_f32_narrow_kernel, so calls on either side of the rule give the same bits.
struct StreamNorm {
    const float *gamma, *beta;
    float2* stats;                           // [rows] (mean, 1 / std)
    float eps;
};

template <int EPI, bool NORM_A, bool NORM_RES>
__global__ __launch_bounds__(256) void gemm_f32_norm_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                            const float* __restrict__ bias,
                                                            const float* __restrict__ residual, float* __restrict__ C,
                                                            int N, int K, StreamNorm in, StreamNorm res, const BatchMeta* meta) {
    __shared__ float s_part[4][32][33];
    __shared__ float s_red[2][4][32];
    const int m0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
    const int total = meta->total_rows;      // looked at when the first loads are on their way (all rows lie in the buffers)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 31, half = lane >> 5, n = n0 + row;
    const int groups = K / 8, g0 = groups * wave / 4, g1 = groups * (wave + 1) / 4;
    const float* ap = A + (int64_t)(m0 + row) * K + 4 * half;
    const float* wp = W + (int64_t)(4 * half) * N + min(n, N - 1);
    // what the epilogue adds, requested with the operands
    float add[4];
    float2 st[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + (threadIdx.x >> 5), c = min(n0 + (int)(threadIdx.x & 31), N - 1);
        add[i] = EPI == F32_RESIDUAL ? residual[(int64_t)(m0 + r) * N + c] : 0.f;
        st[i] = NORM_RES ? res.stats[m0 + r] : make_float2(0.f, 1.f);
    }
    const int col = min(n0 + (int)(threadIdx.x & 31), N - 1);
    const float bv = bias[col], rg = NORM_RES ? res.gamma[col] : 1.f, rb = NORM_RES ? res.beta[col] : 0.f;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    constexpr int U = 8;                     // groups in flight (all of a wavefront's with NORM_A)
    for (int g = g0; g < g1; g += U) {
        float a[U][4], w[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 8 * min(g + u, g1 - 1);               // (past the end: the last group again, not used)
            const float4 v = *(const float4*)(ap + k);
            a[u][0] = v.x; a[u][1] = v.y; a[u][2] = v.z; a[u][3] = v.w;
        }
        if (NORM_A) asm volatile("" ::: "memory");              // (the rows first)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 8 * min(g + u, g1 - 1);
#pragma unroll
            for (int t = 0; t < 4; ++t) w[u][t] = wp[(int64_t)(k + t) * N];
        }
        if (g == g0) {
            asm volatile("" ::: "memory");
            if (m0 >= total) return;                            // the whole workgroup
        }
        if (NORM_A) {
            float4 ga[U], be[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = 8 * min(g + u, g1 - 1) + 4 * half;
                ga[u] = *(const float4*)(in.gamma + k);
                be[u] = *(const float4*)(in.beta + k);
            }
            // a row's elements are in lanes row and row + 32 of the four wavefronts
            auto row_sum = [&](float v, int which) {
                v += __shfl_xor(v, 32, 64);
                if (half == 0) s_red[which][wave][row] = v;
                __syncthreads();
                return (s_red[which][0][row] + s_red[which][1][row]) + (s_red[which][2][row] + s_red[which][3][row]);
            };
            float sum = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (g + u < g1) sum += narrow_quad(a[u][0], a[u][1], a[u][2], a[u][3]);
            const float mean = row_sum(sum, 0) / (float)K;
            float sq = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int t = 0; t < 4; ++t) a[u][t] -= mean;
                if (g + u < g1) sq += narrow_squares(a[u][0], a[u][1], a[u][2], a[u][3]);
            }
            const float rstd = 1.0f / sqrtf(row_sum(sq, 1) / (float)K + in.eps);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u][0] = fmaf(a[u][0] * rstd, ga[u].x, be[u].x);
                a[u][1] = fmaf(a[u][1] * rstd, ga[u].y, be[u].y);
                a[u][2] = fmaf(a[u][2] * rstd, ga[u].z, be[u].z);
                a[u][3] = fmaf(a[u][3] * rstd, ga[u].w, be[u].w);
            }
            if (blockIdx.y == 0 && wave == 0 && half == 0) in.stats[m0 + row] = make_float2(mean, rstd);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g + u < g1) {
#pragma unroll
                for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][t], w[u][t], acc, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) s_part[wave][8 * (e >> 2) + 4 * half + (e & 3)][row] = acc[e];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + (threadIdx.x >> 5), c = threadIdx.x & 31;
        if (n0 + c >= N) continue;
        float v = ((s_part[0][r][c] + s_part[1][r][c]) + (s_part[2][r][c] + s_part[3][r][c])) + bv;
        if (EPI == F32_GELU) v = 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
        if (EPI == F32_RESIDUAL) v += NORM_RES ? fmaf((add[i] - st[i].x) * st[i].y, rg, rb) : add[i];
        C[(int64_t)(m0 + r) * N + n0 + c] = v;
    }
}

// LayerNorm of one row per wavefront (biased variance, two passes over the row).
__global__ __launch_bounds__(256) void layernorm_f32_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                            const float* __restrict__ gamma,
                                                            const float* __restrict__ beta, float eps, int H,
                                                            const BatchMeta* meta) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= meta->total_rows) return;
    const float* x = in + row * H;
    float sum = 0.f;
    for (int i = lane; i < H; i += 64) sum += x[i];
    const float mean = wave_sum(sum) / (float)H;
    float sq = 0.f;
    for (int i = lane; i < H; i += 64) { const float t = x[i] - mean; sq += t * t; }
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)H + eps);
    for (int i = lane; i < H; i += 64) out[row * H + i] = (x[i] - mean) * rstd * gamma[i] + beta[i];
}

// LayerNorm of the rows that the maps above could take themselves, in calls of many rows: eight lanes a row (narrow_moments' parts),
// the same sums in the same order.  A lane has its part of the row, of Q = H / 32 groups (at most QM), in registers: one trip to
// memory, and eight rows make a workgroup (THREADS 64), so that a call of some hundred rows has many units at it.  Two layers of
// hidden 256, 1540 rows: 192 us a call with a wavefront a row, 198 with 32 rows a workgroup and a trip for each pass, 187; 192 wide
// 166, 167, 162; 128 113, 113, 110; 12000 rows of 256 790, 787, 784.  Rows of 64 and less keep 32 a workgroup (1 % of a call).
template <int QM, int THREADS>
__global__ __launch_bounds__(THREADS) void layernorm_f32_narrow_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                                  const float* __restrict__ gamma,
                                                                  const float* __restrict__ beta, float eps, int H,
                                                                  const BatchMeta* meta) {
    const int64_t row = (int64_t)blockIdx.x * (THREADS / 8) + (threadIdx.x >> 3);
    const int total = meta->total_rows;           // looked at when the loads are on their way (all rows lie in the buffers)
    const int part = threadIdx.x & 7, Q = H / 32, at = 8 * Q * (part >> 1) + 4 * (part & 1);
    const float* x = in + row * H + at;
    float4 v[QM], g[QM], b[QM];
#pragma unroll
    for (int u = 0; u < QM; ++u) v[u] = *(const float4*)(x + 8 * min(u, Q - 1));
#pragma unroll
    for (int u = 0; u < QM; ++u) {
        g[u] = *(const float4*)(gamma + at + 8 * min(u, Q - 1));
        b[u] = *(const float4*)(beta + at + 8 * min(u, Q - 1));
    }
    asm volatile("" ::: "memory");
    if (row >= total) return;                     // eight lanes together
    auto all = [](float t) {
        t += __shfl_xor(t, 1, 64);
        t += __shfl_xor(t, 2, 64);
        return t + __shfl_xor(t, 4, 64);
    };
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int u = 0; u < QM; ++u)
        if (u < Q) sum += narrow_quad(v[u].x, v[u].y, v[u].z, v[u].w);
    const float mean = all(sum) / (float)H;
#pragma unroll
    for (int u = 0; u < QM; ++u) {
        v[u].x -= mean; v[u].y -= mean; v[u].z -= mean; v[u].w -= mean;
        if (u < Q) sq += narrow_squares(v[u].x, v[u].y, v[u].z, v[u].w);
    }
    const float rstd = 1.0f / sqrtf(all(sq) / (float)H + eps);
#pragma unroll
    for (int u = 0; u < QM; ++u)
        if (u < Q)
            *(float4*)(out + row * H + at + 8 * u) = make_float4(fmaf(v[u].x * rstd, g[u].x, b[u].x), fmaf(v[u].y * rstd, g[u].y, b[u].y),
                                                                 fmaf(v[u].z * rstd, g[u].z, b[u].z), fmaf(v[u].w * rstd, g[u].w, b[u].w));
}

template <int EPI, int TM>
void gemm_f32_rows(const float* A, const float* W, const float* bias, const float* res, float* C, int64_t max_rows, int N, int K,
                   const BatchMeta* meta, hipStream_t s) {
    const int most = 65535 * 32;                                 // columns a grid holds
    for (int n_first = 0; n_first < N; n_first += most) {
        const dim3 grid((unsigned)(max_rows / (32 * TM)), (unsigned)(((N - n_first < most ? N - n_first : most) + 31) / 32));
        if (K % 8 != 0)
            hipLaunchKernelGGL((gemm_f32_kernel<EPI, TM, true>), grid, dim3(256), 0, s, A, W, bias, res, C, N, K, n_first, meta);
        else
            hipLaunchKernelGGL((gemm_f32_kernel<EPI, TM, false>), grid, dim3(256), 0, s, A, W, bias, res, C, N, K, n_first, meta);
    }
}

template <int EPI>
void gemm_f32(const float* A, const float* W, const float* bias, const float* res, float* C, int64_t max_rows, int N, int K,
              const BatchMeta* meta, hipStream_t s) {
    // enough workgroups to fill the chip twice: a tile of 64 rows reads W half as often
    if (max_rows / 64 * ((N + 31) / 32) >= 512) gemm_f32_rows<EPI, 2>(A, W, bias, res, C, max_rows, N, K, meta, s);
    else gemm_f32_rows<EPI, 1>(A, W, bias, res, C, max_rows, N, K, meta, s);
}

template <int EPI, bool NORM_A, bool NORM_RES>
void gemm_f32_norm(const float* A, const float* W, const float* bias, const float* res, float* C, int64_t max_rows, int N, int K,
                   const StreamNorm& in, const StreamNorm& stream, const BatchMeta* meta, hipStream_t s) {
    hipLaunchKernelGGL((gemm_f32_norm_kernel<EPI, NORM_A, NORM_RES>), dim3((unsigned)(max_rows / 32), (unsigned)((N + 31) / 32)),
                       dim3(256), 0, s, A, W, bias, res, C, N, K, in, stream, meta);
}

}  // namespace

static bool narrow_norms(const ps_model_info& f) { return f.hidden % 32 == 0 && f.hidden <= PS_NARROW_WIDTH && f.ffn % 32 == 0; }

// As long as the widest map does not fill the chip twice (what its other form asks for): every column of its workgroups makes
// the statistics again.
bool f32_maps_take_norms(const ps_model_info& f, int64_t max_rows) {
    const int64_t wide = 3 * f.hidden > f.ffn ? 3 * f.hidden : f.ffn;
    return narrow_norms(f) && wide <= 65535 * 32 && max_rows / 64 * ((wide + 31) / 32) < 512;
}

void run_encoder_f32(const ps_model* m, int32_t n_req, const Workspace& ws, hipStream_t s) {
    const ps_model_info& f = m->info;
    const int H = f.hidden, F = f.ffn, d = H / f.heads;
    float *x = (float*)ws.x, *qkv = (float*)ws.qkv, *att = (float*)ws.att, *y = (float*)ws.y,
          *x1 = (float*)ws.x1, *g = (float*)ws.g;
    const unsigned row_blocks = (unsigned)(ws.max_rows / 4);
    // Keys and values through LDS where a head is whole 16-byte groups and they fit: one row a wavefront (us a launch with
    // hidden 128, 2 heads: 16 prompts, 768 rows, 9.3 without / 7.9 so, 30 prompts 11.9 / 8.5), two from 3072 rows x heads (50
    // prompts, 2304 rows, 12.5 / 9.9); from 8192 on four rows a wavefront without LDS use the vector units better (150 prompts,
    // 6400 rows, 16.9 / 20.0; four rows and LDS 27.0).  Heads of 64 features and more only while all workgroups have a place
    // at once, by the LDS that head size and positions take: a second round costs more than the loads save (two layers, rows x
    // heads: us a call without / through LDS; 64 features of 640 positions, 512 places, 3072: 166 / 156, 7936: 211 / 267; 64 of
    // 512, 768 places, 4096: 156 / 153, 7168: 215 / 250; 100 of 256, 512 places, 3328: 170 / 165, 6912: 206 / 264).  Smaller ones
    // gain there too (32 of 1024, 768 places, 7168: 282 / 179).
    auto staged_lds = [&](int rows) {
        return sizeof(float) * ((size_t)64 * (2 * d + 4) + (size_t)4 * rows * (d + ((f.max_pos + 3) & ~3)));
    };
    const int64_t row_heads = ws.max_rows * f.heads;
    auto one_round = [&](int rows) { return row_heads / (4 * rows) <= 256 * (int64_t)(160 * 1024 / staged_lds(rows)); };
    const int staged_rows = row_heads >= 3072 ? 2 : 1;
    const int staged = d % 4 != 0 || staged_lds(2) > 64 * 1024 || row_heads >= 8192 || (d >= 64 && !one_round(staged_rows)) ? 0 : staged_rows;
    // Four rows a wavefront where there are rows enough to fill the chip all the same and their scores leave room for
    // several workgroups to a unit.  Two layers, hidden 128, us a call, one row / four: 16 prompts (768 rows x 2 heads) 90.5 /
    // 93.8, 50 (2048 x 2) 131 / 128, 150 224 / 196, 512 507 / 419.
    const size_t att_lds = sizeof(float) * 4 * (size_t)(f.max_pos + d);
    const size_t att_lds4 = sizeof(float) * 16 * (size_t)(((f.max_pos + 3) & ~3) + ((d + 3) & ~3));
    const int att_rows = att_lds4 <= 48 * 1024 && ws.max_rows * f.heads >= 3072 ? 4 : 1;
    auto attention = [&]() {
        if (staged == 2)
            hipLaunchKernelGGL(attention_f32_staged_kernel<2>, dim3(row_blocks / 2, (unsigned)f.heads), dim3(256), staged_lds(2), s,
                               qkv, att, H, d, n_req, f.max_pos, ws.meta, ws.seq_len, ws.row_start);
        else if (staged == 1)
            hipLaunchKernelGGL(attention_f32_staged_kernel<1>, dim3(row_blocks, (unsigned)f.heads), dim3(256), staged_lds(1), s,
                               qkv, att, H, d, n_req, f.max_pos, ws.meta, ws.seq_len, ws.row_start);
        else if (att_rows == 4)
            hipLaunchKernelGGL(attention_f32_kernel<4>, dim3(row_blocks / 4, (unsigned)f.heads), dim3(256), att_lds4, s,
                               qkv, att, H, d, n_req, f.max_pos, ws.meta, ws.seq_len, ws.row_start);
        else
            hipLaunchKernelGGL(attention_f32_kernel<1>, dim3(row_blocks, (unsigned)f.heads), dim3(256), att_lds, s,
                               qkv, att, H, d, n_req, f.max_pos, ws.meta, ws.seq_len, ws.row_start);
    };
    if (f32_maps_take_norms(f, ws.max_rows)) {
        // x: the sums entering a layer (the embedding's are normalised already), y: those after the attention; the statistics
        // lie where the normalised rows would
        float2 *sx = (float2*)x1, *sy = sx + ws.max_rows;
        for (int l = 0; l < f.layers; ++l) {
            const LayerWeights& w = m->layers[(size_t)l];
            const StreamNorm nx = {l > 0 ? m->layers[(size_t)l - 1].ln2_g : nullptr, l > 0 ? m->layers[(size_t)l - 1].ln2_b : nullptr, sx, m->ln_eps};
            const StreamNorm ny = {w.ln1_g, w.ln1_b, sy, m->ln_eps}, none = {nullptr, nullptr, nullptr, 0.f};
            if (l == 0)
                gemm_f32_norm<F32_NONE, false, false>(x, (const float*)w.w_qkv, w.b_qkv, nullptr, qkv, ws.max_rows, 3 * H, H, none, none, ws.meta, s);
            else
                gemm_f32_norm<F32_NONE, true, false>(x, (const float*)w.w_qkv, w.b_qkv, nullptr, qkv, ws.max_rows, 3 * H, H, nx, none, ws.meta, s);
            attention();
            if (l == 0)
                gemm_f32_norm<F32_RESIDUAL, false, false>(att, (const float*)w.w_o, w.b_o, x, y, ws.max_rows, H, H, none, none, ws.meta, s);
            else
                gemm_f32_norm<F32_RESIDUAL, false, true>(att, (const float*)w.w_o, w.b_o, x, y, ws.max_rows, H, H, none, nx, ws.meta, s);
            gemm_f32_norm<F32_GELU, true, false>(y, (const float*)w.w_1, w.b_1, nullptr, g, ws.max_rows, F, H, ny, none, ws.meta, s);
            gemm_f32_norm<F32_RESIDUAL, false, true>(g, (const float*)w.w_2, w.b_2, y, x, ws.max_rows, H, F, none, ny, ws.meta, s);
        }
        return;                                                  // (the head takes the last LayerNorm)
    }
    auto layer_norm = [&](float* out, const float* gamma, const float* beta) {
        auto narrow = [&](auto kernel, unsigned threads) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(ws.max_rows / (threads / 8))), dim3(threads), 0, s, y, out, gamma, beta, m->ln_eps, H,
                               ws.meta);
        };
        if (narrow_norms(f)) {
            if (H <= 64) narrow(layernorm_f32_narrow_kernel<2, 256>, 256);
            else if (H <= 128) narrow(layernorm_f32_narrow_kernel<4, 64>, 64);
            else narrow(layernorm_f32_narrow_kernel<8, 64>, 64);
        } else
            hipLaunchKernelGGL(layernorm_f32_kernel, dim3(row_blocks), dim3(256), 0, s, y, out, gamma, beta, m->ln_eps, H, ws.meta);
    };
    for (int l = 0; l < f.layers; ++l) {
        const LayerWeights& w = m->layers[(size_t)l];
        gemm_f32<F32_NONE>(x, (const float*)w.w_qkv, w.b_qkv, nullptr, qkv, ws.max_rows, 3 * H, H, ws.meta, s);
        attention();
        gemm_f32<F32_RESIDUAL>(att, (const float*)w.w_o, w.b_o, x, y, ws.max_rows, H, H, ws.meta, s);
        layer_norm(x1, w.ln1_g, w.ln1_b);
        gemm_f32<F32_GELU>(x1, (const float*)w.w_1, w.b_1, nullptr, g, ws.max_rows, F, H, ws.meta, s);
        gemm_f32<F32_RESIDUAL>(g, (const float*)w.w_2, w.b_2, x1, y, ws.max_rows, H, F, ws.meta, s);
        layer_norm(x, w.ln2_g, w.ln2_b);
    }
}
