// In-window checks of the proactive instance scaler (Sec. 3.4.2) on the look-ahead maps: for each
// instance the number of the next `window` iterations whose usage exceeds over_pct % of its capacity,
// the peak over the window, and whether that count is more than share_pct % of the window; over all
// instances how many are potentially overloaded, whether all stay below idle_pct %, and the number
// to isolate in that case, N_c - sum(max U) / T_f.  Percent thresholds are integers and every
// comparison is done in integers (tokens * 100 against percent * capacity), so the flags are exact.
#include "device_util.h"
#include "internal.h"

namespace {

// one wavefront per instance
__global__ __launch_bounds__(256) void scaler_rows_kernel(const int32_t* __restrict__ kv_tokens,
                                                          const int32_t* __restrict__ capacity, int n_inst,
                                                          int map_len, int window, int over_pct, int share_pct,
                                                          int32_t* __restrict__ over_count,
                                                          int32_t* __restrict__ peak_tokens,
                                                          int32_t* __restrict__ overloaded) {
    const int lane = threadIdx.x & 63;
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= n_inst) return;
    const int w = min(window, map_len);
    const long long M = capacity[k];
    int cnt = 0, pk = (int)0x80000000;
    if (M >= 1) {
        const int32_t* row = kv_tokens + (int64_t)k * map_len;
        for (int t = lane; t < w; t += 64) {
            const int n = row[t];
            cnt += (long long)n * 100 > (long long)over_pct * M ? 1 : 0;
            pk = max(pk, n);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            cnt += __shfl_xor(cnt, o, 64);
            pk = max(pk, __shfl_xor(pk, o, 64));
        }
    } else {
        pk = 0;
    }
    if (lane == 0) {
        over_count[k] = cnt;
        peak_tokens[k] = w >= 1 ? pk : 0;
        overloaded[k] = (long long)cnt * 100 > (long long)share_pct * w ? 1 : 0;
    }
}

// Totals by one wavefront.  The sum of the peak fractions is taken
// in instance order in fp64: the quotients of 64 instances at a time are made by the lanes and added one by one from
// their registers (a loop over memory with a division per instance took 27 us for 256 instances).
__device__ __forceinline__ void scaler_totals(const int32_t* capacity, const int32_t* peak_tokens, const int32_t* overloaded,
                                              int n_inst, int window, int idle_pct, int lane, int32_t* summary, double* scale_down) {
    int n_over = 0, idle = 1;
    double total = 0.0;
    for (int k0 = 0; k0 < n_inst; k0 += 64) {
        const int k = k0 + lane;
        double q = 0.0;                                    // (adding 0 for instances left out leaves the sum as it is)
        if (k < n_inst) {
            const int M = capacity[k], pk = peak_tokens[k];
            n_over += overloaded[k];
            if (M < 1 || window < 1 || !((long long)pk * 100 < (long long)idle_pct * M)) idle = 0;
            if (M >= 1 && window >= 1) q = (double)pk / (double)M;
        }
        const int lo = __double2loint(q), hi = __double2hiint(q);
#pragma unroll
        for (int l = 0; l < 64; ++l) total += __hiloint2double(__builtin_amdgcn_readlane(hi, l), __builtin_amdgcn_readlane(lo, l));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        n_over += __shfl_xor(n_over, o, 64);
        idle &= __shfl_xor(idle, o, 64);
    }
    if (lane == 0) {
        summary[0] = n_over;
        summary[1] = idle;
        scale_down[0] = (double)n_inst - total / ((double)idle_pct / 100.0);
    }
}

__global__ __launch_bounds__(64) void scaler_summary_kernel(const int32_t* __restrict__ capacity,
                                                            const int32_t* __restrict__ peak_tokens,
                                                            const int32_t* __restrict__ overloaded, int n_inst,
                                                            int window, int idle_pct, int32_t* __restrict__ summary,
                                                            double* __restrict__ scale_down) {
    scaler_totals(capacity, peak_tokens, overloaded, n_inst, window, idle_pct, threadIdx.x, summary, scale_down);
}

// Both parts in one launch by one workgroup, 16 lanes per instance and eight slots of a lane requested at a time: for
// clusters whose windows one compute unit reads in a few microseconds, the second launch costs more than it saves.
// Microseconds, two launches / one: 1 instance of 512 and 1000 slots 13 / 10 and 13 / 14, of 4096 13 / 45 (16 lanes read
// what 64 would, a trip to memory per 128 slots); 64 of 512 and 640 slots 13 / 12 and 13 / 14; 128 of 512 18 / 12;
// 256 of 256 31 / 11; 512 of 128 57 / 15.
constexpr int kOneMostInst = 512;
constexpr int kOneMostWindow = 512;
constexpr int kOneMostSlots = 65536;                       // n_inst * window
template <int CTRL>
__device__ __forceinline__ void sixteen(int& cnt, int& pk) {
    cnt += __builtin_amdgcn_update_dpp(0, cnt, CTRL, 0xf, 0xf, false);
    pk = max(pk, __builtin_amdgcn_update_dpp((int)0x80000000, pk, CTRL, 0xf, 0xf, false));
}
// VEC: rows are whole 16-byte groups, a lane takes four slots a load.  The quotients of the totals are made by a thread each and
// added in instance order from LDS, eight requested at a time.  256 instances of 100 slots 7.9 -> 6.9 us a call (slots one by one,
// quotients by one wavefront and added from its registers).
template <bool VEC>
__global__ __launch_bounds__(1024) void scaler_one_kernel(const int32_t* __restrict__ kv_tokens, const int32_t* __restrict__ capacity,
                                                          int n_inst, int map_len, int w, int over_pct, int share_pct, int idle_pct,
                                                          int32_t* __restrict__ over_count, int32_t* __restrict__ peak_tokens,
                                                          int32_t* __restrict__ overloaded, int32_t* __restrict__ summary,
                                                          double* __restrict__ scale_down) {
    __shared__ int32_t s_cap[kOneMostInst], s_peak[kOneMostInst], s_over[kOneMostInst];
    __shared__ __align__(16) double s_q[kOneMostInst];
    const int l = threadIdx.x & 15;
    constexpr int UK = 4;                                  // instances of a group of 16 lanes whose slots are requested together
    for (int k0 = threadIdx.x >> 4; k0 < n_inst; k0 += 64 * UK) {
        int M[UK], cnt[UK], pk[UK];
#pragma unroll
        for (int i = 0; i < UK; ++i) {
            M[i] = capacity[min(k0 + 64 * i, n_inst - 1)];
            cnt[i] = 0;
            pk[i] = (int)0x80000000;
        }
        auto look = [&](int i, int t, int v) {
            if (t < w) {
                cnt[i] += (long long)v * 100 > (long long)over_pct * M[i] ? 1 : 0;
                pk[i] = max(pk[i], v);
            }
        };
        if (VEC) {
            for (int t0 = 4 * l; t0 < w; t0 += 128) {
                int4 v[UK][2];
#pragma unroll
                for (int i = 0; i < UK; ++i) {
                    const int32_t* row = kv_tokens + (int64_t)min(k0 + 64 * i, n_inst - 1) * map_len;
                    v[i][0] = *(const int4*)(row + t0);
                    v[i][1] = *(const int4*)(row + (t0 + 64 < w ? t0 + 64 : t0));
                }
#pragma unroll
                for (int i = 0; i < UK; ++i)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int t = t0 + 64 * u;
                        look(i, t, v[i][u].x);
                        look(i, t + 1, v[i][u].y);
                        look(i, t + 2, v[i][u].z);
                        look(i, t + 3, v[i][u].w);
                    }
            }
        } else {
            for (int t0 = l; t0 < w; t0 += 128) {
                int v[UK][8];
#pragma unroll
                for (int i = 0; i < UK; ++i) {
                    const int32_t* row = kv_tokens + (int64_t)min(k0 + 64 * i, n_inst - 1) * map_len;
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[i][u] = row[min(t0 + 16 * u, w - 1)];
                }
#pragma unroll
                for (int i = 0; i < UK; ++i)
#pragma unroll
                    for (int u = 0; u < 8; ++u) look(i, t0 + 16 * u, v[i][u]);
            }
        }
#pragma unroll
        for (int i = 0; i < UK; ++i) {
            const int k = k0 + 64 * i;
            sixteen<0x111>(cnt[i], pk[i]);                 // row_shr 1, 2, 4, 8: lane 15 has all
            sixteen<0x112>(cnt[i], pk[i]);
            sixteen<0x114>(cnt[i], pk[i]);
            sixteen<0x118>(cnt[i], pk[i]);
            if (M[i] < 1) { cnt[i] = 0; pk[i] = 0; }
            if (w < 1) pk[i] = 0;
            if (l == 15 && k < n_inst) {
                const int over = (long long)cnt[i] * 100 > (long long)share_pct * w ? 1 : 0;
                over_count[k] = cnt[i];
                peak_tokens[k] = pk[i];
                overloaded[k] = over;
                s_cap[k] = M[i];
                s_peak[k] = pk[i];
                s_over[k] = over;
            }
        }
    }
    __syncthreads();
    // the totals, as scaler_totals
    const int k = threadIdx.x;
    bool over = false, busy = false;
    if (k < kOneMostInst) {
        double q = 0.0;                                    // (adding 0 for instances left out leaves the sum as it is)
        if (k < n_inst) {
            const int M = s_cap[k], pk = s_peak[k];
            over = s_over[k] != 0;
            busy = M < 1 || w < 1 || !((long long)pk * 100 < (long long)idle_pct * M);
            if (M >= 1 && w >= 1) q = (double)pk / (double)M;
        }
        s_q[k] = q;
    }
    const int n_over = __syncthreads_count(over), any_busy = __syncthreads_or(busy);
    if (threadIdx.x >= 64) return;
    double total = 0.0;
    for (int k0 = 0; k0 < n_inst; k0 += 8) {               // (512 is a multiple of 8)
        double2 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = *(const double2*)&s_q[k0 + 2 * u];
#pragma unroll
        for (int u = 0; u < 4; ++u) { total += q[u].x; total += q[u].y; }
    }
    if (threadIdx.x == 0) {
        summary[0] = n_over;
        summary[1] = any_busy ? 0 : 1;
        scale_down[0] = (double)n_inst - total / ((double)idle_pct / 100.0);
    }
}

}  // namespace

extern "C" int ps_scaler_scan(const int32_t* kv_tokens, const int32_t* capacity, int32_t n_inst, int32_t map_len,
                              int32_t window, int32_t over_pct, int32_t share_pct, int32_t idle_pct,
                              int32_t* over_count, int32_t* peak_tokens, int32_t* overloaded, int32_t* summary,
                              double* scale_down, void* hip_stream) {
    if (!kv_tokens || !capacity || !over_count || !peak_tokens || !overloaded || !summary || !scale_down) return PS_EINVAL;
    if (n_inst < 1 || map_len < 1 || window < 0 || over_pct < 0 || share_pct < 0 || idle_pct < 1) return PS_EINVAL;
    hipStream_t s = (hipStream_t)hip_stream;
    (void)hipGetLastError();
    const int w = min(window, map_len);
    if (n_inst <= kOneMostInst && w <= kOneMostWindow && (int64_t)n_inst * w <= kOneMostSlots) {
        const bool vec = map_len % 4 == 0 && (uintptr_t)kv_tokens % 16 == 0;
        hipLaunchKernelGGL(vec ? scaler_one_kernel<true> : scaler_one_kernel<false>, dim3(1), dim3(1024), 0, s, kv_tokens, capacity,
                           n_inst, map_len, w, over_pct, share_pct, idle_pct, over_count, peak_tokens, overloaded, summary, scale_down);
        return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
    }
    hipLaunchKernelGGL(scaler_rows_kernel, dim3((unsigned)((n_inst + 3) / 4)), dim3(256), 0, s, kv_tokens, capacity,
                       n_inst, map_len, window, over_pct, share_pct, over_count, peak_tokens, overloaded);
    hipLaunchKernelGGL(scaler_summary_kernel, dim3(1), dim3(64), 0, s, capacity, peak_tokens, overloaded, n_inst,
                       min(window, map_len), idle_pct, summary, scale_down);
    return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
}
