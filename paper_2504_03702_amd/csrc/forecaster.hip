// Online phase of the service workload predictor (Sec. 3.2, Alg. 2): per service, a multiplicative
// LSTM (Krause et al. 2016) for prompt tokens and one for response tokens forecast the current and
// then the next time window from the k past windows, and the forecasts give the number of instances
// N = max(P / mu_p, D / mu_d, (P + D) / mu_t).  A model sees its input sequence min-max normalised
// (Alg. 1's normalisation step): x = (v - min) / (max - min) over the sequence (a flat sequence takes
// the range as 1), and its output y goes back to token counts as min + (max - min) y, not below 0.
// The second step applies the model to the history extended by the first forecast: while that
// forecast lies inside the history's range the normalisation is unchanged and the recurrence simply
// goes on by one input; otherwise the k + 1 values are normalised afresh and the recurrence is run
// again from the start.
//
// The recurrence is a chain of k + 1 steps, each two products with H x H matrices (H <= 64) and two rounds of
// elementwise functions; a wavefront per service that read its matrices anew at every step (L2, 82 KB a step and
// model) took 33 us a step.  Here a workgroup is one service: four wavefronts per model, both models side by side.
// Lane j owns hidden unit j; wavefront g keeps column j of gate g's matrix and a quarter of W_mh's rows in registers
// (read once: the weights' bytes are what the call cannot do without), so a step is 64 + 16 multiply-adds, two
// exchanges through LDS and two barriers (64 units over 24 windows, with the library's functions and a division a step / so:
// 512 services 92 and 88 us, one 32.4 and 30.4).  What takes the time: vector ALU (some 150 instructions a step and
// wavefront, four wavefronts a SIMD) 56 % of it, and the waits in a step's chain of LDS reads (20 of 16 bytes a lane) and two
// barriers.  Broadcasting h and m by the multiply-adds' own lane selection instead of LDS reads: half-rate multiply-adds,
// no faster.
// c and h are kept by all four wavefronts alike.  fp32 arithmetic, four
// partial sums per product.  Matrices are stored input-major ([in][out]: element (out j, in i) at i * H + j), so the
// lanes of a wavefront read consecutive words.
// A model is packed as
//   w_mx[H] W_mh[H][H] w_hx[H] W_hm[H][H] b_h[H] w_ix[H] W_im[H][H] b_i[H] w_ox[H] W_om[H][H] b_o[H]
//   w_fx[H] W_fm[H][H] b_f[H] w_out[H] b_out
#include "device_util.h"
#include "internal.h"

namespace {

__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + expf(-z)); }

// The two functions as the workgroup's kernel takes them, on the hardware's 2^x and 1/x: a step of every wavefront holds
// one or two of each, and the library's forms with a division for the input were over half of its instructions.
// With t = y / ln 2 rounded and l = y - t ln 2 (ln 2 in two parts, or the error grows with |y|), e^y = E = 2^t (1 + l).  A
// Newton step on r = 1 / (1 + E) takes the residual 1 - r - 2^t r - 2^t l r, in which neither 1 + E nor E is rounded.  tanh:
// below 0.6 z + z^3 P(z^2) (P: degree-5 least-squares fit on Chebyshev nodes), from there 1 - 2 / (1 + e^2|z|).
// Largest / rms relative error against 64 bits, library / so, 400 k points a range of |z|: sigmoid below 0.6 1.3e-7 / 4.3e-8
// and 9.9e-8 / 3.3e-8, 0.6 to 8 1.3e-7 / 3.7e-8 and 1.3e-7 / 3.1e-8, 8 to 20 1.5e-7 / 3.6e-8 and 1.3e-7 / 3.0e-8, 20 to 80
// 1.1e-7 / 2.6e-8 and 1.0e-7 / 2.6e-8 (with ln 2 in one part and 1 + E rounded 1.7e-7 / 4.3e-8 at 4 to 8, 3.5e-7 / 1.1e-7
// at 20 to 80); tanh below 0.6 7.2e-8 / 2.5e-8 both, 0.6 to 1 1.5e-7 / 3.8e-8 and 1.3e-7 / 3.8e-8, above 7.6e-8 and 7.0e-8.
__device__ __forceinline__ float one_over_one_plus_exp(float y) {
    // the steps below must meet no infinity, in 2^t nor in t (as far out as this the result is 1 and 0 already); NaN stays
    y = y > 88.0f ? 88.0f : y < -88.0f ? -88.0f : y;
    const float t = y * 1.44269504f, e = __builtin_amdgcn_exp2f(t);
    const float l = e * fmaf(t, 1.90465421e-09f, fmaf(t, -0.693147182f, y));
    const float r = __builtin_amdgcn_rcpf(1.0f + (e + l));
    return fmaf(fmaf(-l, r, fmaf(-e, r, 1.0f - r)), r, r);
}
__device__ __forceinline__ float sigmoid_hw(float z) { return one_over_one_plus_exp(-z); }
__device__ __forceinline__ float tanh_hw(float z) {
    const float u = z * z;
    float q = 2.354979282e-03f;
    q = fmaf(q, u, -8.397393860e-03f);
    q = fmaf(q, u, 2.178482153e-02f);
    q = fmaf(q, u, -5.396116525e-02f);
    q = fmaf(q, u, 1.333331168e-01f);
    q = fmaf(q, u, -3.333333433e-01f);
    const float far = copysignf(fmaf(-2.0f, one_over_one_plus_exp(2.0f * fabsf(z)), 1.0f), z);
    return fabsf(z) < 0.6f ? fmaf(z * u, q, z) : far;
}

// A value that all lanes hold alike, in a scalar register (the weights fill the vector registers).
__device__ __forceinline__ float uniform(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

// HB: hidden rounded up to 32 or 64 (weights beyond `hidden` are zeros).
template <int HB>
__global__ __launch_bounds__(512, 4) void forecast_kernel(const float* __restrict__ weights, int hidden,
                                                       const float* __restrict__ hist_p,
                                                       const float* __restrict__ hist_d, int k,
                                                       const float* __restrict__ mu, float* __restrict__ out) {
    constexpr int Q = HB / 4;                               // rows of W_mh per wavefront
    __shared__ __align__(16) float s_v[8][64];              // a wavefront's own copy of h, then of m
    __shared__ float s_a[2][4][64], s_g[2][4][64];          // partial products with W_mh; gate values
    __shared__ float s_y[2][2];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kind = wave >> 2, gate = wave & 3;            // gates in storage order: hh, i, o, f
    const int s = blockIdx.x, H = hidden;
    const bool unit = lane < H;
    const size_t model_floats = (size_t)5 * H * H + 10 * H + 1;
    const float* w = weights + (size_t)(2 * s + kind) * model_floats;
    const float* W_mh = w + H;
    const float* gates = W_mh + H * H;                      // per gate: input weights [H], matrix [H][H], bias [H]
    const float* gw = gates + (size_t)gate * (H * H + 2 * H);
    const float* w_out = gates + (size_t)4 * (H * H + 2 * H);
    float wm[Q], wg[HB];
#pragma unroll
    for (int i = 0; i < Q; ++i) wm[i] = unit && gate * Q + i < H ? W_mh[(gate * Q + i) * H + lane] : 0.f;
#pragma unroll
    for (int i = 0; i < HB; ++i) wg[i] = unit && i < H ? gw[H + i * H + lane] : 0.f;
    const float w_mx = unit ? w[lane] : 0.f, w_x = unit ? gw[lane] : 0.f, b_x = unit ? gw[H + H * H + lane] : 0.f;
    const float w_o = unit ? w_out[lane] : 0.f, b_out = w_out[H];
    const float* hist = (kind == 0 ? hist_p : hist_d) + (size_t)s * k;
    float lo = hist[min(lane, k - 1)], hi = lo;
    for (int t = lane + 64; t < k; t += 64) {
        lo = fminf(lo, hist[t]);
        hi = fmaxf(hi, hist[t]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o, 64));
        hi = fmaxf(hi, __shfl_xor(hi, o, 64));
    }
    lo = uniform(lo);
    hi = uniform(hi);
    float span = uniform(hi > lo ? hi - lo : 1.0f);
    float y0 = 0.f, y1 = 0.f;                               // this model's forecasts
    // pass 0: the k past windows, then (first forecast inside [lo, hi]) one more input.  pass 1, only if the
    // first forecast left that range: the k + 1 values again under their own normalisation.  Both models of the
    // workgroup meet its barriers the same number of times: if one needs the second pass, the other runs it on
    // its data all the same and discards the result.
    bool needs_second = false;
    for (int pass = 0; pass < 2; ++pass) {
        float h = 0.f, c = 0.f, xs = 0.f;
        for (int t = 0; t <= k; ++t) {
            // the inputs of 64 steps at a time, a lane each
            if ((t & 63) == 0) xs = (hist[min(t + lane, k - 1)] - lo) / span;
            float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(xs), t & 63));
            if (t == k) x = (y0 - lo) / span;
            // m = (w_mx x) * (W_mh h): this wavefront's rows of W_mh
            s_v[wave][lane] = h;
            __builtin_amdgcn_wave_barrier();
            float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < Q; i += 4) {
                const float4 hv = *(const float4*)&s_v[wave][gate * Q + i];
                a[0] = fmaf(wm[i], hv.x, a[0]); a[1] = fmaf(wm[i + 1], hv.y, a[1]);
                a[2] = fmaf(wm[i + 2], hv.z, a[2]); a[3] = fmaf(wm[i + 3], hv.w, a[3]);
            }
            s_a[kind][gate][lane] = (a[0] + a[1]) + (a[2] + a[3]);
            __syncthreads();
            const float am = (s_a[kind][0][lane] + s_a[kind][1][lane]) + (s_a[kind][2][lane] + s_a[kind][3][lane]);
            s_v[wave][lane] = unit ? (w_mx * x) * am : 0.f;
            __builtin_amdgcn_wave_barrier();
            float z[4] = {fmaf(w_x, x, b_x), 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < HB; i += 4) {
                const float4 mv = *(const float4*)&s_v[wave][i];
                z[0] = fmaf(wg[i], mv.x, z[0]); z[1] = fmaf(wg[i + 1], mv.y, z[1]);
                z[2] = fmaf(wg[i + 2], mv.z, z[2]); z[3] = fmaf(wg[i + 3], mv.w, z[3]);
            }
            const float zs = (z[0] + z[1]) + (z[2] + z[3]);
            s_g[kind][gate][lane] = gate == 0 ? tanh_hw(zs) : sigmoid_hw(zs);
            __syncthreads();
            c = s_g[kind][3][lane] * c + s_g[kind][1][lane] * s_g[kind][0][lane];
            h = unit ? tanh_hw(c) * s_g[kind][2][lane] : 0.f;
            if (t >= k - 1) {                               // after the k-th input and after the extension
                const float dot = wave_sum(w_o * h);
                const float f = uniform(fmaxf(0.f, fmaf(span, dot + b_out, lo)));
                if (pass == 0) {
                    if (t == k - 1) {
                        y0 = f;
                        needs_second = f < lo || f > hi;
                    } else {
                        y1 = f;
                    }
                } else if (needs_second && t == k) {
                    y1 = f;
                }
            }
        }
        // neither model needs the second pass (decided by all threads together, so every one leaves or stays)
        if (pass == 0 && !__syncthreads_or((int)needs_second)) break;
        // normalisation of the extended history for the second pass
        if (needs_second) {
            lo = uniform(fminf(lo, y0));
            hi = uniform(fmaxf(hi, y0));
            span = uniform(hi > lo ? hi - lo : 1.0f);
        }
    }
    if (gate == 0 && lane == 0) { s_y[kind][0] = y0; s_y[kind][1] = y1; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const float p2 = s_y[0][1], d2 = s_y[1][1];
        float* o = out + (size_t)s * 5;
        o[0] = s_y[0][0]; o[1] = s_y[1][0]; o[2] = p2; o[3] = d2;
        o[4] = fmaxf(fmaxf(p2 / mu[3 * s], d2 / mu[3 * s + 1]), (p2 + d2) / mu[3 * s + 2]);
    }
}

// Thousands of services with small models: a workgroup each would be mostly barriers and idle lanes (its 512 threads for
// 8 x 8 matrices), so here a wavefront is one service, 32 to a compute unit; it reads its weights, a few KB that stay in
// the caches, anew at every step, and does its two models one after the other.
__global__ __launch_bounds__(256) void forecast_many_kernel(const float* __restrict__ weights, int hidden,
                                                       const float* __restrict__ hist_p,
                                                       const float* __restrict__ hist_d, int n_services, int k,
                                                       const float* __restrict__ mu, float* __restrict__ out) {
    __shared__ float s_h[4][64], s_m[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = blockIdx.x * 4 + wave;
    const bool live = s < n_services;                       // whole wavefront; dead ones still meet the barriers
    const bool unit = lane < hidden;
    const int H = hidden;
    const size_t model_floats = (size_t)5 * H * H + 10 * H + 1;
    float y[2][2] = {{0.f, 0.f}, {0.f, 0.f}};               // [kind][step]
    for (int kind = 0; kind < 2; ++kind) {
        const float* w = weights + (size_t)(2 * (live ? s : 0) + kind) * model_floats;
        const float* w_mx = w;
        const float* W_mh = w_mx + H;
        const float* w_hx = W_mh + H * H;
        const float* W_hm = w_hx + H;
        const float* b_h = W_hm + H * H;
        const float* w_ix = b_h + H;
        const float* W_im = w_ix + H;
        const float* b_i = W_im + H * H;
        const float* w_ox = b_i + H;
        const float* W_om = w_ox + H;
        const float* b_o = W_om + H * H;
        const float* w_fx = b_o + H;
        const float* W_fm = w_fx + H;
        const float* b_f = W_fm + H * H;
        const float* w_out = b_f + H;
        const float b_out = w_out[H];
        const float* hist = (kind == 0 ? hist_p : hist_d) + (size_t)(live ? s : 0) * k;
        // minimum and maximum of the history (every lane scans it: the values are wave-uniform)
        float lo = hist[0], hi = hist[0];
        for (int t = 1; t < k; ++t) {
            lo = fminf(lo, hist[t]);
            hi = fmaxf(hi, hist[t]);
        }
        float span = hi > lo ? hi - lo : 1.0f;
        // pass 0: the k past windows, then (first forecast inside [lo, hi]) one more input.  pass 1, only if the
        // first forecast left that range: the k + 1 values again under their own normalisation.
        // The barriers below are met by all four wavefronts of the workgroup the same number of times whatever
        // their passes: if one of them needs the second pass, the others run it on their data all the same and
        // discard the result (needs_second false: y is not overwritten).
        bool needs_second = false;
        for (int pass = 0; pass < 2; ++pass) {
            float h = 0.f, c = 0.f;
            s_h[wave][lane] = 0.f;
            __syncthreads();
            for (int t = 0; t <= k; ++t) {
                const float v = t < k ? hist[t] : y[kind][0];
                const float x = (v - lo) / span;
                float a = 0.f;
                if (unit) {
#pragma unroll 16
                    for (int j = 0; j < H; ++j) a = fmaf(W_mh[j * H + lane], s_h[wave][j], a);
                }
                s_m[wave][lane] = unit ? (w_mx[lane] * x) * a : 0.f;
                __syncthreads();
                if (unit) {
                    float hh = fmaf(w_hx[lane], x, b_h[lane]), gi = fmaf(w_ix[lane], x, b_i[lane]);
                    float go = fmaf(w_ox[lane], x, b_o[lane]), gf = fmaf(w_fx[lane], x, b_f[lane]);
#pragma unroll 8
                    for (int j = 0; j < H; ++j) {
                        const float mj = s_m[wave][j];
                        hh = fmaf(W_hm[j * H + lane], mj, hh);
                        gi = fmaf(W_im[j * H + lane], mj, gi);
                        go = fmaf(W_om[j * H + lane], mj, go);
                        gf = fmaf(W_fm[j * H + lane], mj, gf);
                    }
                    c = sigmoid_f(gf) * c + sigmoid_f(gi) * tanhf(hh);
                    h = tanhf(c) * sigmoid_f(go);
                }
                s_h[wave][lane] = unit ? h : 0.f;
                __syncthreads();
                if (t >= k - 1) {                           // after the k-th input and after the extension
                    const float dot = wave_sum(unit ? w_out[lane] * h : 0.f);
                    const float f = fmaxf(0.f, fmaf(span, dot + b_out, lo));
                    if (pass == 0) {
                        y[kind][t - (k - 1)] = f;
                        if (t == k - 1) {
                            needs_second = f < lo || f > hi;
                        }
                    } else if (needs_second && t == k) {
                        y[kind][1] = f;
                    }
                }
            }
            // no wavefront of this workgroup needs the second pass (decided by all its threads together, so
            // every one of them leaves or stays)
            if (pass == 0 && !__syncthreads_or((int)needs_second)) break;
            // normalisation of the extended history for the second pass
            const float f1 = y[kind][0];
            if (needs_second) {
                lo = fminf(lo, f1);
                hi = fmaxf(hi, f1);
                span = hi > lo ? hi - lo : 1.0f;
            }
        }
    }
    if (live && lane == 0) {
        const float p2 = y[0][1], d2 = y[1][1];
        float* o = out + (size_t)s * 5;
        o[0] = y[0][0]; o[1] = y[1][0]; o[2] = p2; o[3] = d2;
        o[4] = fmaxf(fmaxf(p2 / mu[3 * s], d2 / mu[3 * s + 1]), (p2 + d2) / mu[3 * s + 2]);
    }
}

// Microseconds, a workgroup each / a wavefront each, over 24 windows unless said: 2048 services 192 / 108 (1 unit), 193 / 157
// (4), 192 / 211 (8); 8192 services 694 / 555 (8), 698 / 742 (16), over 6 windows 259 / 222 (16), over 1 window 276 / 202 (32);
// 1024 services of 1 and 4 units 100 / 103 and 101 / 159, 1536 of 1 unit 148 / 110.
bool many_pays(int32_t n, int32_t hidden, int32_t k) {
    if (n <= 1024) return false;                             // (all of them on the chip at once)
    if (hidden == 1 || hidden * (k + 1ll) <= 16) return true;
    if (n >= 2048 && (hidden <= 4 || hidden * (k + 1ll) <= 32)) return true;
    return n >= 3072 && (hidden <= 8 || (hidden <= 16 && k <= (n >= 16384 ? 12 : 6)) || (hidden <= 32 && k == 1));
}

}  // namespace

extern "C" int ps_forecast(const float* weights, int32_t hidden, const float* hist_p, const float* hist_d,
                           int32_t n_services, int32_t k, const float* mu, float* out, void* hip_stream) {
    if (!weights || !hist_p || !hist_d || !mu || !out || n_services < 0 || k < 1) return PS_EINVAL;
    if (hidden < 1 || hidden > 64) return PS_EUNSUPPORTED;
    if (n_services == 0) return PS_OK;
    (void)hipGetLastError();
    const size_t model_floats = (size_t)5 * hidden * hidden + 10 * hidden + 1;
    const int32_t most = 1 << 22;                            // services per launch (a grid holds fewer than 2^32 threads)
    for (int32_t s0 = 0, n; s0 < n_services; s0 += n) {
        n = n_services - s0 < most ? n_services - s0 : most;
        const dim3 grid((unsigned)n), block(512);
        const float *w = weights + (size_t)2 * s0 * model_floats, *hp = hist_p + (size_t)s0 * k, *hd = hist_d + (size_t)s0 * k;
        const float* mu0 = mu + (size_t)3 * s0;
        float* o = out + (size_t)5 * s0;
        hipStream_t st = (hipStream_t)hip_stream;
        if (many_pays(n_services, hidden, k))
            hipLaunchKernelGGL(forecast_many_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, w, hidden, hp, hd, n, k, mu0, o);
        else if (hidden <= 32)
            hipLaunchKernelGGL(forecast_kernel<32>, grid, block, 0, st, w, hidden, hp, hd, k, mu0, o);
        else
            hipLaunchKernelGGL(forecast_kernel<64>, grid, block, 0, st, w, hidden, hp, hd, k, mu0, o);
    }
    return hipGetLastError() == hipSuccess ? PS_OK : PS_EHIP;
}
