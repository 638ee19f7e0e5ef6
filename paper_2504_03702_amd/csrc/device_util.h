// Small device-side helpers: bf16 conversion, wavefront reductions, fault reporting.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "preserve.h"

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Round to nearest, ties to even.  NaN stays NaN (quiet bit forced).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Two floats -> two bf16 in one dword (lo in the low half).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

typedef __bf16 ps_bf16x2 __attribute__((ext_vector_type(2)));
typedef float ps_f32x2 __attribute__((ext_vector_type(2)));
// Two floats -> packed bf16 pair with the hardware conversion (round to nearest even).
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
    ps_f32x2 f = {lo, hi};
    ps_bf16x2 b = __builtin_convertvector(f, ps_bf16x2);
    return *reinterpret_cast<uint32_t*>(&b);
}

// Four consecutive int32 (16-byte aligned) that will not be read again: the non-temporal hint keeps a stream
// from displacing what the caches hold (a read-only pass over 529 MB ran at 6.7 TB/s with it, 6.0 without).
__device__ __forceinline__ int4 load_stream_int4(const int32_t* p) {
    int4 v;
    v.x = __builtin_nontemporal_load(p);
    v.y = __builtin_nontemporal_load(p + 1);
    v.z = __builtin_nontemporal_load(p + 2);
    v.w = __builtin_nontemporal_load(p + 3);
    return v;
}

// XOR swizzle of the 16-byte chunks of a 128-byte LDS row: chunk c of row r lives at position
// c ^ lds_swz(r).  Any 8 consecutive rows, and any 16 consecutive rows taken modulo two rows, then
// fall in different banks for a 16-byte read per lane.  Depends on r mod 16 only.
__device__ __forceinline__ int lds_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Inclusive prefix sums over the wavefront (rows of 16 lanes with ROWS_ONLY), by the vector unit's own lane moves: a shuffle is a
// trip through LDS a step and half.
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_add64(long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, ROWS, 0xf, false);
    return v + (((long long)hi << 32) | lo);
}
template <bool ROWS_ONLY = false>
__device__ __forceinline__ long long prefix_sum64(long long v) {
    v = dpp_add64<0x111, 0xf>(v);        // row_shr 1, 2, 4, 8
    v = dpp_add64<0x112, 0xf>(v);
    v = dpp_add64<0x114, 0xf>(v);
    v = dpp_add64<0x118, 0xf>(v);
    if (ROWS_ONLY) return v;
    v = dpp_add64<0x142, 0xa>(v);        // row_bcast 15 into rows 1 and 3
    return dpp_add64<0x143, 0xc>(v);     // row_bcast 31 into rows 2 and 3
}
__device__ __forceinline__ long long readlane64(long long v, int l) {
    return ((long long)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) | (unsigned)__builtin_amdgcn_readlane((int)v, l);
}
// Of sixteen wavefronts' values (in LDS): the sum of those in front of wavefront `wave`, and of all.
__device__ __forceinline__ long long sum_in_front(const long long* s_wave, int wave, long long& all) {
    const long long incl = prefix_sum64<true>(s_wave[threadIdx.x & 15]);
    all = readlane64(incl, 15);
    return wave > 0 ? readlane64(incl, wave - 1) : 0;
}

// erf-GELU x * Phi(x) with Phi(x) - 1/2 = x * Q(x^2) on |x| <= 4.5 (Q: degree-8 least-squares fit on Chebyshev
// nodes, coefficients taken to the variable x^2) and Phi clamped beyond; absolute error of the result below
// 6e-5, under the bf16 rounding of the stored value wherever the value is not itself tiny.  Eleven full-rate
// operations instead of the several dozen of a branching erff.
__device__ __forceinline__ float gelu_erf(float v) {
    const float xc = __builtin_amdgcn_fmed3f(v, -4.5f, 4.5f);
    const float s = xc * xc;
    float q = 2.917371829e-11f;
    q = fmaf(q, s, -3.208389305e-09f);
    q = fmaf(q, s, 1.551676639e-07f);
    q = fmaf(q, s, -4.373868311e-06f);
    q = fmaf(q, s, 8.053694228e-05f);
    q = fmaf(q, s, -1.031751237e-03f);
    q = fmaf(q, s, 9.564368315e-03f);
    q = fmaf(q, s, -6.595010928e-02f);
    q = fmaf(q, s, 3.986949891e-01f);
    return v * fmaf(xc, q, 0.5f);
}

// Record a fault found in device data: OR the flag, keep the smallest index.  first_bad holds
// (2^62 - index) so that a maximum over a zero-initialised word finds the smallest index.
// Faults are exceptional, so the two atomics are off the fast path.
__device__ __forceinline__ void report_fault(ps_status* st, int flag, int64_t index) {
    if (!st) return;
    atomicOr(&st->flags, flag);
    atomicMax((long long*)&st->first_bad, (long long)(((int64_t)1 << 62) - index));
}

// ---- The residual stream: 32-bit sums kept as two arrays of 16 bits ------------------------------------------
// The float's bits plus 0x8000 are cut in two: hi, the upper half, is the sum rounded to bf16 (ties away from zero), the
// operand of the next map; hi and lo together are the float.  Two instructions an element either way; hi and lo as two
// bf16 values, which kept 16 significant bits of a sum, took three.  Ties are as rare as one in 2^16 among the sums of
// products, so where they go does not matter; sums of few bits go through stream_ties_to_even first.
#define PS_STREAM_ZERO_LO 0x8000u     // lo of a zero (hi is 0)
__device__ __forceinline__ float stream_join(uint16_t hi, uint16_t lo) {
    return __uint_as_float((((uint32_t)hi << 16) | lo) - 0x8000u);
}
// Two neighbouring elements at a time, of a word of each array.
__device__ __forceinline__ float2 stream_join2(uint32_t hi, uint32_t lo) {
    return make_float2(__uint_as_float(__builtin_amdgcn_perm(hi, lo, 0x05040100u) - 0x8000u),
                       __uint_as_float(__builtin_amdgcn_perm(hi, lo, 0x07060302u) - 0x8000u));
}
__device__ __forceinline__ void stream_split2(float a, float b, uint32_t& hi, uint32_t& lo) {
    const uint32_t x = __float_as_uint(a) + 0x8000u, y = __float_as_uint(b) + 0x8000u;
    hi = __builtin_amdgcn_perm(y, x, 0x07060302u);
    lo = __builtin_amdgcn_perm(y, x, 0x05040100u);
}
// A sum halfway between two bf16 values whose lower one is even, one float step lower, so that stream_split2 rounds ties to
// even.  A fifth of the sums of a token's and a position's bf16 embedding are ties: all of them away from zero, the first
// maps' operand was 0.08 % too large throughout, an error that no sum over keys or features averages out.
__device__ __forceinline__ float stream_ties_to_even(float x) {
    const uint32_t b = __float_as_uint(x);
    return __uint_as_float(b - ((b & 0x1ffffu) == 0x8000u ? 1u : 0u));
}

// ---- LayerNorm pieces that several kernels must compute alike, to the last bit ----------------------------
// A new sum of the residual stream: a map's product, its bias and the LayerNorm of the sum before it, whose row has
// st = (mean, 1 / std); shift: beta + bias.
__device__ __forceinline__ float residual_sum(float product, float y, float2 st, float gamma, float shift) {
    return product + fmaf(fmaf(y, st.y, -st.x * st.y), gamma, shift);
}

// (mean, 1 / std) from a row's sum and sum of squares (biased variance).
__device__ __forceinline__ float2 ln_moments(float sum, float sq, float inv_n, float eps) {
    const float mean = sum * inv_n;
    const float var = fmaxf(fmaf(sq, inv_n, -(mean * mean)), 0.f);
    return make_float2(mean, 1.0f / sqrtf(var + eps));
}

// LayerNorm of a value of the stream.
__device__ __forceinline__ float ln_apply(float y, float2 st, float gamma, float beta) {
    return fmaf((y - st.x) * st.y, gamma, beta);
}

// (mean, 1 / std) of one row of the stream by one wavefront, in two passes.
__device__ __forceinline__ float2 row_moments(const uint16_t* yh, const uint16_t* yl, int H, float eps, int lane) {
    float sum = 0.f;
#pragma unroll 4
    for (int i = lane; i < H; i += 64) sum += stream_join(yh[i], yl[i]);
    const float mean = wave_sum(sum) / (float)H;
    float sq = 0.f;
#pragma unroll 4
    for (int i = lane; i < H; i += 64) {
        const float d = stream_join(yh[i], yl[i]) - mean;
        sq = fmaf(d, d, sq);
    }
    return make_float2(mean, 1.0f / sqrtf(wave_sum(sq) / (float)H + eps));
}

// Sum over 8 consecutive lanes (lanes 8 r .. 8 r + 7) with DPP moves; every one of them gets the total.
// The order of the additions is fixed, so the result does not change from run to run.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row8_sum(float v) {
    v = dpp_add<0xB1>(v);      // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v);      // quad_perm [2, 3, 0, 1]
    return dpp_add<0x141>(v);  // row_half_mirror: lane i of each group of 8 takes lane 7 - i
}

// Whole lines out of an accumulator tile.  Four sets of R registers, each a run of 8 positions of a line of 64: in, set (a, b)
// of lane l holds the run at 32 a + 16 b + 8 (l / 32) of the line that belongs to l % 32; out, it holds the run at
// 32 (l / 8 % 2) + 16 (l / 16 % 2) + 8 (l / 32) of the line that belongs to l % 32 with bit 3 a and bit 4 b: the 8 lanes that
// differ in bits 3 to 5 hold a line, and an access by 16 bytes a lane covers 8 of them.  A store of 16-byte pieces of 32 lines,
// or of halves of 16, keeps the memory pipeline busy several times as long.
template <int R>
__device__ __forceinline__ void gather_runs(uint32_t (&u)[2][2][R]) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // the second and fourth 16 lanes of b = 0 with the first and third of b = 1
            const auto x = __builtin_amdgcn_permlane16_swap(u[a][0][r], u[a][1][r], false, false);
            u[a][0][r] = x[0];
            u[a][1][r] = x[1];
        }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // the upper 8 of every 16 lanes of a = 0 with the lower 8 of a = 1 (row_ror:8, two banks of four)
            const uint32_t x = u[0][b][r], y = u[1][b][r];
            u[0][b][r] = __builtin_amdgcn_update_dpp(x, y, 0x128, 0xf, 0xc, false);
            u[1][b][r] = __builtin_amdgcn_update_dpp(y, x, 0x128, 0xf, 0x3, false);
        }
}

// ---- LayerNorm of narrow fp32 rows (hidden a multiple of 32, at most PS_NARROW_WIDTH) ----------------------------------
// In eight parts: part 2 w + h has the upper (h) or lower four of every eight elements in the w-th quarter of the row, adds
// them up four at a time, and the parts' sums are paired neighbour by neighbour.
__device__ __forceinline__ float narrow_quad(float a, float b, float c, float d) { return (a + b) + (c + d); }
__device__ __forceinline__ float narrow_squares(float a, float b, float c, float d) {
    return fmaf(a, a, b * b) + fmaf(c, c, d * d);
}
// (mean, 1 / std) of row x by eight neighbouring lanes, lane `part` of them; all get it.
__device__ __forceinline__ float2 narrow_moments(const float* x, int H, float eps, int part) {
    const int groups = H / 8, g0 = groups * (part >> 1) / 4, g1 = groups * ((part >> 1) + 1) / 4, at = 4 * (part & 1);
    auto all = [](float v) {
        v += __shfl_xor(v, 1, 64);
        v += __shfl_xor(v, 2, 64);
        return v + __shfl_xor(v, 4, 64);
    };
    float sum = 0.f, sq = 0.f;
    for (int g = g0; g < g1; ++g) {
        const float4 v = *(const float4*)(x + 8 * g + at);
        sum += narrow_quad(v.x, v.y, v.z, v.w);
    }
    const float mean = all(sum) / (float)H;      // (a product would be contracted with what follows, here or there)
    for (int g = g0; g < g1; ++g) {
        const float4 v = *(const float4*)(x + 8 * g + at);
        sq += narrow_squares(v.x - mean, v.y - mean, v.z - mean, v.w - mean);
    }
    return make_float2(mean, 1.0f / sqrtf(all(sq) / (float)H + eps));
}
