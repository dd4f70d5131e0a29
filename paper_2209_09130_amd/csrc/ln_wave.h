// A LayerNorm row held by one wave (H = 64 CPL, CPL consecutive channels per lane): reductions inside DPP rows, loads, and the arithmetic of the
// fused step (rowwise.hip), for the kernels that form a row on the way to something else.
#pragma once
#include "samp_common.h"

namespace samp {
namespace {

template <int CTRL> __device__ __forceinline__ int dpp_mov(int v)
{ return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }

template <int CTRL> __device__ __forceinline__ double dpp_mov(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = dpp_mov<CTRL>((int)b), hi = dpp_mov<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// sum over the 16 lanes of a DPP row; every lane ends with the same bits (the adds commute)
__device__ __forceinline__ double row16_sum(double v)
{
    v += dpp_mov<0xB1>(v);            // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);            // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);           // row_half_mirror
    v += dpp_mov<0x140>(v);           // row_mirror
    return v;
}
template <bool I8, int CPL> __device__ __forceinline__ void load_lane(const void *p, size_t elem, float (&v)[CPL])
{
    static_assert(CPL % 4 == 0, "whole dwords of int8 channels per lane");
#pragma unroll
    for (int d = 0; d < CPL / 4; d++) {
        if (I8) {
            const int q = *reinterpret_cast<const int *>((const int8_t *)p + elem + 4 * d);
#pragma unroll
            for (int e = 0; e < 4; e++) v[4 * d + e] = (float)(int8_t)(q >> (8 * e));
        } else {
            const v4h h = *reinterpret_cast<const v4h *>((const __half *)p + elem + 4 * d);
#pragma unroll
            for (int e = 0; e < 4; e++) v[4 * d + e] = (float)h[e];
        }
    }
}
template <int CPL> __device__ __forceinline__ void load_lane_f32(const float *p, float (&v)[CPL])
{
#pragma unroll
    for (int q = 0; q < CPL / 4; q++) *reinterpret_cast<v4f *>(v + 4 * q) = *reinterpret_cast<const v4f *>(p + 4 * q);
}

__device__ __forceinline__ double lane_double(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | lo);
}
__device__ __forceinline__ double row64_sum(double v)
{
    v = row16_sum(v);
    return (lane_double(v, 0) + lane_double(v, 16)) + (lane_double(v, 32) + lane_double(v, 48));
}

// y = fmaf((z - mu) * rstd, gamma, beta), binary64 mean and variance rounded once
template <int CPL>
__device__ __forceinline__ void ln_normalise_wave(const float (&z)[CPL], double sum, const float (&gamma)[CPL], const float (&beta)[CPL], float eps,
                                                  float (&y)[CPL])
{
    constexpr int H = 64 * CPL;
    const double mu = row64_sum(sum) / (double)H;
    double sq = 0.0;
#pragma unroll
    for (int e = 0; e < CPL; e++) { const double d = (double)z[e] - mu; sq = __builtin_fma(d, d, sq); }
    const double var = row64_sum(sq) / (double)H;
    const float mu32 = (float)mu, rstd32 = (float)(1.0 / sqrt(var + (double)eps));
#pragma unroll
    for (int e = 0; e < CPL; e++) y[e] = __builtin_fmaf((z[e] - mu32) * rstd32, gamma[e], beta[e]);
}
__device__ __forceinline__ int pack_row_codes(const float *y, float inv_s)
{ return pack_codes(code_bits(y[0] * inv_s), code_bits(y[1] * inv_s), code_bits(y[2] * inv_s), code_bits(y[3] * inv_s)); }

// the row's sum of dequantised input, bias and residual (channels c ..): z, this lane's part of its sum; and the row's gamma and beta
template <int CPL, bool IN_I8, bool RES_I8>
__device__ __forceinline__ double ln_row_wave(const AddLnArgs &a, int row, int c, float (&z)[CPL], float (&gamma)[CPL], float (&beta)[CPL])
{
    constexpr int H = 64 * CPL;
    float x[CPL], r[CPL];
    load_lane<IN_I8>(a.in, (size_t)row * H + c, x);
    load_lane<RES_I8>(a.res, (size_t)row * H + c, r);
    load_lane_f32(a.bias + c, z);
    load_lane_f32(a.gamma + c, gamma);
    load_lane_f32(a.beta + c, beta);
    double sum = 0.0;
#pragma unroll
    for (int e = 0; e < CPL; e++) {
        const float u = IN_I8 ? __builtin_fmaf(x[e], a.s_in, z[e]) : x[e] + z[e];
        z[e] = RES_I8 ? __builtin_fmaf(r[e], a.s_res, u) : u + r[e];
        sum += (double)z[e];
    }
    return sum;
}

}  // namespace
}  // namespace samp
