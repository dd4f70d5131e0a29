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
// A row's statistics are a chain of dependent binary64 operations that every launch of few rows waits for.  At width 768, where mean and variance take
// divisions, they have short forms of the divisions and of the root (some 45 operations with the library's) and sums in four chains; at the other
// widths, where dividing is a product, those are no gain (BERT-large 1 x 19 527 / 529, 16 x 64 1013 / 1020).  Forwards, us, before / now: BERT-base Fully-Quant
// 1 x 19 242 / 238, 1 x 64 292 / 286, 16 x 128 538 / 533, FP16 1 x 64 441 / 439.  (With four rows per wave the chain is shared and the kernel's registers are
// what counts: 32 x 128 754 / 761; not used there.)
template <int H> constexpr bool SHORT_STATISTICS = (H & (H - 1)) != 0;
template <int H> struct RowSum {                          // sum of a lane's values
    double part[SHORT_STATISTICS<H> ? 4 : 1] = {};
    __device__ __forceinline__ void add(int e, double v) { part[SHORT_STATISTICS<H> ? e & 3 : 0] += v; }
    __device__ __forceinline__ void add_square(int e, double v) { double &p = part[SHORT_STATISTICS<H> ? e & 3 : 0]; p = __builtin_fma(v, v, p); }
    __device__ __forceinline__ double total() const
    {
        if constexpr (SHORT_STATISTICS<H>) return (part[0] + part[1]) + (part[2] + part[3]);
        else return part[0];
    }
};
// v / H: the product with the reciprocal, corrected once, is the rounding of the division
template <int H> __device__ __forceinline__ double over_width(double v)
{
    constexpr double inv = 1.0 / H;
    if constexpr (!SHORT_STATISTICS<H>) return v * inv;
    const double q = v * inv;
    return __builtin_fma(__builtin_fma(-q, (double)H, v), inv, q);
}
// 1 / sqrt(v); short: one third-order step on the hardware's estimate, relative error below 2^-51 before the rounding to binary32
template <int H> __device__ __forceinline__ float reciprocal_root(double v)
{
    if (!SHORT_STATISTICS<H> || !(v > 0x1p-900 && v < 0x1p900)) return (float)(1.0 / sqrt(v));
    const double y = __builtin_amdgcn_rsq(v), e = __builtin_fma(-v * y, y, 1.0);
    return (float)__builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
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
    const double mu = over_width<H>(row64_sum(sum));
    RowSum<H> sq;
#pragma unroll
    for (int e = 0; e < CPL; e++) sq.add_square(e, (double)z[e] - mu);
    const double var = over_width<H>(row64_sum(sq.total()));
    const float mu32 = (float)mu, rstd32 = reciprocal_root<H>(var + (double)eps);
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
    RowSum<H> sum;
#pragma unroll
    for (int e = 0; e < CPL; e++) {
        const float u = IN_I8 ? __builtin_fmaf(x[e], a.s_in, z[e]) : x[e] + z[e];
        z[e] = RES_I8 ? __builtin_fmaf(r[e], a.s_res, u) : u + r[e];
        sum.add(e, (double)z[e]);
    }
    return sum.total();
}

}  // namespace
}  // namespace samp
