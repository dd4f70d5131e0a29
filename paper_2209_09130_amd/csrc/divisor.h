// Division by a number that the host knows, for the index arithmetic in front of a block's first load: the high half of one product instead of
// some 25 dependent operations.  Plain arithmetic, so that the host can test it.
#pragma once

#ifdef __HIPCC__
#define SAMP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SAMP_HOST_DEVICE inline
#endif

namespace samp {

// For dividends below n: ceil(2^32 / d), whose product with d is off by e < d; the quotient is exact while n e stays below 2^32.  0: d is 1.  1: it is not
// exact over that range (some hundred million items of a ragged batch), divide.
inline unsigned divisor(unsigned long long n, unsigned d)
{
    if (d <= 1) return 0;
    const unsigned by = (unsigned)(((1ull << 32) + d - 1) / d);
    return n * ((unsigned long long)by * d - (1ull << 32)) < 1ull << 32 && n <= 1ull << 32 ? by : 1;
}
SAMP_HOST_DEVICE unsigned over(unsigned n, unsigned by, unsigned d)
{
    if (by > 1) return (unsigned)(((unsigned long long)n * by) >> 32);
    return by ? n / d : n;
}

}  // namespace samp
