// Downstream target on top of the encoder output (Section 3.1, "Downstream Target"): text
// classification on the first token, logits = W_c tanh(W_p h[b, 0] + b_p) + b_c.
// One block per sequence, because the second product needs the whole pooled vector and the entry point has no
// workspace to hand it from block to block.  What bounds it is one CU reading the H x H weights: 1.2 MB at 768, 10 us at
// the 50 bytes per clock a CU pulls out of L2.  So everything serves keeping that stream going: 16 waves, a row is read by
// 32 lanes (768 and 1024 are whole multiples of their 256 channels), and a wave has its eight rows' loads of a channel
// section outstanding at once.  With four waves that finished one row before they asked for the next, the kernel waited
// out 192 memory latencies in a row: one sequence, us per launch, 128 -> 17.2 at 768 and 193 -> 25.7 at 1024.
// A lane keeps one sum for the even and one for the odd 256-channel sections, so that sums are formed in the order of 64 lanes
// that read 512 channels at a time; a single sum per lane is twice as long a chain and its error 14 % larger at 768, 21 % at
// 1024 (it is as fast at 768 and takes 24.4 us at 1024).
#include "samp_common.h"

namespace samp {
namespace {

constexpr int CLASSIFY_WAVES = 16, CLASSIFY_PAIRS = 4;       // a wave works on CLASSIFY_PAIRS pairs of rows at a time

__device__ __forceinline__ float half_wave_sum(float v)
{
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// y[n] = finish(n, W[n] . x) for all rows n of W [N, H]; x in LDS as X (binary16 or binary32), all waves of the block
template <class X, class Finish>
__device__ __forceinline__ void matrix_times_vector(const __half *__restrict__ W, const X *x, int N, int H, Finish finish)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & 31, upper = lane >> 5;
    constexpr int ROWS = 2 * CLASSIFY_PAIRS;
    for (int n0 = wave * ROWS; n0 < N; n0 += CLASSIFY_WAVES * ROWS) {
        float acc[CLASSIFY_PAIRS], odd[CLASSIFY_PAIRS];
        const __half *row[CLASSIFY_PAIRS];
#pragma unroll
        for (int p = 0; p < CLASSIFY_PAIRS; p++) {
            acc[p] = odd[p] = 0.0f;
            row[p] = W + (size_t)min(n0 + 2 * p + upper, N - 1) * H;            // rows past the end repeat the last one
        }
#pragma unroll 2
        for (int k0 = sub * 8; k0 < H; k0 += 512) {
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const int k = k0 + 256 * u;
                if (k < H) {
                    v8h w[CLASSIFY_PAIRS];
#pragma unroll
                    for (int p = 0; p < CLASSIFY_PAIRS; p++) w[p] = *reinterpret_cast<const v8h *>(row[p] + k);
                    float xv[8];
#pragma unroll
                    for (int e = 0; e < 8; e++) xv[e] = (float)x[k + e];
#pragma unroll
                    for (int p = 0; p < CLASSIFY_PAIRS; p++)
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            float &a = u ? odd[p] : acc[p];
                            a = __builtin_fmaf((float)w[p][e], xv[e], a);
                        }
                }
            }
        }
#pragma unroll
        for (int p = 0; p < CLASSIFY_PAIRS; p++) acc[p] += odd[p];
#pragma unroll
        for (int p = 0; p < CLASSIFY_PAIRS; p++) acc[p] = half_wave_sum(acc[p]);
#pragma unroll
        for (int p = 0; p < CLASSIFY_PAIRS; p++) {
            const int n = n0 + 2 * p + upper;
            if (sub == 0 && n < N) finish(n, acc[p]);
        }
    }
}

__global__ __launch_bounds__(64 * CLASSIFY_WAVES) void classify_kernel(const __half *__restrict__ hidden, size_t seq_stride,
                                                       const __half *__restrict__ w_pool, const float *__restrict__ b_pool,
                                                       const __half *__restrict__ w_cls, const float *__restrict__ b_cls,
                                                       int H, int C, float *__restrict__ logits)
{
    extern __shared__ __attribute__((aligned(16))) char sm[];                 // h[H] binary16, then pooled[H] binary32
    _Float16 *h = reinterpret_cast<_Float16 *>(sm);
    float *pooled = reinterpret_cast<float *>(sm + (size_t)H * 2);
    const __half *src = hidden + (size_t)blockIdx.x * seq_stride;           // first token of the sequence
    for (int k = threadIdx.x * 8; k < H; k += 64 * CLASSIFY_WAVES * 8) *reinterpret_cast<v4i *>(h + k) = *reinterpret_cast<const v4i *>(src + k);
    __syncthreads();
    matrix_times_vector(w_pool, h, H, H, [&](int n, float d) { pooled[n] = tanhf(d + b_pool[n]); });
    __syncthreads();
    matrix_times_vector(w_cls, pooled, C, H, [&](int n, float d) { logits[(size_t)blockIdx.x * C + n] = d + b_cls[n]; });
}

}  // namespace

hipError_t launch_classify(const __half *hidden, int B, int S, int H, const __half *w_pool, const float *b_pool,
                           const __half *w_cls, const float *b_cls, int C, float *logits, hipStream_t st)
{
    hipLaunchKernelGGL(classify_kernel, dim3(B), dim3(64 * CLASSIFY_WAVES), (size_t)H * 6, st, hidden, (size_t)S * H, w_pool,
                       b_pool, w_cls, b_cls, H, C, logits);
    return hipGetLastError();
}

}  // namespace samp
