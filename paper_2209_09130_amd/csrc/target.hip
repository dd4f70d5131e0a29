// Downstream target on top of the encoder output (Section 3.1, "Downstream Target"): text
// classification on the first token, logits = W_c tanh(W_p h[b, 0] + b_p) + b_c.
// Two forms.  With a workspace for the pooled vectors (what the Python entry uses): one launch forms them, eight or sixteen
// rows of W_p per block, so that a hundred blocks share the 1.2 MB of weights (768 channels) that bound the step, and a second one the logits.
// Without: one block per sequence, because the second product needs the whole pooled vector; there the step lasts as long as one CU takes to
// read the H x H weights, 10 us at the 50 bytes per clock it pulls out of L2, and everything serves keeping that stream
// going: 16 waves, a row is read by 32 lanes (768 and 1024 are whole multiples of their 256 channels), and a wave has its eight
// rows' loads of a channel section outstanding at once.  (With four waves that finished one row before they asked for the next, the
// kernel waited out 192 memory latencies in a row: one sequence, us per launch, 128 -> 17.2 at 768 and 193 -> 25.7 at 1024.)
// A lane keeps one sum for the even and one for the odd 256-channel sections, so that sums are formed in the order of 64 lanes
// that read 512 channels at a time; a single sum per lane is twice as long a chain and its error 14 % larger at 768, 21 % at
// 1024 (it is as fast at 768 and takes 24.4 us at 1024).  Both forms give the same bits.
#include "samp_common.h"

#include <algorithm>

namespace samp {
namespace {

constexpr int CLASSIFY_WAVES = 16;

__device__ __forceinline__ float half_wave_sum(float v)
{
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// finish(v, n, W[n] . x[v]) for vectors v = 0 .. V - 1 and rows n of W [N, H], n0 + 2 PAIRS wave on by steps of 2 PAIRS waves; x(v, k) reads
// channels k .. k + 7 of vector v.  A wave works on PAIRS pairs of rows at a time.
template <int V, int PAIRS, class Read, class Finish>
__device__ __forceinline__ void matrix_times_vectors(const __half *__restrict__ W, Read x, int N, int H, int n0, int waves, Finish finish)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane & 31, upper = lane >> 5;
    constexpr int ROWS = 2 * PAIRS;
    for (n0 += wave * ROWS; n0 < N; n0 += waves * ROWS) {
        float acc[V][PAIRS], odd[V][PAIRS];
        const __half *row[PAIRS];
#pragma unroll
        for (int p = 0; p < PAIRS; p++) {
#pragma unroll
            for (int v = 0; v < V; v++) acc[v][p] = odd[v][p] = 0.0f;
            row[p] = W + (size_t)min(n0 + 2 * p + upper, N - 1) * H;            // rows past the end repeat the last one
        }
#pragma unroll 2
        for (int k0 = sub * 8; k0 < H; k0 += 512) {
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const int k = k0 + 256 * u;
                if (k < H) {
                    v8h w[PAIRS];
#pragma unroll
                    for (int p = 0; p < PAIRS; p++) w[p] = *reinterpret_cast<const v8h *>(row[p] + k);
#pragma unroll
                    for (int v = 0; v < V; v++) {
                        float xv[8];
                        x(v, k, xv);
#pragma unroll
                        for (int p = 0; p < PAIRS; p++)
#pragma unroll
                            for (int e = 0; e < 8; e++) {
                                float &a = u ? odd[v][p] : acc[v][p];
                                a = __builtin_fmaf((float)w[p][e], xv[e], a);
                            }
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < V; v++)
#pragma unroll
            for (int p = 0; p < PAIRS; p++) acc[v][p] = half_wave_sum(acc[v][p] + odd[v][p]);
#pragma unroll
        for (int p = 0; p < PAIRS; p++) {
            const int n = n0 + 2 * p + upper;
            if (sub == 0 && n < N)
#pragma unroll
                for (int v = 0; v < V; v++) finish(v, n, acc[v][p]);
        }
    }
}
template <class X> __device__ __forceinline__ void read8(const X *x, float (&xv)[8])
{
#pragma unroll
    for (int e = 0; e < 8; e++) xv[e] = (float)x[e];
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
    matrix_times_vectors<1, 4>(w_pool, [&](int, int k, float (&xv)[8]) { read8(h + k, xv); }, H, H, 0, CLASSIFY_WAVES,
                               [&](int, int n, float d) { pooled[n] = tanhf(d + b_pool[n]); });
    __syncthreads();
    matrix_times_vectors<1, 4>(w_cls, [&](int, int k, float (&xv)[8]) { read8(pooled + k, xv); }, C, H, 0, CLASSIFY_WAVES,
                               [&](int, int n, float d) { logits[(size_t)blockIdx.x * C + n] = d + b_cls[n]; });
}

// pooled[b] = tanh(W_p h[b, 0] + b_p), V sequences and POOL_WAVES 2 PAIRS rows per block (a block's rows of W_p are read once for all of
// its sequences).  What is left of the step is the latency of one row's loads and the launch.
constexpr int POOL_WAVES = 4;
template <int V, int PAIRS>
__global__ __launch_bounds__(64 * POOL_WAVES) void pool_kernel(const __half *__restrict__ hidden, size_t seq_stride, int B,
                                                               const __half *__restrict__ w_pool, const float *__restrict__ b_pool, int H,
                                                               float *__restrict__ pooled)
{
    const int b0 = blockIdx.x * V, n0 = blockIdx.y * (POOL_WAVES * 2 * PAIRS);
    const _Float16 *src[V];
#pragma unroll
    for (int v = 0; v < V; v++) src[v] = reinterpret_cast<const _Float16 *>(hidden) + (size_t)min(b0 + v, B - 1) * seq_stride;
    matrix_times_vectors<V, PAIRS>(w_pool, [&](int v, int k, float (&xv)[8]) { read8(src[v] + k, xv); }, H, H, n0, POOL_WAVES * gridDim.y,
                                   [&](int v, int n, float d) { if (b0 + v < B) pooled[(size_t)(b0 + v) * H + n] = tanhf(d + b_pool[n]); });
}

__global__ __launch_bounds__(64 * POOL_WAVES) void logits_kernel(const float *__restrict__ pooled, const __half *__restrict__ w_cls,
                                                                 const float *__restrict__ b_cls, int H, int C, float *__restrict__ logits)
{
    const size_t b = blockIdx.x;
    matrix_times_vectors<1, 1>(w_cls, [&](int, int k, float (&xv)[8]) { read8(pooled + b * H + k, xv); }, C, H, (int)blockIdx.y * (POOL_WAVES * 2),
                               POOL_WAVES * gridDim.y,
                               [&](int, int n, float d) { logits[b * C + n] = d + b_cls[n]; });
}

}  // namespace

hipError_t launch_classify(const __half *hidden, int B, int S, int H, const __half *w_pool, const float *b_pool,
                           const __half *w_cls, const float *b_cls, int C, float *pooled, float *logits, hipStream_t st)
{
    if (!pooled) {
        hipLaunchKernelGGL(classify_kernel, dim3(B), dim3(64 * CLASSIFY_WAVES), (size_t)H * 6, st, hidden, (size_t)S * H, w_pool,
                           b_pool, w_cls, b_cls, H, C, logits);
        return hipGetLastError();
    }
    // few sequences: eight rows per block, to have more of them; else sixteen rows for four sequences
    auto pool = [&](auto kernel, int vectors, int rows) {
        hipLaunchKernelGGL(kernel, dim3((B + vectors - 1) / vectors, (H + rows - 1) / rows), dim3(64 * POOL_WAVES), 0, st, hidden, (size_t)S * H, B,
                           w_pool, b_pool, H, pooled);
    };
    if (B < 4) pool(pool_kernel<1, 1>, 1, POOL_WAVES * 2);
    else pool(pool_kernel<4, 2>, 4, POOL_WAVES * 4);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(logits_kernel, dim3(B, std::min((C + POOL_WAVES * 2 - 1) / (POOL_WAVES * 2), 65535)), dim3(64 * POOL_WAVES), 0, st, pooled, w_cls, b_cls, H,
                       C, logits);
    return hipGetLastError();
}

}  // namespace samp
