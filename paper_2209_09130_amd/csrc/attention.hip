// Softmax attention over packed (padding-free) rows on gfx950 matrix cores.
//
// INT8 flavour (Section 4.2 / Appendix B: the softmax output is quantised with a step fixed at
// calibration, so both batched products are int8 x int8 -> int32):
//     score = float(q.k) * m_sc;  P = softmax(score);  Pq = rne(P / s_p);  ctx = rne(float(Pq.V) * m_ctx)
// Because the step of P is static, P must be fully normalised before it is rounded: a block keeps
// a whole strip of scores on chip (32 queries x all keys of the sequence, <= 2048), so the scores
// never touch memory and no running rescale is needed.  Longer sequences take the three-sweep
// kernels further down, which recompute the scores instead of keeping them.
//
// One block = (sequence, head, 32 queries), 4 waves (8 for INT8 beyond 512 keys); wave w owns key
// tiles w, w+4, ... (32 keys each).  S^T = K.Q^T is computed so that in the 32x32 MFMA result a lane holds ONE query and 16
// keys: after the softmax those 16 values are, as they stand, the lane's operand of the P.V MFMA.
// Its other operand is V^T: V rows lie in the wave's LDS as they come and are transposed by the read.  Row maxima, row sums and the partial
// P.V products are combined across the waves through LDS (integer partial sums: exact).
// Every floating-point value that decides an int8 code follows one fixed sequence of binary32
// operations; exp and the row sum are evaluated in binary64 and rounded once.
#include "samp_common.h"
#include "mfma_tile.h"
#include "exp2_table.h"
#include "divisor.h"
#include "gemm_rules.h"

#include <algorithm>
#include <atomic>
#include <hip/hip_ext.h>

namespace samp {
namespace {

constexpr int QB = 32;                 // queries per block
constexpr int ONE_PASS_MAX_LEN = 512;  // longest sequence that four waves take in the INT8 flavour
constexpr int VT_STRIDE_I8 = 36;       // bytes per V^T row (32 keys + pad), int8

// exp(x) for x <= 0 in binary64: x = k ln2 + r with |r| <= ln2 / 2 (two-part ln2), then
//     exp(r) = 1 + r (1 + r q(r)),
// q a polynomial of degree 8 that interpolates (exp(r) - 1 - r) / r^2 at the nine Chebyshev nodes of
// [-0.34665, 0.34665] (coefficients solved in rational arithmetic and rounded to binary64), scaled by 2^k.
// Checked against a 60-digit exponential with every fused multiply-add emulated exactly: relative error
// below 2^-49 over the whole argument range, far below a binary32 ulp, so rounding the result to binary32
// gives the correctly rounded exponential (up to ties narrower than 2^-49), which is what the quantiser's
// decision is defined on.  One operation shorter than the Taylor polynomial of the same accuracy.
// x must be finite and above -2^30 (the host bounds the score multiplier accordingly): far below -746 the
// scaling by 2^k underflows to 0 like the exponential itself.  The -inf of a masked key is clamped to
// -746 by the caller.  k = rint(x / ln2) comes out of one fma with 1.5 * 2^52: the sum's low dword is k
// as an integer, the sum minus the constant is k as a double.
__device__ __forceinline__ double exp_nonpos(double x)
{
    const double shifted = __builtin_fma(x, 1.44269504088896338700e+00, 6755399441055744.0);
    const int ki = (int)(unsigned)__double_as_longlong(shifted);
    const double k = shifted - 6755399441055744.0;
    double r = __builtin_fma(k, -6.93147180369123816490e-01, x);
    r = __builtin_fma(k, -1.90821492927058770002e-10, r);
    double p = 0x1.28804ab1d4135p-22;
    p = __builtin_fma(p, r, 0x1.72c73b05aa600p-19);
    p = __builtin_fma(p, r, 0x1.a019c99e7c005p-16);
    p = __builtin_fma(p, r, 0x1.a019ad9901febp-13);
    p = __builtin_fma(p, r, 0x1.6c16c17391579p-10);
    p = __builtin_fma(p, r, 0x1.1111111c49a25p-7);
    p = __builtin_fma(p, r, 0x1.5555555554cb5p-5);
    p = __builtin_fma(p, r, 0x1.5555555553b71p-3);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return __builtin_ldexp(p, ki);
}

// The same function, for the kernels that hold EXP2_TABLE in LDS: x = (k + f) ln2 / 256 with |f| <= 1/2,
//     exp(x) = 2^(k/256) + 2^(k/256) f q(f),
// q a polynomial of degree 3 that interpolates (2^(f/256) - 1) / f at the four Chebyshev nodes of [-0.5001, 0.5001]
// (solved and rounded as above).  f is formed with 256 / ln2 in two parts: the rounding of a single constant is multiplied by x and
// alone costs 2^-49.1 at -104.  Relative error below 2^-51.9 over the whole range (the roundings of the table entry and of the last
// operation), checked the same way; the polynomial above reaches 2^-49.6.  The vector arithmetic
// is what bounds the softmax: this takes 13 operations (a clamp among them) for the polynomial's 16, and its table read runs
// beside them (2.4 clocks of LDS time per wave and read where many entries are equal; those are broadcast).  Forward with the
// polynomial and with this: BERT-base 128 x 512 Fully-Quant 12104 / 11603 us, 6 x 500..1100 1933 / 1860, 33 x 40..301 binary16
// softmax 1709 / 1685 (the second part of the constant is 1.1, 1.5 and 0.7 % of that).
// The result underflows to a binary32 zero below -103.98, so the argument may be clamped at -104 or below, also that of a masked key.
// UNIT: the argument is given as its UNIT-th part, a power of two that goes into the constants: with -128 the subtraction of a score from the row's
// maximum (both divided by 128, which is exact) clamps its own result to [0, 1] and no operation is spent on the bound.  Below -128 is 0 like below -104.
typedef uint64_t ExpTable[256];
template <int UNIT> __device__ __forceinline__ float exp_units(double xd, const ExpTable &table);
__device__ __forceinline__ float exp_nonpos(float x, const ExpTable &table)
{ return exp_units<1>((double)__builtin_fmaxf(x, -104.0f), table); }
template <int UNIT> __device__ __forceinline__ float exp_units(double xd, const ExpTable &table)
{
    const double shifted = __builtin_fma(xd, UNIT * 0x1.71547652b82fep+8, 6755399441055744.0);
    const unsigned k = (unsigned)__double_as_longlong(shifted);
    const uint64_t entry = table[k & 255];
    double f = __builtin_fma(xd, UNIT * 0x1.71547652b82fep+8, -(shifted - 6755399441055744.0));
    f = __builtin_fma(xd, UNIT * 0x1.777d0ffda0d24p-48, f);
    double q = 0x1.3b2ab83ecf101p-39;
    q = __builtin_fma(q, f, 0x1.c6b0902ba1a20p-29);
    q = __builtin_fma(q, f, 0x1.ebfbdff82c585p-19);
    q = __builtin_fma(q, f, 0x1.62e42fefa39d9p-9);
    const double scale = __hiloint2double((int)((unsigned)(entry >> 32) + (k << 12)), (int)(unsigned)entry);
    return (float)__builtin_fma(scale, f * q, scale);
}
constexpr float SCORE_UNIT = 0x1p-7f;
// exp(128 (score - max)), score <= max
__device__ __forceinline__ float exp_below(float score, float max, const ExpTable &table)
{ return exp_units<-128>((double)__builtin_amdgcn_fmed3f(max - score, 0.0f, 1.0f), table); }

// The wave's number inside its block, as a scalar: every test on it (does this wave own key tile j?) then is a
// scalar branch instead of a lane mask with copies of the live registers where the paths join.
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// The lane's number, counted anew where it is needed late: what is derived from it then need not stay in registers from the
// kernel's first lines on.
__device__ __forceinline__ int lane_again() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

__device__ __forceinline__ int opaque_zero()
{
    int z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}

// Sum of the V codes a lane holds of one key tile (its channel, the keys of its half), added to `sum`.  The unsigned operand
// forms are fed to the matrix core as code - 128; 128 times the sum over all keys is what they miss.
__device__ __forceinline__ int add_codes(const v4i &vf, int sum)
{
#pragma unroll
    for (int q = 0; q < 4; q++) sum = __builtin_amdgcn_sdot4(vf[q], 0x01010101, sum, false);
    return sum;
}

// The V rows of key tile j0 as a lane transposes them: d[u][t] holds four channels (4 (lane & 15) ..) of key
// j0 + 4 ((lane >> 4) + 4 u) + t; rows past the end repeat the last one.
__device__ __forceinline__ void load_v_tile(const int8_t *vp, unsigned ld, int j0, int n, int lane, unsigned (&d)[2][4])
{
    const int cq = lane & 15;
    if (j0 + 32 <= n) {                                  // wave-uniform; four consecutive key rows: one address, three strides
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int8_t *p0 = vp + (unsigned)(j0 + 4 * ((lane >> 4) + 4 * u)) * ld + 4 * cq;
#pragma unroll
            for (int t = 0; t < 4; t++) d[u][t] = *reinterpret_cast<const unsigned *>(p0 + t * ld);
        }
    } else {
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int t = 0; t < 4; t++)
                d[u][t] = *reinterpret_cast<const unsigned *>(vp + (unsigned)min(j0 + 4 * ((lane >> 4) + 4 * u) + t, n - 1) * ld + 4 * cq);
    }
}

// V^T of that tile into LDS: 4 keys x 4 channels byte blocks transposed in registers (v_perm_b32) and stored as dwords of four
// consecutive keys per channel
__device__ __forceinline__ void store_vt_tile(const unsigned (&d)[2][4], int lane, int8_t *slab)
{
    const int cq = lane & 15;
#pragma unroll
    for (int u = 0; u < 2; u++) {
        const int kq = (lane >> 4) + 4 * u;
        const unsigned t01l = __builtin_amdgcn_perm(d[u][1], d[u][0], 0x05010400u), t23l = __builtin_amdgcn_perm(d[u][3], d[u][2], 0x05010400u);
        const unsigned t01h = __builtin_amdgcn_perm(d[u][1], d[u][0], 0x07030602u), t23h = __builtin_amdgcn_perm(d[u][3], d[u][2], 0x07030602u);
        unsigned *dst = reinterpret_cast<unsigned *>(&slab[(4 * cq) * VT_STRIDE_I8 + 4 * kq]);
        dst[0 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23l, t01l, 0x05040100u);
        dst[1 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23l, t01l, 0x07060302u);
        dst[2 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23h, t01h, 0x05040100u);
        dst[3 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23h, t01h, 0x07060302u);
    }
}

// V rows of a key tile as they lie (32 keys x 64 codes) in LDS, and V^T operands out of it: ds_read_b64_tr_b8 hands lane i of sixteen the byte
// i & 7 of the eight bytes that each lane of parity i >> 3 points at, so that with lanes 2 j and 2 j + 1 at 16 channels of key j a lane gets one
// channel of eight keys.  No transposition in registers (16 byte permutes and eight dword loads per tile), and the rows can come as direct loads.
// 16-byte chunk c of key k lies at position c ^ 2 ((k >> 3) & 1): the 32 lanes of a read's phase hit 64 different banks.
constexpr int V_TILE = 32 * 64;
struct VLane {                                            // what a lane loads and reads of every tile
    unsigned from, at;                                    // offset of its 16 bytes in the first 16 rows; of its first read in a tile
    __device__ __forceinline__ VLane(unsigned ld, int lane)
    {
        from = (unsigned)(lane >> 2) * ld + (((lane & 3) ^ ((lane >> 5) << 1)) << 4);
        const int pair = (lane >> 1) & 7;                 // keys 4 g + (0..3, 8..11) of the half, channels 16 ((lane >> 4) & 1) + 8 (lane & 1) ..
        at = (4 * (lane >> 5) + (pair & 3) + 8 * (pair >> 2)) * 64 + ((((lane >> 4) & 1) ^ (pair >> 2 << 1)) << 4) + 8 * (lane & 1);
    }
};
// channels 32 cb + (lane & 31), keys 4 (lane >> 5) + (0..3, 8..11, 16..19, 24..27)
__device__ __forceinline__ v4i read_vt(const int8_t *tile, unsigned at, int cb)
{
    typedef __attribute__((address_space(3))) v2i *Lds;
    const int8_t *p = tile + (at ^ (cb << 5));
    const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((Lds)p), hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((Lds)(p + 1024));
    return v4i{lo.x, lo.y, hi.x, hi.y};
}
__device__ __forceinline__ void request_v_tile(__amdgpu_buffer_rsrc_t rows, unsigned from, unsigned ld, int8_t *tile)
{
    buffer_to_lds128(rows, from, 0, tile);
    buffer_to_lds128(rows, from + 16 * ld, 0, tile + 1024);
}

// Four softmax codes, rne((e rS) inv_sp): the conversion rounds to the nearest integer, ties to even, saturates to [0, 255] (probabilities are not
// negative) and puts the byte into its place, one operation where clamp, rounding add and byte permutes were 2.75.
__device__ __forceinline__ int softmax_codes(const float (&e)[16], int first, float rS, float inv_sp)
{
    unsigned pk = 0;
#pragma unroll
    for (int t = 0; t < 4; t++) pk = __builtin_amdgcn_cvt_pk_u8_f32((e[first + t] * rS) * inv_sp, t, pk);
    return (int)pk;
}
// Signed codes end at 127.  A row's largest code is that of exp(0) = 1, so as long as no row of the wave (or of the lanes that share its scores) has a
// probability beyond the calibrated range nothing is to be done; otherwise the products are formed and bounded here, and the factors become 1.
template <int NT, class Live>
__device__ __forceinline__ void bound_codes(float (&e)[NT][16], float &rS, float &inv_sp, Live live)
{
    if (__builtin_amdgcn_ballot_w64(rS * inv_sp > 127.0f) == 0) return;
#pragma unroll
    for (int i = 0; i < NT; i++)
        if (live(i)) {
#pragma unroll
            for (int k = 0; k < 16; k++) e[i][k] = __builtin_fminf((e[i][k] * rS) * inv_sp, 127.0f);
        }
    rS = inv_sp = 1.0f;
}

// FETCH: the grid's last blocks ask for the weights of the kernels that follow.
struct NoFetch {};
template <bool FETCH> struct FetchArg { typedef NoFetch type; };
template <> struct FetchArg<true> { typedef FetchAhead type; };
__device__ __forceinline__ bool fetch_instead(const NoFetch &, int) { return false; }
__device__ __forceinline__ bool fetch_instead(const FetchAhead &f, int items)
{
    const int index = (int)blockIdx.x - items;
    if (index < 0) return false;
    fetch_block(f.part, (int)blockIdx.x & 7, (unsigned)index >> 3, (unsigned)f.blocks >> 3);
    return true;
}

// 4 N consecutive codes
template <int N> __device__ __forceinline__ void store_codes(int8_t *dst, const int (&pk)[N])
{
    if constexpr (N >= 4) {
#pragma unroll
        for (int d = 0; d < N / 4; d++) *reinterpret_cast<v4i *>(dst + 16 * d) = v4i{pk[4 * d], pk[4 * d + 1], pk[4 * d + 2], pk[4 * d + 3]};
    } else if constexpr (N == 2) *reinterpret_cast<v2i *>(dst) = v2i{pk[0], pk[1]};
    else *reinterpret_cast<int *>(dst) = pk[0];
}

// Which (sequence, head) pair and which strip of 32 queries a block works on.  Sequences of one length: XCD x takes the x-th eighth of the sequences, whose
// tokens it also owns in the kernels before and after this one.  Ragged: a strip's work grows with the length of its sequence, and an XCD that owns
// long sequences would still be at work when the others are done, so the pairs are dealt out, all strips of a pair to one XCD.  Forward, three encoders in
// turn, us, eighths / dealt out: BERT-base Fully-Quant 6 x 500..1100 1432 / 1318, 33 x 40..301 1117 / 1064, 30 x 20..200 772 / 757, 3 x 300..2000 1927 / 1753,
// binary16 softmax 33 x 40..301 1168 / 1103, Quant-FFN-Only 6 x 500..1100 1716 / 1577, FP16 20 x 30..400 1660 / 1570; of two strips 7 x 5..61 344 / 346.
constexpr int DEALT_MIN_STRIPS = 4;
struct Strip { int pair, strip; };
__device__ __forceinline__ Strip strip_of(int block, int items, int nqb, unsigned by_nqb, bool ragged)
{
    int first = 0, index = block, scale = 1;
    if (ragged) {
        const int dealt = (int)over(items, by_nqb, nqb) & ~7;     // pairs; the last items / nqb % 8 keep their own index
        if (block < dealt * nqb) first = block & 7, index = block >> 3, scale = 8;
        else first = dealt, index = block - dealt * nqb;
    } else {
        index = xcd_contiguous(block, items);
    }
    const int pair = (int)over(index, by_nqb, nqb);
    return {first + scale * pair, index - pair * nqb};
}

struct SeqInfo { int t0, n; };
__device__ __forceinline__ SeqInfo seq_info(const int *cu, int b, int max_len)
{
    if (cu) { const int t0 = cu[b]; return {t0, cu[b + 1] - t0}; }
    return {b * max_len, max_len};
}
// The 32 rows from j0 on of a sequence of n, base: its first row at the head's Q columns.  A row past the end reads as zeros, so no load needs a test or an
// address of its own.  (No more than 32 rows, so that their bytes fit 31 bits at any width.)
template <class T> __device__ __forceinline__ __amdgpu_buffer_rsrc_t strip_rows(const T *base, unsigned ld, int head, int j0, int n)
{ return buffer_of(base + (size_t)j0 * ld, (int)sizeof(T) * max(min(n - j0, 32) * (int)ld - head * 64, 0)); }

// PU: the softmax codes are unsigned, rne(P / s_p) in [0, 255] (the variant that spends all 256 codes
//     on [0, 1]).  The matrix core multiplies signed bytes, so it is fed code - 128 (a flip of the top
//     bit) and the missing 128 * sum_k V[k] of the same V tiles is added back; both are exact in int32.
// HIST: also counts every softmax code of a valid (query, key) pair into p_hist[256] (a diagnostic:
//     which of the 256 integers the softmax output uses, as Appendix B tabulates).
// What bounds it beyond a few hundred keys is vector arithmetic, all of it at four clocks per operation and wave: 20.5 operations per score, and
// per tile of 16 scores some 25 for addresses, loads and V (it was 24 and 65 with V transposed by byte permutes on the way to LDS, row numbers
// clamped per load, an exponential that clamps its argument and codes packed from rounding adds).  All loads of up to four tiles are requested at
// once.  Forward, us, before / now: BERT-base 128 x 512 10850 / 10370, 6 x 500..1100 1690 / 1590, BERT-large 32 x 256 3780 / 3728, 7 x 61 397 / 393.
// At least two waves per SIMD are asked for so that the register budget is one the matrix-core results fit
// without the accumulation registers: the products then land where the vector ALU reads them.
// NW: waves of the block.  Four up to 512 keys; eight up to 2048 (NT = 3 to 8 key tiles per wave), so that the strip of scores of a
// long sequence stays in registers too.  A sequence of 1100 tokens then evaluates each exponential once and forms each
// score once, where three sweeps over recomputed scores (the kernels further down) evaluate it twice and form it three
// times: three sequences of 1100 tokens (twelve heads) 94 -> 52 us, two of 2048 190 -> 118 us.
template <int NT, bool PU, bool HIST, int NW = 4, bool FETCH = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NT <= 5 ? 4 : 2))) void attention_i8_kernel(const int8_t *__restrict__ qkv, const int *__restrict__ cu,
                                                           int max_len, int H, int items, unsigned by_nqb, unsigned by_heads, float m_sc,
                                                           float inv_sp, float m_ctx, int8_t *__restrict__ ctx, unsigned long long *__restrict__ p_hist, typename FetchArg<FETCH>::type fetch)
{
    if (fetch_instead(fetch, items)) return;
    __shared__ unsigned hist[HIST ? 256 : 1];
    // One slab per wave: first its V tiles (written and read by that wave alone), then, once its last P.V
    // product has read them, its partial context for the other waves; sharing the bytes lets a fourth block fit a CU.
    // It holds at most four tiles, requested at the start: a fifth one (and so on) takes the place of a tile that has been multiplied, through
    // registers and two steps before it is used itself.
    constexpr int SO_BYTES = QB * 64 * 4, V_TILES = NT < 4 ? NT : 4;
    constexpr int SLAB = V_TILES * V_TILE > SO_BYTES ? V_TILES * V_TILE : SO_BYTES;
    constexpr int K_AHEAD = NT <= 4 ? NT : NT == 5 && PU ? 1 : 2;   // key tiles whose rows are requested before the first product (as many as registers hold)
    __shared__ __attribute__((aligned(1024))) int8_t slab[NW][SLAB];
    auto so = [&](int wave) { return reinterpret_cast<int(*)[64]>(slab[wave]); };
    __shared__ float smax[NW][QB];
    __shared__ double ssum[NW][QB];
    __shared__ ExpTable exp_table;

    const int nqb = (max_len + QB - 1) / QB, heads = H >> 6;
    const Strip at = strip_of(blockIdx.x, items, nqb, by_nqb, cu && nqb >= DEALT_MIN_STRIPS);
    const int seq = (int)over(at.pair, by_heads, heads), head = at.pair - seq * heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int q0 = at.strip * QB;
    if (q0 >= sq.n) return;
    const int n = sq.n;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), r = lane & 31, g = lane >> 5;
    const unsigned ld = 3u * (unsigned)H;                          // row offsets inside a sequence fit 32 bits
    const int8_t *base = qkv + (size_t)sq.t0 * ld + head * 64;
    auto rows_from = [&](int j0) { return strip_rows(base, ld, head, j0, n); };
    auto first_key = [&](int i) { return (w + NW * i) * 32; };
    constexpr int ENTRIES = NW < 4 ? 4 / NW : 1;                  // of the exponential's table, per thread
    uint64_t table_entry[ENTRIES];
#pragma unroll
    for (int i = 0; i < ENTRIES; i++) table_entry[i] = EXP2_TABLE[(tid + 64 * NW * i) & 255];
    if (HIST && tid < 256) hist[tid] = 0;                                      // ordered before its use by the barriers below

    // lane (row r, half g) holds 16 consecutive bytes of the head dim of a query row (second MFMA operand) or a key row (first)
    const unsigned row_at = (unsigned)r * ld + g * 16, key_at = row_at + H;
    const VLane vl(ld, lane);
    v4i qf[2], kf[K_AHEAD][2];
    auto request_keys = [&](int i) {
        const auto rows = rows_from(first_key(i));
#pragma unroll
        for (int ks = 0; ks < 2; ks++) kf[i % K_AHEAD][ks] = __builtin_amdgcn_raw_buffer_load_b128(rows, key_at + ks * 32, 0, 0);
    };
    {
        const auto rows = rows_from(q0);
#pragma unroll
        for (int ks = 0; ks < 2; ks++) qf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rows, row_at + ks * 32, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < K_AHEAD; i++) request_keys(i);
#pragma unroll
    for (int i = 0; i < V_TILES; i++) request_v_tile(rows_from(first_key(i)), vl.from + 2 * H, ld, &slab[w][i * V_TILE]);

    float sc[NT][16];                                             // scores / 128, then exponentials
    const float m_unit = m_sc * SCORE_UNIT;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NT; i++) {
        const int j0 = first_key(i);
        if (j0 < n) {                                           // wave-uniform
            v16i acc;
#pragma unroll
            for (int e = 0; e < 16; e++) acc[e] = 0;
#pragma unroll
            for (int ks = 0; ks < 2; ks++) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[i % K_AHEAD][ks], qf[ks], acc, 0, 0, 0);
            if (j0 + 32 <= n) {                                  // a full tile needs no masking
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    sc[i][e] = (float)acc[e] * m_unit;
                    mx = __builtin_fmaxf(mx, sc[i][e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int key = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
                    sc[i][e] = key < n ? (float)acc[e] * m_unit : -INFINITY;
                    mx = __builtin_fmaxf(mx, sc[i][e]);
                }
            }
        }                                                        // the scores of a tile past the end are never read
        if (i + K_AHEAD < NT) request_keys(i + K_AHEAD);
    }
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) smax[w][r] = mx;
#pragma unroll
    for (int i = 0; i < ENTRIES; i++)
        if (NW <= 4 || tid < 256) exp_table[tid + 64 * NW * i] = table_entry[i];
    wait_vm<0>();                                                 // the wave's V tiles are in its slab
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NW; u++) mx = __builtin_fmaxf(mx, smax[u][r]);

    // tiles past the end are skipped here and below
    double part = 0.0;
#pragma unroll
    for (int i = 0; i < NT; i++) {
        if (first_key(i) < n) {
#pragma unroll
            for (int e = 0; e < 16; e++) {
                sc[i][e] = exp_below(sc[i][e], mx, exp_table);
                part += (double)sc[i][e];
            }
        }
    }
    part += __shfl_xor(part, 32, 64);
    if (g == 0) ssum[w][r] = part;
    __syncthreads();
    double total = ssum[0][r];
#pragma unroll
    for (int u = 1; u < NW; u++) total += ssum[u][r];
    const float S = (float)total;
    float rS = __fdiv_rn(1.0f, S);
    if (!PU) bound_codes(sc, rS, inv_sp, [&](int i) { return first_key(i) < n; });

    // Every accumulator register starts from a zero of its own that the compiler cannot see through: with literal
    // zeros it gives the first product of each path registers of its own and copies all 32 accumulators where the
    // paths join.
    v16i o[2];
    int vsum[2] = {0, 0};
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) o[cb][e] = opaque_zero();
#pragma unroll
    for (int i = 0; i < NT; i++) {
        const int j0 = first_key(i);
        v4i late[2];                                          // tile i + 2 takes the place of tile i - 2
        const bool refill = i > 1 && i + 2 < NT && first_key(i + 2) < n;
        if (refill) {
            const auto rows = rows_from(first_key(i + 2));
#pragma unroll
            for (int u = 0; u < 2; u++) late[u] = __builtin_amdgcn_raw_buffer_load_b128(rows, vl.from + 2 * H + u * 16 * ld, 0, 0);
        }
        if (j0 < n) {
            v4i pf;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                pf[q] = softmax_codes(sc[i], 4 * q, rS, inv_sp);
                if (HIST) {
#pragma unroll
                    for (int t = 0; t < 4; t++)
                        if (q0 + r < n && j0 + 8 * q + 4 * g + t < n) atomicAdd(&hist[((unsigned)pf[q] >> (8 * t)) & 0xffu], 1u);
                }
                if (PU) pf[q] ^= (int)0x80808080u;             // code - 128 as a signed byte
            }
#pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                const v4i vf = read_vt(&slab[w][(i & 3) * V_TILE], vl.at, cb);
                o[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(pf, vf, o[cb], 0, 0, 0);
                if (PU) vsum[cb] = add_codes(vf, vsum[cb]);
            }
        }
        if (refill) {
#pragma unroll
            for (int u = 0; u < 2; u++) *reinterpret_cast<v4i *>(&slab[w][((i + 2) & 3) * V_TILE + u * 1024 + lane_again() * 16]) = late[u];
        }
    }
    if (PU) {
#pragma unroll
        for (int cb = 0; cb < 2; cb++) {
            vsum[cb] = 128 * (vsum[cb] + __shfl_xor(vsum[cb], 32, 64));          // the other half's keys
#pragma unroll
            for (int e = 0; e < 16; e++) o[cb][e] += vsum[cb];
        }
    }
    // partial context of this wave: lane holds channel cb*32 + r and queries 8q + 4g + t
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) so(w)[8 * (e >> 2) + 4 * g + (e & 3)][cb * 32 + r] = o[cb][e];
    __syncthreads();

    constexpr int CPT = 32 / NW;                                  // channels per thread: 4 to 32
    const int query = tid / (64 / CPT), c0 = tid % (64 / CPT) * CPT;
    if (q0 + query < n) {
        int pk[CPT / 4];
#pragma unroll
        for (int d = 0; d < CPT / 4; d++) {
            float codes[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                int O = 0;
#pragma unroll
                for (int u = 0; u < NW; u++) O += so(u)[query][c0 + 4 * d + e];
                codes[e] = code_bits((float)O * m_ctx);
            }
            pk[d] = pack_codes(codes[0], codes[1], codes[2], codes[3]);
        }
        int8_t *dst = ctx + (size_t)(sq.t0 + q0 + query) * H + head * 64 + c0;
        store_codes(dst, pk);
    }
    if (HIST && tid < 256 && hist[tid]) atomicAdd(&p_hist[tid], (unsigned long long)hist[tid]);   // after the barrier above
}

// ---- QKV GEMM and attention of one (sequence, head) in one kernel ------------------------------------------
// For sequences of at most 128 tokens the QKV tile of one (sequence, head) -- the sequence's token rows times the
// head's 64 query, 64 key and 64 value channels -- is exactly one 128 x 192 block tile of the large-tile GEMM, and it
// is all that head's attention needs (Section 3.2: the QKV GEMM's requantised int8 output is the attention's only
// input).  The block therefore runs that GEMM's main loop (three-deep ring of 64-byte stages, direct global->LDS
// loads, wave tiles of 64 x 96), requantises q, k, v into LDS where the ring was, and goes on as the attention
// kernels above do, one wave per 32 queries over all keys: q, k, v never reach memory and one launch per layer is
// gone.  Every value is produced by the same operations in the same order as in the two separate kernels (row sums
// and, for FP16, partial contexts are accumulated per key tile modulo 4 in ascending order, which is how the four
// waves of those kernels form them), so the context is the same bytes.  QT = 2 is the same for up to 256 tokens: a
// 256 x 192 block tile, wave tiles of 128 x 96, a wave's 64 queries 32 at a time.
//
// The ring holds two 128-byte stages: whole cache lines per operand row (a line that is asked for in two halves, some stages
// apart, is fetched twice).  For QT = 1 two blocks' rings fill a CU's 160 KB of LDS exactly, so the tables of the epilogue
// come last, into the stage that the last one but one leaves free (LATE).  A stand-in that only loads the stages pulls 35 to 41
// bytes per clock and CU like this, 24 with 64-byte stages; forward, three 64-byte stages against two of 128: BERT-base 256 x 128
// Fully-Quant 4.43 / 4.21 ms, 32 x 128 FP16 1.380 / 1.324, BERT-large 64 x 128 Fully-Quant 3.94 / 3.78, Quant-FFN-Only 4.73 / 4.48.  Three 64-byte stages are kept for rows that are no
// multiple of 128 bytes (an odd number of heads in INT8) and for QT = 2, whose registers do not hold 128-byte stages' offsets.
template <int QT, int STAGE>                               // QT 32-query tiles per wave: sequences of at most 128 QT tokens
struct QkvTile {                                           // the block tile both flavours of the kernel share
    static constexpr int TM = 2 * QT, TN = 3, BKB = STAGE, NSTAGE = STAGE == 128 ? 2 : 3, NWAVES = 4, CH = BKB / 16, RPI = 64 / CH, KS = BKB / 32;
    static constexpr bool LATE = QT == 1 && STAGE == 128;
    static constexpr int BM = 128 * QT, BN = 192;
    static constexpr int A_BYTES = BM * BKB, STAGE_BYTES = (BM + BN) * BKB, RING_BYTES = NSTAGE * STAGE_BYTES;
    static constexpr int NLD = (BM + BN) / RPI / NWAVES;          // 1 KiB pieces per wave and stage
};

// The GEMM part: the wave's (64 QT) x 96 accumulators of X[t0 .. t0+n) . W_head^T, rows of Kbytes bytes; HALF: fp16 operands.
// The main loop of the large-tile GEMM kernel (same ring, same waits); load_tables() runs once the first stages are
// requested.  On return the ring is idle.
// VWAVE: the wave's last two channel tiles are value channels.  Their products are formed with the operands the other
// way round (token rows first), so that a lane of the result holds ONE channel and four consecutive tokens per
// register group: exactly a dword (fp16: 8 bytes) of V^T, which the P.V product wants key-contiguous.  The sums are
// the same (the same products over the same k).  ALL_LIVE: every 32-token tile of the block holds tokens (no tests in
// the loop).
template <int QT, int STAGE, bool HALF, bool VWAVE, bool ALL_LIVE, class Acc, class LoadTables>
__device__ __forceinline__ void qkv_tile_gemm(const char *__restrict__ X, const char *__restrict__ W, int t0, int n, int head, int H,
                                              int Kbytes, char *lds, int wave, int lane, Acc (&acc)[3][2 * QT], LoadTables load_tables)
{
    typedef QkvTile<QT, STAGE> Tile;
    constexpr int TM = Tile::TM, TN = Tile::TN, BKB = Tile::BKB, NSTAGE = Tile::NSTAGE, NWAVES = Tile::NWAVES;
    constexpr int CH = Tile::CH, RPI = Tile::RPI, KS = Tile::KS, BM = Tile::BM;
    constexpr int A_BYTES = Tile::A_BYTES, STAGE_BYTES = Tile::STAGE_BYTES, RING_BYTES = Tile::RING_BYTES, NLD = Tile::NLD;
    static_assert((Tile::BM + Tile::BN) % (RPI * NWAVES) == 0, "a stage must split into whole pieces per wave");
    const int wm = (wave >> 1) * 32 * TM, wn = (wave & 1) * 32 * TN;
    const int r = lane & 31, g = lane >> 5;
    // operand rows: the sequence's tokens (rows past its end repeat the last one), and the head's 64 rows of each of
    // the query, key and value thirds of the weight matrix
    // (32-bit offsets from a base that is the same for the whole wave: half the registers of a pointer per load)
    constexpr int NLDA = BM / RPI / NWAVES;                       // the first NLDA pieces hold token rows
    const char *bases[2] = {X + (size_t)t0 * Kbytes, W + (size_t)head * 64 * Kbytes};
    unsigned off[NLD];
#pragma unroll
    for (int j = 0; j < NLD; j++) {
        const int srow = RPI * (wave + NWAVES * j) + lane / CH, row = j < NLDA ? min(srow, n - 1) : srow - BM;
        off[j] = (unsigned)(j < NLDA ? row : (row >> 6) * H + (row & 63)) * (unsigned)Kbytes + (((lane % CH) ^ swz<BKB>(j < NLDA ? srow : row)) << 4);
    }
    const int KT = Kbytes / BKB;
    int fill_slot = 0, fill_kt = 0;
    auto issue = [&]() {
        char *st = lds + fill_slot * STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < NLD; j++) {
            unsigned o = off[j];
            asm volatile("" : "+v"(o));                            // keeps the offset a 32-bit one: scalar base + vector offset
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(bases[j >= NLDA] + (size_t)fill_kt * BKB + o),
                                             (__attribute__((address_space(3))) void *)(st + (wave + NWAVES * j) * 1024), 16, 0, 0);
        }
        fill_kt++;
        fill_slot = fill_slot + 1 == NSTAGE ? 0 : fill_slot + 1;
    };
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    unsigned offa[KS], offw[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
        offa[ks] = lds_base + (wm + r) * BKB + (((2 * ks + g) ^ swz<BKB>(wm + r)) << 4);
        offw[ks] = lds_base + A_BYTES + (wn + r) * BKB + (((2 * ks + g) ^ swz<BKB>(wn + r)) << 4);
    }
    auto fetch = [&](int slot_bytes, int ks, v4i (&fa)[TM], v4i (&fw)[TN]) {
        lds_read_frags<32 * BKB>(offa[ks] + slot_bytes, fa, std::make_integer_sequence<int, TM>());
        lds_read_frags<32 * BKB>(offw[ks] + slot_bytes, fw, std::make_integer_sequence<int, TN>());
    };
    auto ready = [&](v4i (&fa)[TM], v4i (&fw)[TN]) {
        tie(fa, std::make_integer_sequence<int, TM>());
        tie(fw, std::make_integer_sequence<int, TN>());
    };

#pragma unroll
    for (int s = 0; s < NSTAGE - 1; s++)
        if (s < KT) issue();
    if (!Tile::LATE) load_tables();

#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0;
    bool rows_live[TM];                                           // wave-uniform: token tiles past the sequence's end are not multiplied
#pragma unroll
    for (int j = 0; j < TM; j++) rows_live[j] = wm + 32 * j < n;
    auto multiply = [&](const v4i (&fa)[TM], const v4i (&fw)[TN]) {
#pragma unroll
        for (int j = 0; j < TM; j++)
            if (ALL_LIVE || rows_live[j]) {
#pragma unroll
                for (int i = 0; i < TN; i++) {
                    const bool tokens_first = VWAVE && i >= 1;
                    const v4i first = tokens_first ? fa[j] : fw[i], second = tokens_first ? fw[i] : fa[j];
                    if constexpr (HALF)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, first), __builtin_bit_cast(v8h, second), acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(first, second, acc[i][j], 0, 0, 0);
                }
            }
    };

    v4i fa[2][TM], fw[2][TN];
    if (KT > NSTAGE - 2) wait_vm_and_barrier<(NSTAGE - 2) * NLD>(); else wait_vm_and_barrier<0>();
    fetch(0, 0, fa[0], fw[0]);
    int slot_bytes = 0;
    auto next_slot = [&]() { slot_bytes = slot_bytes + STAGE_BYTES == RING_BYTES ? 0 : slot_bytes + STAGE_BYTES; };
    auto step = [&](int ks, bool refill, bool more, auto vm_tag) {
        constexpr int VM = decltype(vm_tag)::value;
        if (ks + 1 < KS) {
            fetch(slot_bytes, ks + 1, fa[(ks + 1) & 1], fw[(ks + 1) & 1]);
            wait_lds_reads<TM + TN>();
        } else if (more) {
            wait_vm_and_barrier<VM>();
            next_slot();
            fetch(slot_bytes, 0, fa[0], fw[0]);
        } else {
            wait_lds_reads<0>();
        }
        ready(fa[ks & 1], fw[ks & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (refill && ks == 0) issue();
        if (Tile::LATE && !more && ks == 0) load_tables();         // direct loads: the last wait below covers them
        multiply(fa[ks & 1], fw[ks & 1]);
        __builtin_amdgcn_sched_barrier(0);
    };
    int kt = 0;
    for (; kt + NSTAGE - 1 < KT; kt++)
#pragma unroll
        for (int ks = 0; ks < KS; ks++) step(ks, true, true, std::integral_constant<int, (NSTAGE - 2) * NLD>());
    if constexpr (NSTAGE > 2)
        for (; kt + 1 < KT; kt++)
#pragma unroll
            for (int ks = 0; ks < KS; ks++) step(ks, false, true, std::integral_constant<int, 0>());
#pragma unroll
    for (int ks = 0; ks < KS; ks++) step(ks, false, false, std::integral_constant<int, 0>());
    wait_vm_and_barrier<0>();                                     // the ring is idle from here on
}

// one of four copies of the loop: by wave column (value channels or not) and by whether all token tiles are live
template <int QT, int STAGE, bool HALF, class Acc, class LoadTables>
__device__ __forceinline__ void qkv_tile_gemm_any(const char *__restrict__ X, const char *__restrict__ W, int t0, int n, int head, int H,
                                                  int Kbytes, char *lds, int wave, int lane, Acc (&acc)[3][2 * QT], LoadTables load_tables)
{
    const bool all_live = n > QkvTile<QT, STAGE>::BM - 32;               // block-uniform; wave & 1 is wave-uniform
    if (wave & 1) {
        if (all_live) qkv_tile_gemm<QT, STAGE, HALF, true, true>(X, W, t0, n, head, H, Kbytes, lds, wave, lane, acc, load_tables);
        else qkv_tile_gemm<QT, STAGE, HALF, true, false>(X, W, t0, n, head, H, Kbytes, lds, wave, lane, acc, load_tables);
    } else {
        if (all_live) qkv_tile_gemm<QT, STAGE, HALF, false, true>(X, W, t0, n, head, H, Kbytes, lds, wave, lane, acc, load_tables);
        else qkv_tile_gemm<QT, STAGE, HALF, false, false>(X, W, t0, n, head, H, Kbytes, lds, wave, lane, acc, load_tables);
    }
}

// `words` dwords into LDS by one wave, 64 per direct load; the caller waits for them (vmcnt) before its next barrier
__device__ __forceinline__ void load_direct(float *dst, const void *src, int words, int lane)
{
    const auto from = buffer_of(src);
    for (int i = 0; i < words; i += 64)
        buffer_to_lds32(from, 4 * (i + lane), (int *)dst + i);
}

// q and k as token rows of 64 codes, v transposed (a channel's codes of all keys in a row): strides of the LDS copies
constexpr int QK_STRIDE_I8 = 80;
template <int QT> constexpr int VT_ROW_I8 = 128 * QT + 4;

// The attention of the QKV + attention kernels, from q, k and V^T in LDS: this wave's 32 QT queries against all keys.
template <int QT, bool PU>
__device__ __forceinline__ void attend_i8(char *lq, const char *lk, const char *lvt, const ExpTable &exp_table, int n, int t0, int head, int H,
                                          float m_sc, float inv_sp, float m_ctx, int8_t *__restrict__ ctx, int wave, int lane)
{
    constexpr int QK_STRIDE = QK_STRIDE_I8, VT_STRIDE = VT_ROW_I8<QT>, NKT = 4 * QT;
    const int r = lane & 31, g = lane >> 5;
    // attention: this wave's 32 QT queries against all keys, 32 queries at a time
#pragma unroll 1
    for (int qt = 0; qt < QT; qt++) {
        const int q0 = (wave * QT + qt) * QB;
        if (q0 >= n) break;                                       // no barrier below
        v4i qf[2];
#pragma unroll
        for (int ks = 0; ks < 2; ks++) qf[ks] = *reinterpret_cast<const v4i *>(lq + (q0 + r) * QK_STRIDE + ks * 32 + g * 16);
        float sc[NKT][16];                                        // scores / 128, then exponentials
        const float m_unit = m_sc * SCORE_UNIT;
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < NKT; i++) {
            const int j0 = 32 * i;
            if (j0 < n) {                                        // wave-uniform
                v4i kf[2];
#pragma unroll
                for (int ks = 0; ks < 2; ks++) kf[ks] = *reinterpret_cast<const v4i *>(lk + (j0 + r) * QK_STRIDE + ks * 32 + g * 16);
                v16i s;
#pragma unroll
                for (int e = 0; e < 16; e++) s[e] = 0;
#pragma unroll
                for (int ks = 0; ks < 2; ks++) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[ks], qf[ks], s, 0, 0, 0);
                if (j0 + 32 <= n) {
#pragma unroll
                    for (int e = 0; e < 16; e++) {
                        sc[i][e] = (float)s[e] * m_unit;
                        mx = __builtin_fmaxf(mx, sc[i][e]);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 16; e++) {
                        const int key = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
                        sc[i][e] = key < n ? (float)s[e] * m_unit : -INFINITY;
                        mx = __builtin_fmaxf(mx, sc[i][e]);
                    }
                }
            }
        }
        mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));

        // row sums: key tile i adds to partial sum i mod 4, in ascending order, as wave i mod 4 of the attention kernel does
        double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < NKT; i++) {
            if (32 * i < n) {
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    sc[i][e] = exp_below(sc[i][e], mx, exp_table);
                    part[i & 3] += (double)sc[i][e];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; u++) part[u] += __shfl_xor(part[u], 32, 64);
        const float S = (float)(((part[0] + part[1]) + part[2]) + part[3]);
        float rS = __fdiv_rn(1.0f, S), per_code = inv_sp;
        if (!PU) bound_codes(sc, rS, per_code, [&](int i) { return 32 * i < n; });

        v16i o[2], o1[PU ? 2 : 1];
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
            for (int e = 0; e < 16; e++) { o[cb][e] = opaque_zero(); if (PU) o1[cb][e] = opaque_zero(); }
        const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
#pragma unroll
        for (int i = 0; i < NKT; i++) {
            const int j0 = 32 * i;
            if (j0 < n) {
                v4i pf;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    pf[q] = softmax_codes(sc[i], 4 * q, rS, per_code);
                    if (PU) pf[q] ^= (int)0x80808080u;             // code - 128 as a signed byte
                }
#pragma unroll
                for (int cb = 0; cb < 2; cb++) {
                    v4i vf;
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        vf[q] = *reinterpret_cast<const int *>(lvt + (cb * 32 + r) * VT_STRIDE + j0 + 8 * q + 4 * g);
                    o[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, pf, o[cb], 0, 0, 0);   // channels x queries: a lane holds ONE query
                    if (PU) o1[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(vf, ones, o1[cb], 0, 0, 0);   // 128 times this is added back below
                }
            }
        }

        if (PU) {
#pragma unroll
            for (int cb = 0; cb < 2; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) o[cb][e] += o1[cb][e] * 128;
        }
        // context codes: the lane's query, channels cb*32 + 8q + 4g + t: four codes per dword into the wave's own query rows
        // in LDS (read into qf above, read by no other wave), from where they leave as 32 bytes per lane
        char *slab = lq + q0 * QK_STRIDE;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<int *>(slab + r * QK_STRIDE + cb * 32 + 8 * q + 4 * g) =
                    pack_codes(code_bits((float)o[cb][4 * q] * m_ctx), code_bits((float)o[cb][4 * q + 1] * m_ctx),
                               code_bits((float)o[cb][4 * q + 2] * m_ctx), code_bits((float)o[cb][4 * q + 3] * m_ctx));
        __builtin_amdgcn_wave_barrier();
        const int query = lane >> 1, half = lane & 1;
        if (q0 + query < n) {
            const v4i lo = *reinterpret_cast<const v4i *>(slab + query * QK_STRIDE + half * 32);
            const v4i hi = *reinterpret_cast<const v4i *>(slab + query * QK_STRIDE + half * 32 + 16);
            int8_t *dst = ctx + (size_t)(t0 + q0 + query) * H + head * 64 + half * 32;
            *reinterpret_cast<v4i *>(dst) = lo;
            *reinterpret_cast<v4i *>(dst + 16) = hi;
        }
    }
}

template <int QT, bool PU, int STAGE>                      // PU: unsigned softmax codes, as in attention_i8_kernel
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(QT == 1 ? 2 : 1, QT == 1 ? 2 : 1)))
void qkv_attention_i8_kernel(const char *__restrict__ X, const char *__restrict__ W, const float *__restrict__ m_tab,
                             const float *__restrict__ b_tab, const int *__restrict__ cu, int max_len, int H, float m_sc,
                             float inv_sp, float m_ctx, int8_t *__restrict__ ctx)
{
    typedef QkvTile<QT, STAGE> Tile;
    constexpr int TM = Tile::TM, TN = Tile::TN, BM = Tile::BM, BN = Tile::BN, RING_BYTES = Tile::RING_BYTES;
    constexpr int QK_STRIDE = QK_STRIDE_I8, VT_STRIDE = VT_ROW_I8<QT>;
    constexpr int TAB_BYTES = 4096;                               // multipliers and offsets of the 192 columns, table of the exponential
    constexpr int Q_OFF = Tile::LATE ? TAB_BYTES : 0, K_OFF = Q_OFF + BM * QK_STRIDE, VT_OFF = K_OFF + BM * QK_STRIDE;
    static_assert(VT_OFF + 64 * VT_STRIDE + Q_OFF <= RING_BYTES, "q, k and V^T take the place of the ring, clear of a table at either end");
    static_assert(2 * BN * 4 + sizeof(ExpTable) <= TAB_BYTES, "");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // LATE: at the end of the ring that the second last of the H / STAGE stages lies in
    float *tab = reinterpret_cast<float *>(lds + (!Tile::LATE ? RING_BYTES : (H / STAGE) & 1 ? RING_BYTES - TAB_BYTES : 0));
    ExpTable &exp_table = *reinterpret_cast<ExpTable *>(tab + 2 * BN);

    const int heads = H >> 6;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);       // sequences outermost, as in the attention kernel
    const int seq = item / heads, head = item % heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int n = sq.n;
    if (n <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int wm = (wave >> 1) * 32 * TM, wn = (wave & 1) * 32 * TN;
    const int r = lane & 31, g = lane >> 5;

    v16i acc[TN][TM];
    qkv_tile_gemm_any<QT, STAGE, false>(X, W, sq.t0, n, head, H, H, lds, wave, lane, acc, [&]() {
        if constexpr (Tile::LATE) {
            load_direct(tab + 2 * BN + wave * 128, (const int *)EXP2_TABLE + wave * 128, 128, lane);
            if (wave < 3) {
                const int col = wave * H + head * 64;
                load_direct(tab + wave * 64, m_tab + col, 64, lane);
                if (b_tab) load_direct(tab + BN + wave * 64, b_tab + col, 64, lane);
                else tab[BN + wave * 64 + lane] = 0.0f;
            }
            return;
        }
        exp_table[tid] = EXP2_TABLE[tid];
        for (int c = tid; c < BN; c += 256) {
            const int col = (c >> 6) * H + head * 64 + (c & 63);
            tab[c] = m_tab[col];
            tab[BN + c] = b_tab ? b_tab[col] : 0.0f;
        }
    });

    // requantise into LDS: q and k as token rows of 64 codes, v transposed (a channel's codes of all keys in a row).
    // In a query / key tile a lane holds one token and groups of four consecutive channels; in a value tile one channel
    // and groups of four consecutive tokens.
#pragma unroll
    for (int io = 0; io < TN; io++) {
        const int nl = wn + io * 32;                              // first of the tile's 32 columns among the block's 192 (scalar)
        const int part = nl >> 6, c0 = nl & 63;                   // 0 query, 1 key, 2 value
        if (part < 2) {
            v4f mm[4], bb[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                mm[q] = *reinterpret_cast<const v4f *>(tab + nl + 8 * q + 4 * g);
                bb[q] = *reinterpret_cast<const v4f *>(tab + BN + nl + 8 * q + 4 * g);
            }
#pragma unroll
            for (int j = 0; j < TM; j++) {
                const int row = wm + 32 * j + r;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const v16i &a = acc[io][j];
                    const int pk = pack_codes(code_bits(__builtin_fmaf((float)a[4 * q + 0], mm[q].x, bb[q].x)),
                                              code_bits(__builtin_fmaf((float)a[4 * q + 1], mm[q].y, bb[q].y)),
                                              code_bits(__builtin_fmaf((float)a[4 * q + 2], mm[q].z, bb[q].z)),
                                              code_bits(__builtin_fmaf((float)a[4 * q + 3], mm[q].w, bb[q].w)));
                    *reinterpret_cast<int *>(lds + (part ? K_OFF : Q_OFF) + row * QK_STRIDE + c0 + 8 * q + 4 * g) = pk;
                }
            }
        } else {
            const float mm = tab[nl + r], bb = tab[BN + nl + r];  // the lane's channel
#pragma unroll
            for (int j = 0; j < TM; j++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const v16i &a = acc[io][j];
                    const int pk = pack_codes(code_bits(__builtin_fmaf((float)a[4 * q + 0], mm, bb)), code_bits(__builtin_fmaf((float)a[4 * q + 1], mm, bb)),
                                              code_bits(__builtin_fmaf((float)a[4 * q + 2], mm, bb)), code_bits(__builtin_fmaf((float)a[4 * q + 3], mm, bb)));
                    *reinterpret_cast<int *>(lds + VT_OFF + (c0 + r) * VT_STRIDE + wm + 32 * j + 8 * q + 4 * g) = pk;
                }
        }
    }
    __syncthreads();

    attend_i8<QT, PU>(lds + Q_OFF, lds + K_OFF, lds + VT_OFF, exp_table, n, sq.t0, head, H, m_sc, inv_sp, m_ctx, ctx, wave, lane);
}

// The same for at most 128 tokens on packed weights (the tile loop that keeps weights out of LDS): wave w owns 16 of the head's 64 channels in
// each of the three parts, so a lane's query and key results are four channels of one token per 16 x 16 tile and its value results, formed
// with the operands the other way round, four tokens of one channel.  Its multipliers and offsets fit 18 registers.  50 KB of LDS for two stages
// of token rows (the row-major kernel: 80 KB).  Every value is formed by the same operations as there.
// Forwards, row-major / packed: BERT-base 32 x 128 Fully-Quant 848 / 822 us, 64 x 16..128 with six Fully-Quant layers 1404 / 1392; three stages
// in flight instead of two: the same.
template <bool PU, int D, bool FETCH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void qkv_attention_i8_packed_kernel(const char *__restrict__ X, const char *__restrict__ Wp, const float *__restrict__ m_tab,
                                    const float *__restrict__ b_tab, const int *__restrict__ cu, int max_len, int H, int items, unsigned by_heads, float m_sc,
                                    float inv_sp, float m_ctx, int8_t *__restrict__ ctx, typename FetchArg<FETCH>::type fetch)
{
    if (fetch_instead(fetch, items)) return;
    constexpr int MT = 8, BM = 16 * MT, RING = stream_ring_bytes<false, MT, D>();
    constexpr int K_OFF = BM * QK_STRIDE_I8, VT_OFF = 2 * K_OFF;
    static_assert(VT_OFF + 64 * VT_ROW_I8<1> <= RING, "q, k and V^T take the place of the ring");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    ExpTable &exp_table = *reinterpret_cast<ExpTable *>(lds + RING);

    const int heads = H >> 6;
    // sequences outermost, as in the attention kernel; ragged ones dealt out to the XCDs (64 x 16..128 Fully-Quant 900 / 886 us, half FP16 1178 / 1168)
    const int item = cu ? (int)blockIdx.x : xcd_contiguous(blockIdx.x, items);
    const int seq = (int)over(item, by_heads, heads), head = item - seq * heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int n = sq.n;
    if (n <= 0) return;
    const int lane = threadIdx.x & 63, wave = wave_index(), r = lane & 15, q = lane >> 4;

    unsigned offa[MT / 2];
#pragma unroll
    for (int j = 0; j < MT / 2; j++) {
        const int srow = 8 * (wave + 4 * j) + (lane >> 3);
        offa[j] = (unsigned)min(srow, n - 1) * (unsigned)H + (((lane & 7) ^ swz<128>(srow)) << 4);
    }
    const int c0 = head * 64 + 16 * wave;                         // the wave's channels in each part
    const char *wbase = Wp + (size_t)c0 * H;
    const unsigned woff[3] = {0, (unsigned)(H * H), (unsigned)(2 * H * H)};
    v4i acc[3][MT];
#pragma unroll
    for (int t = 0; t < 3; t++)
#pragma unroll
        for (int i = 0; i < MT; i++) acc[t][i] = v4i{0, 0, 0, 0};
    v4f mm[2], bb[2];
    float mv = 0.0f, bv = 0.0f;
    auto started = [&]() {
        load_direct(reinterpret_cast<float *>(lds + RING) + wave * 128, reinterpret_cast<const int *>(EXP2_TABLE) + wave * 128, 128, lane);
#pragma unroll
        for (int t = 0; t < 2; t++) {
            mm[t] = *reinterpret_cast<const v4f *>(m_tab + t * H + c0 + 4 * q);
            bb[t] = b_tab ? *reinterpret_cast<const v4f *>(b_tab + t * H + c0 + 4 * q) : v4f{0.f, 0.f, 0.f, 0.f};
        }
        mv = m_tab[2 * H + c0 + r];
        bv = b_tab ? b_tab[2 * H + c0 + r] : 0.0f;
    };
    auto loop = [&](auto live) {                                  // live(i): token tile i holds tokens
        stream_tile_loop<false, MT, 3, D>(X + (size_t)sq.t0 * H, offa, wbase, woff, H / 128, lds, wave, lane, started,
            [&](int t, int i, const v4i &w, const v4i &f) {
                if (live(i)) acc[t][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(t < 2 ? w : f, t < 2 ? f : w, acc[t][i], 0, 0, 0);
            });
    };
    if (n > BM - 16) loop([](int) { return true; });
    else loop([&](int i) { return 16 * i < n; });

#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
        for (int i = 0; i < MT; i++) {
            const v4i a = acc[t][i];
            *reinterpret_cast<int *>(lds + t * K_OFF + (16 * i + r) * QK_STRIDE_I8 + 16 * wave + 4 * q) =
                pack_codes(code_bits(__builtin_fmaf((float)a.x, mm[t].x, bb[t].x)), code_bits(__builtin_fmaf((float)a.y, mm[t].y, bb[t].y)),
                           code_bits(__builtin_fmaf((float)a.z, mm[t].z, bb[t].z)), code_bits(__builtin_fmaf((float)a.w, mm[t].w, bb[t].w)));
        }
#pragma unroll
    for (int i = 0; i < MT; i++) {
        const v4i a = acc[2][i];
        *reinterpret_cast<int *>(lds + VT_OFF + (16 * wave + r) * VT_ROW_I8<1> + 16 * i + 4 * q) =
            pack_codes(code_bits(__builtin_fmaf((float)a.x, mv, bv)), code_bits(__builtin_fmaf((float)a.y, mv, bv)),
                       code_bits(__builtin_fmaf((float)a.z, mv, bv)), code_bits(__builtin_fmaf((float)a.w, mv, bv)));
    }
    __syncthreads();
    attend_i8<1, PU>(lds, lds + K_OFF, lds + VT_OFF, exp_table, n, sq.t0, head, H, m_sc, inv_sp, m_ctx, ctx, wave, lane);
}

constexpr int QKV_F16_PACKED_D = 2, QKV_F16_PACKED_RING = stream_ring_bytes<true, 4, QKV_F16_PACKED_D>();

// The FP16 flavour of the kernel above: fp16 QKV GEMM with its bias, q, k, v rounded to fp16 into LDS, then the
// arithmetic of attention_f16_kernel.  The products P.V of the four key tiles are formed from zero one by one and
// added in the order in which that kernel adds its four waves' partial contexts (tiles past the end add +0), and the
// row sums likewise, so the context is the same bytes as from the two kernels.
// PACKED (at most 128 tokens, weights in the order of the 32 x 32 x 16 product): the tile loop of the GEMMs on packed weights, in the same
// 2 x 2 arrangement of waves (six channel blocks do not deal out over four waves), so two waves each load the same weight rows.  55 KB of
// LDS instead of 80, two stages in flight instead of one; BERT-base 32 x 128 forward, us, row-major / packed: FP16 1240 / 1196, Quant-FFN-Only
// 941 / 891.
template <int QT, int STAGE, bool PACKED, bool FETCH = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(QT == 1 ? 2 : 1, QT == 1 ? 2 : 1)))
void qkv_attention_f16_kernel(const char *__restrict__ X, const char *__restrict__ W, const float *__restrict__ bias,
                              const int *__restrict__ cu, int max_len, int H, int items, unsigned by_heads, float scale, __half *__restrict__ ctx, typename FetchArg<FETCH>::type fetch)
{
    if (fetch_instead(fetch, items)) return;
    typedef QkvTile<QT, STAGE> Tile;
    constexpr bool LATE = Tile::LATE && !PACKED;
    constexpr int TM = Tile::TM, TN = Tile::TN, BM = Tile::BM, BN = Tile::BN, NKT = 4 * QT;
    constexpr int RING_BYTES = PACKED ? QKV_F16_PACKED_RING : Tile::RING_BYTES;
    constexpr int QK_STRIDE = 144, VT_STRIDE = 2 * BM + 8;        // bytes per token row of q / k (64 fp16 + pad), per channel row of V^T (all keys + pad)
    constexpr int TAB_BYTES = 1024;                               // bias of the 192 columns
    constexpr int Q_OFF = LATE ? TAB_BYTES : 0, K_OFF = Q_OFF + BM * QK_STRIDE, VT_OFF = K_OFF + BM * QK_STRIDE;
    constexpr int QKV_BYTES = VT_OFF + 64 * VT_STRIDE;            // q, k and V^T take the place of the ring (and more, for 256 tokens)
    constexpr int TAB_OFF = QKV_BYTES > RING_BYTES ? QKV_BYTES : RING_BYTES;
    static_assert(!LATE || QKV_BYTES + TAB_BYTES <= RING_BYTES, "clear of a table at either end of the ring");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    float *tab = reinterpret_cast<float *>(lds + (!LATE ? TAB_OFF : (H / 64) & 1 ? RING_BYTES - TAB_BYTES : 0));

    const int heads = H >> 6;
    const int item = cu ? (int)blockIdx.x : xcd_contiguous(blockIdx.x, items);
    const int seq = (int)over(item, by_heads, heads), head = item - seq * heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int n = sq.n;
    if (n <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int wm = (wave >> 1) * 32 * TM, wn = (wave & 1) * 32 * TN;
    const int r = lane & 31, g = lane >> 5;

    v16f acc[TN][TM];
    auto load_tables = [&]() {
        if constexpr (LATE || PACKED) {
            if (wave < 3) {
                if (bias) load_direct(tab + wave * 64, bias + wave * H + head * 64, 64, lane);
                else tab[wave * 64 + lane] = 0.0f;
            }
            return;
        }
        for (int c = tid; c < BN; c += 256) tab[c] = bias ? bias[(c >> 6) * H + head * 64 + (c & 63)] : 0.0f;
    };
    if constexpr (PACKED) {
        unsigned offa[stream_loads<true, 4>()];
#pragma unroll
        for (int j = 0; j < stream_loads<true, 4>(); j++) {
            const int srow = 8 * (wave + 4 * j) + (lane >> 3);
            offa[j] = (unsigned)min(srow, n - 1) * (unsigned)(2 * H) + (((lane & 7) ^ swz<128>(srow)) << 4);
        }
        unsigned woff[TN];
#pragma unroll
        for (int io = 0; io < TN; io++) {
            const int nl = wn + 32 * io;
            woff[io] = (unsigned)((nl >> 6) * H + head * 64 + (nl & 63)) * (unsigned)(2 * H);
        }
#pragma unroll
        for (int io = 0; io < TN; io++)
#pragma unroll
            for (int j = 0; j < TM; j++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[io][j][e] = 0.0f;
        // values (the last two channel blocks of odd waves): token rows first, as in qkv_tile_gemm()
        auto loop = [&](auto vwave, auto live) {
            stream_tile_loop<true, TM, TN, QKV_F16_PACKED_D, 2>(X + (size_t)sq.t0 * (2 * H), offa, W, woff, H / 64, lds, wave, lane, load_tables,
                [&](int t, int i, const v4i &w, const v4i &f) {
                    const bool swap = decltype(vwave)::value && t > 0;
                    if (live(i)) acc[t][i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, swap ? f : w),
                                                                                   __builtin_bit_cast(v8h, swap ? w : f), acc[t][i], 0, 0, 0);
                }, wave >> 1);
        };
        auto either = [&](auto vwave) {
            if (n > BM - 32) loop(vwave, [](int) { return true; });
            else loop(vwave, [&](int i) { return wm + 32 * i < n; });
        };
        if (wave & 1) either(std::true_type());
        else either(std::false_type());
    } else {
        qkv_tile_gemm_any<QT, STAGE, true>(X, W, sq.t0, n, head, H, 2 * H, lds, wave, lane, acc, load_tables);
    }

    // fp16(acc + bias) into LDS: q and k as token rows, v transposed (lane layouts as in the INT8 flavour)
#pragma unroll
    for (int io = 0; io < TN; io++) {
        const int nl = wn + io * 32;
        const int part = nl >> 6, c0 = nl & 63;
        if (part < 2) {
            v4f bb[4];
#pragma unroll
            for (int q = 0; q < 4; q++) bb[q] = *reinterpret_cast<const v4f *>(tab + nl + 8 * q + 4 * g);
#pragma unroll
            for (int j = 0; j < TM; j++) {
                const int row = wm + 32 * j + r;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const v16f &a = acc[io][j];
                    const v4h h = {to_half(a[4 * q] + bb[q].x), to_half(a[4 * q + 1] + bb[q].y), to_half(a[4 * q + 2] + bb[q].z),
                                   to_half(a[4 * q + 3] + bb[q].w)};
                    *reinterpret_cast<v4h *>(lds + (part ? K_OFF : Q_OFF) + row * QK_STRIDE + (c0 + 8 * q + 4 * g) * 2) = h;
                }
            }
        } else {
            const float bb = tab[nl + r];                         // the lane's channel
#pragma unroll
            for (int j = 0; j < TM; j++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const v16f &a = acc[io][j];
                    const v4h h = {to_half(a[4 * q] + bb), to_half(a[4 * q + 1] + bb), to_half(a[4 * q + 2] + bb), to_half(a[4 * q + 3] + bb)};
                    *reinterpret_cast<v4h *>(lds + VT_OFF + (c0 + r) * VT_STRIDE + (wm + 32 * j + 8 * q + 4 * g) * 2) = h;
                }
        }
    }
    __syncthreads();

#pragma unroll 1
    for (int qt = 0; qt < QT; qt++) {
        const int q0 = (wave * QT + qt) * QB;
        if (q0 >= n) break;                                       // no barrier below
        v8h qf[4];
#pragma unroll
        for (int ks = 0; ks < 4; ks++) qf[ks] = *reinterpret_cast<const v8h *>(lds + Q_OFF + (q0 + r) * QK_STRIDE + (ks * 16 + g * 8) * 2);
        float sc[NKT][16];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < NKT; i++) {
            const int j0 = 32 * i;
            if (j0 < n) {
                v16f s;
#pragma unroll
                for (int e = 0; e < 16; e++) s[e] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < 4; ks++)
                    s = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const v8h *>(lds + K_OFF + (j0 + r) * QK_STRIDE + (ks * 16 + g * 8) * 2),
                                                               qf[ks], s, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int key = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
                    sc[i][e] = key < n ? s[e] * scale : -INFINITY;
                    mx = __builtin_fmaxf(mx, sc[i][e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) sc[i][e] = -INFINITY;
            }
        }
        mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));

        float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};                // key tile i adds to partial sum i mod 4, in ascending order
#pragma unroll
        for (int i = 0; i < NKT; i++)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const float ev = __builtin_amdgcn_exp2f((sc[i][e] - mx) * 1.44269504088896341f);
                sc[i][e] = ev;
                part[i & 3] += ev;
            }
#pragma unroll
        for (int u = 0; u < 4; u++) part[u] += __shfl_xor(part[u], 32, 64);
        const float S = ((part[0] + part[1]) + part[2]) + part[3];
        const float rS = __fdiv_rn(1.0f, S);

        // partial context u: the key tiles u, u + 4, ... from zero, as wave u of the attention kernel forms it; then added in its order
        v16f o[2];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            v16f ot[2];
#pragma unroll
            for (int cb = 0; cb < 2; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) ot[cb][e] = 0.0f;
#pragma unroll
            for (int ii = 0; ii < QT; ii++) {
                const int i = u + 4 * ii;
                if (32 * i < n) {
#pragma unroll
                    for (int hf = 0; hf < 2; hf++) {                // keys 8q+4g+t for q in {2hf, 2hf+1}
                        v8h pf;
#pragma unroll
                        for (int e = 0; e < 8; e++) pf[e] = to_half(sc[i][8 * hf + e] * rS);
#pragma unroll
                        for (int cb = 0; cb < 2; cb++) {
                            const char *rowp = lds + VT_OFF + (cb * 32 + r) * VT_STRIDE + 32 * i * 2;
                            const v4h lo = *reinterpret_cast<const v4h *>(rowp + (16 * hf + 4 * g) * 2);
                            const v4h hi = *reinterpret_cast<const v4h *>(rowp + (16 * hf + 8 + 4 * g) * 2);
                            const v8h vf = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                            ot[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pf, ot[cb], 0, 0, 0);   // channels x queries: a lane holds ONE query
                        }
                    }
                }
            }
#pragma unroll
            for (int cb = 0; cb < 2; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) o[cb][e] = u == 0 ? ot[cb][e] : o[cb][e] + ot[cb][e];
        }

        // context: the lane's query, channels cb*32 + 8q + 4g + t; through the wave's own query rows in LDS, out as 64 bytes per lane
        char *slab = lds + Q_OFF + q0 * QK_STRIDE;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const v4h h = {to_half(o[cb][4 * q]), to_half(o[cb][4 * q + 1]), to_half(o[cb][4 * q + 2]), to_half(o[cb][4 * q + 3])};
                *reinterpret_cast<v4h *>(slab + r * QK_STRIDE + (cb * 32 + 8 * q + 4 * g) * 2) = h;
            }
        __builtin_amdgcn_wave_barrier();
        const int query = lane >> 1, half = lane & 1;
        if (q0 + query < n) {
            __half *dst = ctx + (size_t)(sq.t0 + q0 + query) * H + head * 64 + half * 32;
#pragma unroll
            for (int u = 0; u < 4; u++)
                *reinterpret_cast<v4i *>(dst + u * 8) = *reinterpret_cast<const v4i *>(slab + query * QK_STRIDE + half * 64 + u * 16);
        }
    }
}

// V rows of a key tile as they lie (32 keys x 64 binary16) in LDS, and V^T operands out of it: ds_read_b64_tr_b16 hands lane i of sixteen the
// half i & 3 of the four halves that lanes (i >> 2) + 4 t, t = 0..3, point at, so that with lanes 4 t .. 4 t + 3 at 16 channels of key t a lane gets
// one channel of four keys.  16-byte chunk c of key k lies at position c ^ 4 ((k >> 1) & 1): the 32 lanes of a read's phase hit 64 different banks.
constexpr int V_TILE_F16 = 32 * 64 * 2;
struct VLaneF16 {                                         // what a lane loads and reads of every tile, in bytes
    unsigned from, at;                                    // offset of its 16 bytes in the first 8 rows (of 2 ld bytes); of its first read in a tile
    __device__ __forceinline__ VLaneF16(unsigned ld, int lane)
    {
        from = (unsigned)(lane >> 3) * 2 * ld + (((lane & 7) ^ (((lane >> 4) & 1) << 2)) << 4);
        const int key = 4 * (lane >> 5) + ((lane >> 2) & 3), chunk = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
        at = key * 128 + ((chunk ^ (((key >> 1) & 1) << 2)) << 4) + 8 * (lane & 1);
    }
};
// channel 32 cb + (lane & 31), keys 16 hf + 4 (lane >> 5) + (0..3, 8..11)
__device__ __forceinline__ v8h read_vt_f16(const char *tile, unsigned at, int hf, int cb)
{
    typedef __attribute__((address_space(3))) v4s *Lds;
    const char *p = tile + (at ^ (cb << 6)) + hf * 2048;
    const v4h lo = __builtin_bit_cast(v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds)p));
    const v4h hi = __builtin_bit_cast(v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds)(p + 1024)));
    return v8h{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}
__device__ __forceinline__ void request_v_tile_f16(__amdgpu_buffer_rsrc_t rows, unsigned from, unsigned ld, char *tile)
{
#pragma unroll
    for (int u = 0; u < 4; u++) buffer_to_lds128(rows, from + u * 16 * ld, 0, tile + u * 1024);
}

// FP16 flavour: fp16 q, k, v; binary32 scores, fast exp; P rounded to fp16 before P.V; binary32
// accumulation of P.V.  Optionally records the largest softmax output (calibration of the P step).
// Up to 2048 keys (NT = 16 key tiles per wave) the strip of scores stays in registers; the order of all sums is that of the
// three-sweep kernel, tile by tile, so both give the same bytes.  Twelve heads, three sequences of 1100 tokens: 76 -> 51 us, 17 of
// 301 36.5 -> 30 us.  V rows are loaded straight into LDS and transposed by the reads, rows past the end are cut off by the buffer
// descriptor, and a full key tile's scores need no mask; tiles beyond the first two take a read tile's place by direct loads, so that four
// tiles of scores leave registers for four waves per SIMD instead of two, which is what bounded them.  Twelve heads, us, before / now: 64 x 512 255 /
// 200, 3 x 1100 51 / 42, 12 x 1250 191 / 170, 20 x 30..400 33.6 / 27.5; 16 x 256 of sixteen heads 27.2 / 26.9 (two tiles: as many waves as before).
template <int NT, bool FETCH = false, int NW = 4>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NT <= 4 ? 4 : NT <= 10 ? 2 : 1))) void attention_f16_kernel(const __half *__restrict__ qkv, const int *__restrict__ cu,
                                                            int max_len, int H, int items, unsigned by_nqb, unsigned by_heads, float scale, __half *__restrict__ ctx,
                                                            float *__restrict__ p_absmax, typename FetchArg<FETCH>::type fetch)
{
    if (fetch_instead(fetch, items)) return;
    // one slab per wave, as in the INT8 kernel: first its V^T tiles (two; a further one takes a tile's place when that one has
    // been read), then its partial context for the other waves.  TIGHT: ten tiles of scores leave two waves per SIMD just
    // enough registers if V rows are requested one tile earlier (four tiles in the slab) and tiles past the end are skipped in
    // the sums of exponentials; without either it takes 20 bytes of scratch (12 heads, 12 sequences of 1250 tokens, when it was 48: 213 -> 194 us).
    // Fewer or more tiles do not need it, and 12 sequences of 1500 would lose 3 %.
    constexpr bool TIGHT = NT == 10;
    constexpr int SO_BYTES = QB * 64 * 4, VT_TILES = TIGHT ? 4 : NT < 2 ? NT : 2, AHEAD = TIGHT ? 2 : 1;
    constexpr int SLAB = VT_TILES * V_TILE_F16 > SO_BYTES ? VT_TILES * V_TILE_F16 : SO_BYTES;
    constexpr int K_AHEAD = NT == 1 || NT == 3 || NT == 4 ? 1 : 2;   // key tiles whose rows are requested before the first product (as many as registers hold)
    __shared__ __attribute__((aligned(1024))) char slab[NW][SLAB];
    auto so = [&](int wave) { return reinterpret_cast<float(*)[64]>(slab[wave]); };
    __shared__ float smax[NW][QB];
    __shared__ float ssum[NW][QB];

    const int nqb = (max_len + QB - 1) / QB, heads = H >> 6;
    const Strip at = strip_of(blockIdx.x, items, nqb, by_nqb, cu && nqb >= DEALT_MIN_STRIPS);
    const int seq = (int)over(at.pair, by_heads, heads), head = at.pair - seq * heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int q0 = at.strip * QB;
    if (q0 >= sq.n) return;
    const int n = sq.n;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), r = lane & 31, g = lane >> 5;
    const unsigned ld = 3u * (unsigned)H;
    const __half *base = qkv + (size_t)sq.t0 * ld + head * 64;
    auto rows_from = [&](int j0) { return strip_rows(base, ld, head, j0, n); };
    auto first_key = [&](int i) { return (w + NW * i) * 32; };

    const unsigned row_at = 2 * (unsigned)r * ld + g * 16, key_at = row_at + 2 * H;
    const VLaneF16 vl(ld, lane);
    v4i qf[4], kf[K_AHEAD][4];
    auto request_keys = [&](int i) {
        const auto rows = rows_from(first_key(i));
#pragma unroll
        for (int ks = 0; ks < 4; ks++) kf[i % K_AHEAD][ks] = __builtin_amdgcn_raw_buffer_load_b128(rows, key_at + ks * 32, 0, 0);
    };
    {
        const auto rows = rows_from(q0);
#pragma unroll
        for (int ks = 0; ks < 4; ks++) qf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rows, row_at + ks * 32, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < K_AHEAD; i++) request_keys(i);
#pragma unroll
    for (int i = 0; i < VT_TILES; i++) request_v_tile_f16(rows_from(first_key(i)), vl.from + 4 * H, ld, &slab[w][i * V_TILE_F16]);

    float sc[NT][16];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NT; i++) {
        const int j0 = first_key(i);
        if (j0 < n) {
            v16f acc;
#pragma unroll
            for (int e = 0; e < 16; e++) acc[e] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < 4; ks++)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, kf[i % K_AHEAD][ks]), __builtin_bit_cast(v8h, qf[ks]), acc, 0, 0, 0);
            if (j0 + 32 <= n) {                                  // a full tile needs no masking
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    sc[i][e] = acc[e] * scale;
                    mx = __builtin_fmaxf(mx, sc[i][e]);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int key = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
                    sc[i][e] = key < n ? acc[e] * scale : -INFINITY;
                    mx = __builtin_fmaxf(mx, sc[i][e]);
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; e++) sc[i][e] = -INFINITY;
        }
        if (i + K_AHEAD < NT) request_keys(i + K_AHEAD);
    }
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) smax[w][r] = mx;
    wait_vm<0>();                                                 // the wave's V tiles are in its slab
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NW; u++) mx = __builtin_fmaxf(mx, smax[u][r]);

    float part = 0.0f;
#pragma unroll
    for (int i = 0; i < NT; i++)
        if (!TIGHT || (w + NW * i) * 32 < n) {                     // tiles past the end add zeros
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const float ev = __builtin_amdgcn_exp2f((sc[i][e] - mx) * 1.44269504088896341f);
                sc[i][e] = ev;
                part += ev;
            }
        }
    part += __shfl_xor(part, 32, 64);
    if (g == 0) ssum[w][r] = part;
    __syncthreads();
    float S = ssum[0][r];
#pragma unroll
    for (int u = 1; u < NW; u++) S += ssum[u][r];
    const float rS = __fdiv_rn(1.0f, S);
    if (p_absmax && w == 0 && g == 0 && q0 + r < n)              // the row's largest P is exp(0) / S
        atomicMax(reinterpret_cast<int *>(p_absmax), __float_as_int((float)(_Float16)rS));

    v16f o[2];
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) o[cb][e] = 0.0f;
#pragma unroll
    for (int i = 0; i < NT; i++) {
        const int j1 = (w + NW * (i + AHEAD)) * 32;                 // the tile that takes the place of tile i - AHEAD
        const bool more = i >= AHEAD && i + AHEAD < NT && j1 < n;
        if (more) {
            wait_lds();                                             // the reads of tile i - AHEAD have returned
            request_v_tile_f16(rows_from(j1), vl.from + 4 * H, ld, &slab[w][(i + AHEAD) % VT_TILES * V_TILE_F16]);
        }
        if ((w + NW * i) * 32 < n) {
#pragma unroll
            for (int hf = 0; hf < 2; hf++) {                    // keys 8q+4g+t for q in {2hf, 2hf+1}
                v8h pf;
#pragma unroll
                for (int e = 0; e < 8; e++) pf[e] = to_half(sc[i][8 * hf + e] * rS);
#pragma unroll
                for (int cb = 0; cb < 2; cb++) {
                    const v8h vf = read_vt_f16(&slab[w][i % VT_TILES * V_TILE_F16], vl.at, hf, cb);
                    o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(pf, vf, o[cb], 0, 0, 0);
                }
            }
        }
        if (NT > VT_TILES) {                                        // tile i + 1 is there
            if (AHEAD > 1 && more) wait_vm<4 * (AHEAD - 1)>();
            else wait_vm<0>();
        }
    }
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) so(w)[8 * (e >> 2) + 4 * g + (e & 3)][cb * 32 + r] = o[cb][e];
    __syncthreads();

    // (fewer waves than four: those without a key tile would have added +0)
#pragma unroll
    for (int i = 0; i < 4 / NW; i++) {
        const int query = (tid >> 3) + 8 * NW * i, c0 = (tid & 7) * 8;
        if (q0 + query < n) {
            v8h outv;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                float o_sum = so(0)[query][c0 + e];
#pragma unroll
                for (int u = 1; u < NW; u++) o_sum += so(u)[query][c0 + e];
                if (NW < 4) o_sum += 0.0f;
                outv[e] = to_half(o_sum);
            }
            *reinterpret_cast<v8h *>(ctx + (size_t)(sq.t0 + q0 + query) * H + head * 64 + c0) = outv;
        }
    }
}


// ---- sequences whose scores do not fit the registers: the same arithmetic as above, tile by tile ---------------------
// Beyond 2048 keys (1536 with the binary16 softmax output) the kernels below sweep the key tiles three
// times: row maxima, row sums, then codes and P.V.  The integer products q.k are recomputed in each
// sweep (two MFMAs per 32 x 32 tile; exact, so all sweeps see the same scores), the exponentials in the
// last two.  A wave still owns key tiles w, w+4, ... and visits them in ascending order, so every
// binary32 / binary64 operation happens in the same order as in the one-pass kernels.

// scores of key tile j0 for the lane's query: sc[e] belongs to key j0 + 8 (e >> 2) + 4 g + (e & 3)
__device__ __forceinline__ void score_tile_i8(const int8_t *base, unsigned ld, int H, int j0, int n, int r, int g,
                                              const v4i (&qf)[2], float m_sc, float (&sc)[16])
{
    const int8_t *kp = base + (unsigned)min(j0 + r, n - 1) * ld + H;
    v16i acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0;
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i *>(kp + ks * 32 + g * 16), qf[ks], acc, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 16; e++) {
        const int key = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
        sc[e] = key < n ? (float)acc[e] * m_sc : -INFINITY;
    }
}

template <bool PU, bool HIST>
__global__ __launch_bounds__(256) void attention_i8_long_kernel(const int8_t *__restrict__ qkv, const int *__restrict__ cu,
                                                                int max_len, int H, float m_sc, float inv_sp, float m_ctx,
                                                                int8_t *__restrict__ ctx, unsigned long long *__restrict__ p_hist)
{
    __shared__ unsigned hist[HIST ? 256 : 1];
    __shared__ __attribute__((aligned(16))) int8_t vt[4][64 * VT_STRIDE_I8];
    __shared__ __attribute__((aligned(16))) int so[4][QB][64];
    __shared__ float smax[4][QB];
    __shared__ double ssum[4][QB];

    const int nqb = (max_len + QB - 1) / QB, heads = H >> 6;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int seq = item / (nqb * heads), head = (item / nqb) % heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int q0 = (item % nqb) * QB;
    if (q0 >= sq.n) return;
    const int n = sq.n;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), r = lane & 31, g = lane >> 5;
    const unsigned ld = 3u * (unsigned)H;
    const int8_t *base = qkv + (size_t)sq.t0 * ld + head * 64;
    if (HIST) hist[tid] = 0;

    const int qrow = min(q0 + r, n - 1);
    v4i qf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ks++) qf[ks] = *reinterpret_cast<const v4i *>(base + (unsigned)qrow * ld + ks * 32 + g * 16);

    float sc[16];
    float mx = -INFINITY;
    for (int j0 = w * 32; j0 < n; j0 += 128) {
        score_tile_i8(base, ld, H, j0, n, r, g, qf, m_sc, sc);
#pragma unroll
        for (int e = 0; e < 16; e++) mx = __builtin_fmaxf(mx, sc[e]);
    }
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) smax[w][r] = mx;
    __syncthreads();
    mx = __builtin_fmaxf(__builtin_fmaxf(smax[0][r], smax[1][r]), __builtin_fmaxf(smax[2][r], smax[3][r]));

    double part = 0.0;
    for (int j0 = w * 32; j0 < n; j0 += 128) {
        score_tile_i8(base, ld, H, j0, n, r, g, qf, m_sc, sc);
#pragma unroll
        for (int e = 0; e < 16; e++) part += (double)(float)exp_nonpos((double)__builtin_fmaxf(sc[e] - mx, -746.0f));
    }
    part += __shfl_xor(part, 32, 64);
    if (g == 0) ssum[w][r] = part;
    __syncthreads();
    const float S = (float)(((ssum[0][r] + ssum[1][r]) + ssum[2][r]) + ssum[3][r]);
    const float rS = __fdiv_rn(1.0f, S);

    v16i o[2], o1[PU ? 2 : 1];
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) { o[cb][e] = 0; if (PU) o1[cb][e] = 0; }
    const float lo = PU ? 0.0f : -127.0f, hi = PU ? 255.0f : 127.0f;
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const int8_t *vp = base + 2 * H;
    for (int j0 = w * 32; j0 < n; j0 += 128) {
        score_tile_i8(base, ld, H, j0, n, r, g, qf, m_sc, sc);
        // V^T of this key tile into the wave's own LDS slab (4 keys x 4 channels byte blocks transposed in
        // registers); the slab is written and read by this wave only, in program order
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int cq = lane & 15, kq = (lane >> 4) + 4 * u;
            unsigned d[4];
#pragma unroll
            for (int t = 0; t < 4; t++)
                d[t] = *reinterpret_cast<const unsigned *>(vp + (unsigned)min(j0 + 4 * kq + t, n - 1) * ld + 4 * cq);
            const unsigned t01l = __builtin_amdgcn_perm(d[1], d[0], 0x05010400u), t23l = __builtin_amdgcn_perm(d[3], d[2], 0x05010400u);
            const unsigned t01h = __builtin_amdgcn_perm(d[1], d[0], 0x07030602u), t23h = __builtin_amdgcn_perm(d[3], d[2], 0x07030602u);
            unsigned *dst = reinterpret_cast<unsigned *>(&vt[w][(4 * cq) * VT_STRIDE_I8 + 4 * kq]);
            dst[0 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23l, t01l, 0x05040100u);
            dst[1 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23l, t01l, 0x07060302u);
            dst[2 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23h, t01h, 0x05040100u);
            dst[3 * (VT_STRIDE_I8 / 4)] = __builtin_amdgcn_perm(t23h, t01h, 0x07060302u);
        }
        __builtin_amdgcn_wave_barrier();
        v4i pf;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float f[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const float ev = (float)exp_nonpos((double)__builtin_fmaxf(sc[4 * q + t] - mx, -746.0f));
                f[t] = __builtin_amdgcn_fmed3f((ev * rS) * inv_sp, lo, hi) + SAMP_RNE_MAGIC;
                if (HIST && q0 + r < n && j0 + 8 * q + 4 * g + t < n) atomicAdd(&hist[__float_as_uint(f[t]) & 0xffu], 1u);
            }
            pf[q] = pack_codes(f[0], f[1], f[2], f[3]);
            if (PU) pf[q] ^= (int)0x80808080u;
        }
#pragma unroll
        for (int cb = 0; cb < 2; cb++) {
            v4i vf;
#pragma unroll
            for (int q = 0; q < 4; q++)
                vf[q] = *reinterpret_cast<const int *>(&vt[w][(cb * 32 + r) * VT_STRIDE_I8 + 8 * q + 4 * g]);
            o[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(pf, vf, o[cb], 0, 0, 0);
            if (PU) o1[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ones, vf, o1[cb], 0, 0, 0);
        }
    }
    if (PU) {
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
            for (int e = 0; e < 16; e++) o[cb][e] += o1[cb][e] * 128;
    }
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) so[w][8 * (e >> 2) + 4 * g + (e & 3)][cb * 32 + r] = o[cb][e];
    __syncthreads();

    const int query = tid >> 3, c0 = (tid & 7) * 8;
    if (q0 + query < n) {
        int codes[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int O = ((so[0][query][c0 + e] + so[1][query][c0 + e]) + so[2][query][c0 + e]) + so[3][query][c0 + e];
            codes[e] = qcode((float)O * m_ctx);
        }
        v2i pk = {pack4(codes[0], codes[1], codes[2], codes[3]), pack4(codes[4], codes[5], codes[6], codes[7])};
        *reinterpret_cast<v2i *>(ctx + (size_t)(sq.t0 + q0 + query) * H + head * 64 + c0) = pk;
    }
    if (HIST && hist[tid]) atomicAdd(&p_hist[tid], (unsigned long long)hist[tid]);
}

// ---- INT8 attention block whose softmax output stays binary16 (not on the 8-bit grid) ---------------
// P16 = fl16(e * rS), ctx = rne(fl32(sum_k P16[k] V[k]) * m) with m = s_v / s_ctx.  The sum is evaluated
// exactly: a binary16 value in [0, 1] is an integer multiple of 2^-24, so P16 * 2^24 is an integer below
// 2^25 that splits into four bytes; each byte plane is one more int8 operand for the matrix core (the lower
// three as byte - 128, with 128 times the sum of V added back; the top byte is 0 or 1), the int32
// products recombine in 64-bit integers, and one conversion rounds the true sum to binary32.  That is the kernel for any length;
// up to 1536 keys two binary16 parts do it with less arithmetic (below).

// V^T of key tile j0 into a wave's own LDS slab
__device__ __forceinline__ void stage_vt_i8(const int8_t *vp, unsigned ld, int j0, int n, int lane, int8_t *slab)
{
    unsigned d[2][4];
    load_v_tile(vp, ld, j0, n, lane, d);
    store_vt_tile(d, lane, slab);
}

// digit planes of one key tile: ev[e] = fl32(exp(score - max)) of the lane's 16 keys; pf[k] is the int8 operand
// holding byte k of P16 * 2^24 for those keys, bytes 0..2 with the top bit flipped (byte - 128 as a signed byte)
__device__ __forceinline__ void p16_digits(const float (&ev)[16], float rS, v4i (&pf)[4])
{
#pragma unroll
    for (int q = 0; q < 4; q++) {
        unsigned fixed[4];                                        // P16 * 2^24 of four consecutive keys
#pragma unroll
        for (int t = 0; t < 4; t++) fixed[t] = (unsigned)((float)to_half(ev[4 * q + t] * rS) * 16777216.0f);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const unsigned sel = 0x0c0c0000u | (unsigned)((4 + k) << 8) | (unsigned)k;
            const unsigned lo = __builtin_amdgcn_perm(fixed[1], fixed[0], sel), hi = __builtin_amdgcn_perm(fixed[3], fixed[2], sel);
            pf[k][q] = (int)(__builtin_amdgcn_perm(hi, lo, 0x05040100u) ^ (k < 3 ? 0x80808080u : 0u));
        }
    }
}

// digit planes times the V^T tile in the slab, channel block cb: o[k] += pf[k] . V; vsum: the sum of the lane's V codes
__device__ __forceinline__ void p16_mfma(const v4i (&pf)[4], const int8_t *slab, int cb, int r, int g, v16i (&o)[4], int &vsum)
{
    v4i vf;
#pragma unroll
    for (int q = 0; q < 4; q++) vf[q] = *reinterpret_cast<const int *>(&slab[(cb * 32 + r) * VT_STRIDE_I8 + 8 * q + 4 * g]);
#pragma unroll
    for (int k = 0; k < 4; k++) o[k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(pf[k], vf, o[k], 0, 0, 0);
    vsum = add_codes(vf, vsum);
}

// adds 2^24 times a wave's partial context of one channel block to the block's 64-bit sums (exact in any order)
__device__ __forceinline__ void p16_add(const v16i (&o)[4], int vsum, long long (&so)[QB][32], int r, int g)
{
    const long long ones = (long long)(vsum + __shfl_xor(vsum, 32, 64)) * (128 * (1 + 256 + 65536));     // the 128s taken off three digits
#pragma unroll
    for (int e = 0; e < 16; e++) {
        const long long v = ((((long long)o[3][e] * 256 + o[2][e]) * 256 + o[1][e]) * 256) + o[0][e] + ones;
        atomicAdd(reinterpret_cast<unsigned long long *>(&so[8 * (e >> 2) + 4 * g + (e & 3)][r]), (unsigned long long)v);
    }
}

// The block's sums, complete after a barrier: scaled back (exact) and rounded once to binary32.
__device__ __forceinline__ void p16_store(const long long (&so)[2][QB][32], float m_ctx, int8_t *ctx_rows, int H, int rows_left, int tid)
{
    const int query = tid >> 3, c0 = (tid & 7) * 8;
    if (query >= rows_left) return;
    int codes[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int c = c0 + e;
        codes[e] = qcode((float)((double)so[c >> 5][query][c & 31] * 5.9604644775390625e-08) * m_ctx);      // * 2^-24
    }
    *reinterpret_cast<v2i *>(ctx_rows + (size_t)query * H + c0) =
        v2i{pack4(codes[0], codes[1], codes[2], codes[3]), pack4(codes[4], codes[5], codes[6], codes[7])};
}

// Up to 1536 keys the strip of scores stays in registers (one pass, as attention_i8_kernel), and the exact sum needs no digits: P16 splits into two
// binary16 numbers, hi = (P16 + C) - C with C = 1.5 / 16 and lo = P16 - hi, both exact, whose products with the V codes (as binary16) the FP16 matrix
// instruction adds up exactly in binary32, whatever its order:
//     hi is a multiple of 2^-14 and sum |hi V| <= 128 (1.001 + 2^-15 keys) < 2^24 2^-14;
//     lo is a multiple of 2^-24 with |lo| <= 2^-15 + P16 / 2^10, so sum |lo V| <= 128 (2^-15 keys + 1.01 / 2^10) < 2^24 2^-24 as long as a wave has at most
//     192 keys.
// The waves' parts meet in int32 in units of 2^-24, modulo 2^32: hi sums in their own unit, shifted up, lo sums as they are.  With S = sum P16 <= 1.001
// the whole sum lies in [-128 S, 127 S], which is wider than int32's [-128, 128) to the left and shorter to the right, so the parts are added to a half
// (P16_HALF) that is taken off again in binary64.
// What bounds the kernel is vector arithmetic: 19 operations of the softmax per score, then 3 for the parts and 2.5 for V as binary16, where the
// digits took 9.3 and the recombination of the waves' sums twice the operations; it also fits four blocks to a CU instead of two.  Forward,
// BERT-base 33 x 40..301, us, digits / parts: 1458 / 1265.
constexpr int P16_WAVE_KEYS = 192, P16_HALF = 1 << 23;
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// one key tile's operands, from ev[e] = fl32(exp(score - max)): keys 16 u + 8 q + 4 g + t of half u
__device__ __forceinline__ void p16_split(const float (&ev)[16], float rS, v8h (&hi)[2], v8h (&lo)[2])
{
    const v2h c = {(_Float16)0.09375f, (_Float16)0.09375f};
#pragma unroll
    for (int k = 0; k < 8; k++) {
        v2f v = {ev[2 * k] * rS, ev[2 * k + 1] * rS};
        asm("" : "+v"(v));                                        // (binary32 first, as to_half)
        const v2h p = __builtin_convertvector(v, v2h), h = (p + c) - c, l = p - h;
#pragma unroll
        for (int t = 0; t < 2; t++) { hi[k >> 2][2 * (k & 3) + t] = h[t]; lo[k >> 2][2 * (k & 3) + t] = l[t]; }
    }
}
// eight codes as binary16: byte u = code + 128 under the exponent of 1024 is 1024 + u
__device__ __forceinline__ v8h codes_to_half(int d0, int d1)
{
    const v2h bias = {(_Float16)1152.0f, (_Float16)1152.0f};
    v4i raw;
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const unsigned x = (unsigned)(k ? d1 : d0) ^ 0x80808080u;
        raw[2 * k] = (int)__builtin_amdgcn_perm(0x64646464u, x, 0x04010400u);
        raw[2 * k + 1] = (int)__builtin_amdgcn_perm(0x64646464u, x, 0x04030402u);
    }
    v4i out;
#pragma unroll
    for (int k = 0; k < 4; k++) out[k] = __builtin_bit_cast(int, __builtin_bit_cast(v2h, (int)raw[k]) - bias);
    return __builtin_bit_cast(v8h, out);
}

template <int NT, int NW = 4, bool FETCH = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NT <= 3 ? 4 : 2))) void
attention_i8_p16_kernel(const int8_t *__restrict__ qkv, const int *__restrict__ cu, int max_len, int H, int items, unsigned by_nqb, unsigned by_heads, float m_sc, float m_ctx,
                        int8_t *__restrict__ ctx, typename FetchArg<FETCH>::type fetch)
{
    if (fetch_instead(fetch, items)) return;
    static_assert(32 * NT <= P16_WAVE_KEYS, "the bound on the sum of the low parts");
    constexpr int K_AHEAD = NT <= 4 ? NT : 2;
    __shared__ __attribute__((aligned(1024))) int8_t slab[NW][NT * V_TILE];
    __shared__ __attribute__((aligned(16))) unsigned so[QB][64];
    __shared__ float smax[NW][QB];
    __shared__ double ssum[NW][QB];
    __shared__ ExpTable exp_table;

    const int nqb = (max_len + QB - 1) / QB, heads = H >> 6;
    const Strip at = strip_of(blockIdx.x, items, nqb, by_nqb, cu && nqb >= DEALT_MIN_STRIPS);
    const int seq = (int)over(at.pair, by_heads, heads), head = at.pair - seq * heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int q0 = at.strip * QB;
    if (q0 >= sq.n) return;
    const int n = sq.n;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), r = lane & 31, g = lane >> 5;
    const unsigned ld = 3u * (unsigned)H;
    const int8_t *base = qkv + (size_t)sq.t0 * ld + head * 64;
    auto rows_from = [&](int j0) { return strip_rows(base, ld, head, j0, n); };
    auto first_key = [&](int i) { return (w + NW * i) * 32; };
    const uint64_t table_entry = EXP2_TABLE[tid & 255];

    const unsigned row_at = (unsigned)r * ld + g * 16, key_at = row_at + H;
    const VLane vl(ld, lane);
    v4i qf[2], kf[K_AHEAD][2];
    auto request_keys = [&](int i) {
        const auto rows = rows_from(first_key(i));
#pragma unroll
        for (int ks = 0; ks < 2; ks++) kf[i % K_AHEAD][ks] = __builtin_amdgcn_raw_buffer_load_b128(rows, key_at + ks * 32, 0, 0);
    };
    {
        const auto rows = rows_from(q0);
#pragma unroll
        for (int ks = 0; ks < 2; ks++) qf[ks] = __builtin_amdgcn_raw_buffer_load_b128(rows, row_at + ks * 32, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < K_AHEAD; i++) request_keys(i);
#pragma unroll
    for (int i = 0; i < NT; i++) request_v_tile(rows_from(first_key(i)), vl.from + 2 * H, ld, &slab[w][i * V_TILE]);
#pragma unroll
    for (int i = 0; i < QB * 64 / 4 / (64 * NW); i++) reinterpret_cast<v4i *>(&so[0][0])[i * 64 * NW + tid] = v4i{P16_HALF, P16_HALF, P16_HALF, P16_HALF};      // used after two barriers

    float sc[NT][16];                                             // scores / 128, then exponentials
    const float m_unit = m_sc * SCORE_UNIT;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < NT; i++) {
        const int j0 = first_key(i);
        if (j0 < n) {
            v16i acc;
#pragma unroll
            for (int e = 0; e < 16; e++) acc[e] = 0;
#pragma unroll
            for (int ks = 0; ks < 2; ks++) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(kf[i % K_AHEAD][ks], qf[ks], acc, 0, 0, 0);
            if (j0 + 32 <= n) {
#pragma unroll
                for (int e = 0; e < 16; e++) sc[i][e] = (float)acc[e] * m_unit;
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) sc[i][e] = j0 + 8 * (e >> 2) + 4 * g + (e & 3) < n ? (float)acc[e] * m_unit : -INFINITY;
            }
#pragma unroll
            for (int e = 0; e < 16; e++) mx = __builtin_fmaxf(mx, sc[i][e]);
        }
        if (i + K_AHEAD < NT) request_keys(i + K_AHEAD);
    }
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) smax[w][r] = mx;
    if (NW == 4 || tid < 256) exp_table[tid] = table_entry;
    wait_vm<0>();                                                 // the wave's V tiles are in its slab
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NW; u++) mx = __builtin_fmaxf(mx, smax[u][r]);

    double part = 0.0;
#pragma unroll
    for (int i = 0; i < NT; i++)
        if (first_key(i) < n) {
#pragma unroll
            for (int e = 0; e < 16; e++) {
                sc[i][e] = exp_below(sc[i][e], mx, exp_table);
                part += (double)sc[i][e];
            }
        }
    part += __shfl_xor(part, 32, 64);
    if (g == 0) ssum[w][r] = part;
    __syncthreads();
    double total = ssum[0][r];
#pragma unroll
    for (int u = 1; u < NW; u++) total += ssum[u][r];
    const float S = (float)total;
    const float rS = __fdiv_rn(1.0f, S);

    // the operands of all tiles take the exponentials' registers; one channel block at a time halves the accumulators
    v8h hi[NT][2], lo[NT][2];
#pragma unroll
    for (int i = 0; i < NT; i++)
        if (first_key(i) < n) p16_split(sc[i], rS, hi[i], lo[i]);
    if (w * 32 < n) {
#pragma unroll
        for (int cb = 0; cb < 2; cb++) {
            v16f o[2];
#pragma unroll
            for (int k = 0; k < 2; k++)
#pragma unroll
                for (int e = 0; e < 16; e++) o[k][e] = __int_as_float(opaque_zero());
#pragma unroll
            for (int i = 0; i < NT; i++)
                if (first_key(i) < n) {
                    const v4i vf = read_vt(&slab[w][i * V_TILE], vl.at, cb);
#pragma unroll
                    for (int u = 0; u < 2; u++) {
                        const v8h v = codes_to_half(vf[2 * u], vf[2 * u + 1]);
                        o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hi[i][u], v, o[0], 0, 0, 0);
                        o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(lo[i][u], v, o[1], 0, 0, 0);
                    }
                }
#pragma unroll
            for (int e = 0; e < 16; e++)
                atomicAdd(&so[8 * (e >> 2) + 4 * g + (e & 3)][cb * 32 + r], ((unsigned)(int)(o[0][e] * 0x1p14f) << 10) + (unsigned)(int)(o[1][e] * 0x1p24f));
        }
    }
    __syncthreads();

    // the block's sums: scaled back (exact) and rounded once to binary32
    constexpr int CPT = 32 / NW;
    const int query = tid / (64 / CPT), c0 = tid % (64 / CPT) * CPT;
    if (q0 + query >= n) return;
    int pk[CPT / 4];
#pragma unroll
    for (int d = 0; d < CPT / 4; d++) {
        float codes[4];
#pragma unroll
        for (int e = 0; e < 4; e++) codes[e] = code_bits((float)((double)(int)so[query][c0 + 4 * d + e] - P16_HALF) * 0x1p-24f * m_ctx);
        pk[d] = pack_codes(codes[0], codes[1], codes[2], codes[3]);
    }
    int8_t *dst = ctx + (size_t)(sq.t0 + q0 + query) * H + head * 64 + c0;
    store_codes(dst, pk);
}

// Any length: three sweeps (as attention_i8_long_kernel), digit planes.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void
attention_i8_p16_long_kernel(const int8_t *__restrict__ qkv, const int *__restrict__ cu, int max_len, int H, float m_sc, float m_ctx,
                             int8_t *__restrict__ ctx)
{
    constexpr int NW = 4;
    __shared__ __attribute__((aligned(16))) int8_t vt[NW][64 * VT_STRIDE_I8];
    __shared__ long long so[2][QB][32];
    __shared__ float smax[NW][QB];
    __shared__ double ssum[NW][QB];
    __shared__ ExpTable exp_table;

    const int nqb = (max_len + QB - 1) / QB, heads = H >> 6;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int seq = item / (nqb * heads), head = (item / nqb) % heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int q0 = (item % nqb) * QB;
    if (q0 >= sq.n) return;
    const int n = sq.n;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), r = lane & 31, g = lane >> 5;
    const unsigned ld = 3u * (unsigned)H;
    const int8_t *base = qkv + (size_t)sq.t0 * ld + head * 64;
    const int8_t *vp = base + 2 * H;
    const uint64_t table_entry = EXP2_TABLE[tid & 255];

    const int qrow = min(q0 + r, n - 1);
    v4i qf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ks++) qf[ks] = *reinterpret_cast<const v4i *>(base + (unsigned)qrow * ld + ks * 32 + g * 16);
#pragma unroll
    for (int i = 0; i < 2 * QB * 32 / (64 * NW); i++) (&so[0][0][0])[i * 64 * NW + tid] = 0;      // used after two barriers

    float sc[16];
    float mx = -INFINITY;
    for (int j0 = w * 32; j0 < n; j0 += 32 * NW) {
        score_tile_i8(base, ld, H, j0, n, r, g, qf, m_sc, sc);
#pragma unroll
        for (int e = 0; e < 16; e++) mx = __builtin_fmaxf(mx, sc[e]);
    }
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) smax[w][r] = mx;
    exp_table[tid] = table_entry;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NW; u++) mx = __builtin_fmaxf(mx, smax[u][r]);

    double part = 0.0;
    for (int j0 = w * 32; j0 < n; j0 += 32 * NW) {
        score_tile_i8(base, ld, H, j0, n, r, g, qf, m_sc, sc);
#pragma unroll
        for (int e = 0; e < 16; e++) part += (double)exp_nonpos(sc[e] - mx, exp_table);
    }
    part += __shfl_xor(part, 32, 64);
    if (g == 0) ssum[w][r] = part;
    __syncthreads();
    double total = ssum[0][r];
#pragma unroll
    for (int u = 1; u < NW; u++) total += ssum[u][r];
    const float S = (float)total;
    const float rS = __fdiv_rn(1.0f, S);

    v16i o[2][4];                                         // [channel block][digit plane]
    int vsum[2] = {0, 0};
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int e = 0; e < 16; e++) o[cb][k][e] = 0;
    for (int j0 = w * 32; j0 < n; j0 += 32 * NW) {
        score_tile_i8(base, ld, H, j0, n, r, g, qf, m_sc, sc);
        // the slab is written and read by this wave only, in program order
        __builtin_amdgcn_wave_barrier();
        stage_vt_i8(vp, ld, j0, n, lane, vt[w]);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int e = 0; e < 16; e++) sc[e] = exp_nonpos(sc[e] - mx, exp_table);
        v4i pf[4];
        p16_digits(sc, rS, pf);
        p16_mfma(pf, vt[w], 0, r, g, o[0], vsum[0]);
        p16_mfma(pf, vt[w], 1, r, g, o[1], vsum[1]);
    }
    p16_add(o[0], vsum[0], so[0], r, g);
    p16_add(o[1], vsum[1], so[1], r, g);
    __syncthreads();
    p16_store(so, m_ctx, ctx + (size_t)(sq.t0 + q0) * H + head * 64, H, n - q0, tid);
}

__device__ __forceinline__ void score_tile_f16(const __half *base, unsigned ld, int H, int j0, int n, int r, int g,
                                               const v8h (&qf)[4], float scale, float (&sc)[16])
{
    const __half *kp = base + (unsigned)min(j0 + r, n - 1) * ld + H;
    v16f acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.0f;
#pragma unroll
    for (int ks = 0; ks < 4; ks++)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const v8h *>(kp + ks * 16 + g * 8), qf[ks], acc, 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 16; e++) {
        const int key = j0 + 8 * (e >> 2) + 4 * g + (e & 3);
        sc[e] = key < n ? acc[e] * scale : -INFINITY;
    }
}

__global__ __launch_bounds__(256) void attention_f16_long_kernel(const __half *__restrict__ qkv, const int *__restrict__ cu,
                                                                 int max_len, int H, float scale, __half *__restrict__ ctx,
                                                                 float *__restrict__ p_absmax)
{
    __shared__ __attribute__((aligned(1024))) char vt[4][V_TILE_F16];
    __shared__ __attribute__((aligned(16))) float so[4][QB][64];
    __shared__ float smax[4][QB];
    __shared__ float ssum[4][QB];

    const int nqb = (max_len + QB - 1) / QB, heads = H >> 6;
    const int item = xcd_contiguous(blockIdx.x, gridDim.x);
    const int seq = item / (nqb * heads), head = (item / nqb) % heads;
    const SeqInfo sq = seq_info(cu, seq, max_len);
    const int q0 = (item % nqb) * QB;
    if (q0 >= sq.n) return;
    const int n = sq.n;
    const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), r = lane & 31, g = lane >> 5;
    const unsigned ld = 3u * (unsigned)H;
    const __half *base = qkv + (size_t)sq.t0 * ld + head * 64;

    const int qrow = min(q0 + r, n - 1);
    v8h qf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) qf[ks] = *reinterpret_cast<const v8h *>(base + (unsigned)qrow * ld + ks * 16 + g * 8);

    float sc[16];
    float mx = -INFINITY;
    for (int j0 = w * 32; j0 < n; j0 += 128) {
        score_tile_f16(base, ld, H, j0, n, r, g, qf, scale, sc);
#pragma unroll
        for (int e = 0; e < 16; e++) mx = __builtin_fmaxf(mx, sc[e]);
    }
    mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (g == 0) smax[w][r] = mx;
    __syncthreads();
    mx = __builtin_fmaxf(__builtin_fmaxf(smax[0][r], smax[1][r]), __builtin_fmaxf(smax[2][r], smax[3][r]));

    float part = 0.0f;
    for (int j0 = w * 32; j0 < n; j0 += 128) {
        score_tile_f16(base, ld, H, j0, n, r, g, qf, scale, sc);
#pragma unroll
        for (int e = 0; e < 16; e++) part += __builtin_amdgcn_exp2f((sc[e] - mx) * 1.44269504088896341f);
    }
    part += __shfl_xor(part, 32, 64);
    if (g == 0) ssum[w][r] = part;
    __syncthreads();
    const float S = ((ssum[0][r] + ssum[1][r]) + ssum[2][r]) + ssum[3][r];
    const float rS = __fdiv_rn(1.0f, S);
    if (p_absmax && w == 0 && g == 0 && q0 + r < n)
        atomicMax(reinterpret_cast<int *>(p_absmax), __float_as_int((float)(_Float16)rS));

    v16f o[2];
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) o[cb][e] = 0.0f;
    const VLaneF16 vl(ld, lane);
    for (int j0 = w * 32; j0 < n; j0 += 128) {
        const auto rows = strip_rows(base, ld, head, j0, n);
        v4i d[4];
#pragma unroll
        for (int u = 0; u < 4; u++) d[u] = __builtin_amdgcn_raw_buffer_load_b128(rows, vl.from + 4 * H + u * 16 * ld, 0, 0);
        score_tile_f16(base, ld, H, j0, n, r, g, qf, scale, sc);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 4; u++) *reinterpret_cast<v4i *>(&vt[w][u * 1024 + lane * 16]) = d[u];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int hf = 0; hf < 2; hf++) {
            v8h pf;
#pragma unroll
            for (int e = 0; e < 8; e++)
                pf[e] = to_half(__builtin_amdgcn_exp2f((sc[8 * hf + e] - mx) * 1.44269504088896341f) * rS);
#pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                const v8h vf = read_vt_f16(vt[w], vl.at, hf, cb);
                o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(pf, vf, o[cb], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int cb = 0; cb < 2; cb++)
#pragma unroll
        for (int e = 0; e < 16; e++) so[w][8 * (e >> 2) + 4 * g + (e & 3)][cb * 32 + r] = o[cb][e];
    __syncthreads();

    const int query = tid >> 3, c0 = (tid & 7) * 8;
    if (q0 + query < n) {
        v8h outv;
#pragma unroll
        for (int e = 0; e < 8; e++)
            outv[e] = to_half(((so[0][query][c0 + e] + so[1][query][c0 + e]) + so[2][query][c0 + e]) + so[3][query][c0 + e]);
        *reinterpret_cast<v8h *>(ctx + (size_t)(sq.t0 + q0 + query) * H + head * 64 + c0) = outv;
    }
}

}  // namespace

// One or two key tiles and blocks enough for the chip: no waves without a tile.  Forward, us, four waves / as many as tiles: BERT-base Fully-Quant 512 x 8
// 878 / 738, 256 x 16 782 / 720, 128 x 32 734 / 715, 24 x 48 413 / 413, BERT-large 128 x 32 2075 / 2002; FP16 512 x 8 1351 / 1299, 256 x 16 1264 / 1262, 128 x 32
// 1258 / 1231, Quant-FFN-Only 256 x 16 968 / 921; with fewer blocks Fully-Quant 16 x 24 345 / 345, 1 x 19 241 / 242, BERT-large 64 x 32 1256 / 1275.  (The binary16
// softmax output keeps four waves: 256 x 16 774 / 786.)
// Blocks that ask for weights beside them change nothing about it, us, three encoders in turn, four waves / as many as tiles: BERT-base Fully-Quant 64 x 16
// 400 / 395, 128 x 16 545 / 511, 80 x 32 560 / 537, 40 x 48 535 / 517, FP16 128 x 16 834 / 788, Quant-FFN-Only 128 x 16 676 / 634, BERT-large 100 x 16
// 1327 / 1255.
static int waves_of(unsigned blocks, int max_len) { return blocks < 768 || max_len > 64 ? 4 : max_len <= 32 ? 1 : 2; }
// blocks that ask with as many threads as blocks of four waves would
static FetchAhead fetch_with(FetchAhead fetch, int waves)
{
    fetch.blocks *= 4 / waves;
    return fetch;
}

// 513 to 2048 tokens: eight waves, a wave's NT key tiles as few as the longest sequence allows (registers and LDS, and with
// them the blocks per CU, follow NT)
template <bool PU>
static void launch_attention_i8_8waves(const int8_t *qkv, const int *cu, int max_len, int H, float m_sc, float inv_sp, float m_ctx,
                                       int8_t *ctx, dim3 grid, hipStream_t st, const Timing *tm)
{
    const unsigned by_nqb = divisor(grid.x + 1u, (max_len + QB - 1) / QB), by_heads = divisor(grid.x, H / 64);
    auto go = [&](auto kern) {
        launch_kernel(kern, grid, dim3(512), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, inv_sp, m_ctx, ctx,
                      (unsigned long long *)nullptr, NoFetch());
    };
    switch ((max_len + 255) / 256) {
    case 3: return go(attention_i8_kernel<3, PU, false, 8>);
    case 4: return go(attention_i8_kernel<4, PU, false, 8>);
    case 5: return go(attention_i8_kernel<5, PU, false, 8>);
    case 6: return go(attention_i8_kernel<6, PU, false, 8>);
    default: return go(attention_i8_kernel<8, PU, false, 8>);
    }
}

template <bool PU, bool HIST>
static void launch_attention_i8_variant(const int8_t *qkv, const int *cu, int B, int max_len, int H, int heads, float m_sc,
                                        float inv_sp, float m_ctx, int8_t *ctx, unsigned long long *p_hist, hipStream_t st,
                                        const Timing *tm, const FetchAhead *fetch)
{
    dim3 grid((unsigned)((max_len + QB - 1) / QB) * heads * B);
    const unsigned by_nqb = divisor(grid.x + 1u, (max_len + QB - 1) / QB), by_heads = divisor(grid.x, H / 64);
    if constexpr (!HIST) {
        auto go = [&](auto kern, int waves, unsigned more, auto what) {
            launch_kernel(kern, dim3(grid.x + more), dim3(64 * waves), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, inv_sp, m_ctx, ctx,
                          p_hist, what);
        };
        const int waves = waves_of(grid.x, max_len);
        if (fetch && max_len <= ATTENTION_FETCH_MAX_LEN) {
            const FetchAhead f = fetch_with(*fetch, waves);
            if (waves == 1) return go(attention_i8_kernel<1, PU, HIST, 1, true>, 1, f.blocks, f);
            if (waves == 2) return go(attention_i8_kernel<1, PU, HIST, 2, true>, 2, f.blocks, f);
            if (max_len <= 128) return go(attention_i8_kernel<1, PU, HIST, 4, true>, 4, f.blocks, f);
            return go(attention_i8_kernel<2, PU, HIST, 4, true>, 4, f.blocks, f);
        }
        if (waves == 1) return go(attention_i8_kernel<1, PU, HIST, 1>, 1, 0, NoFetch());
        if (waves == 2) return go(attention_i8_kernel<1, PU, HIST, 2>, 2, 0, NoFetch());
    }
    if (max_len <= 128)
        launch_kernel(attention_i8_kernel<1, PU, HIST>, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, inv_sp, m_ctx, ctx, p_hist, NoFetch());
    else if (max_len <= 256)
        launch_kernel(attention_i8_kernel<2, PU, HIST>, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, inv_sp, m_ctx, ctx, p_hist, NoFetch());
    else if (max_len <= 384)
        launch_kernel(attention_i8_kernel<3, PU, HIST>, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, inv_sp, m_ctx, ctx, p_hist, NoFetch());
    else if (max_len <= ONE_PASS_MAX_LEN)
        launch_kernel(attention_i8_kernel<4, PU, HIST>, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, inv_sp, m_ctx, ctx, p_hist, NoFetch());
    else if (!HIST && max_len <= 8 * 256)
        launch_attention_i8_8waves<PU>(qkv, cu, max_len, H, m_sc, inv_sp, m_ctx, ctx, grid, st, tm);
    else
        launch_kernel(attention_i8_long_kernel<PU, HIST>, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, m_sc, inv_sp, m_ctx, ctx, p_hist);
}

hipError_t launch_attention_i8(const int8_t *qkv, const int *cu, int B, int max_len, int H, int heads, float m_sc,
                               float inv_sp, float m_ctx, bool p_unsigned, int8_t *ctx, unsigned long long *p_hist,
                               hipStream_t st, const Timing *tm, const FetchAhead *fetch)
{
    if (p_unsigned) {
        if (p_hist) launch_attention_i8_variant<true, true>(qkv, cu, B, max_len, H, heads, m_sc, inv_sp, m_ctx, ctx, p_hist, st, tm, nullptr);
        else launch_attention_i8_variant<true, false>(qkv, cu, B, max_len, H, heads, m_sc, inv_sp, m_ctx, ctx, p_hist, st, tm, fetch);
    } else {
        if (p_hist) launch_attention_i8_variant<false, true>(qkv, cu, B, max_len, H, heads, m_sc, inv_sp, m_ctx, ctx, p_hist, st, tm, nullptr);
        else launch_attention_i8_variant<false, false>(qkv, cu, B, max_len, H, heads, m_sc, inv_sp, m_ctx, ctx, p_hist, st, tm, fetch);
    }
    return hipGetLastError();
}

template <int QT, bool PU, int STAGE>
static hipError_t launch_qkv_attention_i8_stages(const int8_t *x, const int8_t *w_qkv, const float *m, const float *b, const int *cu,
                                                  int B, int max_len, int H, float m_sc, float inv_sp, float m_ctx, int8_t *ctx,
                                                  hipStream_t st, const Timing *tm)
{
    typedef QkvTile<QT, STAGE> Tile;
    const size_t lds = Tile::RING_BYTES + (Tile::LATE ? 0 : 2 * 192 * sizeof(float) + sizeof(ExpTable));
    if (lds > 64 * 1024) {
        static std::atomic<bool> attr_set{false};
        if (!attr_set.load(std::memory_order_acquire)) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(qkv_attention_i8_kernel<QT, PU, STAGE>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            attr_set.store(true, std::memory_order_release);
        }
    }
    launch_kernel(qkv_attention_i8_kernel<QT, PU, STAGE>, dim3((unsigned)(B * (H / 64))), dim3(256), lds, st, tm, (const char *)x,
                  (const char *)w_qkv, m, b, cu, max_len, H, m_sc, inv_sp, m_ctx, ctx);
    return hipGetLastError();
}

template <int QT, bool PU>
static hipError_t launch_qkv_attention_i8_variant(const int8_t *x, const int8_t *w_qkv, const float *m, const float *b, const int *cu,
                                                  int B, int max_len, int H, float m_sc, float inv_sp, float m_ctx, int8_t *ctx,
                                                  hipStream_t st, const Timing *tm)
{
    if constexpr (QT == 1)
        if (H % 128 == 0) return launch_qkv_attention_i8_stages<QT, PU, 128>(x, w_qkv, m, b, cu, B, max_len, H, m_sc, inv_sp, m_ctx, ctx, st, tm);
    return launch_qkv_attention_i8_stages<QT, PU, 64>(x, w_qkv, m, b, cu, B, max_len, H, m_sc, inv_sp, m_ctx, ctx, st, tm);
}

hipError_t launch_qkv_attention_i8(const int8_t *x, const int8_t *w_qkv, const float *m, const float *b, const int *cu, int B,
                                   int max_len, int H, float m_sc, float inv_sp, float m_ctx, bool p_unsigned, int8_t *ctx,
                                   hipStream_t st, const Timing *tm)
{
    if (max_len > 256 || H % 64 || B <= 0) return hipErrorInvalidValue;
    if (max_len <= 128)
        return p_unsigned ? launch_qkv_attention_i8_variant<1, true>(x, w_qkv, m, b, cu, B, max_len, H, m_sc, inv_sp, m_ctx, ctx, st, tm)
                          : launch_qkv_attention_i8_variant<1, false>(x, w_qkv, m, b, cu, B, max_len, H, m_sc, inv_sp, m_ctx, ctx, st, tm);
    return p_unsigned ? launch_qkv_attention_i8_variant<2, true>(x, w_qkv, m, b, cu, B, max_len, H, m_sc, inv_sp, m_ctx, ctx, st, tm)
                      : launch_qkv_attention_i8_variant<2, false>(x, w_qkv, m, b, cu, B, max_len, H, m_sc, inv_sp, m_ctx, ctx, st, tm);
}

hipError_t launch_qkv_attention_i8_packed(const int8_t *x, const int8_t *w_packed, const float *m, const float *b, const int *cu, int B,
                                          int max_len, int H, float m_sc, float inv_sp, float m_ctx, bool p_unsigned, int8_t *ctx,
                                          hipStream_t st, const Timing *tm, const FetchAhead *fetch)
{
    if (!qkv_attention_packed(true, w_packed, max_len, H) || B <= 0) return hipErrorNotSupported;
    auto go = [&](auto kern, unsigned more, auto what) {
        launch_kernel(kern, dim3((unsigned)(B * (H / 64)) + more), dim3(256), stream_ring_bytes<false, 8, 2>() + sizeof(ExpTable), st, tm, (const char *)x,
                      (const char *)w_packed, m, b, cu, max_len, H, B * (H / 64), divisor((unsigned)B * (H / 64), H / 64), m_sc, inv_sp, m_ctx, ctx, what);
        return hipGetLastError();
    };
    if (fetch)
        return p_unsigned ? go(qkv_attention_i8_packed_kernel<true, 2, true>, fetch->blocks, *fetch)
                          : go(qkv_attention_i8_packed_kernel<false, 2, true>, fetch->blocks, *fetch);
    return p_unsigned ? go(qkv_attention_i8_packed_kernel<true, 2, false>, 0, NoFetch()) : go(qkv_attention_i8_packed_kernel<false, 2, false>, 0, NoFetch());
}

hipError_t launch_qkv_attention_f16(const __half *x, const __half *w_qkv, const __half *w_packed, const float *bias, const int *cu, int B,
                                    int max_len, int H, float scale, __half *ctx, hipStream_t st, const Timing *tm, const FetchAhead *fetch)
{
    if (max_len > 256 || H % 64 || B <= 0) return hipErrorInvalidValue;
    const bool packed = qkv_attention_packed(false, w_packed, max_len, H);
    if (!packed && !w_qkv) return hipErrorNotSupported;
    const dim3 grid((unsigned)(B * (H / 64)));
    auto go = [&](auto kern, size_t lds, std::atomic<bool> &attr_set, unsigned more, auto what) {
        if (!attr_set.load(std::memory_order_acquire)) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            attr_set.store(true, std::memory_order_release);
        }
        launch_kernel(kern, dim3(grid.x + more), dim3(256), lds, st, tm, (const char *)x, (const char *)(packed ? w_packed : w_qkv), bias, cu, max_len, H, (int)grid.x, divisor(grid.x, H / 64), scale, ctx, what);
        return hipGetLastError();
    };
    static std::atomic<bool> attr_set[4];
    constexpr size_t tab = 192 * sizeof(float);
    constexpr auto qkv_bytes = [](size_t BM) { return 2 * BM * 144 + 64 * (2 * BM + 8); };
    constexpr size_t packed_lds = std::max<size_t>(qkv_bytes(128), QKV_F16_PACKED_RING) + tab;
    if (packed && fetch) return go(qkv_attention_f16_kernel<1, 128, true, true>, packed_lds, attr_set[3], fetch->blocks, *fetch);
    if (packed) return go(qkv_attention_f16_kernel<1, 128, true>, packed_lds, attr_set[1], 0, NoFetch());
    if (max_len > 128) return go(qkv_attention_f16_kernel<2, 64, false>, std::max<size_t>(qkv_bytes(256), QkvTile<2, 64>::RING_BYTES) + tab, attr_set[2], 0, NoFetch());
    return go(qkv_attention_f16_kernel<1, 128, false>, QkvTile<1, 128>::RING_BYTES, attr_set[0], 0, NoFetch());
}

hipError_t launch_attention_i8_p16(const int8_t *qkv, const int *cu, int B, int max_len, int H, int heads, float m_sc,
                                   float m_ctx, int8_t *ctx, hipStream_t st, const Timing *tm, const FetchAhead *fetch)
{
    dim3 grid((unsigned)((max_len + QB - 1) / QB) * heads * B);
    const unsigned by_nqb = divisor(grid.x + 1u, (max_len + QB - 1) / QB), by_heads = divisor(grid.x, H / 64);
    auto go = [&](auto kern, int waves, unsigned more, auto what) {
        launch_kernel(kern, dim3(grid.x + more), dim3(64 * waves), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, m_sc, m_ctx, ctx, what);
    };
    if (fetch && max_len <= 128) go(attention_i8_p16_kernel<1, 4, true>, 4, fetch->blocks, *fetch);
    else if (fetch && max_len <= ATTENTION_FETCH_MAX_LEN) go(attention_i8_p16_kernel<2, 4, true>, 4, fetch->blocks, *fetch);
    else if (max_len <= 128) go(attention_i8_p16_kernel<1>, 4, 0, NoFetch());
    else if (max_len <= 256) go(attention_i8_p16_kernel<2>, 4, 0, NoFetch());
    else if (max_len <= 384) go(attention_i8_p16_kernel<3>, 4, 0, NoFetch());
    else if (max_len <= ONE_PASS_MAX_LEN) go(attention_i8_p16_kernel<4>, 4, 0, NoFetch());
    else if (max_len <= 1024) go(attention_i8_p16_kernel<4, 8>, 8, 0, NoFetch());
    else if (max_len <= 1536) go(attention_i8_p16_kernel<6, 8>, 8, 0, NoFetch());      // (beyond, V and the sums do not fit LDS together)
    else launch_kernel(attention_i8_p16_long_kernel, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, m_sc, m_ctx, ctx);
    return hipGetLastError();
}

hipError_t launch_attention_f16(const __half *qkv, const int *cu, int B, int max_len, int H, int heads, float scale,
                                __half *ctx, float *p_absmax, hipStream_t st, const Timing *tm, const FetchAhead *fetch)
{
    dim3 grid((unsigned)((max_len + QB - 1) / QB) * heads * B);
    const unsigned by_nqb = divisor(grid.x + 1u, (max_len + QB - 1) / QB), by_heads = divisor(grid.x, H / 64);
    const int few = waves_of(grid.x, max_len);
    auto go = [&](auto kern, int waves = 4) {
        launch_kernel(kern, grid, dim3(64 * waves), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, scale, ctx, p_absmax, NoFetch());
    };
    if (fetch && max_len <= ATTENTION_FETCH_MAX_LEN) {
        const FetchAhead f = fetch_with(*fetch, few);
        auto with = [&](auto kern) {
            launch_kernel(kern, dim3(grid.x + f.blocks), dim3(64 * few), 0, st, tm, qkv, cu, max_len, H, (int)grid.x, by_nqb, by_heads, scale, ctx, p_absmax, f);
        };
        if (few == 1) with(attention_f16_kernel<1, true, 1>);
        else if (few == 2) with(attention_f16_kernel<1, true, 2>);
        else if (max_len <= 128) with(attention_f16_kernel<1, true>);
        else with(attention_f16_kernel<2, true>);
        return hipGetLastError();
    }
    if (few < 4) {
        if (few == 1) go(attention_f16_kernel<1, false, 1>, 1); else go(attention_f16_kernel<1, false, 2>, 2);
        return hipGetLastError();
    }
    switch ((max_len + 127) / 128) {                              // key tiles per wave
    case 1: go(attention_f16_kernel<1>); break;
    case 2: go(attention_f16_kernel<2>); break;
    case 3: go(attention_f16_kernel<3>); break;
    case 4: go(attention_f16_kernel<4>); break;
    case 5: case 6: go(attention_f16_kernel<6>); break;
    case 7: case 8: go(attention_f16_kernel<8>); break;
    case 9: case 10: go(attention_f16_kernel<10>); break;
    case 11: case 12: go(attention_f16_kernel<12>); break;
    case 13: case 14: case 15: case 16: go(attention_f16_kernel<16>); break;
    default: launch_kernel(attention_f16_long_kernel, grid, dim3(256), 0, st, tm, qkv, cu, max_len, H, scale, ctx, p_absmax);
    }
    return hipGetLastError();
}

}  // namespace samp
