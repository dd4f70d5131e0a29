// INT8 and FP16 "NT" GEMMs on gfx950 matrix cores with fused epilogues (Section 3.2: the four
// GEMMs of a layer run as INT8 with int32 accumulation or as FP16; quantise / dequantise, bias and
// GELU are fused into the producing kernel so that only int8 or fp16 tensors reach memory).
//
//   C[m,n] = sum_k A[m,k] * W[n,k]      A [M,K] and W [N,K] both K-contiguous.
//
// Byte geometry is the same for both element types: one MFMA consumes 32 bytes of K per row
// (v_mfma_i32_32x32x32_i8: 32 int8; v_mfma_f32_32x32x16_f16: 16 fp16), 16 bytes per lane.  The
// weight rows are the MFMA's first operand and the activation rows its second, so that in the
// 32x32 result a lane owns ONE token row and four consecutive output channels per register
// group -- which is what the per-channel epilogue tables and the packed int8/fp16 stores want.
//
// A block of 4 waves (2 x 2) computes a (64 TM) x (64 TN) tile, each wave (32 TM) x (32 TN).
// K is consumed 64 bytes per stage through an NSTAGE-deep ring of LDS tiles that is filled by
// direct global->LDS loads (global_load_lds_dwordx4, no register staging), so that NSTAGE-1
// stages of loads are in flight while one is being multiplied: the memory round trip of a step
// is several times longer than its MFMA work, and only a deep ring hides it.  A direct load puts
// lane i's 16 bytes at LDS position i of a 1 KiB run; the XOR swizzle that keeps the operand
// fetches (ds_read_b128) conflict-free is therefore applied to the global address instead.
// Work-groups are renumbered so that each XCD (own L2) owns a contiguous range of tiles.
// What the first loads need comes first among a kernel's arguments: the launch puts 14 dwords of them into registers (up to the first struct),
// the rest is loaded.  A load of arguments costs a launch 0.2 to 0.4 us, which is what a small forward consists of (build.py has the figures).
// That is the row-major kernels.  An encoder keeps its weights packed as well and runs most of its GEMMs on those (gemm_nt_stream_kernel):
// the row-major ones are left with few rows (gemm_rules.h), INT8 rows that are no whole pairs of 128-byte stages (widths 384, 640, 896, ...), GELU
// without a table, the step entries, forced configurations and encoders whose arena has no room for packed copies.
#include "samp_common.h"
#include "mfma_tile.h"
#include "ln_wave.h"
#include "gemm_rules.h"
#include "divisor.h"

#include <atomic>
#include <type_traits>
#include <utility>

namespace samp {
namespace {

// Where tile `tile` lies when the row tiles of a channel tile come one after the other.  by_m: divisor() of the row tiles that the host counted; a ragged
// batch may have fewer.  Forward, us, three encoders in turn, with divisions in the GEMM and attention kernels / with these: BERT-base 7 x 61 354 / 349,
// 16 x 128 529 / 523, 32 x 128 685 / 676, 33 x 40..301 1233 / 1216.
struct TileAt { int m, n; };
__device__ __forceinline__ TileAt tile_channels_first(int tile, int tiles_m, int host_tiles_m, unsigned by_m)
{
    const int n = (int)over(tile, tiles_m == host_tiles_m ? by_m : 1u, tiles_m);
    return {tile - n * tiles_m, n};
}
__device__ __forceinline__ TileAt tile_rows_first(int tile, int tiles_n, unsigned by_n)
{
    const int m = (int)over(tile, by_n, tiles_n);
    return {m, tile - m * tiles_n};
}

struct I8 {
    typedef v16i acc_t;
    static constexpr int ELEM = 1;
    __device__ static __forceinline__ acc_t mma(v4i a, v4i b, acc_t c)
    { return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0); }
};
struct F16 {
    typedef v16f acc_t;
    static constexpr int ELEM = 2;
    __device__ static __forceinline__ acc_t mma(v4i a, v4i b, acc_t c)
    { return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0); }
};

// ---- epilogues -------------------------------------------------------------------------------
// A 32x32 result tile gives each lane 16 accumulators: register 4q+t holds channel
// n_tile + 8q + 4g + t (g = lane >> 5) of the lane's token row.  tile() turns them into the four
// packed output groups of the lane (q = 0..3).  The per-channel tables of the block's BN channels
// are copied into LDS when the block starts (load_tables), so that their memory latency is hidden
// behind the main loop.  load_tab() fetches the table entries of one 32-channel tile from there into registers
// (a Tab) and tile() works from those: the kernels request the Tab of the next tile before they work on the
// current one, because a wave that waits for every LDS read where it needs it spends more time in the
// epilogue of a small problem than in its main loop.
struct EpiRawI32 {                                // test hook: the exact int32 accumulators
    int32_t *out; int N;
    static constexpr int OUT_BYTES = 4;
    static constexpr bool STAGED = false;
    static constexpr int NTAB = 0;
    struct Tab {};
    __device__ __forceinline__ void load_tables(float *, int, int, int, int) const {}
    __device__ __forceinline__ void load_tables_direct(float *, int, int, int, int, int) const {}
    __device__ __forceinline__ Tab load_tab(const float *, int, int, int) const { return {}; }
    __device__ __forceinline__ void direct(int row, int n, int a0, int a1, int a2, int a3) const
    { *reinterpret_cast<v4i *>(out + (size_t)row * N + n) = v4i{a0, a1, a2, a3}; }
};

__device__ __forceinline__ void copy_table(float *dst, const float *src, int n0, int bn, int tid, int nthreads)
{
    for (int c = tid * 4; c < bn; c += nthreads * 4)
        *reinterpret_cast<v4f *>(dst + c) = src ? *reinterpret_cast<const v4f *>(src + n0 + c) : v4f{0.f, 0.f, 0.f, 0.f};
}

// The same copies as direct loads, which the caller waits for (vmcnt) before its next barrier: `words` dwords, 64 per
// instruction, the instructions dealt out over the waves.
__device__ __forceinline__ void copy_direct(void *dst, const void *src, int words, int wave, int nwaves, int lane)
{
    const auto from = buffer_of(src);
    for (int i = wave * 64; i < words; i += nwaves * 64)             // wave-uniform
        if (i + lane < words)
            buffer_to_lds32(from, 4 * (i + lane), (int *)dst + i);
}
__device__ __forceinline__ void copy_table_direct(float *dst, const float *src, int n0, int bn, int wave, int nwaves, int lane)
{
    if (src) copy_direct(dst, src + n0, bn, wave, nwaves, lane);
    else
        for (int c = wave * 64 + lane; c < bn; c += nwaves * 64) dst[c] = 0.0f;
}

// the multiplier and offset vectors of one 32-channel tile: group q holds channels n_loc + 8q + 4g .. + 3
template <class Tab> __device__ __forceinline__ Tab load_tab_mb(const float *tab, int bn, int n_loc, int g)
{
    Tab t;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int n = n_loc + 8 * q + 4 * g;
        t.m[q] = *reinterpret_cast<const v4f *>(tab + n);
        t.b[q] = *reinterpret_cast<const v4f *>(tab + bn + n);
    }
    return t;
}

struct EpiRequant {                               // code = rne(fmaf(acc, m[n], b[n]))
    const float *m, *b;
    __device__ __forceinline__ const float *offsets() const { return b; }
    __device__ __forceinline__ void load_lut_direct(v2i *, int, int, int) const {}
    static constexpr int OUT_BYTES = 1;
    static constexpr bool STAGED = true;
    static constexpr int NTAB = 2;
    typedef int pack_t;
    __device__ __forceinline__ void load_tables(float *tab, int n0, int bn, int tid, int nthreads) const
    { copy_table(tab, m, n0, bn, tid, nthreads); copy_table(tab + bn, b, n0, bn, tid, nthreads); }
    __device__ __forceinline__ void load_tables_direct(float *tab, int n0, int bn, int wave, int nwaves, int lane) const
    { copy_table_direct(tab, m, n0, bn, wave, nwaves, lane); copy_table_direct(tab + bn, b, n0, bn, wave, nwaves, lane); }
    // four consecutive channels of one token
    __device__ __forceinline__ int four(const v4i &acc, const float *tab, int bn, int n) const
    {
        const v4f mm = *reinterpret_cast<const v4f *>(tab + n), bb = *reinterpret_cast<const v4f *>(tab + bn + n);
        return pack_codes(code_bits(__builtin_fmaf((float)acc.x, mm.x, bb.x)), code_bits(__builtin_fmaf((float)acc.y, mm.y, bb.y)),
                          code_bits(__builtin_fmaf((float)acc.z, mm.z, bb.z)), code_bits(__builtin_fmaf((float)acc.w, mm.w, bb.w)));
    }
    struct Tab { v4f m[4], b[4]; };
    __device__ __forceinline__ Tab load_tab(const float *tab, int bn, int n_loc, int g) const { return load_tab_mb<Tab>(tab, bn, n_loc, g); }
    __device__ __forceinline__ void tile(const v16i &acc, const Tab &t, const float *tab, int bn, int n_loc, int g, int (&pk)[4]) const
    {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const v4f mm = t.m[q], bb = t.b[q];
            pk[q] = pack_codes(code_bits(__builtin_fmaf((float)acc[4 * q + 0], mm.x, bb.x)),
                               code_bits(__builtin_fmaf((float)acc[4 * q + 1], mm.y, bb.y)),
                               code_bits(__builtin_fmaf((float)acc[4 * q + 2], mm.z, bb.z)),
                               code_bits(__builtin_fmaf((float)acc[4 * q + 3], mm.w, bb.w)));
        }
    }
    // the same four channels of N tokens
    template <int N>
    __device__ __forceinline__ void quads(const v4i (&acc)[N], const v4f &mm, const v4f &bb, const v2i *, int (&pk)[N]) const
    {
#pragma unroll
        for (int i = 0; i < N; i++)
            pk[i] = pack_codes(code_bits(__builtin_fmaf((float)acc[i].x, mm.x, bb.x)), code_bits(__builtin_fmaf((float)acc[i].y, mm.y, bb.y)),
                               code_bits(__builtin_fmaf((float)acc[i].z, mm.z, bb.z)), code_bits(__builtin_fmaf((float)acc[i].w, mm.w, bb.w)));
    }
};

// y = fmaf(acc, m[n], bias[n]); code = rne(GELU(y) / s_out), decided exactly: the fast binary32
// GELU is used wherever it provably rounds like the binary64 definition.  The tie tests leave one
// wave-wide lane mask per accumulator in scalar registers and cost no vector work; only when some
// mask is non-zero (a few percent of the tiles) are they turned into a per-lane bit mask, and the
// flagged elements redone in binary64 by one compact loop (one copy of the slow code per tile).
struct EpiGeluQuant {
    const float *m, *bias; float inv_s;
    static constexpr int OUT_BYTES = 1;
    static constexpr bool STAGED = true;
    static constexpr int NTAB = 2;
    typedef int pack_t;
    __device__ __forceinline__ void load_tables(float *tab, int n0, int bn, int tid, int nthreads) const
    { copy_table(tab, m, n0, bn, tid, nthreads); copy_table(tab + bn, bias, n0, bn, tid, nthreads); }
    __device__ __forceinline__ void load_tables_direct(float *tab, int n0, int bn, int wave, int nwaves, int lane) const
    { copy_table_direct(tab, m, n0, bn, wave, nwaves, lane); copy_table_direct(tab + bn, bias, n0, bn, wave, nwaves, lane); }
    struct Tab { v4f m[4], b[4]; };
    __device__ __forceinline__ Tab load_tab(const float *tab, int bn, int n_loc, int g) const { return load_tab_mb<Tab>(tab, bn, n_loc, g); }
    __device__ __forceinline__ void tile(const v16i &acc, const Tab &tb, const float *tab, int bn, int n_loc, int g, int (&pk)[4]) const
    {
        unsigned long long tie[16], any = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const v4f mm = tb.m[q], bb = tb.b[q];
            float f[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const float y = __builtin_fmaf((float)acc[4 * q + t], mm[t], bb[t]);
                bool near_tie;
                f[t] = gelu_code_bits_fast(y, inv_s, near_tie);
                tie[4 * q + t] = __builtin_amdgcn_ballot_w64(near_tie);
                any |= tie[4 * q + t];
            }
            pk[q] = pack_codes(f[0], f[1], f[2], f[3]);
        }
        if (any == 0) return;                                          // wave-uniform
        const int lane = threadIdx.x & 63;
        unsigned slow = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) slow |= (unsigned)((tie[k] >> lane) & 1) << k;
        while (__builtin_amdgcn_ballot_w64(slow != 0) != 0) {          // wave-uniform loop
            const bool active = slow != 0;
            const int e = active ? __builtin_ctz(slow) : 0;
            int a = acc[0];
#pragma unroll
            for (int k = 1; k < 16; k++) a = (e == k) ? acc[k] : a;
            const int n = n_loc + 8 * (e >> 2) + 4 * g + (e & 3);
            const float y = __builtin_fmaf((float)a, tab[n], tab[bn + n]);
            const int code = qcode(gelu_exact(y) * inv_s);
            const int sh = 8 * (e & 3);
#pragma unroll
            for (int q = 0; q < 4; q++)
                if (active && (e >> 2) == q) pk[q] = (pk[q] & ~(0xff << sh)) | ((code & 0xff) << sh);
            slow &= slow - 1;
        }
    }
};

// The same decision through the threshold table of gelu_table.hip: the bin of y comes out of one fused
// multiply-add (the addend carries 2^23, so the adder rounds to an integer that sits in the low mantissa
// bits), the bin's entry holds the binary32 number at which the code changes inside the bin and the codes
// on either side.  Exact by construction (the table is built from the binary64 definition), about ten
// vector operations and one 8-byte LDS read per element, no transcendental and no slow path.
// The table (at most 16 KiB) is copied into LDS behind the per-channel tables when the block starts.
struct EpiGeluTable {
    const float *m, *bias; const uint32_t *entries; float rate, offset, t_max; int bins;
    static constexpr int OUT_BYTES = 1;
    static constexpr bool STAGED = true;
    static constexpr int NTAB = 2;
    typedef int pack_t;
    __host__ __device__ int extra_lds_bytes() const { return bins * 8; }
    __device__ __forceinline__ const float *offsets() const { return bias; }
    __device__ __forceinline__ void load_lut_direct(v2i *lut, int wave, int nwaves, int lane) const
    { copy_direct(lut, entries, 2 * bins, wave, nwaves, lane); }
    __device__ __forceinline__ void load_tables(float *tab, int n0, int bn, int tid, int nthreads) const
    {
        copy_table(tab, m, n0, bn, tid, nthreads);
        copy_table(tab + bn, bias, n0, bn, tid, nthreads);
        v2i *lut = reinterpret_cast<v2i *>(tab + 2 * bn);
        for (int i = tid; i < bins; i += nthreads) lut[i] = reinterpret_cast<const v2i *>(entries)[i];
    }
    __device__ __forceinline__ void load_tables_direct(float *tab, int n0, int bn, int wave, int nwaves, int lane) const
    {
        copy_table_direct(tab, m, n0, bn, wave, nwaves, lane);
        copy_table_direct(tab + bn, bias, n0, bn, wave, nwaves, lane);
        copy_direct(tab + 2 * bn, entries, 2 * bins, wave, nwaves, lane);
    }
    __device__ __forceinline__ int four(const v4i &acc, const float *tab, int bn, int n) const
    {
        const v2i *lut = reinterpret_cast<const v2i *>(tab + 2 * bn);
        const v4f mm = *reinterpret_cast<const v4f *>(tab + n), bb = *reinterpret_cast<const v4f *>(tab + bn + n);
        unsigned c[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const float y = __builtin_fmaf((float)acc[k], mm[k], bb[k]);
            const v2i e = lut[__float_as_uint(__builtin_amdgcn_fmed3f(__builtin_fmaf(y, rate, offset), 8388608.0f, t_max)) - 0x4B000000u];
            c[k] = (y >= __int_as_float(e.x) ? (unsigned)e.y >> 8 : (unsigned)e.y) & 0xffu;
        }
        return (int)(c[0] | c[1] << 8 | c[2] << 16 | c[3] << 24);
    }
    struct Tab { v4f m[4], b[4]; };
    __device__ __forceinline__ Tab load_tab(const float *tab, int bn, int n_loc, int g) const { return load_tab_mb<Tab>(tab, bn, n_loc, g); }
    __device__ __forceinline__ void tile(const v16i &acc, const Tab &t, const float *tab, int bn, int n_loc, int g, int (&pk)[4]) const
    {
        const v2i *lut = reinterpret_cast<const v2i *>(tab + 2 * bn);
        // all sixteen bins first, then the sixteen table reads, then the comparisons: one wait instead of sixteen
        float y[16];
        unsigned bin[16];
        v2i e[16];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            y[k] = __builtin_fmaf((float)acc[k], t.m[k >> 2][k & 3], t.b[k >> 2][k & 3]);
            bin[k] = __float_as_uint(__builtin_amdgcn_fmed3f(__builtin_fmaf(y[k], rate, offset), 8388608.0f, t_max)) - 0x4B000000u;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 16; k++) e[k] = lut[bin[k]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            unsigned c[4];
#pragma unroll
            for (int k = 0; k < 4; k++)
                c[k] = y[4 * q + k] >= __int_as_float(e[4 * q + k].x) ? (unsigned)e[4 * q + k].y >> 8 : (unsigned)e[4 * q + k].y;
            const unsigned lo = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm(c[3], c[2], 0x0c0c0400u);
            pk[q] = (int)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
        }
    }
    template <int N>
    __device__ __forceinline__ void quads(const v4i (&acc)[N], const v4f &mm, const v4f &bb, const v2i *lut, int (&pk)[N]) const
    {
        float y[4 * N];
        unsigned bin[4 * N];
        v2i e[4 * N];
#pragma unroll
        for (int k = 0; k < 4 * N; k++) {
            y[k] = __builtin_fmaf((float)acc[k >> 2][k & 3], mm[k & 3], bb[k & 3]);
            bin[k] = __float_as_uint(__builtin_amdgcn_fmed3f(__builtin_fmaf(y[k], rate, offset), 8388608.0f, t_max)) - 0x4B000000u;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 4 * N; k++) e[k] = lut[bin[k]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < N; q++) {
            unsigned c[4];
#pragma unroll
            for (int k = 0; k < 4; k++)
                c[k] = y[4 * q + k] >= __int_as_float(e[4 * q + k].x) ? (unsigned)e[4 * q + k].y >> 8 : (unsigned)e[4 * q + k].y;
            const unsigned lo = __builtin_amdgcn_perm(c[1], c[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm(c[3], c[2], 0x0c0c0400u);
            pk[q] = (int)__builtin_amdgcn_perm(hi, lo, 0x05040100u);
        }
    }
};

struct EpiF16 {                                   // fp16(act(acc + bias[n]))
    const float *bias; bool gelu;
    static constexpr int OUT_BYTES = 2;
    static constexpr bool STAGED = true;
    static constexpr int NTAB = 1;
    typedef v2i pack_t;
    __device__ __forceinline__ void load_tables(float *tab, int n0, int bn, int tid, int nthreads) const
    { copy_table(tab, bias, n0, bn, tid, nthreads); }
    __device__ __forceinline__ void load_tables_direct(float *tab, int n0, int bn, int wave, int nwaves, int lane) const
    { copy_table_direct(tab, bias, n0, bn, wave, nwaves, lane); }
    struct Tab { v4f b[4]; };
    __device__ __forceinline__ Tab load_tab(const float *tab, int bn, int n_loc, int g) const
    {
        Tab t;
#pragma unroll
        for (int q = 0; q < 4; q++) t.b[q] = *reinterpret_cast<const v4f *>(tab + n_loc + 8 * q + 4 * g);
        return t;
    }
    __device__ __forceinline__ void tile(const v16f &acc, const Tab &t, const float *tab, int bn, int n_loc, int g, v2i (&pk)[4]) const
    {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const v4f bb = t.b[q];
            float a0 = acc[4 * q] + bb.x, a1 = acc[4 * q + 1] + bb.y, a2 = acc[4 * q + 2] + bb.z, a3 = acc[4 * q + 3] + bb.w;
            if (gelu) { a0 = gelu_fast(a0); a1 = gelu_fast(a1); a2 = gelu_fast(a2); a3 = gelu_fast(a3); }
            const v4h h = {to_half(a0), to_half(a1), to_half(a2), to_half(a3)};
            pk[q] = __builtin_bit_cast(v2i, h);
        }
    }
};

template <class Epi> auto extra_lds_of(const Epi &e, int) -> decltype(e.extra_lds_bytes()) { return e.extra_lds_bytes(); }
template <class Epi> int extra_lds_of(const Epi &, long) { return 0; }

// A block is WGM x WGN waves, each computing 32 TM tokens x 32 TN channels.
template <class T, class Epi, int TM, int TN, int BKB, int NSTAGE, int WAVES_PER_EU, int WGM = 2, int WGN = 2>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(WAVES_PER_EU, 8)))
void gemm_nt_kernel(const char *__restrict__ A, const char *__restrict__ W, const int *__restrict__ dev_rows, int host_rows, int N, int Kbytes,
                    int tiles_n, char *__restrict__ out, Epi epi)
{
    constexpr int NWAVES = WGM * WGN, NT = 64 * NWAVES;
    constexpr int BM = 32 * WGM * TM, BN = 32 * WGN * TN;
    constexpr int A_BYTES = BM * BKB, W_BYTES = BN * BKB, STAGE_BYTES = A_BYTES + W_BYTES;
    constexpr int CH = BKB / 16, RPI = 64 / CH;                  // chunks per row; rows per direct-load instruction
    static_assert(BKB == 64 || BKB == 128, "stage depth");
    static_assert(BM % RPI == 0 && BN % RPI == 0, "operand tiles must be whole 1 KiB pieces");
    // a stage is (BM + BN) / RPI pieces of 1 KiB (the token tile first, then the channel tile), dealt to the
    // waves in turn; when they do not divide evenly the first NPIECE % NWAVES waves issue one load more
    constexpr int NPIECE = (BM + BN) / RPI, NLD = (NPIECE + NWAVES - 1) / NWAVES, NLD_FEWER = NPIECE / NWAVES;
    constexpr int RING_BYTES = NSTAGE * STAGE_BYTES;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    float *tab = reinterpret_cast<float *>(lds + RING_BYTES);

    // each XCD owns a contiguous range of the tiles of the rows that exist (tile order: token rows, then
    // channel tiles), i.e. the same eighth of the token rows as in every other kernel of the path
    const int M = dev_rows ? *dev_rows : host_rows;
    const int tiles = ((M + BM - 1) / BM) * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave / WGN) * 32 * TM, wn = (wave % WGN) * 32 * TN;    // wave tile origin inside the block tile
    const int r = lane & 31, g = lane >> 5;

    // direct loads: instruction j of this wave fills RPI consecutive rows (1 KiB) of an operand tile;
    // lane i supplies row (i / CH), LDS chunk (i % CH), i.e. global chunk (i % CH) ^ swz(row).
    const char *src[NLD];
    const bool fewer = NLD_FEWER != NLD && wave >= NPIECE % NWAVES;   // this wave has no last piece
#pragma unroll
    for (int j = 0; j < NLD; j++) {
        const int piece = min(wave + NWAVES * j, NPIECE - 1);
        const int srow = RPI * piece + lane / CH;                // row inside the stage
        if (srow < BM) {
            int am = m0 + srow; if (am > M - 1) am = M - 1;      // rows past the end re-read the last row
            src[j] = A + (size_t)am * Kbytes + (((lane % CH) ^ swz<BKB>(srow)) << 4);
        } else {
            const int row = srow - BM;
            src[j] = W + (size_t)(n0 + row) * Kbytes + (((lane % CH) ^ swz<BKB>(row)) << 4);
        }
    }
    auto issue = [&](int kt) {
        char *st = lds + (kt % NSTAGE) * STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < NLD; j++)
            if (j < NLD_FEWER || !fewer)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[j] + (size_t)kt * BKB),
                                                 (__attribute__((address_space(3))) void *)(st + (wave + NWAVES * j) * 1024), 16, 0, 0);
    };
    // stage kt has landed when at most the loads of the (NSTAGE - 2) later stages are outstanding
    auto wait_stage = [&](bool later_stages_in_flight) {
        if (!later_stages_in_flight) wait_vm_and_barrier<0>();
        else if (fewer) wait_vm_and_barrier<(NSTAGE - 2) * NLD_FEWER>();
        else wait_vm_and_barrier<(NSTAGE - 2) * NLD>();
    };

    const int KT = Kbytes / BKB;
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; s++)
        if (s < KT) issue(s);
    epi.load_tables(tab, n0, BN, tid, NT);            // ordinary loads; consumed after the main loop

    typename T::acc_t acc[TN][TM];                                // [channel tile][token tile]
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0;

    for (int kt = 0; kt < KT; kt++) {
        // stage kt must have landed: all but the loads of the (up to NSTAGE-2) later stages
        wait_stage(kt + NSTAGE - 2 < KT);
        if (kt + NSTAGE - 1 < KT) issue(kt + NSTAGE - 1);        // refills the buffer consumed at kt-1
        const char *cur = lds + (kt % NSTAGE) * STAGE_BYTES;
#pragma unroll
        for (int ks = 0; ks < CH / 2; ks++) {
            v4i fa[TM], fw[TN];
#pragma unroll
            for (int j = 0; j < TM; j++) {
                const int row = wm + j * 32 + r;
                fa[j] = *reinterpret_cast<const v4i *>(cur + row * BKB + (((2 * ks + g) ^ swz<BKB>(row)) << 4));
            }
#pragma unroll
            for (int i = 0; i < TN; i++) {
                const int row = wn + i * 32 + r;
                fw[i] = *reinterpret_cast<const v4i *>(cur + A_BYTES + row * BKB + (((2 * ks + g) ^ swz<BKB>(row)) << 4));
            }
#pragma unroll
            for (int i = 0; i < TN; i++)
#pragma unroll
                for (int j = 0; j < TM; j++) acc[i][j] = T::mma(fw[i], fa[j], acc[i][j]);
        }
    }
    typename Epi::Tab tabs[TN];                                   // the epilogue's table entries arrive while the waves gather
#pragma unroll
    for (int io = 0; io < TN; io++) tabs[io] = epi.load_tab(tab, BN, wn + io * 32, g);
    wait_vm_and_barrier<0>();                                     // the ring is idle from here on

    if constexpr (!Epi::STAGED) {
#pragma unroll
        for (int io = 0; io < TN; io++)
#pragma unroll
            for (int j = 0; j < TM; j++) {
                const int row = m0 + wm + j * 32 + r;
                if (row < M) {
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const int n = n0 + wn + io * 32 + 8 * q + 4 * g;
                        epi.direct(row, n, acc[io][j][4 * q], acc[io][j][4 * q + 1], acc[io][j][4 * q + 2], acc[io][j][4 * q + 3]);
                    }
                }
            }
    } else {
        // stage the output tile in LDS, then write full rows, 16 bytes per lane
        constexpr int OB = Epi::OUT_BYTES;
        constexpr int STRIDE = BN * OB + 16;
        static_assert(BM * STRIDE <= RING_BYTES, "staging tile does not fit in the ring");
#pragma unroll
        for (int io = 0; io < TN; io++)
#pragma unroll
            for (int j = 0; j < TM; j++) {
                typename Epi::pack_t pk[4];
                const int lrow = wm + j * 32 + r;
                const int nl = wn + io * 32;
                epi.tile(acc[io][j], tabs[io], tab, BN, nl, g, pk);
#pragma unroll
                for (int q = 0; q < 4; q++)
                    *reinterpret_cast<typename Epi::pack_t *>(lds + lrow * STRIDE + (nl + 8 * q + 4 * g) * OB) = pk[q];
            }
        __syncthreads();
        constexpr int CHUNKS = BN * OB / 16;                      // 16-byte chunks per output row
        static_assert((BM * CHUNKS) % NT == 0, "output chunks must split evenly over the threads");
#pragma unroll
        for (int p = 0; p < BM * CHUNKS / NT; p++) {
            const int idx = p * NT + tid;
            const int lrow = idx / CHUNKS, ochunk = idx % CHUNKS;
            if (m0 + lrow < M) {
                const v4i v = *reinterpret_cast<const v4i *>(lds + lrow * STRIDE + ochunk * 16);
                *reinterpret_cast<v4i *>(out + ((size_t)(m0 + lrow) * N + n0) * OB + ochunk * 16) = v;
            }
        }
    }
}

template <class T, class Epi, int TM, int TN, int BKB, int NSTAGE, int WPE, int WGM = 2, int WGN = 2>
hipError_t launch_cfg(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st,
                      const Timing *tm)
{
    constexpr int BM = 32 * WGM * TM, BN = 32 * WGN * TN;
    constexpr size_t LDS_FIXED = (size_t)NSTAGE * (BM + BN) * BKB + (size_t)Epi::NTAB * BN * sizeof(float);
    const size_t LDS = LDS_FIXED + extra_lds_of(epi, 0);
    if (N % BN) return hipErrorInvalidValue;
    if ((K * T::ELEM) % BKB) return hipErrorInvalidValue;
    auto kern = gemm_nt_kernel<T, Epi, TM, TN, BKB, NSTAGE, WPE, WGM, WGN>;
    // > 64 KiB of dynamic LDS must be enabled once per kernel (for the largest table an epilogue may bring);
    // setting it twice from two threads is harmless
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(LDS_FIXED + GELU_TABLE_MAX_BINS * 8));
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_n = N / BN, tiles_m = (rows.host_rows + BM - 1) / BM, total = tiles_n * tiles_m;
    launch_kernel(kern, dim3(total), dim3(64 * WGM * WGN), LDS, st, tm,
                          (const char *)A, (const char *)W, rows.dev_rows, rows.host_rows, N, K * T::ELEM, tiles_n, (char *)out, epi);
    return hipGetLastError();
}


// ---- large tiles ---------------------------------------------------------------------------------
// For many tokens the block tile grows to (64 TM) x (64 TN) with wave tiles of (32 TM) x (32 TN), up to
// 256 x 256 with 128 x 128 per wave: a 32 x 32 x 32 MFMA takes 32 clocks and eats 2 KiB of LDS operands,
// so a wave tile of TM x TN such products needs (TM + TN) / (TM TN) KiB per 32 clocks -- with 2 x 2 the
// four SIMDs of a CU ask for the whole LDS bandwidth, with 4 x 4 for half of it -- and a block tile of
// BM x BN pulls (BM + BN) bytes per BM BN multiply-adds out of L2.  One wave per SIMD, so the latencies
// are hidden by software pipelining instead of by other waves: the K stages (64 or 128 bytes) travel through
// an NSTAGE-deep ring of direct global->LDS loads, and the operand fragments of the next 32-byte step
// are fetched from LDS into a second register set while the MFMAs of the current one run.
//
// 128-byte stages read whole cache lines: a stand-in that only loads the stages of 128 x 256 tiles (32768 x 3072 x 768) pulls 35 to
// 41 bytes per clock and CU with them and 24 with 64-byte stages, whose lines are fetched twice.  They cost a deeper ring or a
// resident block: 128 x 192 tiles are the largest of which two blocks keep two such stages each (2 x 80 KB, all of a CU's
// LDS), so their epilogue tables have to wait for a free stage (LATE).  Forward, three 64-byte stages against two of 128 bytes:
// BERT-base 32 x 128 -1.1 %, 64 ragged -2.7 %, BERT-large 32 x 256 Fully-Quant (QKV alone) -2.1 %; as 192 x 128 tiles for FFN1 of
// BERT-large (128 x 256 and 64-byte stages now) +0.7 %.
template <class Epi> constexpr int late_table_bytes(int bn)
{
    return (Epi::NTAB * bn * (int)sizeof(float) + (std::is_same<Epi, EpiGeluTable>::value ? GELU_TABLE_MAX_BINS * 8 : 0) + 1023) / 1024 * 1024;
}
template <class Epi> constexpr bool big_tables_late(int bm, int bn, int bkb, int nstage)
{
    return Epi::STAGED && nstage == 2 && (bm + bn) * bkb * nstage == 80 * 1024;
}

template <class T, class Epi, int TM, int TN, int BKB, int NSTAGE, int WPE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void gemm_nt_big_kernel(const char *__restrict__ A, const char *__restrict__ W, const int *__restrict__ dev_rows, int host_rows, int N, int Kbytes,
                        int tiles_n, char *__restrict__ out, Epi epi)
{
    constexpr int CH = BKB / 16, RPI = 64 / CH, KS = BKB / 32, NWAVES = 4, NT = 256;
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int A_BYTES = BM * BKB, STAGE_BYTES = (BM + BN) * BKB;
    constexpr int NLD = (BM + BN) / RPI / NWAVES;                 // 1 KiB pieces per wave and stage
    constexpr int RING_BYTES = NSTAGE * STAGE_BYTES;
    static_assert(BKB == 64 || BKB == 128, "stage depth");
    static_assert(NSTAGE >= 2, "the ring must hold the stage in use and one in flight");
    static_assert((BM + BN) % (RPI * NWAVES) == 0, "a stage must split into whole pieces per wave");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    float *tab = reinterpret_cast<float *>(lds + RING_BYTES);
    // Two 128-byte stages of which two blocks exactly fill a CU's LDS: the epilogue's tables go into the stage that the last
    // one but one leaves free, at the end of the ring that lies in it; the output slabs keep clear of both ends.
    constexpr bool LATE = big_tables_late<Epi>(BM, BN, BKB, NSTAGE);
    constexpr int LATE_BYTES = LATE ? late_table_bytes<Epi>(BN) : 0;

    const int M = dev_rows ? *dev_rows : host_rows;
    const int tiles = ((M + BM - 1) / BM) * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * 32 * TM, wn = (wave & 1) * 32 * TN;
    const int r = lane & 31, g = lane >> 5;

    // 32-bit offsets from a base that is the same for the whole wave: half the registers of a pointer per load, and the step to
    // the next stage is scalar
    constexpr int NLDA = BM / RPI / NWAVES;                       // the first NLDA pieces hold token rows
    static_assert(BM % (RPI * NWAVES) == 0, "a piece of every wave holds rows of one operand");
    const char *bases[2] = {A + (size_t)m0 * Kbytes, W + (size_t)n0 * Kbytes};
    unsigned off[NLD];
#pragma unroll
    for (int j = 0; j < NLD; j++) {
        const int srow = RPI * (wave + NWAVES * j) + lane / CH, row = j < NLDA ? min(srow, M - 1 - m0) : srow - BM;
        off[j] = (unsigned)row * (unsigned)Kbytes + (((lane % CH) ^ swz<BKB>(j < NLDA ? srow : row)) << 4);
    }
    const int KT = Kbytes / BKB;
    int fill_slot = 0, fill_kt = 0;                               // next stage to request and the ring slot it goes to
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
    // LDS address of this lane's first fragment of either operand inside a stage, for each 32-byte step of a
    // stage; the fragments of the other 32-row tiles of the wave lie whole multiples of 32 rows further on (the
    // swizzle only looks at row bits 0..3)
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
    if constexpr (LATE) tab = reinterpret_cast<float *>(lds + ((KT & 1) ? RING_BYTES - LATE_BYTES : 0));
    else epi.load_tables(tab, n0, BN, tid, NT);

    typename T::acc_t acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0;
    auto multiply = [&](const v4i (&fa)[TM], const v4i (&fw)[TN]) {
#pragma unroll
        for (int i = 0; i < TN; i++)
#pragma unroll
            for (int j = 0; j < TM; j++) acc[i][j] = T::mma(fw[i], fa[j], acc[i][j]);
    };

    v4i fa[2][TM], fw[2][TN];                                     // fragments of the current and of the next 32-byte step
    // stage 0 has landed when only the later prologue stages are outstanding
    if (KT > NSTAGE - 2) wait_vm_and_barrier<(NSTAGE - 2) * NLD>(); else wait_vm_and_barrier<0>();
    fetch(0, 0, fa[0], fw[0]);
    // One iteration per stage.  Its first step refills the ring slot that was read last in the iteration before
    // (that iteration's barrier lies between); every step first requests the fragments of the step after it --
    // the last one from the next stage, after waiting for that stage -- then waits for its own fragments only
    // (requested a step ago: the TM + TN requests just made stay outstanding) and multiplies.  The scheduling
    // fences keep the steps apart.  Three copies of the body (stages that still refill the ring, stages that
    // only drain it, the last stage) keep every wait count a constant.
    int slot_bytes = 0;
    auto next_slot = [&]() { slot_bytes = slot_bytes + STAGE_BYTES == RING_BYTES ? 0 : slot_bytes + STAGE_BYTES; };
    auto step = [&](int ks, bool refill, bool more, auto vm_tag) {
        constexpr int VM = decltype(vm_tag)::value;
        if (ks + 1 < KS) {
            fetch(slot_bytes, ks + 1, fa[(ks + 1) & 1], fw[(ks + 1) & 1]);
            wait_lds_reads<TM + TN>();
        } else if (more) {
            wait_vm_and_barrier<VM>();                            // own fragments too (lgkmcnt 0): the slot may be refilled after this
            next_slot();
            fetch(slot_bytes, 0, fa[0], fw[0]);
        } else {
            wait_lds_reads<0>();
        }
        ready(fa[ks & 1], fw[ks & 1]);
        __builtin_amdgcn_sched_barrier(0);
        if (refill && ks == 0) issue();
        if (LATE && !more && ks == 0) epi.load_tables_direct(tab, n0, BN, wave, NWAVES, lane);
        multiply(fa[ks & 1], fw[ks & 1]);
        __builtin_amdgcn_sched_barrier(0);
    };
    int kt = 0;
    for (; kt + NSTAGE - 1 < KT; kt++)
#pragma unroll
        for (int ks = 0; ks < KS; ks++) step(ks, true, true, std::integral_constant<int, (NSTAGE - 2) * NLD>());
    for (; kt + 1 < KT; kt++)
#pragma unroll
        for (int ks = 0; ks < KS; ks++) step(ks, false, true, std::integral_constant<int, 0>());
#pragma unroll
    for (int ks = 0; ks < KS; ks++) step(ks, false, false, std::integral_constant<int, 0>());
    typename Epi::Tab first_tab;
    if (!LATE) first_tab = epi.load_tab(tab, BN, wn, g);          // arrives while the waves gather
    wait_vm_and_barrier<0>();                                     // the ring is idle from here on
    if (LATE) first_tab = epi.load_tab(tab, BN, wn, g);

    if constexpr (!Epi::STAGED) {
#pragma unroll
        for (int io = 0; io < TN; io++)
#pragma unroll
            for (int j = 0; j < TM; j++) {
                const int row = m0 + wm + j * 32 + r;
                if (row < M) {
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const int n = n0 + wn + io * 32 + 8 * q + 4 * g;
                        epi.direct(row, n, acc[io][j][4 * q], acc[io][j][4 * q + 1], acc[io][j][4 * q + 2], acc[io][j][4 * q + 3]);
                    }
                }
            }
    } else {
        // the output tile goes through LDS 64 token rows at a time (32 of each wave row), then out as full rows
        constexpr int OB = Epi::OUT_BYTES;
        constexpr int STRIDE = BN * OB + 16;
        constexpr int CHUNKS = BN * OB / 16;
        static_assert(2 * 64 * STRIDE + 2 * LATE_BYTES <= RING_BYTES, "two staging slabs must fit in the ring");
        static_assert((64 * CHUNKS) % NT == 0, "output chunks must split evenly over the threads");
#pragma unroll
        for (int j = 0; j < TM; j++) {
            char *slab = lds + LATE_BYTES + (j & 1) * 64 * STRIDE;             // alternate slabs: one barrier per pass
            const int lrow = (wave >> 1) * 32 + r;
            typename Epi::Tab cur = j == 0 ? first_tab : epi.load_tab(tab, BN, wn, g);
#pragma unroll
            for (int io = 0; io < TN; io++) {
                typename Epi::pack_t pk[4];
                const int nl = wn + io * 32;
                typename Epi::Tab nxt;                            // the next tile's entries travel while this tile is worked on
                if (io + 1 < TN) nxt = epi.load_tab(tab, BN, nl + 32, g);
                __builtin_amdgcn_sched_barrier(0);
                epi.tile(acc[io][j], cur, tab, BN, nl, g, pk);
#pragma unroll
                for (int q = 0; q < 4; q++)
                    *reinterpret_cast<typename Epi::pack_t *>(slab + lrow * STRIDE + (nl + 8 * q + 4 * g) * OB) = pk[q];
                if (io + 1 < TN) cur = nxt;
            }
            __syncthreads();
            constexpr int PASSES = 64 * CHUNKS / NT;
            v4i v[PASSES];                                        // all reads of the pass, then the stores
#pragma unroll
            for (int p = 0; p < PASSES; p++) {
                const int idx = p * NT + tid;
                v[p] = *reinterpret_cast<const v4i *>(slab + (idx / CHUNKS) * STRIDE + (idx % CHUNKS) * 16);
            }
#pragma unroll
            for (int p = 0; p < PASSES; p++) {
                const int idx = p * NT + tid;
                const int srow = idx / CHUNKS, ochunk = idx % CHUNKS;
                const int grow = m0 + (srow >> 5) * 32 * TM + j * 32 + (srow & 31);
                if (grow < M) *reinterpret_cast<v4i *>(out + ((size_t)grow * N + n0) * OB + ochunk * 16) = v[p];
            }
        }
    }
}

template <class T, class Epi, int TM, int TN, int BKB, int NSTAGE, int WPE = 1>
hipError_t launch_big(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st,
                      const Timing *tm)
{
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr bool LATE = big_tables_late<Epi>(BM, BN, BKB, NSTAGE);
    constexpr size_t LDS_FIXED = (size_t)NSTAGE * (BM + BN) * BKB + (LATE ? 0 : (size_t)Epi::NTAB * BN * sizeof(float));
    const size_t LDS = LDS_FIXED + (LATE ? 0 : extra_lds_of(epi, 0));
    if (N % BN || (K * T::ELEM) % BKB || LDS > 160 * 1024) return hipErrorInvalidValue;
    auto kern = gemm_nt_big_kernel<T, Epi, TM, TN, BKB, NSTAGE, WPE>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        const size_t cap = std::min<size_t>(LDS_FIXED + GELU_TABLE_MAX_BINS * 8, 160 * 1024);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)cap);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_n = N / BN, tiles_m = (rows.host_rows + BM - 1) / BM;
    launch_kernel(kern, dim3(tiles_n * tiles_m), dim3(256), LDS, st, tm,
                  (const char *)A, (const char *)W, rows.dev_rows, rows.host_rows, N, K * T::ELEM, tiles_n, (char *)out, epi);
    return hipGetLastError();
}


// ---- packed weights, straight into registers ---------------------------------------------------
// The tile loops above move both operands through LDS, and LDS is what the large ones run out of: a 128 x 192 tile of four 64 x 96
// wave tiles reads 20 KB of fragments and writes 10 KB for every 192 clocks of matrix work, and its ring holds one stage in flight
// (40 KB per block).  Here the block's four waves stand side by side, each with all 16 MT tokens and 16 NTW channels of its own: no
// other wave wants a wave's weight rows, so they go from L2 into registers, D stages ahead, and only the token rows are staged in
// LDS (a ring of D + 1 stages of 128 bytes a row).
// What makes that pay is the order of the weights in memory (pack_weight_kernel): 16 rows x 64 bytes, what one 16 x 16 x 64 product
// takes, are 1 KB in the order of the lanes.  A probe that reads a 3 MB matrix from L2 into registers gets 130 bytes per ns and CU
// in that order and 38 from 16 rows of 64 bytes where they lie in the matrix (each lane of a quad in a line of its own); rows
// of 128 bytes into LDS get 125.
// A lane's results are four channels of one token per 16 x 16 tile, the same four for all its tokens: its entries of the epilogue's
// vectors are loaded once, into registers, and a wave's table lookups are the only LDS reads of the epilogue beside the output tile's.
// FP16: 32 x 32 x 16 products, as in the row-major kernels and so with their bytes; blocks of 32 rows x 32 bytes; four products' weights
// per 128-byte stage.  The bias goes to LDS: in registers (16 NTW) it makes the 128 x 256 tile spill.
template <class T, class Epi, int MT, int NTW, int D> struct StreamTile {
    static constexpr bool HALF = std::is_same<T, F16>::value;
    static constexpr int ROWS = StreamGeometry<HALF>::ROWS, BM = ROWS * MT, BN = 4 * ROWS * NTW;
    static constexpr int RING = stream_ring_bytes<HALF, MT, D>(), STRIDE = BN * Epi::OUT_BYTES + 16, OUT = BM * STRIDE;
    static constexpr int LUT_OFF = RING > OUT ? RING : OUT;       // the output tile takes the ring's place
};

template <class T, class Epi, int MT, int NTW, int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_nt_stream_kernel(const char *__restrict__ A, const char *__restrict__ Wp, const int *__restrict__ dev_rows, int host_rows, int N, int Kbytes,
                           int tiles_n, unsigned by, int channels_first, char *__restrict__ out, Epi epi)
{
    typedef StreamTile<T, Epi, MT, NTW, D> Tile;
    constexpr bool HALF = Tile::HALF;
    constexpr int ROWS = Tile::ROWS, BM = Tile::BM, BN = Tile::BN, G = MT < 4 ? MT : 4, H = MT / G, NLDA = stream_loads<HALF, MT>();
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    v2i *lut = reinterpret_cast<v2i *>(lds + Tile::LUT_OFF);

    const int M = dev_rows ? *dev_rows : host_rows;
    const int tiles_m = (M + BM - 1) / BM, tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    const TileAt at = channels_first ? tile_channels_first(tile, tiles_m, (host_rows + BM - 1) / BM, by) : tile_rows_first(tile, tiles_n, by);
    const int m0 = at.m * BM, n0 = at.n * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & (ROWS - 1), q = lane / ROWS;

    unsigned offa[NLDA];
#pragma unroll
    for (int j = 0; j < NLDA; j++) {
        const int srow = 8 * (wave + 4 * j) + (lane >> 3);
        offa[j] = (unsigned)min(srow, M - 1 - m0) * (unsigned)Kbytes + (((lane & 7) ^ swz<128>(srow)) << 4);
    }
    const char *wbase = Wp + (size_t)(n0 + ROWS * NTW * wave) * Kbytes;
    unsigned woff[NTW];
#pragma unroll
    for (int t = 0; t < NTW; t++) woff[t] = ROWS * t * Kbytes;
    typedef typename std::conditional<HALF, v16f, v4i>::type Acc;
    Acc acc[NTW][MT];
#pragma unroll
    for (int t = 0; t < NTW; t++)
#pragma unroll
        for (int i = 0; i < MT; i++)
#pragma unroll
            for (int e = 0; e < (HALF ? 16 : 4); e++) acc[t][i][e] = 0;
    constexpr int OB = Epi::OUT_BYTES, STRIDE = Tile::STRIDE;
    if constexpr (HALF) {
        float *tab = reinterpret_cast<float *>(lds + Tile::LUT_OFF);
        stream_tile_loop<HALF, MT, NTW, D>(A + (size_t)m0 * Kbytes, offa, wbase, woff, Kbytes / 128, lds, wave, lane,
            [&]() { epi.load_tables_direct(tab, n0, BN, wave, 4, lane); },
            [&](int t, int i, const v4i &w, const v4i &f) { acc[t][i] = T::mma(w, f, acc[t][i]); });
#pragma unroll
        for (int t = 0; t < NTW; t++) {
            const typename Epi::Tab b = epi.load_tab(tab, BN, 32 * (NTW * wave + t), q);
#pragma unroll
            for (int i = 0; i < MT; i++) {
                v2i pk[4];
                epi.tile(acc[t][i], b, nullptr, BN, 0, q, pk);
#pragma unroll
                for (int u = 0; u < 4; u++)
                    *reinterpret_cast<v2i *>(lds + (32 * i + r) * STRIDE + (32 * (NTW * wave + t) + 8 * u + 4 * q) * OB) = pk[u];
            }
        }
    } else {
        v4f mm[NTW], bb[NTW];
        stream_tile_loop<HALF, MT, NTW, D>(A + (size_t)m0 * Kbytes, offa, wbase, woff, Kbytes / 128, lds, wave, lane,
            [&]() {
                epi.load_lut_direct(lut, wave, 4, lane);
#pragma unroll
                for (int t = 0; t < NTW; t++) {
                    const int n = n0 + 16 * (NTW * wave + t) + 4 * q;
                    mm[t] = *reinterpret_cast<const v4f *>(epi.m + n);
                    bb[t] = *reinterpret_cast<const v4f *>((epi.offsets() ? epi.offsets() : epi.m) + n);
                }
            },
            [&](int t, int i, const v4i &w, const v4i &f) { acc[t][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, f, acc[t][i], 0, 0, 0); });
#pragma unroll
        for (int t = 0; t < NTW; t++) {
            if (!epi.offsets()) bb[t] = v4f{0.f, 0.f, 0.f, 0.f};   // (here: a choice before the loop would wait for the loads)
#pragma unroll
            for (int h = 0; h < H; h++) {
                v4i group[G];
                int pk[G];
#pragma unroll
                for (int i = 0; i < G; i++) group[i] = acc[t][G * h + i];
                epi.quads(group, mm[t], bb[t], lut, pk);
#pragma unroll
                for (int i = 0; i < G; i++)
                    *reinterpret_cast<int *>(lds + (16 * (G * h + i) + r) * STRIDE + 16 * (NTW * wave + t) + 4 * q) = pk[i];
            }
        }
    }
    __syncthreads();
    constexpr int CHUNKS = BN * OB / 16, PASSES = (BM * CHUNKS + 255) / 256;
    constexpr bool EVEN = BM * CHUNKS % 256 == 0;
    constexpr int BATCH = PASSES < 8 ? PASSES : 8;                // all reads of a batch, then its stores
    static_assert(PASSES % BATCH == 0, "whole batches");
#pragma unroll
    for (int p0 = 0; p0 < PASSES; p0 += BATCH) {
        v4i v[BATCH];
#pragma unroll
        for (int p = 0; p < BATCH; p++) {
            const int idx = EVEN ? (p0 + p) * 256 + tid : min((p0 + p) * 256 + tid, BM * CHUNKS - 1);
            v[p] = *reinterpret_cast<const v4i *>(lds + (idx / CHUNKS) * STRIDE + (idx % CHUNKS) * 16);
        }
#pragma unroll
        for (int p = 0; p < BATCH; p++) {
            const int idx = (p0 + p) * 256 + tid, row = m0 + idx / CHUNKS;
            if (row < M && (EVEN || idx < BM * CHUNKS)) *reinterpret_cast<v4i *>(out + ((size_t)row * N + n0) * OB + (idx % CHUNKS) * 16) = v[p];
        }
    }
}

template <class T, class Epi, int MT, int NTW, int D>
hipError_t launch_stream(const void *A, const void *Wp, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    typedef StreamTile<T, Epi, MT, NTW, D> Tile;
    const size_t LDS = Tile::LUT_OFF + (Tile::HALF ? Tile::BN * 4 : extra_lds_of(epi, 0));
    if (N % Tile::BN || K * T::ELEM % (128 * D)) return hipErrorInvalidValue;
    auto kern = gemm_nt_stream_kernel<T, Epi, MT, NTW, D>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           Tile::LUT_OFF + GELU_TABLE_MAX_BINS * 8);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    // An XCD takes the tiles of an eighth of the token rows, as in every other kernel of the path, unless the weights
    // are more than its L2 holds beside them and the rows are few: then it takes an eighth of the channels and all of the rows (us, token
    // rows first / channels first: 1024 x 4096, 256 rows 7.8 / 6.4, 512 rows 10.6 / 7.1, 1024 rows 11.3 / 11.6, 2048 rows 13.9 / 14.5;
    // 4096 x 1024, 512 rows 6.9 / 6.1, 1024 rows 10.6 / 8.6; 768 x 3072 and 3072 x 768 +-2 % up to 1024 rows)
    const bool channels_first = (long)N * K * T::ELEM >= 3 << 20 && rows.host_rows <= 1024;
    const int tiles_n = N / Tile::BN, tiles_m = (rows.host_rows + Tile::BM - 1) / Tile::BM;
    launch_kernel(kern, dim3(tiles_n * tiles_m), dim3(256), LDS, st, tm, (const char *)A, (const char *)Wp, rows.dev_rows,
                  rows.host_rows, N, K * T::ELEM, tiles_n, divisor(tiles_n * tiles_m, channels_first ? tiles_m : tiles_n), (int)channels_first,
                  (char *)out, epi);
    return hipGetLastError();
}

// Stages in flight: a small tile's stage is short next to the latency of its loads (the weights of a layer come from beyond L2), so it asks
// for more of them (us, 2 stages / as chosen here: 32 x 64 tiles, 768 x 768 at 427 rows 4.1 / 3.5, 1024 x 4096 at 427 rows 9.1 / 6.4; 64 x 64,
// 768 x 3072 at 1024 rows 8.5 / 7.2; 64 x 128, 768 x 3072 at 2048 rows 10.2 / 9.0; 64 x 192, 768 x 3072 at 4096 rows 12.2 / 11.7; the
// larger tiles are +-3 %).  KT, the number of stages, has to be a multiple.
template <class Epi>
hipError_t launch_packed(const void *A, const void *Wp, void *out, const Epi &epi, Rows rows, int N, int K, int tile, hipStream_t st, const Timing *tm)
{
    if (K % 256 || N % 64) return hipErrorNotSupported;
    switch (tile < 0 ? stream_tile(rows.host_rows, rows.dev_rows && !rows.beside, N, K) : tile) {
    case 0:
        if (K % 512 == 0) return launch_stream<I8, Epi, 2, 1, 4>(A, Wp, out, epi, rows, N, K, st, tm);
        if (K % 768 == 0) return launch_stream<I8, Epi, 2, 1, 6>(A, Wp, out, epi, rows, N, K, st, tm);
        return launch_stream<I8, Epi, 2, 1, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 1:
        if (K % 512 == 0) return launch_stream<I8, Epi, 4, 1, 4>(A, Wp, out, epi, rows, N, K, st, tm);
        if (K % 384 == 0) return launch_stream<I8, Epi, 4, 1, 3>(A, Wp, out, epi, rows, N, K, st, tm);
        return launch_stream<I8, Epi, 4, 1, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 2:
        if (K % 512 == 0) return launch_stream<I8, Epi, 4, 2, 4>(A, Wp, out, epi, rows, N, K, st, tm);
        if (K % 384 == 0) return launch_stream<I8, Epi, 4, 2, 3>(A, Wp, out, epi, rows, N, K, st, tm);
        return launch_stream<I8, Epi, 4, 2, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 3:
        if (K % 384 == 0) return launch_stream<I8, Epi, 4, 3, 3>(A, Wp, out, epi, rows, N, K, st, tm);
        return launch_stream<I8, Epi, 4, 3, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 4: return launch_stream<I8, Epi, 4, 4, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 5: return launch_stream<I8, Epi, 8, 2, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 6: return launch_stream<I8, Epi, 8, 3, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    }
    return hipErrorInvalidValue;
}

// The same for FP16: tiles of 32 mt tokens x 128 ntw channels.  Here the operand bytes alone decide (a fit gives the other terms no weight;
// the choice costs 0.3 % on average over the best of the four, from 256 rows on; fewer rows read the weights as they lie, gemm_rules.h).
constexpr StreamShape STREAM_TILES_F16[] = {{1, 1}, {2, 1}, {2, 2}, {4, 2}};
constexpr int STREAM_TILE_F16_COUNT = sizeof(STREAM_TILES_F16) / sizeof(STREAM_TILES_F16[0]);
int stream_tile_f16(Rows rows, int N, int K)
{
    int best = -1;
    long best_cost = 0;
    for (int i = 0; i < STREAM_TILE_F16_COUNT; i++) {
        const int bm = 32 * STREAM_TILES_F16[i].mt, bn = 128 * STREAM_TILES_F16[i].ntw;
        if (N % bn) continue;
        const long tiles = (long)(N / bn) * ((rows.host_rows + bm - 1) / bm), cost = (tiles + 255) / 256 * (bm + bn);
        if (best < 0 || cost < best_cost) { best = i; best_cost = cost; }
    }
    return best;
}
hipError_t launch_packed_f16(const void *A, const void *Wp, void *out, const EpiF16 &epi, Rows rows, int N, int K, int tile, hipStream_t st, const Timing *tm)
{
    if (K % 128 || N % 128) return hipErrorNotSupported;
    // four stages in flight (two where K is no multiple): 32 x 128 tiles 768 x 3072 at 1024 rows 14.8 / 13.1, 128 x 128 4096 x 1024 at 4096
    // rows 58.0 / 50.7, 3072 x 768 there 34.1 / 31.0.  The wide tiles have no registers for more than two.
    const bool deep = K % 256 == 0;
    switch (tile < 0 ? stream_tile_f16(rows, N, K) : tile) {
    case 0:
        if (deep) return launch_stream<F16, EpiF16, 1, 1, 4>(A, Wp, out, epi, rows, N, K, st, tm);
        return launch_stream<F16, EpiF16, 1, 1, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 1:
        if (deep) return launch_stream<F16, EpiF16, 2, 1, 4>(A, Wp, out, epi, rows, N, K, st, tm);
        return launch_stream<F16, EpiF16, 2, 1, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 2: return launch_stream<F16, EpiF16, 2, 2, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    case 3: return launch_stream<F16, EpiF16, 4, 2, 2>(A, Wp, out, epi, rows, N, K, st, tm);
    }
    return hipErrorInvalidValue;
}

// ---- long operand rows on few tiles ------------------------------------------------------------------
// FFN2 at small batch: 24 (FP16: 48) stages of 128 bytes, 64 x 96 tiles that no more than fill the chip once.  Such
// a block is a chain of dependent stages whose pace is set by bytes in flight over load latency, and LDS for a
// deeper ring is what the other batch group's kernels on the same CU need.  Here the stages in flight wait in
// REGISTERS instead (a 32 x 32 tile per wave leaves most of them idle): every wave keeps DEPTH stages of its share
// of the loads outstanding, writes the oldest one to one of two LDS buffers when it lands, and requests the stage
// DEPTH ahead into the registers just freed.  One barrier per stage: a buffer is rewritten two stages after it
// was read, and the barrier of the stage between lies between.  Deeper is faster for the kernel alone and slower
// for the forward (the loads in flight compete with the other group's kernels), so the launcher takes DEPTH = 2:
// what is won is the LDS (40 KB against 61 KB for the three-deep ring).
template <class T, class Epi, int WGN, int DEPTH>
__global__ __launch_bounds__(128 * WGN)
void gemm_nt_longk_kernel(const char *__restrict__ A, const char *__restrict__ W, const int *__restrict__ dev_rows, int host_rows, int N, int Kbytes,
                          int tiles_n, char *__restrict__ out, Epi epi)
{
    constexpr int BKB = 128, BM = 64, BN = 32 * WGN, NWAVES = 2 * WGN, NT = 64 * NWAVES;
    constexpr int NPIECE = (BM + BN) / 8, NLD = (NPIECE + NWAVES - 1) / NWAVES;      // 1 KiB pieces of 8 rows; loads per wave and stage
    constexpr int STAGE_BYTES = (BM + BN) * BKB, A_BYTES = BM * BKB;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    float *tab = reinterpret_cast<float *>(lds + 2 * STAGE_BYTES);

    const int M = dev_rows ? *dev_rows : host_rows;
    const int tiles = ((M + BM - 1) / BM) * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave / WGN) * 32, wn = (wave % WGN) * 32;
    const int r = lane & 31, g = lane >> 5;

    // this wave's pieces: where they come from and where they go (a surplus slot repeats the last piece)
    const char *src[NLD];
    int dst[NLD];
#pragma unroll
    for (int j = 0; j < NLD; j++) {
        const int piece = min(wave + NWAVES * j, NPIECE - 1);
        const int srow = 8 * piece + (lane >> 3), chunk = lane & 7;
        if (srow < BM) {
            int am = m0 + srow; if (am > M - 1) am = M - 1;
            src[j] = A + (size_t)am * Kbytes + chunk * 16;
            dst[j] = srow * BKB + ((chunk ^ swz<BKB>(srow)) << 4);
        } else {
            const int row = srow - BM;
            src[j] = W + (size_t)(n0 + row) * Kbytes + chunk * 16;
            dst[j] = A_BYTES + row * BKB + ((chunk ^ swz<BKB>(row)) << 4);
        }
    }
    const int KT = Kbytes / BKB;                                  // a multiple of DEPTH (the launcher checks)
    // (scheduling fences keep the loads in stage order: the wait for a stage's registers counts the loads behind it)
    v4i held[DEPTH][NLD];
    epi.load_tables(tab, n0, BN, tid, NT);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < DEPTH; d++) {
#pragma unroll
        for (int j = 0; j < NLD; j++) held[d][j] = *reinterpret_cast<const v4i *>(src[j] + (size_t)d * BKB);
        __builtin_amdgcn_sched_barrier(0);
    }

    typename T::acc_t acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0;
    const int offa = (wm + r) * BKB, offw = A_BYTES + (wn + r) * BKB;
    const int sa = swz<BKB>(wm + r), sw = swz<BKB>(wn + r);

    auto stage = [&](int kt, int d, bool refill) {
        char *buf = lds + (kt & 1) * STAGE_BYTES;
#pragma unroll
        for (int j = 0; j < NLD; j++) *reinterpret_cast<v4i *>(buf + dst[j]) = held[d][j];    // waits for these loads only
        __builtin_amdgcn_sched_barrier(0);
        if (refill) {
#pragma unroll
            for (int j = 0; j < NLD; j++) held[d][j] = *reinterpret_cast<const v4i *>(src[j] + (size_t)(kt + DEPTH) * BKB);
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            const v4i fa = *reinterpret_cast<const v4i *>(buf + offa + (((2 * ks + g) ^ sa) << 4));
            const v4i fw = *reinterpret_cast<const v4i *>(buf + offw + (((2 * ks + g) ^ sw) << 4));
            acc = T::mma(fw, fa, acc);
        }
    };
    int kt = 0;
    for (; kt + DEPTH < KT; kt += DEPTH)
#pragma unroll
        for (int d = 0; d < DEPTH; d++) stage(kt + d, d, true);
#pragma unroll
    for (int d = 0; d < DEPTH; d++) stage(kt + d, d, false);
    const typename Epi::Tab tb = epi.load_tab(tab, BN, wn, g);     // arrives while the waves gather
    __syncthreads();                                              // both buffers are idle from here on

    constexpr int OB = Epi::OUT_BYTES;
    constexpr int STRIDE = BN * OB + 16;
    static_assert(BM * STRIDE <= 2 * STAGE_BYTES, "staging tile does not fit");
    {
        typename Epi::pack_t pk[4];
        epi.tile(acc, tb, tab, BN, wn, g, pk);
#pragma unroll
        for (int q = 0; q < 4; q++)
            *reinterpret_cast<typename Epi::pack_t *>(lds + (wm + r) * STRIDE + (wn + 8 * q + 4 * g) * OB) = pk[q];
    }
    __syncthreads();
    constexpr int CHUNKS = BN * OB / 16;
    for (int idx = tid; idx < BM * CHUNKS; idx += NT) {
        const int lrow = idx / CHUNKS, ochunk = idx % CHUNKS;
        if (m0 + lrow < M)
            *reinterpret_cast<v4i *>(out + ((size_t)(m0 + lrow) * N + n0) * OB + ochunk * 16) =
                *reinterpret_cast<const v4i *>(lds + lrow * STRIDE + ochunk * 16);
    }
}

template <class T, class Epi, int WGN, int DEPTH>
hipError_t launch_longk(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st,
                        const Timing *tm)
{
    constexpr int BN = 32 * WGN;
    const int kbytes = K * T::ELEM;
    if (N % BN || kbytes % (128 * DEPTH)) return hipErrorInvalidValue;
    const size_t LDS = 2 * (size_t)(64 + BN) * 128 + (size_t)Epi::NTAB * BN * sizeof(float);
    const int tiles_n = N / BN, tiles_m = (rows.host_rows + 63) / 64;
    launch_kernel(gemm_nt_longk_kernel<T, Epi, WGN, DEPTH>, dim3(tiles_n * tiles_m), dim3(128 * WGN), LDS, st, tm,
                  (const char *)A, (const char *)W, rows.dev_rows, rows.host_rows, N, kbytes, tiles_n, (char *)out, epi);
    return hipGetLastError();
}

// ---- few token rows ----------------------------------------------------------------------------------
// Up to a few hundred token rows a GEMM of the path is a chain of latencies, not of work: the matrix instructions of a tile
// take tens of nanoseconds, the loop over K stages above pays one memory latency per ring refill.  Here a block computes a small
// tile (16 MT tokens x 16 NT channels) with its NWAVES waves splitting K: every wave streams its own share of the 128-byte
// slabs of both operands through LDS of its own (direct loads, up to R slabs requested before the first is used, no barrier
// in the loop) and forms the whole tile for that share; the int32 partial tiles meet in LDS behind the block's only
// barrier.  Integer sums do not depend on the order, so the result is the same bytes as from every other configuration.
// Blocks are numbered channels outermost, so that an XCD reads an eighth of the weights and all of the few token rows.
template <class Epi, int MT, int NT, int NWAVES, int R>
struct SmallGemm {
    static constexpr int BM = 16 * MT, BN = 16 * NT, SLAB = (BM + BN) * 128, PIECES = SLAB / 1024;
    static constexpr int TAB_OFF = NWAVES * R * SLAB;             // behind the rings
};

template <class Epi, int MT, int NT, int NWAVES, int R>
__global__ __launch_bounds__(64 * NWAVES)
void gemm_nt_small_kernel(const char *__restrict__ A, const char *__restrict__ W, const int *__restrict__ dev_rows, int host_rows, int N, int Kbytes,
                          int tiles_n, char *__restrict__ out, Epi epi)
{
    typedef SmallGemm<Epi, MT, NT, NWAVES, R> G;
    constexpr int BM = G::BM, BN = G::BN;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    float *tab = reinterpret_cast<float *>(lds + G::TAB_OFF);
    const int M = dev_rows ? *dev_rows : host_rows;
    const int tiles_m = (M + BM - 1) / BM, tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    const int m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // pieces of 8 rows x 128 bytes, the token rows first; the wave takes slabs wave, wave + NWAVES, ...
    const char *src[G::PIECES];
#pragma unroll
    for (int j = 0; j < G::PIECES; j++) {
        const int row = 8 * j + (lane >> 3), chunk = ((lane & 7) ^ swz<128>(row)) << 4;
        src[j] = (j < BM / 8 ? A + (size_t)min(m0 + row, M - 1) * Kbytes : W + (size_t)(n0 + row - BM) * Kbytes) + chunk + wave * 128;
    }
    char *ring = lds + wave * (R * G::SLAB);
    auto issue = [&](int s, int slot) {
#pragma unroll
        for (int j = 0; j < G::PIECES; j++)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[j] + (size_t)s * (NWAVES * 128)),
                                             (__attribute__((address_space(3))) void *)(ring + slot * G::SLAB + j * 1024), 16, 0, 0);
    };
    const int slabs = Kbytes / (128 * NWAVES);                                   // of this wave (the launcher checks that they are whole)
#pragma unroll
    for (int s = 0; s < R; s++)
        if (s < slabs) issue(s, s);
    epi.load_tables(tab, n0, BN, tid, 64 * NWAVES);

    v4i acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int j = 0; j < NT; j++) acc[i][j] = v4i{0, 0, 0, 0};
    const int r = lane & 15, q = lane >> 4;
    auto consume = [&](int slot) {
        const char *a = ring + slot * G::SLAB;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            v4i fa[MT], fw[NT];
#pragma unroll
            for (int i = 0; i < MT; i++) fa[i] = *reinterpret_cast<const v4i *>(a + (16 * i + r) * 128 + (((4 * k + q) ^ swz<128>(16 * i + r)) << 4));
#pragma unroll
            for (int j = 0; j < NT; j++)
                fw[j] = *reinterpret_cast<const v4i *>(a + (BM + 16 * j + r) * 128 + (((4 * k + q) ^ swz<128>(BM + 16 * j + r)) << 4));
#pragma unroll
            for (int i = 0; i < MT; i++)
#pragma unroll
                for (int j = 0; j < NT; j++) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[j], fa[i], acc[i][j], 0, 0, 0);
        }
    };
    // a wave waits for its own loads only; every wait below lets the slabs behind the one needed stay in flight
    int s = 0;
    for (; s + R < slabs; s += R)
#pragma unroll
        for (int u = 0; u < R; u++) {
            if (s + u + R - 1 < slabs) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 1) * G::PIECES) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            consume(u);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                  // the slot has been read
            if (s + u + R < slabs) issue(s + u + R, u);
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < R; u++)
        if (s + u < slabs) consume(u);

    // a wave's partial tiles take the place of its own part of the ring, which no other wave reads: [tile][lane]
    static_assert(MT * NT * 1024 <= R * G::SLAB, "");
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
        for (int j = 0; j < NT; j++) *reinterpret_cast<v4i *>(ring + (i * NT + j) * 1024 + lane * 16) = acc[i][j];
    __syncthreads();
    // lane: token 16 i + (lane & 15), channels 16 j + 4 (lane >> 4) .. + 3
    for (int t = wave; t < MT * NT; t += NWAVES) {
        v4i sum = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < NWAVES; w++) sum += *reinterpret_cast<const v4i *>(lds + w * (R * G::SLAB) + t * 1024 + lane * 16);
        const int i = t / NT, j = t % NT, row = m0 + 16 * i + r, nl = 16 * j + 4 * q;
        const int pk = epi.four(sum, tab, BN, nl);
        if (row < M) *reinterpret_cast<int *>(out + (size_t)row * N + n0 + nl) = pk;
    }
}

template <class Epi, int MT, int NT, int NWAVES, int R>
hipError_t launch_small(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    typedef SmallGemm<Epi, MT, NT, NWAVES, R> G;
    const size_t LDS = G::TAB_OFF + (size_t)Epi::NTAB * G::BN * sizeof(float) + extra_lds_of(epi, 0);
    if (N % G::BN || K % (128 * NWAVES) || LDS > 160 * 1024) return hipErrorInvalidValue;
    auto kern = gemm_nt_small_kernel<Epi, MT, NT, NWAVES, R>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_n = N / G::BN, tiles_m = (rows.host_rows + G::BM - 1) / G::BM;
    launch_kernel(kern, dim3(tiles_n * tiles_m), dim3(64 * NWAVES), LDS, st, tm, (const char *)A, (const char *)W, rows.dev_rows,
                  rows.host_rows, N, K, tiles_n, (char *)out, epi);
    return hipGetLastError();
}

// The smallest of four tiles that the chip holds all at once (blocks per CU by LDS): a second round of blocks costs more than a
// larger tile.  hipErrorNotSupported: none, the problem has enough rows for the kernels above (or a K they split differently).
// Measured, us per launch in a chain (before: the 64 x 96 and 64 x 128 tiles of configuration 2): N x K = 768 x 3072, 19 rows
// 9.9 -> 3.7, 256 rows 10.7 -> 4.7, 1024 rows 10.7 -> 7.7; 768 x 768, 19 rows 4.3 -> 2.5, 1024 rows 5.3 -> 4.1; 2304 x 768,
// 128 rows 5.2 -> 3.4.
// Beside another batch group half of the chip is there for it (few rows beside another group: forced groups, or no packed copies; us, forward of 6 layers of width 512, counting on the whole chip / on
// half of it: FP16 at 2048 and 1920 rows 540 / 486, Fully-Quant at 2 x 2048 rows 386 / 372).
constexpr int CUS = 256;
long cus_for(Rows rows) { return rows.beside ? CUS / 2 : CUS; }
template <class Epi, int MT, int NT, int NWAVES, int R>
bool small_fits(const Epi &epi, Rows rows, int N)
{
    typedef SmallGemm<Epi, MT, NT, NWAVES, R> G;
    if (N % G::BN) return false;
    const size_t lds = G::TAB_OFF + (size_t)Epi::NTAB * G::BN * sizeof(float) + extra_lds_of(epi, 0);
    const long per_cu = std::min<long>((long)(160 * 1024 / lds), 2048 / (64 * NWAVES));
    return (long)(N / G::BN) * ((rows.host_rows + G::BM - 1) / G::BM) <= cus_for(rows) * per_cu;
}
template <class Epi, int NWAVES, int R1, int R2>
hipError_t launch_small_waves(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    if (small_fits<Epi, 2, 1, NWAVES, R1>(epi, rows, N)) return launch_small<Epi, 2, 1, NWAVES, R1>(A, W, out, epi, rows, N, K, st, tm);
    if (small_fits<Epi, 2, 2, NWAVES, R2>(epi, rows, N)) return launch_small<Epi, 2, 2, NWAVES, R2>(A, W, out, epi, rows, N, K, st, tm);
    if (small_fits<Epi, 4, 2, NWAVES, 1>(epi, rows, N)) return launch_small<Epi, 4, 2, NWAVES, 1>(A, W, out, epi, rows, N, K, st, tm);
    if (small_fits<Epi, 4, 4, NWAVES, 1>(epi, rows, N)) return launch_small<Epi, 4, 4, NWAVES, 1>(A, W, out, epi, rows, N, K, st, tm);
    return hipErrorNotSupported;
}
template <class Epi>
hipError_t launch_small_any(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    if (i8_small_waves(K) == 8) {                                 // eight waves; rings as deep as LDS allows where a wave has more than one slab
        if (K > 1024) return launch_small_waves<Epi, 8, 3, 2>(A, W, out, epi, rows, N, K, st, tm);
        return launch_small_waves<Epi, 8, 1, 1>(A, W, out, epi, rows, N, K, st, tm);
    }
    // (other numbers of waves are not instantiated: i8_small_waves)
    if (i8_small_waves(K) == 6) return launch_small_waves<Epi, 6, 1, 1>(A, W, out, epi, rows, N, K, st, tm);
    return hipErrorNotSupported;
}

// ---- LayerNorm step and the GEMM behind it, few rows -------------------------------------------------------------
// Up to some dozens of tokens a layer is a chain of launches, each 3.6 us long whatever it does.  Here every block forms the LayerNorm rows
// that it multiplies by itself: a wave one row (int8 in, residual and out; the arithmetic of add_ln_wave_kernel), its codes into LDS, then the
// wave's 128 channels of K times 64 channels of packed weights, which were requested before the row was; the waves' partial sums meet in
// LDS.  K = 128 NW: six and eight waves, the widths of the two BERT models; two and four (256, 512) are not built, nor is an FP16 input or
// output (Quant-FFN-Only layers take the two launches).  The blocks of the first 64 channels store the codes for the next residual.  What a launch and its gap cost (3.9 us) is
// replaced by the row's arithmetic (0.7 us), done again by every block of its row.
template <class Epi, int NW>
struct LnGemm {
    static constexpr int K = 128 * NW, STRIDE = K + 16, A_OFF = NW * 4096, TAB_OFF = A_OFF + NW * STRIDE;
};

template <class Epi, int NW>
__global__ __launch_bounds__(64 * NW)
void gemm_nt_ln_kernel(const char *__restrict__ Wp, const int *a_dev_rows, const void *a_in, const void *a_res, const float *a_bias,
                       const float *a_gamma, int a_host_rows, int tiles_n, AddLnArgs a, char *__restrict__ out, Epi epi, int N)
{
    a.in = a_in, a.res = a_res, a.bias = a_bias, a.gamma = a_gamma;
    a.rows.dev_rows = a_dev_rows, a.rows.host_rows = a_host_rows;
    typedef LnGemm<Epi, NW> G;
    constexpr int K = G::K, CPL = K / 64;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    float *tab = reinterpret_cast<float *>(lds + G::TAB_OFF);
    const int M = a.rows.dev_rows ? *a.rows.dev_rows : a.rows.host_rows;
    const int tiles_m = (M + NW - 1) / NW, tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    // (a divisor among the preloaded arguments would take the place of a vector's address: BERT-large 1 x 19 529 / 540 us)
    const int m0 = (tile % tiles_m) * NW, n0 = (tile / tiles_m) * 64;          // channels outermost: an XCD reads an eighth of the weights
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, q = lane >> 4;

    const auto weights = buffer_of(Wp);
    v4i w[2][4];
#pragma unroll
    for (int t = 0; t < 4; t++)
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
            w[ks][t] = __builtin_amdgcn_raw_buffer_load_b128(weights, 16 * lane, ((n0 / 16 + t) * (K / 64) + 2 * wave + ks) * 1024, 0);
    epi.load_tables_direct(tab, n0, 64, wave, NW, lane);

    const int row = m0 + wave, c = lane * CPL;
    float z[CPL], gamma[CPL], beta[CPL], y[CPL];
    const double sum = ln_row_wave<CPL, true, true>(a, min(row, M - 1), c, z, gamma, beta);
    ln_normalise_wave<CPL>(z, sum, gamma, beta, a.eps, y);
    const float inv_s = 1.0f / a.s_out;
#pragma unroll
    for (int d = 0; d < CPL / 4; d++) {
        const int codes = pack_row_codes(y + 4 * d, inv_s);
        *reinterpret_cast<int *>(lds + G::A_OFF + wave * G::STRIDE + c + 4 * d) = codes;
        if (n0 == 0 && row < M) *reinterpret_cast<int *>((int8_t *)a.out + (size_t)row * K + c + 4 * d) = codes;
    }
    wait_vm_and_barrier<0>();                                     // the rows and the direct loads of the tables are in LDS

    v4i acc[4];
#pragma unroll
    for (int t = 0; t < 4; t++) acc[t] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {                              // (a product has sixteen rows; those past the block's NW repeat the last one)
        const v4i f = *reinterpret_cast<const v4i *>(lds + G::A_OFF + min(r, NW - 1) * G::STRIDE + wave * 128 + ks * 64 + q * 16);
#pragma unroll
        for (int t = 0; t < 4; t++) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[ks][t], f, acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 4; t++) *reinterpret_cast<v4i *>(lds + (wave * 4 + t) * 1024 + lane * 16) = acc[t];
    __syncthreads();
    if (wave >= 4) return;                                        // lane: token r, channels 16 wave + 4 q .. + 3
    v4i total = {0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < NW; u++) total += *reinterpret_cast<const v4i *>(lds + (u * 4 + wave) * 1024 + lane * 16);
    const int nl = 16 * wave + 4 * q, pk = epi.four(total, tab, 64, nl);
    if (r < NW && m0 + r < M) *reinterpret_cast<int *>(out + (size_t)(m0 + r) * N + n0 + nl) = pk;
}

template <class Epi, int NW>
hipError_t launch_ln_gemm(const AddLnArgs &a, const void *Wp, void *out, const Epi &epi, int N, hipStream_t st)
{
    typedef LnGemm<Epi, NW> G;
    // 57984 bytes at most (1024 channels, 2048 bins); a launch gets 64 KB without asking for more
    static_assert(G::TAB_OFF + 2 * 64 * sizeof(float) + GELU_TABLE_MAX_BINS * 8 <= 64 * 1024, "");
    const size_t LDS = G::TAB_OFF + 2 * 64 * sizeof(float) + extra_lds_of(epi, 0);
    const int tiles_n = N / 64, tiles_m = (a.rows.host_rows + NW - 1) / NW;
    launch_kernel(gemm_nt_ln_kernel<Epi, NW>, dim3(tiles_n * tiles_m), dim3(64 * NW), LDS, st, nullptr, (const char *)Wp, a.rows.dev_rows,
                  a.in, a.res, a.bias, a.gamma, a.rows.host_rows, tiles_n, a, (char *)out, epi, N);
    return hipGetLastError();
}
template <class Epi>
hipError_t launch_ln_gemm_width(const AddLnArgs &a, const void *Wp, void *out, const Epi &epi, int N, hipStream_t st)
{
    if (a.H == 768) return launch_ln_gemm<Epi, 6>(a, Wp, out, epi, N, st);
    if (a.H == 1024) return launch_ln_gemm<Epi, 8>(a, Wp, out, epi, N, st);
    return hipErrorNotSupported;
}

// The FP16 counterpart.  Binary32 sums are formed in K order whatever the tile, so K is not split; what four waves share is the
// issue of the loads (one wave that loads and multiplies spends most of its time issuing loads: 768 x 3072, 19 rows, 13 us).
// A block of four waves computes 32 tokens x 32 CW channels: all waves stream the operands through an R-deep ring of stages of
// four 128-byte slabs, wave w loading slab w, and the first CW waves each multiply one 32 x 32 tile.
template <int CW, int R>
__global__ __launch_bounds__(256)
void gemm_nt_small_f16_kernel(const char *__restrict__ A, const char *__restrict__ W, const int *__restrict__ dev_rows, int host_rows, int N, int Kbytes,
                              int tiles_n, unsigned by_m, char *__restrict__ out, EpiF16 epi)
{
    constexpr int BM = 32, BN = 32 * CW, SLAB = (BM + BN) * 128, PIECES = SLAB / 1024, STAGE = 4 * SLAB;
    static_assert(R >= 2 && (R - 1) * PIECES < 64, "wait count range");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int M = dev_rows ? *dev_rows : host_rows;
    const int tiles_m = (M + BM - 1) / BM, tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= tiles) return;
    const int tile = xcd_contiguous(blockIdx.x, tiles);
    const TileAt at = tile_channels_first(tile, tiles_m, (host_rows + BM - 1) / BM, by_m);
    const int m0 = at.m * BM, n0 = at.n * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 31, g = lane >> 5;
    const char *src[PIECES];
#pragma unroll
    for (int j = 0; j < PIECES; j++) {
        const int row = 8 * j + (lane >> 3), chunk = ((lane & 7) ^ swz<128>(row)) << 4;
        src[j] = (j < BM / 8 ? A + (size_t)min(m0 + row, M - 1) * Kbytes : W + (size_t)(n0 + row - BM) * Kbytes) + chunk + wave * 128;
    }
    auto issue = [&](int st, int slot) {
#pragma unroll
        for (int j = 0; j < PIECES; j++)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[j] + (size_t)st * 512),
                                             (__attribute__((address_space(3))) void *)(lds + slot * STAGE + wave * SLAB + j * 1024), 16, 0, 0);
    };
    const int stages = Kbytes / 512;
#pragma unroll
    for (int s = 0; s < R - 1; s++)
        if (s < stages) issue(s, s);
    v16f acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.0f;
    const unsigned lbase = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    unsigned off[4];
#pragma unroll
    for (int k = 0; k < 4; k++) off[k] = lbase + r * 128 + (((2 * k + g) ^ swz<128>(r)) << 4);
    const int w_off = (BM + 32 * wave) * 128;
    int slot = 0, fill = R - 1;
    for (int st = 0; st < stages; st++) {
        if (st + R - 2 < stages) wait_vm_and_barrier<(R - 2) * PIECES>(); else wait_vm_and_barrier<0>();
        if (st + R - 1 < stages) issue(st + R - 1, fill);          // takes the place of the stage read before the barrier
        if (wave < CW) {
            // fragments of slab u + 1 are on their way from LDS while slab u is multiplied
            v4i fa[2][4], fw[2][4];
            auto fetch = [&](int u) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    fa[u & 1][k] = lds_read128<0>(off[k] + slot * STAGE + u * SLAB);
                    fw[u & 1][k] = lds_read128<0>(off[k] + slot * STAGE + u * SLAB + w_off);
                }
            };
            fetch(0);
#pragma unroll
            for (int u = 0; u < 4; u++) {
                if (u < 3) { fetch(u + 1); wait_lds_reads<8>(); } else wait_lds_reads<0>();
                tie(fa[u & 1], std::make_integer_sequence<int, 4>());
                tie(fw[u & 1], std::make_integer_sequence<int, 4>());
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 4; k++) acc = F16::mma(fw[u & 1][k], fa[u & 1][k], acc);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        slot = slot + 1 == R ? 0 : slot + 1;
        fill = fill + 1 == R ? 0 : fill + 1;
    }
    if (wave >= CW) return;
    const int row = m0 + r, n = n0 + 32 * wave + 4 * g;
    EpiF16::Tab t;
#pragma unroll
    for (int q = 0; q < 4; q++) t.b[q] = epi.bias ? *reinterpret_cast<const v4f *>(epi.bias + n + 8 * q) : v4f{0.f, 0.f, 0.f, 0.f};
    v2i pk[4];
    epi.tile(acc, t, nullptr, BN, 0, g, pk);
    if (row < M) {
#pragma unroll
        for (int q = 0; q < 4; q++) *reinterpret_cast<v2i *>(out + ((size_t)row * N + n + 8 * q) * 2) = pk[q];
    }
}

template <int CW, int R>
hipError_t launch_small_f16(const void *A, const void *W, void *out, const EpiF16 &epi, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    const size_t LDS = (size_t)R * (32 + 32 * CW) * 512;
    if (N % (32 * CW) || K % 256) return hipErrorInvalidValue;
    auto kern = gemm_nt_small_f16_kernel<CW, R>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_n = N / (32 * CW), tiles_m = (rows.host_rows + 31) / 32;
    launch_kernel(kern, dim3(tiles_n * tiles_m), dim3(256), LDS, st, tm, (const char *)A, (const char *)W, rows.dev_rows,
                  rows.host_rows, N, K * 2, tiles_n, divisor(tiles_n * tiles_m, tiles_m), (char *)out, epi);
    return hipGetLastError();
}

// As for INT8: the smallest tile that the chip holds all at once.  Us per launch in a chain (before: 64 x 96 tiles): 768 x 3072,
// 19 rows 17.4 -> 10.8, 427 rows 17.8 -> 11.8; 768 x 768, 19 rows 6.0 -> 4.2; 2304 x 768, 128 rows 7.6 -> 5.6.  The widest tile
// reads its operands too slowly for long rows (768 x 3072, 1024 rows: 19.5 against 17.9 us).
hipError_t launch_small_f16_any(const void *A, const void *W, void *out, const EpiF16 &epi, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    if (K % 256) return hipErrorNotSupported;
    const long tiles_m = (rows.host_rows + 31) / 32;
    if (N % 32 == 0 && f16_small_tiles(rows.host_rows, N) <= 2 * cus_for(rows)) return launch_small_f16<1, 2>(A, W, out, epi, rows, N, K, st, tm);      // two blocks per CU
    if (N % 64 == 0 && tiles_m * (N / 64) <= cus_for(rows)) return launch_small_f16<2, 2>(A, W, out, epi, rows, N, K, st, tm);
    if (N % 128 == 0 && K <= 1024 && tiles_m * (N / 128) <= cus_for(rows)) return launch_small_f16<4, 2>(A, W, out, epi, rows, N, K, st, tm);
    return hipErrorNotSupported;
}

// Tile configuration per problem shape, for weights as they lie (who comes here: the top of this file; figures of the widths 768 and 1024 were
// taken when every encoder did).  What bounds the main loop on this chip is the rate at which
// a CU pulls operand stages out of L2 (20 to 40 bytes per clock per CU, whichever way they are loaded),
// so small problems want many small tiles (more CUs pulling), large ones the larger tile (less traffic):
//   0: 128 x 128 tile, 64-byte stages, 4-deep ring  (any K that is a multiple of 64 bytes)
//   1: 128 x 128 tile, 128-byte stages (whole cache lines per row), 2-deep ring, 2 blocks per CU
//   2: 64 tokens x 128 channels, otherwise as 1: up to about two and a half 128 x 128 tiles per CU; rows of
//      3072 bytes or more (FFN2) get a 3-deep ring (72 KB, still two blocks per CU) when there is at most one
//      block per CU: -4 % on the BERT-base forward (with more blocks than CUs it measured slower); a 4-deep ring is faster for the kernel alone but crowds out the other group's kernels
constexpr int LONG_K_BYTES = 3072;
// From 2048 rows the wide GEMMs fill the chip with 128 x 192 tiles; below they leave most CUs idle (us per launch in a chain, 128 x
// 192 against 64 x 128 tiles at 1024 rows: 2304 x 768 9.8 / 7.4, FFN1 3072 x 768 12.1 / 9.1, FFN1 4096 x 1024 17.3 / 11.8, FP16 2304 x
// 768 17.9 / 12.1; at 1536 rows 9.9 / 7.8, 12.3 / 11.7, 17.5 / 15.2, 18.2 / 13.0).  With another batch group on the chip the idle CUs
// are that group's, and the forward crosses earlier (us, 6 layers of width 768, Fully-Quant / MHA-only / Quant-FFN-Only / FP16, 128 x 192
// against 64 x 128 tiles: two groups of 1280 and 1408 rows 424 / 582 / 533 / 653 against 412 / 581 / 499 / 635, of 1408 rows
// 401 / 555 / 443 / 594 against 405 / 575 / 447 / 609, of 1792 rows 412 / 598 / 476 / 668 against 447 / 659 / 503 / 690), where the rows
// are all there: ragged batches, whose padded rows are counted here, stay at 2048 (two groups of 1536 with 984 tokens each:
// Fully-Quant 390 against 384, FP16 570 against 551).
constexpr int WIDE_TILE_MIN_ROWS = 2048, WIDE_TILE_MIN_ROWS_BESIDE = 1408;
constexpr int BIG_TILE_MIN_ROWS = 16384;                         // from here on the 256 x 256 tiles fill the chip several times over

constexpr int big_tile_width(int cfg) { return cfg == 6 ? 192 : 256; }

template <class T, class Epi>
hipError_t launch(const void *A, const void *W, void *out, const Epi &epi, Rows rows, int N, int K, hipStream_t st,
                  const Timing *tm)
{
    int cfg = gemm_config_override.load(std::memory_order_relaxed);
    const bool forced = cfg >= 0;
    const int kbytes = K * T::ELEM;
    if (cfg >= 3 && cfg < 8 && (N % big_tile_width(cfg) || kbytes % 128)) cfg = -1;   // whole columns of tiles, whole 128-byte stages
    if (cfg >= 0 && cfg < 3 && kbytes % 128) cfg = 0;
    if (cfg < 0) {
        if (kbytes % 128) cfg = 0;
        else {
            const int wide_min_rows = rows.beside && !rows.dev_rows ? WIDE_TILE_MIN_ROWS_BESIDE : WIDE_TILE_MIN_ROWS;
            const long tiles = (long)(N / 128) * ((rows.host_rows + 127) / 128);
            // fewer 128 x 128 tiles than CUs: the smaller tiles of configuration 2 (BERT-large's 1024-wide GEMMs at
            // 4096 tokens, 256 tiles, measured -4.4 % on that forward with 128 x 128 against 64 x 128)
            cfg = tiles < 256 ? 2 : 1;
            // wide GEMMs (QKV, FFN1): 128 x 192 tiles, 64 x 96 per wave, two blocks
            // per CU.  Measured in the BERT-base forward at 2 x 2048 tokens: -5 % with FFN1 (whose table-lookup epilogue
            // in the 64 x 128 configuration costs more than it saves: its table in LDS takes the third resident block
            // away), another -1.4 % with QKV; the FP16 forward gains 2 %
            if (N % 192 == 0 && N >= 2304 && rows.host_rows >= wide_min_rows) cfg = 6;
            // widths that 192 does not divide (FFN1 of BERT-large, 4096): 128 x 256 tiles (-3.5 % on that forward
            // at 2 x 4096 tokens against 128 x 128; 256 x 128 -0.5 %, 64 x 128 +5.5 %)
            else if (N % 256 == 0 && N >= 2304 && rows.host_rows >= wide_min_rows) cfg = 4;
            // many tokens (INT8): the 128 x 192 tiles also where few rows of tiles would do with larger ones (BERT-base 128 x 512,
            // 128 x 256 tiles of 64-byte stages: +0.5 %); long operand rows amortise the epilogue of a 256 x 256 tile by
            // themselves (FFN2 there on 128 x 192: +1.4 %); 128 x 256 where 192 does not divide the width
            if (std::is_same<T, I8>::value && N % 256 == 0 && rows.host_rows >= BIG_TILE_MIN_ROWS)
                cfg = kbytes >= LONG_K_BYTES ? 7 : N % 192 == 0 ? 6 : 4;
        }
    }
    if constexpr (std::is_same<T, I8>::value && (std::is_same<Epi, EpiRequant>::value || std::is_same<Epi, EpiGeluTable>::value)) {
        if (!forced) {
            const hipError_t e = launch_small_any<Epi>(A, W, out, epi, rows, N, K, st, tm);
            if (e != hipErrorNotSupported) return e;
        }
    }
    if constexpr (std::is_same<T, F16>::value) {
        if (!forced) {
            const hipError_t e = launch_small_f16_any(A, W, out, epi, rows, N, K, st, tm);
            if (e != hipErrorNotSupported) return e;
        }
    }
    switch (cfg) {
    case 3: return launch_big<T, Epi, 4, 4, 128, 2>(A, W, out, epi, rows, N, K, st, tm);      // 256 x 256, two 128-byte stages
    case 4: return launch_big<T, Epi, 2, 4, 64, 3, 2>(A, W, out, epi, rows, N, K, st, tm);    // 128 tokens x 256 channels, two blocks per CU
    case 5: return launch_big<T, Epi, 4, 2, 64, 3, 2>(A, W, out, epi, rows, N, K, st, tm);    // 256 tokens x 128 channels, two blocks per CU
    case 6: return launch_big<T, Epi, 2, 3, 128, 2, 2>(A, W, out, epi, rows, N, K, st, tm);   // 128 x 192, two 128-byte stages, two blocks per CU
    case 7: return launch_big<T, Epi, 4, 4, 64, 4>(A, W, out, epi, rows, N, K, st, tm);       // 256 x 256, four 64-byte stages
    case 1:
        // the GELU epilogue is as much vector work as the main loop is matrix work: 64-byte stages leave room
        // for three resident blocks per CU, whose epilogues and main loops overlap (-3 % on the large forwards)
        if constexpr (std::is_same<Epi, EpiGeluQuant>::value || std::is_same<Epi, EpiGeluTable>::value)
            return launch_cfg<T, Epi, 2, 2, 64, 3, 3>(A, W, out, epi, rows, N, K, st, tm);
        else return launch_cfg<T, Epi, 2, 2, 128, 2, 2>(A, W, out, epi, rows, N, K, st, tm);
    case 2: {
        const long row_tiles = (rows.host_rows + 63) / 64;
        const bool long_k = K * T::ELEM >= LONG_K_BYTES;
        // 64 x 96 tiles (six waves of 32 x 32) when they put the problem on more CUs without exceeding one block
        // per CU: the rate at which one CU pulls operands is what bounds these small problems
        if (!forced && N % 96 == 0 && (N / 96) * row_tiles <= 256) {
            // (measured in the BERT-base forward at 2 x 2048 tokens: two stages held in registers -2 %, three +11 %,
            // six +3 % against the three-deep LDS ring, although six is the fastest alone: 12.3 against 14.2 us)
            if constexpr (Epi::STAGED && !std::is_same<Epi, EpiGeluTable>::value) {
                // (also for short rows: the attention-output GEMM; same speed in the batch-32 forward, -4 % for one sequence)
                if (kbytes % 256 == 0) return launch_longk<T, Epi, 3, 2>(A, W, out, epi, rows, N, K, st, tm);
            }
            if (long_k) return launch_cfg<T, Epi, 1, 1, 128, 3, 2, 2, 3>(A, W, out, epi, rows, N, K, st, tm);
            return launch_cfg<T, Epi, 1, 1, 128, 2, 2, 2, 3>(A, W, out, epi, rows, N, K, st, tm);
        }
        if constexpr (Epi::STAGED && !std::is_same<Epi, EpiGeluTable>::value) {
            if (!forced && long_k && kbytes % 256 == 0 && (N / 128) * row_tiles <= 256)
                return launch_longk<T, Epi, 4, 2>(A, W, out, epi, rows, N, K, st, tm);
        }
        if (long_k && (N / 128) * row_tiles <= 256) return launch_cfg<T, Epi, 1, 2, 128, 3, 2>(A, W, out, epi, rows, N, K, st, tm);
        return launch_cfg<T, Epi, 1, 2, 128, 2, 2>(A, W, out, epi, rows, N, K, st, tm);
    }
    default: return launch_cfg<T, Epi, 2, 2, 64, 4, 2>(A, W, out, epi, rows, N, K, st, tm);
    }
}

}  // namespace

std::atomic<int> gemm_config_override{-1};                    // tuning aid: force one tile configuration (see launch())

bool gemm_i8_reads_rows(Rows rows, int N, int K) { return i8_reads_rows(rows.host_rows, N, K); }

hipError_t launch_gemm_i8(GemmEpilogue epi, const int8_t *A, const int8_t *W, const int8_t *Wp, void *out, const float *m, const float *b,
                          float inv_s_out, const GeluTable *gt, Rows rows, int N, int K, hipStream_t st, const Timing *tm)
{
    if (Wp && gemm_config_override.load(std::memory_order_relaxed) < 0 && !gemm_i8_reads_rows(rows, N, K)) {
        const hipError_t e = launch_gemm_i8_packed(epi, A, Wp, out, m, b, gt, rows, N, K, -1, st, tm);
        if (e != hipErrorNotSupported) return e;
    }
    switch (epi) {
    case EPI_RAW_I32: return launch<I8>(A, W, out, EpiRawI32{(int32_t *)out, N}, rows, N, K, st, tm);
    case EPI_REQUANT: return launch<I8>(A, W, out, EpiRequant{m, b}, rows, N, K, st, tm);
    case EPI_GELU_QUANT:
        if (gt && gt->entries)
            return launch<I8>(A, W, out, EpiGeluTable{m, b, gt->entries, gt->spec.rate, gt->spec.offset, gt->spec.t_max, gt->spec.bins},
                              rows, N, K, st, tm);
        return launch<I8>(A, W, out, EpiGeluQuant{m, b, inv_s_out}, rows, N, K, st, tm);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_i8_packed(GemmEpilogue epi, const int8_t *A, const int8_t *Wp, void *out, const float *m, const float *b,
                                 const GeluTable *gt, Rows rows, int N, int K, int tile, hipStream_t st, const Timing *tm)
{
    if (epi == EPI_REQUANT) return launch_packed(A, Wp, out, EpiRequant{m, b}, rows, N, K, tile, st, tm);
    if (epi == EPI_GELU_QUANT && gt && gt->entries)
        return launch_packed(A, Wp, out, EpiGeluTable{m, b, gt->entries, gt->spec.rate, gt->spec.offset, gt->spec.t_max, gt->spec.bins},
                             rows, N, K, tile, st, tm);
    return hipErrorNotSupported;
}

// Beyond, the two launches are faster: the rows' arithmetic is done once per 64 channels of the result.  One sequence, Fully-Quant, us per
// forward, two launches / one: BERT-base 1 token 289 / 265, 19 302 / 275, 32 307 / 293, 48 317 / 304, 64 328 / 328; BERT-large 1 660 / 597, 19 707 / 621,
// 32 747 / 644, 48 739 / 724, 64 761 / 755
constexpr int LN_GEMM_MAX_ROWS = 64;
hipError_t launch_ln_gemm_i8(const AddLnArgs &a, GemmEpilogue epi, const int8_t *Wp, void *out, const float *m, const float *b, const GeluTable *gt,
                             int N, hipStream_t st)
{
    if (a.rows.host_rows > LN_GEMM_MAX_ROWS || !Wp || N % 64 || !a.in_i8 || !a.res_i8 || !a.out_i8 || a.row_map || a.absmax_out ||
        gemm_config_override.load(std::memory_order_relaxed) >= 0)
        return hipErrorNotSupported;
    if (epi == EPI_REQUANT) return launch_ln_gemm_width(a, Wp, out, EpiRequant{m, b}, N, st);
    if (epi == EPI_GELU_QUANT && gt && gt->entries)
        return launch_ln_gemm_width(a, Wp, out, EpiGeluTable{m, b, gt->entries, gt->spec.rate, gt->spec.offset, gt->spec.t_max, gt->spec.bins}, N, st);
    return hipErrorNotSupported;
}

hipError_t launch_gemm_f16_packed(const __half *A, const __half *Wp, const float *bias, bool gelu, __half *out, Rows rows, int N, int K,
                                  int tile, hipStream_t st, const Timing *tm)
{
    return launch_packed_f16(A, Wp, out, EpiF16{bias, gelu}, rows, N, K, tile, st, tm);
}

bool gemm_f16_reads_rows(Rows rows, int N, int K) { return f16_reads_rows(rows.host_rows, N, K, cus_for(rows)); }

hipError_t launch_gemm_f16(const __half *A, const __half *W, const __half *Wp, const float *bias, bool gelu, __half *out, Rows rows,
                           int N, int K, hipStream_t st, const Timing *tm)
{
    if (Wp && gemm_config_override.load(std::memory_order_relaxed) < 0 && !gemm_f16_reads_rows(rows, N, K)) {
        const hipError_t e = launch_gemm_f16_packed(A, Wp, bias, gelu, out, rows, N, K, -1, st, tm);
        if (e != hipErrorNotSupported) return e;
    }
    return launch<F16>(A, W, out, EpiF16{bias, gelu}, rows, N, K, st, tm);
}

}  // namespace samp
