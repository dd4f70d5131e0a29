// Pieces of the LDS-staged MFMA tile loop that more than one kernel file uses: the chunk swizzle of a stage row,
// explicit waits, and operand-fragment reads with waits of their own.
#pragma once
#include "samp_common.h"

#include <type_traits>
#include <utility>

namespace samp {
namespace {

// XOR swizzle of the 16-byte chunk index inside an LDS row of BKB bytes (BKB = 64: 4 chunks,
// BKB = 128: 8 chunks), chosen so that the lanes of one ds_read_b128 phase hit distinct banks.
template <int BKB>
__device__ __forceinline__ int swz(int row)
{
    if constexpr (BKB == 64) return ((row >> 1) & 3) ^ ((row >> 3) & 1);
    else return (row & 7) ^ ((row >> 3) & 1);
}

// wait until at most N vector-memory operations of this wave are outstanding and all of its LDS
// reads have returned, then barrier.  The "memory" clobber keeps the compiler from moving LDS
// accesses across it.
template <int N>
__device__ __forceinline__ void wait_vm_and_barrier()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int N> __device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// all LDS reads of the wave have returned: what they read may be overwritten by direct loads
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Loads through a buffer descriptor: scalar base + 32-bit vector offset + scalar offset, so no address arithmetic in vector registers.  The
// compiler counts such loads one by one when it waits for a register; after a direct load of the global_load_lds kind, which it takes for
// one that may return out of order, it waits for all that are in flight.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base)          // no bounds check
{ return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, 0xffffffffu, 0x00027000); }
// `bytes` of it are there: beyond, loads return zeros
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, int bytes)
{ return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00027000); }
// 16 or 4 bytes per lane, one lane's behind the other's in LDS
__device__ __forceinline__ void buffer_to_lds128(__amdgpu_buffer_rsrc_t from, unsigned offset, unsigned scalar_offset, void *lds)
{ __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)lds, 16, offset, scalar_offset, 0, 0); }
__device__ __forceinline__ void buffer_to_lds32(__amdgpu_buffer_rsrc_t from, unsigned offset, void *lds)
{ __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)lds, 4, offset, 0, 0, 0); }

// Fragment fetches of the large-tile kernel are written as ds_read_b128 instructions of its own, with
// explicit waits: left to the compiler, every group of MFMAs is preceded by a wait for ALL outstanding
// LDS reads, including the ones just issued for the step after it, which puts the LDS latency in front
// of every step instead of behind the MFMAs of the step before.  tie() makes later uses of a fragment
// depend on the wait that precedes it (an empty instruction that "rewrites" the register).
template <int OFFSET> __device__ __forceinline__ v4i lds_read128(unsigned addr)
{
    v4i v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET));
    return v;
}
template <int STRIDE, int N, int... I>
__device__ __forceinline__ void lds_read_frags(unsigned addr, v4i (&f)[N], std::integer_sequence<int, I...>)
{
    ((f[I] = lds_read128<I * STRIDE>(addr)), ...);
}
__device__ __forceinline__ int tie_one(v4i &f)
{
    asm volatile("" : "+v"(f));
    return 0;
}
template <int N, int... I> __device__ __forceinline__ void tie(v4i (&f)[N], std::integer_sequence<int, I...>)
{
    (void)(tie_one(f[I]) + ... + 0);
}
template <int N> __device__ __forceinline__ void wait_lds_reads()
{
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}

// ---- tile loop on packed weights -----------------------------------------------------------------
// A block's four waves stand side by side: each multiplies all token rows of the block by weight rows of its own.  The token rows travel
// through LDS (a ring of D + 1 stages of 128 bytes a row, direct loads); the weight rows, which no other wave wants, come straight into
// registers, D stages ahead, in the order of the matrix product (pack_weight_kernel: 1 KB per 16 rows x 64 bytes for the 16 x 16 x 64 product
// of INT8, per 32 rows x 32 bytes for the 32 x 32 x 16 product of FP16, whose sums are formed in the order of every other FP16 kernel).
template <class F, int... I> __device__ __forceinline__ void each_index(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>()), ...);
}
template <bool HALF> struct StreamGeometry {
    static constexpr int ROWS = HALF ? 32 : 16;                   // token rows of a product, and weight rows
    static constexpr int KS = HALF ? 4 : 2;                       // products along a stage
};
template <bool HALF, int MT, int D> constexpr int stream_ring_bytes() { return (D + 1) * StreamGeometry<HALF>::ROWS * MT * 128; }
template <bool HALF, int MT> constexpr int stream_loads() { return StreamGeometry<HALF>::ROWS * MT / 32; }     // token-row loads of a wave and stage

// MT token tiles, NTW weight blocks per wave.  SPLIT: the block's token rows are split over that many groups of waves (this wave's: part), so
// that waves of different groups load the same weights.  abase: first token row; offa: this lane's offsets into the rows of its pieces (8 rows x 128
// bytes, swizzled); wbase: the wave's packed row blocks; KT: stages of 128 bytes, a multiple of D.  started() runs once the first stage is
// requested; what it loads into LDS is there for all waves behind the barrier that ends the first stage, so it is for use after the loop, not in
// mma (KT >= 2); mma(t, i, w, f) adds the product of weight block t and token tile i.
// On return the ring is idle.
template <bool HALF, int MT, int NTW, int D, int SPLIT = 1, class Started, class Mma>
__device__ __forceinline__ void stream_tile_loop(const char *abase, const unsigned (&offa)[stream_loads<HALF, MT * SPLIT>()], const char *wbase,
                                                 const unsigned (&woff)[NTW], int KT, char *lds, int wave, int lane, Started started, Mma mma,
                                                 int part = 0)
{
    constexpr int ROWS = StreamGeometry<HALF>::ROWS, KS = StreamGeometry<HALF>::KS, TILE = ROWS * 128;
    constexpr int SLOT = TILE * MT * SPLIT, RING = stream_ring_bytes<HALF, MT * SPLIT, D>();
    constexpr int G = MT < 4 ? MT : 4, H = MT / G, STEPS = KS * H;         // token tiles per step; steps of a stage
    constexpr int NLDA = stream_loads<HALF, MT * SPLIT>(), PER = NLDA + KS * NTW;  // loads of a wave and stage: token rows; all
    static_assert(MT % G == 0 && H <= 2 && D >= 2 && NLDA >= 1, "whole steps, whole pieces per wave");
    const int r = lane & (ROWS - 1), q = lane / ROWS;
    const unsigned offw = 16 * lane;
    int fill = 0;                                                 // ring position of the next stage to request
    const auto rows = buffer_of(abase), weights = buffer_of(wbase);
    auto issue_a = [&](int kt, int first, int last) {
#pragma unroll
        for (int j = first; j < last; j++) buffer_to_lds128(rows, offa[j], kt * 128, lds + fill + (wave + 4 * j) * 1024);
        if (last == NLDA) fill = fill + SLOT == RING ? 0 : fill + SLOT;
    };
    v4i w[D][KS][NTW];
    auto load_w = [&](int kt, int ks, v4i (&d)[NTW]) {
#pragma unroll
        for (int t = 0; t < NTW; t++) d[t] = __builtin_amdgcn_raw_buffer_load_b128(weights, offw, woff[t] + (KS * kt + ks) * 1024, 0);
    };
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    unsigned addr[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++) addr[ks] = lds_base + part * (MT * TILE) + r * 128 + (((8 / KS * ks + q) ^ swz<128>(r)) << 4);

#pragma unroll
    for (int s = 0; s < D; s++) {
        issue_a(s, 0, NLDA);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ks++) load_w(s, ks, w[s][ks]);
        if (s == 0) {
            started();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    v4i fa[2][G];
    int slot = 0;
    auto fetch = [&](auto idx_tag, v4i (&f)[G]) {
        constexpr int OFF = (decltype(idx_tag)::value % H) * G * TILE;
        lds_read_frags<TILE>(addr[decltype(idx_tag)::value / H] + slot + OFF, f, std::make_integer_sequence<int, G>());
    };
    constexpr std::integral_constant<int, 0> c0;
    // One step multiplies G token tiles by the wave's channels along one product's K, with the token fragments of the step after it on
    // their way from LDS.  The loads of the stage D further on are dealt out over the steps (a burst of them would hold the wave up
    // at its issue, with the matrix cores idle): token rows in each, weights into the registers that the step before has read last.
    // LEFT: stages after this one, D where there are that many or more (copies of the code instead of tests: the waits are constants).
    // The compiler waits for the weights.  For the token rows, which it does not see in LDS, each stage lets stay in flight what was
    // requested behind them: no less than this stage's loads so far, those of the stages in between, and the next stage's last weights
    // (load order inside a step is the compiler's; across the scheduling barriers it stays).
    auto step = [&](auto left_tag, auto b_tag, auto idx_tag, int kt) {
        constexpr int LEFT = decltype(left_tag)::value, B = decltype(b_tag)::value, IDX = decltype(idx_tag)::value, ks = IDX / H, h = IDX % H;
        constexpr bool MORE = LEFT == D;
        if constexpr (MORE) {
            issue_a(kt + D, NLDA * IDX / STEPS, NLDA * (IDX + 1) / STEPS);
            if constexpr (ks > 0 && h == 0) load_w(kt + D, ks - 1, w[B][ks - 1]);
        }
        if constexpr (IDX + 1 < STEPS) {
            fetch(std::integral_constant<int, IDX + 1>(), fa[(IDX + 1) & 1]);
            wait_lds_reads<G>();
        } else if constexpr (LEFT > 0) {                          // the next stage's token rows have landed
            wait_vm_and_barrier<NTW + (MORE ? (D - 2) * PER + NLDA + (KS - 1) * NTW : (LEFT - 1) * PER)>();
            slot = slot + SLOT == RING ? 0 : slot + SLOT;
            fetch(c0, fa[0]);
        } else {
            wait_lds_reads<0>();
        }
        tie(fa[IDX & 1], std::make_integer_sequence<int, G>());
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NTW; t++)
#pragma unroll
            for (int i = 0; i < G; i++) mma(t, G * h + i, w[B][ks][t], fa[IDX & 1][i]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE && IDX + 1 == STEPS) load_w(kt + D, KS - 1, w[B][KS - 1]);
    };
    auto stage = [&](auto left_tag, auto b_tag, int kt) {
        each_index([&](auto idx) { step(left_tag, b_tag, idx, kt); }, std::make_integer_sequence<int, STEPS>());
    };
    wait_vm_and_barrier<(KS - 1) * NTW + (D - 1) * PER>();
    fetch(c0, fa[0]);
    const auto all = std::make_integer_sequence<int, D>();
    for (int kt = 0; kt + D < KT; kt += D) each_index([&](auto b) { stage(std::integral_constant<int, D>(), b, kt + b); }, all);
    each_index([&](auto b) { stage(std::integral_constant<int, D - 1 - decltype(b)::value>(), b, 0); }, all);
    __syncthreads();
}

}  // namespace
}  // namespace samp
