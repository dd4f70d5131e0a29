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

// ---- tile loop on packed weights (INT8) ----------------------------------------------------------
// A block's four waves stand side by side: each multiplies all 16 MT token rows of the block by 16 NTW weight rows of its own.  The token rows
// travel through LDS (a ring of D + 1 stages of 128 bytes a row, direct loads); the weight rows, which no other wave wants, come straight
// into registers, D stages ahead, in the order of the 16 x 16 x 64 product (pack_weight_kernel: 1 KB per 16 rows x 64 bytes).
template <class F, int... I> __device__ __forceinline__ void each_index(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>()), ...);
}
template <int MT, int D> constexpr int stream_ring_bytes() { return (D + 1) * 16 * MT * 128; }

// abase: first token row; offa: this lane's offsets into the rows of its pieces (8 rows x 128 bytes, swizzled); wbase: the wave's packed
// row blocks; KT: stages of 128 bytes, a multiple of D.  started() runs once the first stage is requested (what it loads has arrived when
// the first product runs); mma(t, i, w, f) adds the product of weight block t and token tile i.  On return the ring is idle.
template <int MT, int NTW, int D, class Started, class Mma>
__device__ __forceinline__ void stream_tile_loop(const char *abase, const unsigned (&offa)[MT / 2], const char *const (&wbase)[NTW], int KT, char *lds,
                                                 int wave, int lane, Started started, Mma mma)
{
    constexpr int SLOT = 16 * MT * 128, RING = stream_ring_bytes<MT, D>();
    constexpr int G = MT < 4 ? MT : 4, H = MT / G, STEPS = 2 * H;          // token tiles per step; steps per 64 bytes of K
    constexpr int NLDA = MT / 2, PER = NLDA + 2 * NTW;                     // loads of a wave and stage: token rows; all
    static_assert(MT % G == 0 && H <= 2 && D >= 2, "whole steps");
    const int r = lane & 15, q = lane >> 4;
    const unsigned offw = 16 * lane;
    int fill = 0;                                                 // ring position of the next stage to request
    auto issue_a = [&](int kt, int first, int last) {
        const char *from = abase + (size_t)kt * 128;
        asm volatile("" : "+s"(from));
#pragma unroll
        for (int j = first; j < last; j++) {
            unsigned o = offa[j];
            asm volatile("" : "+v"(o));                            // keeps the offset a 32-bit one: scalar base + vector offset
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(from + o),
                                             (__attribute__((address_space(3))) void *)(lds + fill + (wave + 4 * j) * 1024), 16, 0, 0);
        }
        if (last == NLDA) fill = fill + SLOT == RING ? 0 : fill + SLOT;
    };
    // (written out so that the compiler does not wait for them: step() does, and ties the registers to its wait)
    v4i w[D][2][NTW];
    auto load_w = [&](int kt, int ks, v4i (&d)[NTW]) {
#pragma unroll
        for (int t = 0; t < NTW; t++)
            asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(d[t]) : "v"(offw), "s"(wbase[t] + (size_t)(2 * kt + ks) * 1024));
    };
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    unsigned addr[2];
#pragma unroll
    for (int ks = 0; ks < 2; ks++) addr[ks] = lds_base + r * 128 + (((4 * ks + q) ^ swz<128>(r)) << 4);

#pragma unroll
    for (int s = 0; s < D; s++) {
        issue_a(s, 0, NLDA);
        load_w(s, 0, w[s][0]);
        load_w(s, 1, w[s][1]);
        if (s == 0) {
            started();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    v4i fa[2][G];
    int slot = 0;
    auto fetch = [&](auto idx_tag, v4i (&f)[G]) {
        constexpr int OFF = (decltype(idx_tag)::value % H) * G * 2048;
        lds_read_frags<2048>(addr[decltype(idx_tag)::value / H] + slot + OFF, f, std::make_integer_sequence<int, G>());
    };
    constexpr std::integral_constant<int, 0> c0;
    constexpr std::integral_constant<int, 1> c1;
    constexpr std::integral_constant<int, 2> c2;
    constexpr std::integral_constant<int, 3> c3;
    // One step multiplies G token tiles by the wave's channels over 64 bytes of K, with the token fragments of the step after it on
    // their way from LDS.  The loads of the stage D further on are dealt out over the steps (a burst of them would hold the wave up
    // at its issue, with the matrix cores idle): token rows in each, weights into the registers that the step before has read last.
    // LEFT: stages after this one, D where there are that many or more (copies of the code instead of tests: the waits are constants).
    auto step = [&](auto left_tag, auto b_tag, auto idx_tag, int kt) {
        constexpr int LEFT = decltype(left_tag)::value, B = decltype(b_tag)::value, IDX = decltype(idx_tag)::value, ks = IDX / H, h = IDX % H;
        constexpr bool MORE = LEFT == D;
        if constexpr (IDX == H) {                                 // the second half of this stage's weights has landed
            wait_vm<MORE ? (D - 1) * PER + NLDA * H / STEPS : LEFT * PER>();
            tie(w[B][1], std::make_integer_sequence<int, NTW>());
        }
        if constexpr (MORE) {
            issue_a(kt + D, NLDA * IDX / STEPS, NLDA * (IDX + 1) / STEPS);
            if constexpr (IDX == H) load_w(kt + D, 0, w[B][0]);
        }
        if constexpr (IDX + 1 < STEPS) {
            fetch(std::integral_constant<int, IDX + 1>(), fa[(IDX + 1) & 1]);
            wait_lds_reads<G>();
        } else if constexpr (LEFT > 0) {                          // so have the next stage's token rows and the first half of its weights
            wait_vm_and_barrier<MORE ? (D - 1) * PER : NTW + (LEFT - 1) * PER>();
            slot = slot + SLOT == RING ? 0 : slot + SLOT;
            fetch(c0, fa[0]);
        } else {
            wait_lds_reads<0>();
        }
        tie(fa[IDX & 1], std::make_integer_sequence<int, G>());
        if constexpr (IDX == 0) tie(w[B][0], std::make_integer_sequence<int, NTW>());
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NTW; t++)
#pragma unroll
            for (int i = 0; i < G; i++) mma(t, G * h + i, w[B][ks][t], fa[IDX & 1][i]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE && IDX + 1 == STEPS) load_w(kt + D, 1, w[B][1]);
    };
    auto stage = [&](auto left_tag, auto b_tag, int kt) {
        step(left_tag, b_tag, c0, kt);
        step(left_tag, b_tag, c1, kt);
        if constexpr (H == 2) { step(left_tag, b_tag, c2, kt); step(left_tag, b_tag, c3, kt); }
    };
    wait_vm_and_barrier<NTW + (D - 1) * PER>();
    fetch(c0, fa[0]);
    const auto all = std::make_integer_sequence<int, D>();
    for (int kt = 0; kt + D < KT; kt += D) each_index([&](auto b) { stage(std::integral_constant<int, D>(), b, kt + b); }, all);
    each_index([&](auto b) { stage(std::integral_constant<int, D - 1 - decltype(b)::value>(), b, 0); }, all);
    __syncthreads();
}

}  // namespace
}  // namespace samp
