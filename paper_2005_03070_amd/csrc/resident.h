// Building blocks of the chip-resident kernels (gfx950): kernels that keep a
// solver's state in registers and LDS for a whole solve and let their
// workgroups talk through memory instead of ending the launch.
//
// Exchange.  A phase's per-workgroup sums and the edge values its neighbours
// need are published as 64-bit words and polled by their readers; a slot
// holds RES_EMPTY (a signalling-NaN pattern that no arithmetic produces)
// until its value arrives, so the value is its own flag and one memory hop
// carries it.  Three buffers alternate by phase.  A workgroup that holds all
// sums of phase q knows that every workgroup has published q, hence finished
// reading q - 1: it then empties its own slots of buffer q - 1 (= q + 2 mod
// 3), and its own sums of q + 1 are published only after those stores have
// completed (s_waitcnt, then the workgroup barrier), so a reader that has
// seen them finds the slots of q + 2 empty or new.  Every access is a relaxed
// device-scope atomic: on gfx950 it bypasses the per-XCD caches, so no fence
// is needed; an acquire/release pair per phase measured 44 us with 256
// workgroups (it writes back and invalidates whole L2s), a flag word beside
// the data 6.4 us, an arrival counter 5.0 us, this exchange 3.6 us (64
// workgroups: 11.5, 4.0, 2.4 and 2.3 us).  Past 32 workgroups the sums take a
// second hop, each value gathered by one workgroup and its total read by all
// (2.6 us with 256): 256 readers of 256 slots a value crowd the memory.
//
// Every workgroup of a team must be resident: the kernels are launched
// cooperatively with at most one workgroup per compute unit, and a team begins
// at a gate that all its workgroups have to reach (res_gate): a kernel of
// another stream or process may hold a unit for as long as it likes.  A team
// that waits there for RES_GATE_TICKS ends without having touched anything, and
// where no team began the host takes the kernels that need no residency.  Past
// the gate a poll that outlasts RES_WAIT_TICKS raises the grid's abort word,
// which every poll watches, so the kernel ends (the host reports an error).
#pragma once

#include "device_common.h"

namespace tgdk {

typedef unsigned long long u64;

constexpr u64 RES_EMPTY = 0x7ff4badc0ffee123ull;
constexpr long long RES_WAIT_TICKS = 20LL * 100000000;  // 20 s of the 100 MHz wall clock

__device__ __forceinline__ u64 res_load(const u64* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_store_bits(u64* p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_store(u64* p, double v) { res_store_bits(p, __builtin_bit_cast(u64, v)); }
// Whether all `team` workgroups of a team reached the gate (thread 0 of each
// calls it).  The word counts arrivals; one that has waited too long closes the
// gate, which it can only while some are missing, so all get the same answer:
// the word is `team` once and for all, or has RES_GATE_CLOSED set.  About 5 us
// with 256 workgroups, once a launch.
constexpr long long RES_GATE_TICKS = 100000000;  // 1 s
__device__ __forceinline__ bool res_gate(unsigned* word, unsigned team) {
    unsigned v = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    const long long t0 = wall_clock64();
    while (v < team) {
        v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v < team && wall_clock64() - t0 > RES_GATE_TICKS &&
            __hip_atomic_compare_exchange_strong(word, &v, v | RES_GATE_CLOSED, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return false;
    }
    return v == team;
}
// A caller's vector may hold any bit pattern: the empty one becomes another NaN.
__device__ __forceinline__ double res_quiet(double v) {
    const u64 b = __builtin_bit_cast(u64, v);
    return __builtin_bit_cast(double, b == RES_EMPTY ? b | (1ull << 51) : b);
}

// Waits until every *p[i] (i < N; null: no slot) holds a value; gives up
// (dead set) when the grid aborts.  All first loads are in flight together.
template <int N>
__device__ __forceinline__ void res_poll(const u64* const (&p)[N], double (&v)[N], unsigned* abort_word, int* dead) {
    u64 x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = p[i] ? res_load(p[i]) : 0;
    long long t0 = 0;
    int n = 0;
    for (;;) {
        bool wait = false;
#pragma unroll
        for (int i = 0; i < N; ++i) wait = wait || x[i] == RES_EMPTY;
        if (!wait) break;
        if ((++n & 255) == 0) {
            const long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            const bool late = now - t0 > RES_WAIT_TICKS;
            if (late) __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (late || __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                *dead = 1;
                break;
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (x[i] == RES_EMPTY) x[i] = res_load(p[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_bit_cast(double, x[i]);
}
__device__ __forceinline__ double res_poll(const u64* p, unsigned* abort_word, int* dead) {
    const u64* const a[1] = {p};
    double v[1];
    res_poll<1>(a, v, abort_word, dead);
    return v[0];
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uniform(double v) {
    const u64 b = __builtin_bit_cast(u64, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
}

template <class T>
__device__ __forceinline__ const T* uniform(const T* p) {
    const u64 b = (u64)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return (const T*)(((u64)hi << 32) | lo);
}

// The value of the lane before / after this one in the wave; `edge` in the
// lane that has none (the move leaves it as it was).
template <int CTRL>
__device__ __forceinline__ int dpp_shift(int edge, int v) {
    return __builtin_amdgcn_update_dpp(edge, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp_shift(float edge, float v) {
    return __builtin_bit_cast(float, dpp_shift<CTRL>(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_shift(double edge, double v) {
    const u64 a = __builtin_bit_cast(u64, edge), b = __builtin_bit_cast(u64, v);
    const unsigned lo = (unsigned)dpp_shift<CTRL>((int)(unsigned)a, (int)(unsigned)b);
    const unsigned hi = (unsigned)dpp_shift<CTRL>((int)(unsigned)(a >> 32), (int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
}
template <class T>
__device__ __forceinline__ T lane_before(T v, T edge) {
    return dpp_shift<0x138>(edge, v);  // wave_shr:1
}
template <class T>
__device__ __forceinline__ T lane_after(T v, T edge) {
    return dpp_shift<0x130>(edge, v);  // wave_shl:1
}

// Sums over the 16 lanes of a row.  row_sum: every lane gets the sum of v.
__device__ __forceinline__ double row_sum(double v) {
    v += dpp_move<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
    v += dpp_move<0x124, 0xf>(v);  // row_ror:4
    v += dpp_move<0x128, 0xf>(v);  // row_ror:8
    return v;
}
// Several values at once: lane i of a row gets value i's sum over the row (i <
// NV <= 9).  Two values share a register from the first step on (each lane
// keeps one and hands the other to its neighbour), four from the second, so
// five sums take 39 vector instructions instead of 60.
template <int NV>
__device__ __forceinline__ double row_sums(const double* a) {
    const int lane = threadIdx.x & 63;
    const bool odd = lane & 1, hi = lane & 2;
    auto pair = [&](double x, double y) { return (odd ? y : x) + dpp_move<0xB1, 0xf>(odd ? x : y); };
    if constexpr (NV == 1) {
        return row_sum(a[0]);
    } else if constexpr (NV <= 4) {
        double r;
        const double ab = pair(a[0], a[1]);
        if constexpr (NV == 2) {
            r = ab + dpp_move<0x4E, 0xf>(ab);
        } else {
            const double cd = pair(a[2], NV > 3 ? a[NV > 3 ? 3 : 0] : 0.0);
            r = (hi ? cd : ab) + dpp_move<0x4E, 0xf>(hi ? ab : cd);
        }
        r += dpp_move<0x124, 0xf>(r);
        r += dpp_move<0x128, 0xf>(r);
        return r;
    } else {
        static_assert(NV <= 9, "values");
        const double r = row_sums<4>(a);
        if constexpr (NV <= 8) {
            const double x = row_sums<NV - 4>(a + 4);  // lane i of four: value 4 + i
            return (lane & 15) < 4 ? r : x;
        } else {
            const double x = row_sums<4>(a + 4), y = row_sum(a[8]);
            return (lane & 15) < 4 ? r : (lane & 15) < 8 ? x : y;
        }
    }
}
// The same value, unknown to the compiler: what is computed from it stays
// where it is written.  (Hoisted out of the iteration loop, the addresses and
// offsets of every exchange filled the register file and spilled.)
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ int opaque_uniform(int v) {
    asm volatile("" : "+s"(v));
    return v;
}
// Lane I's value, in scalar registers.
template <int I>
__device__ __forceinline__ double lane_value(double v) {
    const u64 b = __builtin_bit_cast(u64, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, I);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), I);
    return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
}
// Sum over lanes 0 .. 31.
__device__ __forceinline__ double lanes32_sum(double v) {
    v = row_sum(v);
    return lane_value<0>(v) + lane_value<16>(v);
}

}  // namespace tgdk
