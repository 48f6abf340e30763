// device_common.hpp -- device helpers shared by the DROP kernels of the
// single-image and batched sweeps.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <cstdint>
#include <type_traits>

#include "tvs_internal.hpp"

namespace tvs {
namespace dev {

constexpr uint32_t kNoRow = 0xffffffffu;

// Row (within its block) of an entry tag.
__device__ inline uint32_t row_of(const TileBlock &t, uint32_t m)
{
    return (m >> kTileShift) & t.rowmask;
}

// Chord of entry e (index into the block's arrays) with tag m: float32,
// float16, or fixed point (the low 16 bits of the code in chq, the high bits
// in the tag above the row field) in units of qunit mm.
template <typename CH>
__device__ inline float entry_chord(const TileBlock &t, int64_t e, uint32_t m)
{
    if constexpr (sizeof(CH) == 4) {
        return t.ch32[e];
    } else if constexpr (std::is_same<CH, uint16_t>::value) {
        const uint32_t code = ((m >> t.qshift) << 16) | (uint32_t)t.chq[e];
        return (float)((double)code * t.qunit);
    } else {
        return __half2float(t.ch16[e]);
    }
}

// A lane's value moved along the wavefront by DPP (no LDS round trip); `old`
// where there is no source lane.
template <int CTRL, int ROWS>
__device__ inline uint32_t dpp(uint32_t old, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}

// Wavefront bookkeeping for sums over runs of equal keys: lanes holding the
// same key in consecutive lanes form a run (the entries of one row inside
// one tile are consecutive in its list).
struct Runs {
    int start;     // first lane of this lane's run
    bool tail;     // this lane ends its run
};

__device__ inline Runs wave_runs(uint32_t key)
{
    const int lane = threadIdx.x & 63;
    const uint32_t prev = dpp<0x138, 0xf>(0u, key);      // from lane - 1
    const bool head = (lane == 0) || (prev != key);
    const unsigned long long heads = __ballot(head);
    const unsigned long long upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    Runs r;
    r.start = 63 - __clzll((long long)(heads & upto));
    r.tail = lane == 63 || ((heads >> (lane + 1)) & 1ull);
    return r;
}

template <int CTRL, int ROWS>
__device__ inline long long dpp_add(long long v)
{
    const uint32_t lo = dpp<CTRL, ROWS>(0u, (uint32_t)v);
    const uint32_t hi = dpp<CTRL, ROWS>(0u, (uint32_t)((unsigned long long)v >> 32));
    return v + (long long)(((unsigned long long)hi << 32) | lo);
}

// Sum of v over this lane's run up to this lane: the wavefront's prefix sums
// (within rows of 16 lanes, then across them) less the one before the run.
// Integers: exact, so the total does not depend on how runs are cut, and the
// prefix may wrap.  Six steps of four instructions and one read of another
// lane, in place of six conditional 64-bit shuffles through LDS (with the
// settings' planes of batch.hip: 102.9 -> 83.4 us a step of 24 settings).
__device__ inline long long run_sum(long long v, const Runs &r)
{
    v = dpp_add<0x111, 0xf>(v);      // row_shr:1
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);      // row_bcast:15 to rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);      // row_bcast:31 to rows 2 and 3
    const long long before = __shfl(v, r.start > 0 ? r.start - 1 : 0, 64);
    return r.start > 0 ? v - before : v;
}

// v * scale rounded to nearest (ties to even) as an integer, for a scale that
// is a power of two and |v * scale| < 2^51: the product is exact, and adding
// 1.5 2^52 leaves the integer in the low mantissa bits.
__device__ inline long long round_scaled(double v, double scale)
{
    return __double_as_longlong(fma(v, scale, 6755399441055744.0)) - 0x4338000000000000ll;
}

// This wave's memory operations are complete; its agent-scope stores and atomics
// are then visible to the whole device.
__device__ inline void drain_memory() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

}  // namespace dev
}  // namespace tvs
