// What the trace check makes of a trace: sums over all requests, and the words and the status that follow from them.
#pragma once

#include "host_util.h"
#include "wave.h"

namespace stalloc {

constexpr uint32_t kNever = 0xffffffffu;

// Sums of the high and low halves of the sizes, whether a request is malformed, all bits set in any size, the
// largest size, the sum of the lifetimes, first allocation and last release.
struct TraceSums {
    uint64_t hi, lo, bad, bits, largest, lives;
    uint32_t t_first, t_last;
    static __device__ __forceinline__ TraceSums none() { return TraceSums{0, 0, 0, 0, 0, 0, kNever, 0}; }
    __device__ __forceinline__ void add(uint64_t s, uint32_t a, uint32_t f, uint32_t t_end)
    {
        bad |= (s == 0) | (a >= f) | (f > t_end);
        hi += s >> 32;                 // n < 2^31 terms below 2^32 each: cannot wrap
        lo += s & 0xffffffffull;
        bits |= s;
        largest = umax64(largest, s);
        lives += f - a;                // n terms below 2^32 each
        t_first = umin(t_first, a);
        t_last = umax(t_last, f);
    }
    __device__ __forceinline__ void add(const TraceSums& o)
    {
        hi += o.hi; lo += o.lo; bad |= o.bad; bits |= o.bits; largest = umax64(largest, o.largest);
        lives += o.lives; t_first = umin(t_first, o.t_first); t_last = umax(t_last, o.t_last);
    }
    __device__ __forceinline__ void over_wave()                       // in all lanes
    {
        hi = wave_sum64(hi); lo = wave_sum64(lo); bad = wave_or64(bad); bits = wave_or64(bits); largest = wave_max64(largest);
        lives = wave_sum64(lives);
        t_first = ~read_lane(wave_scan_max(~t_first), kWave - 1); t_last = read_lane(wave_scan_max(t_last), kWave - 1);
    }
};
static_assert(sizeof(TraceSums) == 7 * sizeof(uint64_t), "kAccSpace holds one per workgroup");

// The accumulators (the other words are zero), from the sums over all requests; returns the status.
__device__ __forceinline__ uint32_t verdict(const TraceSums& t, uint32_t n, uint32_t t_end, uint64_t (&words)[kAccWords])
{
    uint32_t code = STALLOC_OK;
    for (int k = 0; k < kAccWords; ++k) words[k] = 0;
    words[0] = t.hi; words[1] = t.lo; words[2] = t.bad; words[3] = t.bits;
    words[kAccMaxSize] = t.largest;
    const float span = (float)(t.t_last - t.t_first);                // (a choice between two ways to the same answer: rounding does not matter)
    words[kAccCrowded] = ((float)t.lives * 5.0f > (float)n * span || span * 16.0f < (float)t_end ? kCrowded : 0) |
                         ((float)t.lives < 80.0f * span ? kFewAlive : 0) | ((float)t.lives < 24.0f * span ? kHardlyAnyAlive : 0);
    if (t.hi + (t.lo >> 32) < (1ull << 31) && t.bits != 0) {
        const uint64_t total = (t.hi << 32) + t.lo;                  // below 2^63 here
        const uint32_t shift = (uint32_t)__builtin_ctzll(t.bits);
        const uint64_t narrow = (total >> shift) < (1ull << 31) ? kModeNarrow : 0;
        const uint64_t compact = (total >> shift) < (1ull << 16) ? kModeCompact : 0;
        const uint64_t bitmap = (total >> shift) <= kBitmapGranules && (t.largest >> shift) <= kBitmapMaxSize ? kModeBitmap : 0;
        // The sum of sizes bounds every address, but plans worth having end far below it: when the
        // sum is too large for 32-bit granule counts and no single request is, the 32-bit placement
        // kernel takes each plan as far as its extent allows and hands the rest to the 64-bit one.
        const uint64_t try32 = (!narrow && (t.largest >> shift) < (1ull << 30)) ? kModeTry32 : 0;
        words[kAccMode] = shift | narrow | compact | bitmap | try32;
        words[kAccGranules] = total >> shift;
    }
    // total = hi * 2^32 + lo  >= 2^63  <=>  hi + (lo >> 32) >= 2^31
    if (t.hi + (t.lo >> 32) >= (1ull << 31)) code = STALLOC_ERR_OVERFLOW;
    if (t.bad) code = STALLOC_ERR_BAD_TRACE;
    return code;
}

}  // namespace stalloc
