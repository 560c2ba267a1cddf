// Two-word sort keys (compared word by word) and the in-LDS sort of one tile of 1024 of them,
// shared by the kernels that order requests: placement orders, HomoSize groups, decisions by
// address.  The tiles are merged by launch_merge_tiles (host_util.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace stalloc {

constexpr int kSortTile = 1024;
constexpr int kSortThreads = 512;                // two keys a thread

__device__ __forceinline__ bool key_before(const ulonglong2& x, const ulonglong2& y)
{
    return x.x < y.x || (x.x == y.x && x.y < y.y);
}

// The key of slot e past the end of a row: behind every real key as long as no real key starts
// with ~0 and carries all ones in the upper half of its second word; distinct from slot to slot.
__device__ __forceinline__ ulonglong2 filler_key(uint32_t e) { return make_ulonglong2(~0ull, 0xffffffff00000000ull | e); }

// Bitonic network over k[0..1023] in LDS; called by all 512 threads of the workgroup with the keys
// already stored (each thread its own two, t and 512 + t); sorted when it returns.  Merges begin by
// comparing mirrored places, so that every exchange goes the same way.  Up to a distance of 64 the 64
// pairs of a wave are a run of 128 places of their own: no barrier between such steps.
// Only the first `real` keys need sorting: those behind them are fillers, larger than any of them and in order
// (with few of them the network is shorter: 300 requests take 45 of the 55 steps, 100 take 28).
__device__ __forceinline__ void sort_tile(ulonglong2 (&k)[kSortTile], uint32_t real)
{
    const uint32_t t = threadIdx.x;
    __syncthreads();
    for (uint32_t span = 2; span <= (uint32_t)kSortTile && span < 2 * real; span <<= 1) {
        for (uint32_t gap = span >> 1; gap > 0; gap >>= 1) {
            const uint32_t x = 2 * t - (t & (gap - 1)), y = gap == span >> 1 ? x ^ (span - 1) : x ^ gap;
            const ulonglong2 a = k[x], b = k[y];
            if (key_before(b, a)) { k[x] = b; k[y] = a; }
            // (the next step reads what other waves wrote if this one or the next reaches beyond the wave's run)
            const uint32_t next = gap > 1 ? gap >> 1 : span;
            if (gap > 64 || next > 64) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
}

// Real keys of the tile that starts at `first`, of `all` (first < all).
__device__ __forceinline__ uint32_t keys_of_tile(uint32_t first, uint32_t all) { return all - first < (uint32_t)kSortTile ? all - first : (uint32_t)kSortTile; }

}  // namespace stalloc
