// stalloc_make_orders: candidate placement orders, produced on the device.
//
// Row p is a permutation of the request numbers, the stable sort of the requests by a key:
//   p = 0          size descending, then allocation time  (large requests first, so that smaller
//                  ones fill the intervals they leave: Sec. 5.1, Global Planning)
//   p = 1          lifetime descending, then size descending
//   p = 2          allocation time  (the order Algorithm 1 takes a group's requests in)
//   p >= 3, odd    a 64-bit pseudo-random key k(p, i): a uniform random permutation
//   p >= 4, even   (c(i) + 1) * 2^32 + (k(p, i) >> 31), c(i) = number of distinct sizes larger than
//                  request i's: size descending with a random order inside each size and a shift
//                  of up to one size to either side
// k(p, i) = mix(i * 0xD1342543DE82EF95 + mix(seed + p)) modulo 2^64; mix(x) is the output of the
// SplitMix64 generator (Steele, Lea, Flood, OOPSLA 2014) whose state before the step is x.
//
// Every key is packed, with the request number in its lowest 32 bits, into two 64-bit words
// compared in turn; keys of a row are therefore distinct and no tie rule is needed.
//
// Rows 0 .. 2 (and all rows of traces beyond kOrMostBuckets buckets) are sorted as tiles of 1024 keys
// in LDS (bitonic network) followed by passes that merge four runs at a time: an element's place in
// the merged run is its place in its own run plus the numbers of elements of the three other runs
// that sort before it, found by binary search.  log4(n / 1024) passes, all rows of a batch side
// by side in every launch.  A pass is a chain of dependent loads, whatever the number of searches:
// 199 748 keys take 4 passes of 13 us where merging in pairs from tiles of 256 took 10 of 13 us.
//
// The keys of the other rows are spread in a way that is known in advance -- uniformly, or uniformly
// inside steps of 2^32 whose counts follow from the sizes -- so that where a key will end up is known to
// within a few places without comparing it to any other: or_scatter drops the request numbers of a
// row into buckets of about 1536 by expected place, or_buckets sorts a bucket in LDS by counting
// the keys per expected place (2048 cells) and comparing inside a cell only.  A key is worked out
// from the request number wherever it is needed; memory only sees the numbers, once out and
// once in between.
//   256 rows of 199 748 requests: 8.72 (all rows merged) -> 0.65 -> 0.53 ms, of which or_scatter 0.10 (key arithmetic; 0.22 with a
// scattered 4-byte store per number), or_buckets 0.28 (LDS counting and key arithmetic), rows 0 .. 2 and the size
// classes 0.17; the sorted numbers alone take 0.04 ms to write.  Merging moved 16-byte keys ten times.
#include "host_util.h"
#include "sort_keys.h"
#include "wave.h"

namespace stalloc {

constexpr int kOrTile = kSortTile;

constexpr uint64_t kOrStream = 0xD1342543DE82EF95ull;

__device__ __forceinline__ uint64_t splitmix64_out(uint64_t x)
{
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

struct OrTrace {
    const uint64_t* size;
    const uint32_t* ta;
    const uint32_t* tf;
    const uint32_t* larger;      // [n] c(i); only read for even rows >= 4
    uint32_t n;
};

// The two key words of request i in row p; slot e past the end gets a key behind every real one.
__device__ __forceinline__ ulonglong2 order_key(const OrTrace& t, uint64_t p, uint64_t stream, uint32_t i, uint32_t e)
{
    ulonglong2 k;
    if (i >= t.n) return filler_key(e);
    if (p == 0) {
        k.x = ~t.size[i];
        k.y = ((uint64_t)t.ta[i] << 32) | i;
    } else if (p == 1) {
        const uint64_t inv_size = ~t.size[i];
        const uint32_t inv_life = ~(t.tf[i] - t.ta[i]);
        k.x = ((uint64_t)inv_life << 32) | (inv_size >> 32);
        k.y = (inv_size << 32) | i;
    } else if (p == 2) {
        k.x = t.ta[i];
        k.y = i;
    } else {
        const uint64_t r = splitmix64_out((uint64_t)i * kOrStream + stream);
        k.x = (p & 1) ? r : (((uint64_t)t.larger[i] + 1) << 32) + (r >> 31);
        k.y = i;
    }
    return k;
}

// grid (tiles, rows): the keys of one tile of one row, sorted in LDS.
__global__ void __launch_bounds__(kSortThreads)
or_sort_tiles(OrTrace t, uint64_t first_plan, uint64_t seed, uint32_t n_pad, ulonglong2* keys, const uint32_t* status)
{
    __shared__ ulonglong2 k[kOrTile];
    if (*status != STALLOC_OK) return;
    const uint64_t p = first_plan + blockIdx.y, stream = splitmix64_out(seed + p);
    ulonglong2* out = keys + (size_t)blockIdx.y * n_pad + blockIdx.x * kOrTile;
    for (uint32_t th = threadIdx.x; th < (uint32_t)kOrTile; th += kSortThreads) {
        const uint32_t e = blockIdx.x * kOrTile + th;
        k[th] = order_key(t, p, stream, e, e);
    }
    sort_tile(k, keys_of_tile(blockIdx.x * kOrTile, t.n));
    for (uint32_t th = threadIdx.x; th < (uint32_t)kOrTile; th += kSortThreads) out[th] = k[th];
}

// Element e of a row whose runs of `run` keys (a power of two) are merged four at a time: where it goes.
// The three searches go side by side; a wave's lanes hold neighbours of a run and take nearly the same steps.
__device__ __forceinline__ uint32_t merged_place(const ulonglong2* row, uint32_t n_pad, uint32_t run, uint32_t e,
                                                 const ulonglong2& me)
{
    const uint32_t mine = e / run, group0 = (mine & ~3u) * run;         // my run; its partners are the others of its four
    uint32_t from[3], left[3];                                          // first key of a partner; keys of it still in question
#pragma unroll
    for (uint32_t v = 0; v < 3; ++v) {
        const uint64_t at = (uint64_t)(mine & ~3u) * run + (uint64_t)(v + (v >= (mine & 3u) ? 1u : 0u)) * run;
        from[v] = at < n_pad ? (uint32_t)at : 0u;
        left[v] = at < n_pad ? (n_pad - from[v] < run ? n_pad - from[v] : run) : 0u;
    }
    uint32_t place = group0 + (e - mine * run) - (from[0] + from[1] + from[2]);
    while (left[0] | left[1] | left[2]) {
#pragma unroll
        for (uint32_t v = 0; v < 3; ++v) {
            if (left[v] == 0) continue;
            const uint32_t half = left[v] >> 1;
            const bool before = key_before(row[from[v] + half], me);
            from[v] = before ? from[v] + half + 1 : from[v];
            left[v] = before ? left[v] - half - 1 : half;
        }
    }
    return place + from[0] + from[1] + from[2];
}

// grid (256-key pieces, rows): runs of `run` keys merged four at a time, src -> dst.
__global__ void __launch_bounds__(256)
or_merge(const ulonglong2* __restrict__ src, ulonglong2* dst, uint32_t n_pad, uint32_t run, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    const ulonglong2* row = src + (size_t)blockIdx.y * n_pad;
    const ulonglong2 me = row[e];
    dst[(size_t)blockIdx.y * n_pad + merged_place(row, n_pad, run, e, me)] = me;
}

__global__ void __launch_bounds__(256)
or_emit(const ulonglong2* __restrict__ keys, uint32_t n_pad, uint32_t n, uint32_t* orders, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    const ulonglong2* row = keys + (size_t)blockIdx.y * n_pad;
    uint32_t* out = orders + (size_t)blockIdx.y * n;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) out[k] = (uint32_t)row[k].y;
}

// Sorted by size descending (row 0): flag[k] = 1 where a new size starts.
__global__ void __launch_bounds__(256)
or_size_flags(const ulonglong2* __restrict__ keys, uint32_t n, uint32_t* flag, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
        flag[k] = (k > 0 && keys[k].x != keys[k - 1].x) ? 1u : 0u;
}

// larger[request at sorted position k] = distinct sizes in front of position k; class_start[c] = the
// first position with c of them.
__global__ void __launch_bounds__(256)
or_size_classes(const ulonglong2* __restrict__ keys, const uint32_t* __restrict__ flag,
                const uint32_t* __restrict__ flags_before, uint32_t n, uint32_t* larger, uint32_t* class_start,
                const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        const uint32_t c = flags_before[k] + flag[k];
        larger[(uint32_t)keys[k].y] = c;
        if (k == 0 || flag[k]) class_start[c] = k;
    }
}

// ------------------------------------------------------------------------------------------
// Rows from 3 on: buckets by expected place.
constexpr uint32_t kOrCells = 2048;              // cells of a bucket, and the request numbers it has room for
#ifndef STALLOC_OR_BUCKET_MEAN
#define STALLOC_OR_BUCKET_MEAN 1536              // (test builds raise it so that buckets do not hold all their numbers)
#endif
constexpr uint32_t kOrBucketMean = STALLOC_OR_BUCKET_MEAN;         // numbers a bucket is meant for: 13 standard deviations below its room
constexpr uint32_t kOrMostBuckets = 4096;
constexpr int kOrScatterThreads = 512, kOrPerThread = 16;
constexpr int kOrBucketThreads = 512;
// Numbers are put in order of bucket in LDS before they are stored (or_scatter) from this many numbers a launch on, in rows of more than two
// buckets or so: below, there are few waves that stores could hold up, and two barriers and a sum more are 1.5 us a launch (directly /
// staged: 4096 requests, 1024 rows 82 / 83 us; 16 384, 64 rows 76.6 / 77.7, 256 rows 97.7 / 97.3; 49 920, 64 rows 109.5 / 107.9).
constexpr uint64_t kOrStagedFrom = 4000 * 1000;
constexpr uint32_t kOrStagedRow = 4096;

struct OrBuckets {
    const uint32_t* step;        // [classes + 3] first cell of the keys k * 2^32 .. of an even row (OrTrace::larger counts the classes)
    uint32_t* filled;            // [rows][buckets] numbers dropped into a bucket
    uint32_t* number;            // [rows][buckets][kOrCells]
    uint32_t buckets;
};
// (4096 buckets are 6.3 million requests; the room counters of or_scatter for more would not fit LDS)

// Request i of row p (>= 3): its key, and the cell of the row in which it is expected (never
// descending with the key; bucket = cell / kOrCells).
// `at`: i * kOrStream + stream.
__device__ __forceinline__ uint64_t spread_key_at(const OrTrace& t, const OrBuckets& b, uint64_t p, uint64_t at, uint32_t i,
                                                  uint32_t& cell)
{
    const uint64_t r = splitmix64_out(at);
    if (p & 1) {                                                  // (uniform)
        cell = __umulhi((uint32_t)(r >> 32), b.buckets * kOrCells);
        return r;
    }
    const uint64_t key = (((uint64_t)t.larger[i] + 1) << 32) + (r >> 31);
    const uint32_t k = (uint32_t)(key >> 32), first = b.step[k];
    cell = first + __umulhi((uint32_t)key, b.step[k + 1] - first);
    return key;
}

__device__ __forceinline__ uint64_t spread_key(const OrTrace& t, const OrBuckets& b, uint64_t p, uint64_t stream, uint32_t i,
                                               uint32_t& cell)
{
    return spread_key_at(t, b, p, (uint64_t)i * kOrStream + stream, i, cell);
}

// step[k], k = 0 .. classes + 2: a request of class c is at [c + 1, c + 3) * 2^32, half of them in either
// step, so 2 * (requests expected in front of step k) = requests of classes below k - 1 + of classes
// below k - 2.  class_start[c] = requests of classes below c.
__global__ void __launch_bounds__(256)
or_steps(const uint32_t* __restrict__ class_start, const uint32_t* later_classes, uint32_t n, uint32_t cells, uint32_t* step,
         const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    const uint32_t classes = *later_classes + 1;
    auto below = [&](uint32_t c) -> uint64_t { return c < classes ? class_start[c] : n; };
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < classes + 3; k += gridDim.x * blockDim.x) {
        const uint64_t twice = (k >= 1 ? below(k - 1) : 0u) + (k >= 2 ? below(k - 2) : 0u);
        step[k] = (uint32_t)(twice * cells / (2ull * n));
    }
}

__global__ void __launch_bounds__(256) or_empty(uint32_t* filled, uint32_t m)
{
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < m; k += gridDim.x * blockDim.x) filled[k] = 0;
}

// grid (pieces of 8192 requests, rows): a piece reserves its room in every bucket with one atomic.  Staged, its numbers are put in order of bucket in
// LDS first, so that the lanes of a store mostly write beside one another: each by itself they were a line per lane, and the L2s,
// which take some 270 of them a nanosecond, set the time (256 rows of 199 748 requests: 220 us, now 98).  The multiplication by the stream's
// constant is an addition from one request of a thread to the next.
template <bool kStaged>
__global__ void __launch_bounds__(kOrScatterThreads)
or_scatter(OrTrace t, OrBuckets b, uint64_t first_plan, uint64_t seed, const uint32_t* status)
{
    constexpr uint32_t kPiece = kOrScatterThreads * kOrPerThread, kOwn = kOrMostBuckets / kOrScatterThreads;
    static_assert((uint64_t)kPiece * kOrMostBuckets <= 1ull << 32, "a request of the piece and its bucket share a word");
    __shared__ uint32_t staged[kStaged ? kPiece : 1];             // bucket * kPiece + request of the piece, by bucket
    __shared__ uint32_t part[kOrScatterThreads / kWave];
    extern __shared__ uint32_t room[];                            // [buckets] numbers of the piece; where they begin in `staged`; from there to the bucket
    if (*status != STALLOC_OK) return;
    const uint64_t p = first_plan + blockIdx.y, stream = splitmix64_out(seed + p);
    const uint32_t piece = blockIdx.x * kPiece, i0 = piece + threadIdx.x;
    const uint32_t many = t.n - piece < kPiece ? t.n - piece : kPiece;
    for (uint32_t k = threadIdx.x; k < b.buckets; k += kOrScatterThreads) room[k] = 0;
    __syncthreads();
    uint32_t bucket[kOrPerThread], place[kOrPerThread];
    uint64_t at = (uint64_t)i0 * kOrStream + stream;
#pragma unroll
    for (int u = 0; u < kOrPerThread; ++u) {
        const uint32_t i = i0 + u * kOrScatterThreads;
        bucket[u] = 0;
        if (i < t.n) {
            uint32_t cell;
            spread_key_at(t, b, p, at, i, cell);
            bucket[u] = cell / kOrCells;
            place[u] = atomicAdd(&room[bucket[u]], 1u);
        }
        at += kOrScatterThreads * kOrStream;
    }
    __syncthreads();
    uint32_t* filled = b.filled + (size_t)blockIdx.y * b.buckets;
    uint32_t* number = b.number + (size_t)blockIdx.y * b.buckets * kOrCells;
    if constexpr (!kStaged) {
        for (uint32_t k = threadIdx.x; k < b.buckets; k += kOrScatterThreads) {
            const uint32_t mine = room[k];
            room[k] = mine ? atomicAdd(&filled[k], mine) : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kOrPerThread; ++u) {
            const uint32_t i = i0 + u * kOrScatterThreads;
            if (i >= t.n) break;
            const uint32_t to = room[bucket[u]] + place[u];
            if (to < kOrCells) number[(size_t)bucket[u] * kOrCells + to] = i;     // (or_buckets sees from `filled` when it did not fit)
        }
        return;
    }
    // a thread sees to `own` buckets in a row
    const uint32_t own = (b.buckets + kOrScatterThreads - 1) / kOrScatterThreads, k0 = threadIdx.x * own;
    uint32_t count[kOwn], reserved[kOwn], mine = 0;
#pragma unroll
    for (uint32_t q = 0; q < kOwn; ++q) {
        const uint32_t k = k0 + q;
        count[q] = q < own && k < b.buckets ? room[k] : 0u;
        reserved[q] = count[q] ? atomicAdd(&filled[k], count[q]) : 0u;
        mine += count[q];
    }
    const uint32_t incl = wave_scan_add(mine);
    if (lane_id() == kWave - 1) part[wave_id()] = incl;
    __syncthreads();
    uint32_t begin = incl - mine;
    for (int w = 0; w < wave_id(); ++w) begin += part[w];
#pragma unroll
    for (uint32_t q = 0; q < kOwn; ++q) {
        if (q < own && k0 + q < b.buckets) room[k0 + q] = begin;
        reserved[q] -= begin;
        begin += count[q];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kOrPerThread; ++u) {
        const uint32_t e = threadIdx.x + u * kOrScatterThreads;
        if (e < many) staged[room[bucket[u]] + place[u]] = bucket[u] * kPiece + e;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kOwn; ++q)
        if (q < own && k0 + q < b.buckets) room[k0 + q] = reserved[q];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kOrPerThread; ++u) {
        const uint32_t e = threadIdx.x + u * kOrScatterThreads;
        if (e >= many) break;
        const uint32_t to_bucket = staged[e] / kPiece, to = room[to_bucket] + e;
        if (to < kOrCells) number[(size_t)to_bucket * kOrCells + to] = piece + staged[e] % kPiece;     // (or_buckets sees from `filled` when it did not fit)
    }
}

// grid (buckets, rows): one bucket sorted in LDS.  With a single bucket nothing has been dropped: it
// holds all requests.
__global__ void __launch_bounds__(kOrBucketThreads)
or_buckets(OrTrace t, OrBuckets b, uint64_t first_plan, uint64_t seed, uint32_t* orders, const uint32_t* status)
{
    constexpr int kPer = kOrCells / kOrBucketThreads;             // cells, and numbers, of a thread
    constexpr int kWaves = kOrBucketThreads / kWave;
    __shared__ uint64_t key_at[kOrCells];
    __shared__ uint32_t number_at[kOrCells];
    __shared__ uint32_t cells[kOrCells + 1];
    __shared__ uint32_t part[kWaves];
    if (*status != STALLOC_OK) return;
    const uint64_t p = first_plan + blockIdx.y, stream = splitmix64_out(seed + p);
    const uint32_t own = blockIdx.x, tid = threadIdx.x;
    const uint32_t* filled = b.filled + (size_t)blockIdx.y * b.buckets;
    const uint32_t m = b.buckets == 1 ? t.n : filled[own];
    // numbers in the buckets below
    uint32_t first = 0;
    for (uint32_t k = tid; k < own; k += kOrBucketThreads) first += filled[k];
    first = wave_sum32(first);
    if (lane_id() == 0) part[wave_id()] = first;
#pragma unroll
    for (int u = 0; u < kPer; ++u) cells[tid + u * kOrBucketThreads] = 0;
    __syncthreads();
    first = 0;
    for (int w = 0; w < kWaves; ++w) first += part[w];
    uint32_t* out = orders + (size_t)blockIdx.y * t.n + first;
    if (m > kOrCells) {
        // (a bucket that got more than it has room for, 13 standard deviations off) its keys are found one
        // after another, each the smallest of the row's keys in this bucket behind the last one
        __shared__ ulonglong2 least;
        ulonglong2 last = make_ulonglong2(0ull, 0ull);            // (key, number + 1)
        for (uint32_t k = 0; k < m; ++k) {
            ulonglong2 mine = make_ulonglong2(~0ull, ~0ull);
            for (uint32_t i = tid; i < t.n; i += kOrBucketThreads) {
                uint32_t cell;
                const ulonglong2 q = make_ulonglong2(spread_key(t, b, p, stream, i, cell), (uint64_t)i + 1);
                if (cell / kOrCells == own && key_before(last, q) && key_before(q, mine)) mine = q;
            }
            for (int d = 1; d < kWave; d <<= 1) {
                const ulonglong2 other = make_ulonglong2(lane_gather((uint64_t)mine.x, lane_id() ^ d),
                                                         lane_gather((uint64_t)mine.y, lane_id() ^ d));
                if (key_before(other, mine)) mine = other;
            }
            __syncthreads();
            if (lane_id() == 0) { key_at[wave_id()] = mine.x; key_at[kWaves + wave_id()] = mine.y; }
            __syncthreads();
            if (tid == 0) {
                for (int w = 1; w < kWaves; ++w) {
                    const ulonglong2 other = make_ulonglong2(key_at[w], key_at[kWaves + w]);
                    if (key_before(other, mine)) mine = other;
                }
                least = mine;
                out[k] = (uint32_t)(mine.y - 1);
            }
            __syncthreads();
            last = least;
        }
        return;
    }
    const uint32_t* number = b.number + ((size_t)blockIdx.y * b.buckets + own) * kOrCells;
    uint64_t key[kPer];
    uint32_t id[kPer], cell[kPer], rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const uint32_t k = tid + u * kOrBucketThreads;
        id[u] = 0;
        if (k < m) id[u] = b.buckets == 1 ? k : number[k];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        cell[u] = 0;
        key[u] = 0;
        if (tid + u * kOrBucketThreads < m) {
            key[u] = spread_key(t, b, p, stream, id[u], cell[u]);
            cell[u] %= kOrCells;
            rank[u] = atomicAdd(&cells[cell[u]], 1u);
        }
    }
    __syncthreads();
    // counts -> first places
    uint32_t c[kPer], mine = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) { c[u] = cells[tid * kPer + u]; mine += c[u]; }
    const uint32_t incl = wave_scan_add(mine);
    if (lane_id() == kWave - 1) part[wave_id()] = incl;
    __syncthreads();
    uint32_t run = incl - mine;
    for (int w = 0; w < wave_id(); ++w) run += part[w];
#pragma unroll
    for (int u = 0; u < kPer; ++u) { cells[tid * kPer + u] = run; run += c[u]; }
    if (tid == kOrBucketThreads - 1) cells[kOrCells] = run;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (tid + u * kOrBucketThreads >= m) continue;
        const uint32_t to = cells[cell[u]] + rank[u];
        key_at[to] = key[u];
        number_at[to] = id[u];
    }
    __syncthreads();
    // inside a cell by key, then by number
    uint32_t place[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (tid + u * kOrBucketThreads >= m) continue;
        const uint32_t from = cells[cell[u]], to = cells[cell[u] + 1];
        uint32_t before = 0;
        for (uint32_t k = from; k < to; ++k)
            before += key_at[k] < key[u] || (key_at[k] == key[u] && number_at[k] < id[u]) ? 1u : 0u;
        place[u] = from + before;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (tid + u * kOrBucketThreads < m) number_at[place[u]] = id[u];
    __syncthreads();
    for (uint32_t k = tid; k < m; k += kOrBucketThreads) out[k] = number_at[k];
}

ulonglong2* launch_merge_tiles(ulonglong2* keys, ulonglong2* spare, uint32_t n_pad, uint32_t rows, const uint32_t* status,
                               hipStream_t stream)
{
    ulonglong2 *src = keys, *dst = spare;
    for (uint64_t run = kOrTile; run < n_pad; run <<= 2) {
        hipLaunchKernelGGL(or_merge, dim3(n_pad / 256, rows), dim3(256), 0, stream, src, dst, n_pad, (uint32_t)run, status);
        ulonglong2* s = src; src = dst; dst = s;
    }
    return src;
}

// Sorts `rows` rows starting at plan first_plan; returns the buffer that holds the result.
static ulonglong2* sort_rows(const OrTrace& t, uint64_t first_plan, uint32_t rows, uint64_t seed, uint32_t n_pad,
                             ulonglong2* buf_a, ulonglong2* buf_b, const uint32_t* status, hipStream_t stream)
{
    hipLaunchKernelGGL(or_sort_tiles, dim3(n_pad / kOrTile, rows), dim3(kSortThreads), 0, stream, t, first_plan, seed, n_pad, buf_a,
                       status);
    return launch_merge_tiles(buf_a, buf_b, n_pad, rows, status, stream);
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_make_orders(const stalloc_trace* tr, uint32_t first_plan, uint32_t P, uint64_t seed,
                                   uint32_t* orders, uint32_t* device_status, void* workspace,
                                   size_t* workspace_bytes, void* hip_stream)
{
    if (!trace_args_ok(tr) || P == 0 || (uint64_t)first_plan + P > 0xffffffffull || !workspace_bytes)
        return STALLOC_ERR_INVALID_ARG;
    const uint32_t n = tr->n;
    const uint32_t tiles = (n + kOrTile - 1) / kOrTile;
    const uint32_t n_pad = tiles * kOrTile;
    const uint64_t last = (uint64_t)first_plan + P - 1;
    const uint32_t buckets = n <= kOrCells ? 1u : (n + kOrBucketMean - 1) / kOrBucketMean;
    const bool spread = buckets <= kOrMostBuckets;
    // rows sorted side by side: as many as fit 1 GiB of key buffers, 256 MiB of buckets (which then stay in
    // the memory-side cache between the two launches), at most 32768 (grid.y)
    uint64_t batch = spread ? (256ull << 20) / ((uint64_t)buckets * kOrCells * sizeof(uint32_t))
                            : (1ull << 30) / (2ull * n_pad * sizeof(ulonglong2));
    if (batch < 1) batch = 1;
    if (batch > 32768) batch = 32768;
    if (batch > P) batch = P;
    const uint32_t chunks = (n + 1023) / 1024;
    // rows that are merged: all of a batch, or rows 0 .. 2 as far as they are asked for, and row 0 for the
    // classes of the even rows
    uint32_t merged = (uint32_t)batch;
    if (spread) merged = first_plan <= 2 ? (uint32_t)(last < 2 ? last + 1 : 3) : (last >= 4 ? 1u : 0u);

    // (the size depends on n and P only: a workspace serves one window of rows after another)
    const uint32_t merged_room = spread ? 3u : merged;
    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    ulonglong2* buf_a = cv.take<ulonglong2>((size_t)merged_room * n_pad);
    ulonglong2* buf_b = cv.take<ulonglong2>((size_t)merged_room * n_pad);
    uint32_t* larger = cv.take<uint32_t>(n);
    uint32_t* flag = cv.take<uint32_t>(n);
    uint32_t* flags_before = cv.take<uint32_t>(n);
    uint32_t* chunk_sum = cv.take<uint32_t>(chunks);
    uint32_t* total = cv.take<uint32_t>(1);
    uint32_t* class_start = cv.take<uint32_t>(n);
    uint32_t* step = cv.take<uint32_t>((size_t)n + 3);
    OrBuckets ob = {step, nullptr, nullptr, buckets};
    if (spread && buckets > 1) {
        ob.filled = cv.take<uint32_t>((size_t)batch * buckets);
        ob.number = cv.take<uint32_t>((size_t)batch * buckets * kOrCells);
    }
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    if (!orders || !device_status || *workspace_bytes < cv.used || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    launch_trace_check(*tr, acc, device_status, stream);

    OrTrace t;
    t.size = tr->size; t.ta = tr->t_alloc; t.tf = tr->t_free; t.larger = larger; t.n = n;
    uint32_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    const uint32_t eb = blocks > 64 ? 64 : blocks;
    const ulonglong2* by_rule = nullptr;                  // rows 0 .. merged - 1
    if (spread ? merged != 0 : last >= 4)
        by_rule = sort_rows(t, 0, spread ? merged : 1u, seed, n_pad, buf_a, buf_b, device_status, stream);
    // c(i) for the rows that sort by size with jitter: from the order of row 0
    if (last >= 4) {
        hipLaunchKernelGGL(or_size_flags, dim3(blocks), dim3(256), 0, stream, by_rule, n, flag, device_status);
        launch_scan(flag, n, flags_before, chunk_sum, total, device_status, stream);
        hipLaunchKernelGGL(or_size_classes, dim3(blocks), dim3(256), 0, stream, by_rule, flag, flags_before, n, larger,
                           class_start, device_status);
        if (spread)
            hipLaunchKernelGGL(or_steps, dim3(blocks), dim3(256), 0, stream, class_start, total, n, buckets * kOrCells, step,
                               device_status);
    }
    if (!spread) {
        for (uint64_t p0 = 0; p0 < P; p0 += batch) {
            const uint32_t rows = (uint32_t)(P - p0 < batch ? P - p0 : batch);
            const ulonglong2* sorted = sort_rows(t, (uint64_t)first_plan + p0, rows, seed, n_pad, buf_a, buf_b, device_status, stream);
            hipLaunchKernelGGL(or_emit, dim3(eb, rows), dim3(256), 0, stream, sorted, n_pad, n, orders + (size_t)p0 * n,
                               device_status);
        }
        return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
    }
    uint64_t p0 = 0;
    if (first_plan <= 2) {
        p0 = merged - first_plan;
        hipLaunchKernelGGL(or_emit, dim3(eb, (uint32_t)p0), dim3(256), 0, stream, by_rule + (size_t)first_plan * n_pad, n_pad, n, orders,
                           device_status);
    }
    constexpr uint32_t kPiece = kOrScatterThreads * kOrPerThread;
    for (; p0 < P; p0 += batch) {
        const uint32_t rows = (uint32_t)(P - p0 < batch ? P - p0 : batch);
        if (buckets > 1) {
            const uint32_t m = rows * buckets;
            hipLaunchKernelGGL(or_empty, dim3(m < 262144 ? (m + 255) / 256 : 1024), dim3(256), 0, stream, ob.filled, m);
            const bool staged = n > kOrStagedRow && (uint64_t)n * rows >= kOrStagedFrom;
            hipLaunchKernelGGL((staged ? or_scatter<true> : or_scatter<false>), dim3((n + kPiece - 1) / kPiece, rows), dim3(kOrScatterThreads), buckets * sizeof(uint32_t),
                               stream, t, ob, (uint64_t)first_plan + p0, seed, device_status);
        }
        hipLaunchKernelGGL(or_buckets, dim3(buckets, rows), dim3(kOrBucketThreads), 0, stream, t, ob, (uint64_t)first_plan + p0, seed,
                           orders + (size_t)p0 * n, device_status);
    }
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}
