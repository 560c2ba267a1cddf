// stalloc_validate: pairwise check of the planning constraint of Sec. 5.1 -- no two
// allocation decisions may conflict in lifespan and in address range at once.
//
// Three forms of the same count.  val_pairs tests all n(n-1)/2 unordered pairs of every plan: the
// pair space is cut into 256 x 256 tiles (upper triangle only); one workgroup owns one tile of
// one plan: each thread keeps its own request i in registers and walks the 256 requests j of the
// tile, which sit in LDS and are read as broadcasts.  val_near puts the short-lived requests in order of
// time and the long-lived ones in order of address first and leaves out what cannot meet (see there); val_four goes through four
// plans together in order of time.  Per plan all accumulate the number of conflicting pairs and the smallest key (i << 32 | j),
// i < j, which is the lexicographically first conflicting pair.
#include "host_util.h"
#include "wave.h"

namespace stalloc {

constexpr int kValTile = 256;

// val_near is part of calls of at least this many requests^2 x plans: its seven further launches cost some 35 us, all pairs
// take 50 us and more from here on (all pairs / val_near: 6144 requests, 10 plans 65 / 50 us; 19 612 requests, one plan 65 / 43;
// 960 requests, 440 plans 87 / 59; of an expert-parallel trace, where all requests go into buckets by address, 6144 and 8 plans 58 / 63,
// 10 plans 66 / 63).
#ifndef STALLOC_VAL_NEAR_FROM
#define STALLOC_VAL_NEAR_FROM (300ull * 1000 * 1000)
#endif
constexpr uint64_t kVnFrom = STALLOC_VAL_NEAR_FROM;
// Four plans a wave (val_four) where a look at the lifetimes is most of the work, from four plans on: in short traces; and, up to some length
// and from some requests x plans on, in traces of which few requests are alive at a time, which only the device knows, so that both forms
// are enqueued and one of them returns at once (3 us).
constexpr uint32_t kVfPlans = 4;
constexpr uint32_t kVfShort = 224, kVfMiddling = 2048, kVfLongest = 8192;
constexpr uint64_t kVfFrom = 1000 * 1000, kVfLongFrom = 4000 * 1000;
constexpr uint32_t kVfGroups = 32768;          // workgroups: several times what is resident; they take further plans in turn
constexpr size_t kVnRoom = (size_t)128 << 20;    // what the plans that are gone through together take of the workspace
constexpr uint32_t kVnGroup = 65535;             // (largest grid.y)
// Waves that are resident.  They take the units of work of a few plans (199 748 requests, one plan 12 us more with twice as many);
// with many plans a wave has few units, and twice as many even out (6144 requests, 512 plans 217 -> 206 us).
constexpr uint64_t kVnResident = 256 * 24;
// With fewer units than this a unit takes 64 boxes instead of 256, so that there are enough of them (49 920 requests, one plan,
// val_near alone 65 -> 35 us).
constexpr uint64_t kVnFewUnits = 4 * kVnResident;

__global__ void val_init(uint64_t* conflicts, uint64_t* first_key, uint32_t P)
{
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < P; p += gridDim.x * blockDim.x) {
        conflicts[p] = 0;
        first_key[p] = ~0ull;
    }
}

// One tile of one plan.
__global__ void __launch_bounds__(kValTile)
val_pairs(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf,
          const uint64_t* __restrict__ offsets, uint32_t n, uint32_t tiles, uint32_t plan0,
          uint64_t* conflicts, uint64_t* first_key, uint32_t* status)
{
    __shared__ uint64_t j_lo[kValTile];
    __shared__ uint64_t j_hi[kValTile];
    __shared__ uint32_t j_ta[kValTile];
    __shared__ uint32_t j_tf[kValTile];
    const uint32_t p = plan0 + blockIdx.y, lin = blockIdx.x;
    // linear tile index -> (ti, tj) with ti <= tj, row-major over the upper triangle
    const double nt = (double)tiles;
    uint32_t ti = (uint32_t)((2.0 * nt + 1.0 - sqrt((2.0 * nt + 1.0) * (2.0 * nt + 1.0) - 8.0 * (double)lin)) * 0.5);
    if (ti >= tiles) ti = tiles - 1;
    // row ti starts at ti*tiles - ti*(ti-1)/2; fix rounding either way
    auto row_start = [&](uint32_t r) { return (uint64_t)r * tiles - (uint64_t)r * (r - 1) / 2; };
    while (ti > 0 && row_start(ti) > lin) --ti;
    while (ti + 1 < tiles && row_start(ti + 1) <= lin) ++ti;
    const uint32_t tj = ti + (uint32_t)(lin - row_start(ti));

    const uint64_t* off = offsets + (size_t)p * n;

    const uint32_t j0 = tj * kValTile;
    {
        uint32_t j = j0 + threadIdx.x;
        bool ok = j < n;
        uint64_t o = ok ? off[j] : 0, s = ok ? size[j] : 0;
        // an address range that would run past 2^64 is reported, and kept from wrapping so that
        // what it covers still counts
        if (o + s < o) { atomicMax(status, (uint32_t)STALLOC_ERR_OVERFLOW); s = ~o; }
        j_lo[threadIdx.x] = o;
        j_hi[threadIdx.x] = o + s;
        j_ta[threadIdx.x] = ok ? ta[j] : 0;
        j_tf[threadIdx.x] = ok ? tf[j] : 0;     // empty lifetime [0,0): conflicts with nothing
    }
    const uint32_t i = ti * kValTile + threadIdx.x;
    const bool i_ok = i < n;
    const uint64_t i_lo = i_ok ? off[i] : 0;
    const uint64_t i_size = i_ok ? size[i] : 0;
    const uint64_t i_hi = i_lo + i_size < i_lo ? ~0ull : i_lo + i_size;
    const uint32_t i_ta = i_ok ? ta[i] : 0;
    const uint32_t i_tf = i_ok ? tf[i] : 0;
    __syncthreads();

    uint32_t count = 0;
    uint32_t min_j = 0xffffffffu;
    // on the diagonal tile only j > i counts
    const uint32_t first = (ti == tj) ? threadIdx.x + 1 : 0;
#pragma unroll 8
    for (uint32_t q = 0; q < kValTile; ++q) {
        bool hit = (q >= first) & (j_ta[q] < i_tf) & (i_ta < j_tf[q]) & (j_lo[q] < i_hi) & (i_lo < j_hi[q]);
        if (hit) {
            ++count;
            uint32_t j = j0 + q;
            min_j = j < min_j ? j : min_j;
        }
    }
    uint64_t key = count ? (((uint64_t)i << 32) | min_j) : ~0ull;
    uint32_t wave_count = wave_sum32(count);
    uint64_t wave_key = wave_min64(key);
    if (lane_id() == 0 && wave_count) {
        atomicAdd((unsigned long long*)&conflicts[p], (unsigned long long)wave_count);
        atomicMin((unsigned long long*)&first_key[p], (unsigned long long)wave_key);
    }
}

// ------------------------------------------------------------------------------------------
// Pairs that can meet.  In a plan worth checking few pairs meet in time and in address range, and which of the two says
// so sooner depends on the pair.  Requests that live shortly meet few others in time, whatever their addresses are (thousands
// of them share the lowest addresses); requests that live long meet a large part of all others in time, but few in
// address range (that is what keeps the plan free of conflicts).  So the requests are put, once per call, into buckets of (lifetime
// class, allocation time), and the long-lived ones, which come last, into buckets by address for each plan.  64 neighbours are a
// tile with a box, a span of time and of addresses: short spans of time for the short-lived, of addresses for the long-lived.
// A wave takes a tile, a request a lane, and holds it against the boxes of the tiles at and behind it: few of its requests meet a
// box, most of them none.  Only then is the other tile looked at, request by request.
// Which request of a bucket comes first does not matter: the results are a sum and a minimum over the request numbers.
//   Bound by chains of loads (a tile, its boxes, the tiles that it meets) with few waves, by vector issue with many.  All
// tiles of requests that meet in time, by request / this: 199 748 requests, one plan 228 / 68 us, of which val_near 29 (before 185);
// 6144 requests, 512 plans 599 / 200; 49 920 requests, 8 plans 474 / 165.  With the long-lived tile in the lanes and the short ones
// loaded one after the other, each a round trip to memory, val_near took 216 us on the first of these.
constexpr uint32_t kVnTile = 64;
constexpr uint32_t kVnWaves = 4;
constexpr uint32_t kVnRow = kVnTile + 4;         // (the walk over a tile's requests takes four at a time)

// Lifetimes below 2^base (about the time in which 64 requests are allocated) form class 0, whose
// buckets are 2^base wide; class k holds the lifetimes of [2^(base+k-1), 2^(base+k)) in buckets of a
// half of the smallest of them.
struct VnBuckets {
    uint32_t base, t_end, count;
    uint32_t apart;              // counters lie 2^apart words apart: on a coarse clock there are few, and atomics on one line of memory queue up
    uint32_t lasting;            // classes from here on are long-lived
    __host__ __device__ uint32_t shift_of(uint32_t k) const { return k == 0 ? base : (base + k > 2 ? base + k - 2 : 0u); }
    __host__ __device__ uint32_t in_class(uint32_t k) const { return (t_end >> shift_of(k)) + 1; }
    __device__ uint32_t of(uint32_t ta, uint32_t tf) const            // place of the counter
    {
        const uint32_t bits = 32u - (uint32_t)__builtin_clz((tf - ta) | 1u);
        const uint32_t cls = bits > base ? bits - base : 0u;
        uint32_t first = 0;
        for (uint32_t k = 0; k < cls; ++k) first += in_class(k);
        return (first + ((ta < t_end ? ta : t_end) >> shift_of(cls))) << apart;
    }
    __host__ __device__ uint32_t words() const { return count << apart; }
    __device__ uint32_t longest_short() const { return base + lasting > 32 ? 0xffffffffu : 1u << (base + lasting - 1); }   // (and what is shorter)
    __host__ __device__ uint32_t before_lasting() const               // buckets of the short-lived classes
    {
        uint32_t first = 0;
        for (uint32_t k = 0; k < lasting && k <= 32 - base; ++k) first += in_class(k);
        return first;
    }
};

static VnBuckets vn_buckets(uint32_t n, uint32_t t_end)
{
    VnBuckets b = {0, t_end, 0, 0, 1};
    while (b.base < 31 && ((uint64_t)n << b.base) < (uint64_t)t_end * kVnTile) ++b.base;
    for (uint32_t k = 0; k <= 32 - b.base; ++k) b.count += b.in_class(k);
    while (b.apart < 5 && b.count << b.apart < 4096) ++b.apart;
    // With c requests alive at once a request meets about 2 c others in time and, as each of them has a c-th of the
    // addresses, 2 n / c in address range: long-lived is what lives while more than the square root of n are allocated.
    while (b.lasting < 31 && ((uint64_t)kVnTile << b.lasting) * (kVnTile << b.lasting) <= n) ++b.lasting;
    return b;
}

struct VnSorted {
    uint32_t* bucket;        // [buckets.words()] requests per bucket, then where the next one of the bucket goes
    uint32_t* shorts_in;     // [n / 256] short-lived requests among 256 (and then: in front of them)
    uint2* shorts;           // [1] x: how many requests are short-lived: the first ones in bucket order; y: whether val_four has the plans
    uint2* life;             // [n] in bucket order: lifetime,
    uint64_t* size;          //     size
    uint32_t* id;            //     and number of the request
};

struct Range { uint64_t lo, hi; };
struct VnBox { uint64_t lo, hi; uint32_t t_first, t_last; };
// Of every plan of a group: address ranges in bucket order, those of the long-lived in order of their start; the latter's lifetimes
// and numbers.
struct VnPlans {
    uint64_t* top;           // [plans] highest end of a long-lived request
    uint64_t* start;         // [plans][n] start addresses of the long-lived in bucket order (from place 0)
    Range* range;            // [plans][n] short-lived in bucket order, then long-lived by address
    uint2* life;             // [plans][n] of the long-lived (from place 0)
    uint32_t* id;            // [plans][n]
    VnBox* box;              // [plans][tiles] of the short-lived, then of the long-lived
};

// Most traces number their requests by allocation time.  Then the short-lived ones are in the order they are wanted in, and only have
// to be told from the others: shorts_in[k] of the requests 256 k .. are short-lived.
__device__ __forceinline__ bool vn_short(const VnBuckets& b, uint32_t ta, uint32_t tf) { return tf - ta < b.longest_short(); }

__global__ void __launch_bounds__(256) vn_clear(const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n, VnBuckets b, VnSorted s,
                                                uint64_t* conflicts, uint64_t* first_key, uint32_t P, uint64_t* top, uint32_t group, uint64_t* acc)
{
    const uint32_t buckets = b.words(), first = blockIdx.x * 256 + threadIdx.x;
    for (uint32_t k = first; k < buckets || k < P; k += gridDim.x * 256) {
        if (k < buckets) s.bucket[k] = 0;
        if (k < P) { conflicts[k] = 0; first_key[k] = ~0ull; }
        if (k < group) top[k] = 0;                                    // (group <= P)
    }
    const bool crowded = (acc[kAccCrowded] & kCrowded) != 0;
    for (uint32_t i0 = blockIdx.x * 256; i0 < n; i0 += gridDim.x * 256) {                      // (uniform trip count)
        const uint32_t i = i0 + threadIdx.x;
        const uint32_t a = i < n ? ta[i] : 0u, f = i < n ? tf[i] : 0u;
        if (__builtin_amdgcn_ballot_w64(i + 1 < n && a > ta[i + 1 < n ? i + 1 : 0]) && lane_id() == 0) acc[kAccUnsorted] = 1;
        const int many = __syncthreads_count(i < n && !crowded && vn_short(b, a, f));
        if (threadIdx.x == 0) s.shorts_in[i0 / 256] = (uint32_t)many;
    }
}

// One atomic for all lanes of the wave that name the same bucket, as far as the first four buckets
// go (requests are numbered by allocation time in most traces, so that few buckets meet in a
// wave and many lanes in a bucket); returns what the bucket held in front of the lane's request.
__device__ __forceinline__ uint32_t vn_take(uint32_t* bucket, uint32_t mine, bool valid)
{
    uint32_t place = 0;
    uint64_t left = __builtin_amdgcn_ballot_w64(valid);
    for (int round = 0; round < 4 && left; ++round) {
        const uint32_t b = read_lane(mine, __builtin_ctzll(left));
        const uint64_t same = __builtin_amdgcn_ballot_w64(valid && mine == b) & left;
        uint32_t first = 0;
        if (lane_id() == __builtin_ctzll(same)) first = atomicAdd(&bucket[b], (uint32_t)__builtin_popcountll(same));
        first = read_lane(first, __builtin_ctzll(same));
        if ((same >> lane_id()) & 1) place = first + lanes_below(same);
        left &= ~same;
    }
    if ((left >> lane_id()) & 1) place = atomicAdd(&bucket[mine], 1u);
    return place;
}

// A crowded trace (a fifth of all requests alive at once, or a clock of which it covers little) has no short-lived requests
// worth the name: all count as long-lived, in the order that they have.
__global__ void __launch_bounds__(256)
vn_count(const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n, VnBuckets b, uint32_t* bucket, const uint64_t* acc)
{
    const uint64_t alive = acc[kAccCrowded], unsorted = acc[kAccUnsorted];        // (loaded together: mostly that is all the kernel does)
    if ((alive & kCrowded) | (unsorted == 0)) return;
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {        // (uniform trip count)
        const uint32_t i = i0 + threadIdx.x;
        vn_take(bucket, i < n ? b.of(ta[i], tf[i]) : 0u, i < n);
    }
}

// Exclusive sums of the bucket sizes (of shorts_in, when that is all), in place; one workgroup, four a thread and step.
// `form`: val_four has the plans (2: if few requests are alive at a time).
__global__ void __launch_bounds__(1024) vn_starts(VnBuckets b, VnSorted s, uint32_t n, uint32_t form, const uint64_t* acc)
{
    __shared__ uint32_t part[16];
    const uint64_t alive = acc[kAccCrowded], unsorted = acc[kAccUnsorted];
    const bool by_bucket = (unsorted != 0) & !(alive & kCrowded);
    uint32_t* counted = by_bucket ? s.bucket : s.shorts_in;
    const uint32_t many = by_bucket ? b.count : (n + 255) / 256, apart = by_bucket ? b.apart : 0u, lasting = by_bucket ? b.before_lasting() : many;
    uint32_t carry = 0;
    for (uint32_t k0 = 0; k0 < many; k0 += 4096) {
        const uint32_t k = k0 + 4 * threadIdx.x;
        uint32_t v[4], mine = 0;
        for (int u = 0; u < 4; ++u) { v[u] = k + u < many ? counted[(k + u) << apart] : 0u; mine += v[u]; }
        const uint32_t incl = wave_scan_add(mine);
        __syncthreads();                                              // (the step before has read part[])
        if (lane_id() == kWave - 1) part[wave_id()] = incl;
        __syncthreads();
        uint32_t before = carry + incl - mine;
        for (int w = 0; w < 16; ++w) { if (w < wave_id()) before += part[w]; carry += part[w]; }
        for (int u = 0; u < 4; ++u) {
            if (k + u < many) counted[(k + u) << apart] = before;
            if (k + u == lasting && k + u < many) s.shorts->x = before;
            before += v[u];
        }
    }
    if (threadIdx.x != 0) return;
    if (lasting >= many) s.shorts->x = carry;
    // (long traces of which hardly any are alive have so few tiles that meet that val_near is the faster)
    s.shorts->y = form == 1 || (form == 2 && (alive & kFewAlive) && (n <= kVfMiddling || !(alive & kHardlyAnyAlive))) ? 1u : 0u;
}

__global__ void __launch_bounds__(256)
vn_scatter(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n,
           VnBuckets b, VnSorted s, const uint64_t* acc)
{
    __shared__ uint32_t part[4];
    const uint64_t alive = acc[kAccCrowded], unsorted = acc[kAccUnsorted];
    const uint32_t shorts = s.shorts->x;
    const bool crowded = (alive & kCrowded) != 0, sorted = crowded | (unsorted == 0);         // (uniform)
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {        // (uniform trip count)
        const uint32_t i = i0 + threadIdx.x;
        const bool valid = i < n;
        const uint32_t a = valid ? ta[i] : 0u, f = valid ? tf[i] : 0u;
        uint32_t at;                                                   // < n: every place is taken once
        if (sorted) {
            const bool brief = valid && !crowded && vn_short(b, a, f);
            const uint64_t wave_shorts = __builtin_amdgcn_ballot_w64(brief);
            __syncthreads();                                           // (the step before has read part[])
            if (lane_id() == 0) part[wave_id()] = (uint32_t)__builtin_popcountll(wave_shorts);
            __syncthreads();
            uint32_t before = s.shorts_in[i0 / 256] + lanes_below(wave_shorts);
            for (int w = 0; w < wave_id(); ++w) before += part[w];
            at = brief ? before : shorts + (i - before);
        } else {
            at = vn_take(s.bucket, b.of(a, f), valid);
        }
        if (!valid) continue;
        s.life[at] = make_uint2(a, f);
        s.size[at] = size[i];
        s.id[at] = i;
    }
}

__device__ __forceinline__ VnBox vn_box(bool ok, const Range& r, const uint2& life)     // of the requests in a wave's lanes
{
    return VnBox{wave_min64(ok ? r.lo : ~0ull), wave_max64(ok ? r.hi : 0ull),
                 ~read_lane(wave_scan_max(ok ? ~life.x : 0u), kWave - 1), read_lane(wave_scan_max(ok ? life.y : 0u), kWave - 1)};
}

// The address ranges of a plan in bucket order, and the boxes of its short-lived tiles.
__global__ void __launch_bounds__(256)
vn_ranges(VnSorted s, const uint64_t* __restrict__ offsets, uint32_t n, uint32_t tiles, uint32_t plan0, VnPlans v, uint32_t* status)
{
    const uint2 parted = *s.shorts;
    if (parted.y) return;
    const uint32_t k = blockIdx.x * 256 + threadIdx.x, p = blockIdx.y, shorts = parted.x;
    const size_t row = (size_t)p * n;
    uint64_t hi = 0;                                                  // of a long-lived request
    Range r = {0, 0};
    if (k < n) {
        const uint64_t lo = offsets[(size_t)(plan0 + p) * n + s.id[k]], size = s.size[k];
        // an address range that would run past 2^64 is reported, and kept from wrapping so that what
        // it covers still counts
        const bool wraps = lo + size < lo;
        if (wraps) atomicMax(status, (uint32_t)STALLOC_ERR_OVERFLOW);
        r = Range{lo, wraps ? ~0ull : lo + size};
        if (k < shorts) v.range[row + k] = r;
        else { v.start[row + k - shorts] = lo; hi = r.hi; }
    }
    const uint64_t top = wave_max64(hi);
    if (lane_id() == 0 && top) atomicMax((unsigned long long*)&v.top[p], (unsigned long long)top);
    if (k - lane_id() >= shorts) return;                              // (uniform in a wave, and the rest is by waves)
    const VnBox box = vn_box(k < shorts, r, k < shorts ? s.life[k] : make_uint2(0u, 0u));
    if (lane_id() == 0) v.box[(size_t)p * tiles + k / kVnTile] = box;
}

// Start addresses to buckets of one width.  They cover what nearly all starts lie in, as a sample of 64 shows, with as much again to either
// side; the first and the last bucket take what lies beyond, so that an address that is far off (a damaged decision, what a validator is
// for) or a large one that all have in common costs little.  (In buckets from 0 to the highest end one address near 2^62 puts all others
// into one: 49 920 requests of an expert-parallel trace, one plan 351 us with a decision at 2^62, 107 without; here 112 and 107.)
struct VnPlaces {
    uint64_t from, width;
    uint32_t shift;
    __device__ __forceinline__ uint32_t of(uint64_t start) const { return (uint32_t)(umin64(start > from ? start - from : 0ull, width) >> shift); }
};
__device__ __forceinline__ VnPlaces vn_places(uint64_t sample, uint64_t top, uint32_t place_bits)     // one start per lane
{
    const uint64_t x = read_lane(sample, 10), y = read_lane(sample, 31), z = read_lane(sample, 52), high = umax64(x, y), low = umin64(x, y);
    const uint64_t middle = umax64(low, umin64(high, z));
    const uint64_t away = sample > middle ? sample - middle : middle - sample, most = umax64(middle, top - middle);
    uint32_t bits = most ? 64 - (uint32_t)__builtin_clzll(most) : 0u;                          // all but two are less than 2^bits away
    while (bits > 0 && __builtin_popcountll(__builtin_amdgcn_ballot_w64(away >> (bits - 1) == 0)) >= kWave - 2) --bits;
    const uint64_t far = bits < 63 ? 2ull << bits : ~0ull;
    const uint64_t from = middle > far ? middle - far : 0ull, to = top - middle < far ? top : middle + far;
    const uint64_t width = to - from;                                 // (no start is above the highest end)
    const uint32_t width_bits = width ? 64 - (uint32_t)__builtin_clzll(width) : 0u;
    return VnPlaces{from, width, width_bits > place_bits ? width_bits - place_bits : 0u};
}

// The long-lived requests of a plan in buckets of their start addresses, and their tiles' boxes; one workgroup a plan.
__global__ void __launch_bounds__(1024) vn_by_address(VnSorted s, uint32_t n, uint32_t tiles, uint32_t place_bits, VnPlans v)
{
    extern __shared__ uint32_t bucket[];                              // 2^place_bits
    __shared__ uint32_t part[16];
    const uint2 parted = *s.shorts;
    const uint32_t p = blockIdx.x, shorts = parted.x, longs = n - shorts, step = blockDim.x, waves = step / kWave;
    if (longs == 0 || parted.y) return;
    const size_t row = (size_t)p * n;
    const uint64_t top = v.top[p], sample = v.start[row + (uint32_t)((uint64_t)longs * lane_id() / kWave)];
    constexpr int kAhead = 4;                                         // requests a thread, or tiles a wave, has under way together
    uint64_t lo[kAhead];
    auto load_starts = [&](uint32_t k) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) lo[u] = v.start[row + umin(k + u * step, longs - 1)];
    };
    load_starts(threadIdx.x);
    const uint32_t buckets = 1u << place_bits, per = (buckets + step - 1) / step;       // (buckets a thread sums up)
    for (uint32_t k = threadIdx.x; k < buckets; k += step) bucket[k] = 0;
    const VnPlaces places = vn_places(sample, top, place_bits);
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < longs; k += kAhead * step) {
        if (k != threadIdx.x) load_starts(k);
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (k + u * step < longs) atomicAdd(&bucket[places.of(lo[u])], 1u);
    }
    __syncthreads();
    const uint32_t k0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t u = 0; u < per; ++u) mine += k0 + u < buckets ? bucket[k0 + u] : 0u;
    const uint32_t incl = wave_scan_add(mine);
    if (lane_id() == kWave - 1) part[wave_id()] = incl;
    __syncthreads();
    uint32_t before = incl - mine;
    for (int w = 0; w < wave_id(); ++w) before += part[w];
    for (uint32_t u = 0; u < per && k0 + u < buckets; ++u) {
        const uint32_t many = bucket[k0 + u];
        bucket[k0 + u] = before;
        before += many;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < longs; k += kAhead * step) {
        uint64_t size[kAhead];
        uint2 life[kAhead];
        uint32_t id[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t at = umin(k + u * step, longs - 1);
            lo[u] = v.start[row + at]; size[u] = s.size[shorts + at]; life[u] = s.life[shorts + at]; id[u] = s.id[shorts + at];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (k + u * step >= longs) break;
            const uint32_t at = atomicAdd(&bucket[places.of(lo[u])], 1u);      // < longs: the buckets hold every one of them once
            v.range[row + shorts + at] = Range{lo[u], lo[u] + size[u] < lo[u] ? ~0ull : lo[u] + size[u]};
            v.life[row + at] = life[u];
            v.id[row + at] = id[u];
        }
    }
    __syncthreads();                                                  // (what this workgroup has written is read by itself)
    VnBox* box = v.box + (size_t)p * tiles + (shorts + kVnTile - 1) / kVnTile;
    for (uint32_t t0 = (uint32_t)wave_id(); t0 * kVnTile < longs; t0 += kAhead * waves) {
        Range r[kAhead];
        uint2 l[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t k = umin((t0 + u * waves) * kVnTile + lane_id(), longs - 1);
            r[u] = v.range[row + shorts + k];
            l[u] = v.life[row + k];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t t = t0 + u * waves;
            const VnBox of = vn_box(t * kVnTile + lane_id() < longs, r[u], l[u]);
            if (lane_id() == 0 && t * kVnTile < longs) box[t] = of;
        }
    }
    if (threadIdx.x == 0) v.top[p] = 0;                               // (for the next group of plans)
}

// All pairs of a plan that can meet.  A unit of work is a first tile and 64 kBoxes second tiles at or behind it, whose boxes the
// wave takes in turn as scalars; `waves` waves a plan take the units in turn (how many tiles there are is known on the device only).
struct ValNearLds {
    uint4 who[kVnWaves][kVnRow];                                      // t_alloc, t_free, number, place in the tile
    Range range[kVnWaves][kVnRow];
};
struct VnRecord { uint2 life; Range range; uint32_t id; };

template <uint32_t kBoxes>
__global__ void __launch_bounds__(kVnWaves * kWave, 6)
val_near(VnSorted s, VnPlans v, uint32_t n, uint32_t box_row, uint32_t plan0, uint32_t plans, uint32_t waves, uint64_t* conflicts,
         uint64_t* first_key)
{
    __shared__ ValNearLds sh;
    const int lane = lane_id(), wave = wave_id();
    const uint32_t nth = blockIdx.x * kVnWaves + (uint32_t)wave, p = nth / waves;
    const uint2 parted = *s.shorts;
    const uint32_t shorts = parted.x;
    if (p >= plans || parted.y) return;                               // (uniform; the waves do not meet)
    const uint32_t st = (shorts + kVnTile - 1) / kVnTile, tiles = st + (n - shorts + kVnTile - 1) / kVnTile;
    const size_t row = (size_t)p * n;
    const VnBox* box = v.box + (size_t)p * box_row;
    auto record_of = [&](uint32_t t) -> VnRecord {                    // (t uniform) this lane's request of tile t
        const bool brief = t < st;
        const uint32_t at = (brief ? t : t - st) * kVnTile + lane, many = brief ? shorts : n - shorts, k = at < many ? at : many - 1;
        VnRecord r = {brief ? s.life[k] : v.life[row + k], v.range[row + (brief ? 0u : shorts) + k], brief ? s.id[k] : v.id[row + k]};
        if (at >= many) r.life = make_uint2(0xffffffffu, 0u);         // (meets nothing)
        return r;
    };
    uint64_t count = 0;                                               // (a wave's units hold more than 2^32 pairs from 7.3 million requests on)
    uint64_t key = ~0ull;
    const uint32_t blocks = (tiles + kBoxes * kWave - 1) / (kBoxes * kWave);
    for (uint32_t u = nth % waves; u < tiles * blocks; u += waves) {
        const uint32_t it = u % tiles, jn = u / tiles * kBoxes * kWave;
        if (jn + kBoxes * kWave <= it) continue;                    // (uniform)
        const VnBox own = box[it];
        const VnRecord mine = record_of(it);
        VnBox other[kBoxes];
#pragma unroll
        for (uint32_t c = 0; c < kBoxes; ++c) other[c] = box[umin(jn + c * kWave + lane, tiles - 1)];
#pragma unroll
        for (uint32_t c = 0; c < kBoxes; ++c) {
            const uint32_t j0 = jn + c * kWave;
            const VnBox& o = other[c];
            uint64_t near = __builtin_amdgcn_ballot_w64(j0 + lane < tiles && j0 + lane >= it && o.t_first < own.t_last && own.t_first < o.t_last &&
                                                        o.lo < own.hi && own.lo < o.hi);
            auto meets = [&](int f) -> uint64_t {                     // requests of the first tile that meet the box of lane f
                return lanes_lt(mine.life.x, read_lane(o.t_last, f)) & lanes_lt(read_lane(o.t_first, f), mine.life.y) &
                       lanes_lt(mine.range.lo, read_lane(o.hi, f)) & lanes_lt(read_lane(o.lo, f), mine.range.hi);
            };
            uint64_t hit = 0;
            for (; near; near &= near - 1)
                if (meets(__builtin_ctzll(near))) hit |= near & -near;
            if (hit == 0) continue;                                   // (uniform)
            VnRecord next = record_of(j0 + (uint32_t)__builtin_ctzll(hit));
            while (hit) {
                const int f = __builtin_ctzll(hit);
                const uint32_t jt = j0 + (uint32_t)f;
                hit &= hit - 1;
                const VnRecord now = next;
                if (hit) next = record_of(j0 + (uint32_t)__builtin_ctzll(hit));
                const uint64_t left = meets(f);
                const uint32_t many = (uint32_t)__builtin_popcountll(left);
                __builtin_amdgcn_wave_barrier();                      // (the wave's own LDS: its accesses complete in order)
                if (lane_in(left)) {
                    const uint32_t to = lanes_below(left);
                    sh.who[wave][to] = make_uint4(mine.life.x, mine.life.y, mine.id, (uint32_t)lane);
                    sh.range[wave][to] = mine.range;
                }
                if (lane < 4) sh.who[wave][many + lane] = make_uint4(0xffffffffu, 0u, 0u, 0u);      // up to a multiple of four
                __builtin_amdgcn_wave_barrier();
                for (uint32_t k = 0; k < many; k += 4) {
                    uint64_t pair[4], any = 0;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const uint4 who = sh.who[wave][k + w];
                        const Range r = sh.range[wave][k + w];
                        pair[w] = lanes_lt(who.x, now.life.y) & lanes_lt(now.life.x, who.y) & lanes_lt(r.lo, now.range.hi) & lanes_lt(now.range.lo, r.hi);
                        if (jt == it) pair[w] &= ~1ull << uniform(who.w);     // inside one tile: the second one lies behind
                        any |= pair[w];
                    }
                    if (any == 0) continue;                           // (uniform) the usual case
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const uint32_t i = sh.who[wave][k + w].z, j = now.id;
                        count += (uint32_t)__builtin_popcountll(pair[w]);
                        if (lane_in(pair[w])) key = umin64(key, i < j ? ((uint64_t)i << 32) | j : ((uint64_t)j << 32) | i);
                    }
                }
            }
        }
    }
    if (count == 0) return;                                           // (uniform)
    const uint64_t wave_key = wave_min64(key);
    if (lane == 0) {
        atomicAdd((unsigned long long*)&conflicts[plan0 + p], (unsigned long long)count);
        atomicMin((unsigned long long*)&first_key[plan0 + p], (unsigned long long)wave_key);
    }
}

// All pairs of four plans that meet in time, in the order of VnSorted: a wave takes a tile of first requests, a request a lane, and
// holds it against four tiles of second requests at or behind it, request by request as broadcasts from LDS: two lifetime compares for all
// plans, two address compares a plan, and neither address ranges nor boxes are written first.  Tiles whose spans of time do not
// meet drop out together, requests of the others that do not meet the first tile's span 64 at a time.  The records of the next tile
// but one and the addresses of the next are on their way meanwhile.  A group of plans beyond the last plan repeats that one, and leaves out its results.
//   Bound by vector issue.  Whole calls with val_near / this: 500 requests of which 29 are alive at a time, 10 000 plans 287 / 215 us; 2000
// and 48, 2500 plans 395 / 293; 4000 and 67, 5000 plans 1784 / 1229; 8000 and 71, 2500 plans 2136 / 1403; 256 of an interleaved
// schedule, 24 414 plans 400 / 237.  With more alive it looks at more pairs, and val_near, which leaves out what is apart in address, catches up: 256
// requests and 92 equal, 384 and 139 val_near 7 to 15 % faster.  With hardly any alive so few tiles meet that val_near is the faster
// from some length on: 8000 and 11, 2500 plans 820 / 1120, 2000 and 11, 10 000 plans 835 / 772.
struct ValFourLds {
    uint4 who[kVnWaves][kVnRow];                                      // t_alloc, t_free, number, place in the tile
    Range range[kVnWaves][kVfPlans][kVnRow];
};

// The four tiles of a workgroup's waves and four second ones at or behind them: groups of four tiles in pairs (g, c), g <= c, numbered from c (c + 1) / 2 on.
__global__ void __launch_bounds__(kVnWaves * kWave, 5)
val_four(VnSorted s, const uint64_t* __restrict__ offsets, uint32_t n, uint32_t tiles, uint32_t plans, uint64_t* conflicts,
         uint64_t* first_key, uint32_t* status)
{
    __shared__ ValFourLds sh;
    __shared__ uint2 spans[kVnWaves];
    if (!s.shorts->y) return;                                         // (left to val_near)
    const int lane = lane_id(), wave = wave_id();
    // (with one tile or two, the workgroup's waves share them out four times or twice)
    const uint32_t per = tiles <= 2 ? tiles : kVnWaves, shares = kVnWaves / per, tile = (uint32_t)wave % per, share = (uint32_t)wave / per;
    uint32_t c = (uint32_t)((sqrt(1.0 + 8.0 * (double)blockIdx.x) - 1.0) * 0.5);
    while (c * (c + 1) / 2 > blockIdx.x) --c;
    while ((c + 1) * (c + 2) / 2 <= blockIdx.x) ++c;
    const uint32_t g = blockIdx.x - c * (c + 1) / 2, it = g * kVnWaves + tile, first_jt = c * kVnWaves;
    struct Record { uint2 life; uint64_t size; uint32_t id; };
    auto record_of = [&](uint32_t t) -> Record {                      // (t uniform) this lane's request of tile t
        const uint32_t at = t * kVnTile + lane;
        const bool ok = t < tiles && at < n;
        const uint32_t k = ok ? at : 0u;
        Record q = {s.life[k], s.size[k], s.id[k]};
        if (!ok) { q.life = make_uint2(0xffffffffu, 0u); q.size = 0; }        // (meets nothing)
        return q;
    };
    auto span_of = [&](const uint2& life) -> uint2 {
        return make_uint2(~read_lane(wave_scan_max(~life.x), kWave - 1), read_lane(wave_scan_max(life.y), kWave - 1));
    };
    const Record own = record_of(it);
    const uint2 span = span_of(own.life);
    {
        const uint2 second = g == c ? span : span_of(record_of(first_jt + tile).life);
        if (lane == 0) spans[wave] = second;
    }
    __syncthreads();
    uint64_t meets = 0;
    {
        const uint2 other = spans[lane & (kVnWaves - 1)];
        meets = __builtin_amdgcn_ballot_w64(lane < (int)per && first_jt + lane >= it && other.x < span.y && span.x < other.y);
    }
    // the requests with a malformed lifetime meet nothing, but an address range that would wrap is looked for in all
    if (meets == 0 && g != c) return;                                 // (uniform; the waves do not meet from here on)
    auto next_record = [&](uint64_t tiles_left) -> Record { return record_of(tiles_left ? first_jt + (uint32_t)__builtin_ctzll(tiles_left) : tiles); };
    for (uint64_t next_plan = (uint64_t)(blockIdx.y * shares + share) * kVfPlans; next_plan < plans; next_plan += gridDim.y * shares * kVfPlans) {
        const uint32_t p0 = (uint32_t)next_plan;
        auto addresses_of = [&](const Record& q, uint64_t (&lo)[kVfPlans]) {
#pragma unroll
            for (uint32_t p = 0; p < kVfPlans; ++p) lo[p] = offsets[(size_t)umin(p0 + p, plans - 1) * n + q.id];
        };
        uint64_t near = meets, ahead = near & (near - 1);
        Record now = next_record(near), next = next_record(ahead);
        uint64_t now_lo[kVfPlans], next_lo[kVfPlans], own_lo[kVfPlans];
        addresses_of(now, now_lo);
        addresses_of(own, own_lo);
        Range mine[kVfPlans];
        uint32_t count[kVfPlans];
        uint64_t key[kVfPlans];
#pragma unroll
        for (uint32_t p = 0; p < kVfPlans; ++p) {
            // an address range that would run past 2^64 is reported, and kept from wrapping so that what
            // it covers still counts
            const bool wraps = own_lo[p] + own.size < own_lo[p];
            if (g == c && wraps) atomicMax(status, (uint32_t)STALLOC_ERR_OVERFLOW);
            mine[p] = Range{own_lo[p], wraps ? ~0ull : own_lo[p] + own.size};
            count[p] = 0; key[p] = ~0ull;
        }
        for (; near; near &= near - 1) {
            const uint32_t jt = first_jt + (uint32_t)__builtin_ctzll(near);
            ahead &= ahead - 1;
            const Record after = next_record(ahead);
            addresses_of(next, next_lo);
            const uint64_t left = lanes_lt(now.life.x, span.y) & lanes_lt(span.x, now.life.y);
            const uint32_t many = (uint32_t)__builtin_popcountll(left);
            __builtin_amdgcn_wave_barrier();                              // (the wave's own LDS: its accesses complete in order)
            if (lane_in(left)) {
                const uint32_t to = lanes_below(left);
                sh.who[wave][to] = make_uint4(now.life.x, now.life.y, now.id, (uint32_t)lane);
#pragma unroll
                for (uint32_t p = 0; p < kVfPlans; ++p)
                    sh.range[wave][p][to] = Range{now_lo[p], now_lo[p] + now.size < now_lo[p] ? ~0ull : now_lo[p] + now.size};
            }
            now = next;
            next = after;
#pragma unroll
            for (uint32_t p = 0; p < kVfPlans; ++p) now_lo[p] = next_lo[p];
            if (lane < 4) sh.who[wave][many + lane] = make_uint4(0xffffffffu, 0u, 0u, 0u);      // up to a multiple of four
            __builtin_amdgcn_wave_barrier();
            for (uint32_t k = 0; k < many; k += 2) {
                uint64_t hit[2][kVfPlans], any = 0;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint4 who = sh.who[wave][k + u];
                    const uint64_t together = lanes_lt(who.x, own.life.y) & lanes_lt(own.life.x, who.y);
#pragma unroll
                    for (uint32_t p = 0; p < kVfPlans; ++p) {
                        const Range r = sh.range[wave][p][k + u];
                        hit[u][p] = together & lanes_lt(r.lo, mine[p].hi) & lanes_lt(mine[p].lo, r.hi);
                        any |= hit[u][p];
                    }
                }
                if (any == 0) continue;                                   // (uniform) the usual case
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint4 who = sh.who[wave][k + u];
                    const uint32_t j = who.z;
                    const uint64_t once = jt == it ? (1ull << uniform(who.w)) - 1 : ~0ull;      // inside one tile: the first one lies in front
#pragma unroll
                    for (uint32_t p = 0; p < kVfPlans; ++p) {
                        const uint64_t h = hit[u][p] & once;
                        count[p] += (uint32_t)__builtin_popcountll(h);     // (at most 64 * 256)
                        if (lane_in(h)) key[p] = umin64(key[p], own.id < j ? ((uint64_t)own.id << 32) | j : ((uint64_t)j << 32) | own.id);
                    }
                }
            }
        }
#pragma unroll
        for (uint32_t p = 0; p < kVfPlans; ++p) {
            if (count[p] == 0 || p0 + p >= plans) continue;            // (uniform)
            const uint64_t wave_key = wave_min64(key[p]);
            if (lane == 0) {
                atomicAdd((unsigned long long*)&conflicts[p0 + p], (unsigned long long)count[p]);
                atomicMin((unsigned long long*)&first_key[p0 + p], (unsigned long long)wave_key);
            }
        }
    }
}

__global__ void val_finish(const uint64_t* first_key, uint32_t* first_pair, uint32_t P)
{
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < P; p += gridDim.x * blockDim.x) {
        uint64_t k = first_key[p];
        first_pair[2 * p] = (uint32_t)(k >> 32);
        first_pair[2 * p + 1] = (uint32_t)k;
    }
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_validate(const stalloc_trace* tr, const uint64_t* offsets, uint32_t P, uint64_t* conflicts,
                                uint32_t* first_pair, uint32_t* device_status, void* workspace,
                                size_t* workspace_bytes, void* hip_stream)
{
    if (!trace_args_ok(tr) || P == 0 || !workspace_bytes) return STALLOC_ERR_INVALID_ARG;
    const uint64_t tiles = ((uint64_t)tr->n + kValTile - 1) / kValTile;
    const uint64_t tri = tiles * (tiles + 1) / 2;
    if (tri >= 0x7fffffffull) return STALLOC_ERR_INVALID_ARG;   // n beyond ~16.7 million requests
    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    uint64_t* first_key = cv.take<uint64_t>(P);
    bool near = (uint64_t)tr->n * tr->n * P >= kVnFrom;
    VnBuckets buckets = {};
    VnSorted sorted = {};
    VnPlans plans = {};
    const uint32_t near_tiles = (tr->n + kVnTile - 1) / kVnTile;
    // plans that are gone through together
    const size_t of_plan = (sizeof(Range) + sizeof(uint2) + sizeof(uint64_t) + sizeof(uint32_t)) * (size_t)tr->n;
    const size_t most = kVnRoom / of_plan;
    const uint32_t group_room = P < most ? P : most < 1 ? 1u : most < kVnGroup ? (uint32_t)most : kVnGroup;
    const size_t all_pairs = cv.used;
    const bool four_only = P >= kVfPlans && tr->n <= kVfShort;
    const bool four = four_only || (P >= kVfPlans && tr->n <= kVfLongest && (uint64_t)tr->n * P >= (tr->n <= kVfMiddling ? kVfFrom : kVfLongFrom));
    const uint32_t group = four_only ? 0 : group_room;
    if (near) {
        buckets = vn_buckets(tr->n, tr->t_end);
        sorted.bucket = cv.take<uint32_t>(buckets.words());
        sorted.shorts_in = cv.take<uint32_t>((tr->n + 255) / 256);
        sorted.shorts = cv.take<uint2>(1);
        sorted.life = cv.take<uint2>(tr->n);
        sorted.size = cv.take<uint64_t>(tr->n);
        sorted.id = cv.take<uint32_t>(tr->n);
        plans.top = cv.take<uint64_t>(group);
        plans.start = cv.take<uint64_t>((size_t)group * tr->n);
        plans.range = cv.take<Range>((size_t)group * tr->n);
        plans.life = cv.take<uint2>((size_t)group * tr->n);
        plans.id = cv.take<uint32_t>((size_t)group * tr->n);
        plans.box = cv.take<VnBox>((size_t)group * (near_tiles + 1));
    }
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    // (the first two pieces are all that P asks for; a workspace with room for no more gets the all-pairs form)
    if (near && *workspace_bytes < cv.used) near = false;
    if (!offsets || !conflicts || !first_pair || !device_status || *workspace_bytes < (near ? cv.used : all_pairs) ||
        (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    launch_trace_check(*tr, acc, device_status, stream);
    uint32_t pb = (P + 255) / 256;
    if (pb > 1024) pb = 1024;
    if (near) {
        uint32_t blocks = (tr->n + 255) / 256;
        if (blocks > 1024) blocks = 1024;
        uint32_t cb = ((buckets.words() > P ? buckets.words() : P) + 255) / 256;
        if (cb > 1024) cb = 1024;
        hipLaunchKernelGGL(vn_clear, dim3(cb > blocks ? cb : blocks), dim3(256), 0, stream, tr->t_alloc, tr->t_free, tr->n, buckets, sorted, conflicts,
                           first_key, P, plans.top, group, acc);
        hipLaunchKernelGGL(vn_count, dim3(blocks), dim3(256), 0, stream, tr->t_alloc, tr->t_free, tr->n, buckets, sorted.bucket, acc);
        hipLaunchKernelGGL(vn_starts, dim3(1), dim3(1024), 0, stream, buckets, sorted, tr->n, four_only ? 1u : four ? 2u : 0u, acc);
        hipLaunchKernelGGL(vn_scatter, dim3(blocks), dim3(256), 0, stream, tr->size, tr->t_alloc, tr->t_free, tr->n, buckets, sorted, acc);
        const uint32_t box_row = near_tiles + 1;                      // (the short-lived and the long-lived may each end with part of a tile)
        const uint64_t blocks_of_boxes = (box_row + kWave - 1) / kWave;
        // (short traces come with many plans: small workgroups, with little LDS, of which many are resident)
        const uint32_t threads = tr->n <= 512 ? 64 : tr->n <= 1024 ? 256 : 1024;
        uint32_t place_bits = 6;
        while (place_bits < 12 && (1u << place_bits) < tr->n) ++place_bits;
        const uint32_t fours = (near_tiles + kVnWaves - 1) / kVnWaves;
        if (four) {
            const uint32_t pairs = fours * (fours + 1) / 2, rows = (P - 1) / (kVfPlans * (near_tiles <= 2 ? kVnWaves / near_tiles : 1u)) + 1, most_rows = (kVfGroups + pairs - 1) / pairs;
            hipLaunchKernelGGL(val_four, dim3(pairs, rows < most_rows ? rows : most_rows), dim3(kVnWaves * kWave), 0, stream, sorted, offsets, tr->n,
                               near_tiles, P, conflicts, first_key, device_status);
        }
        for (uint32_t p0 = 0; !four_only && p0 < P; p0 += group) {
            const uint32_t many = P - p0 < group ? P - p0 : group;
            const bool few = blocks_of_boxes == 1 || blocks_of_boxes * box_row * many < kVnFewUnits;
            const uint64_t units = box_row * (few ? blocks_of_boxes : (blocks_of_boxes + 3) / 4);
            uint64_t waves = (many < 64 ? 1 : 2) * kVnResident / many;
            if (waves < 1) waves = 1;
            if (waves > units) waves = units;
            hipLaunchKernelGGL(vn_ranges, dim3((tr->n + 255) / 256, many), dim3(256), 0, stream, sorted, offsets, tr->n, box_row, p0, plans,
                               device_status);
            hipLaunchKernelGGL(vn_by_address, dim3(many), dim3(threads), sizeof(uint32_t) << place_bits, stream, sorted, tr->n, box_row,
                               place_bits, plans);
            hipLaunchKernelGGL(few ? val_near<1> : val_near<4>, dim3((uint32_t)((waves * many + kVnWaves - 1) / kVnWaves)), dim3(kVnWaves * kWave), 0,
                               stream, sorted, plans, tr->n, box_row, p0, many, (uint32_t)waves, conflicts, first_key);
        }
    } else {
        hipLaunchKernelGGL(val_init, dim3(pb), dim3(256), 0, stream, conflicts, first_key, P);
        for (uint32_t p0 = 0; p0 < P; p0 += 32768) {          // grid.y is limited to 65535
            uint32_t py = P - p0 < 32768 ? P - p0 : 32768;
            hipLaunchKernelGGL(val_pairs, dim3((uint32_t)tri, py), dim3(kValTile), 0, stream, tr->size, tr->t_alloc,
                               tr->t_free, offsets, tr->n, (uint32_t)tiles, p0, conflicts, first_key,
                               device_status);
        }
    }
    hipLaunchKernelGGL(val_finish, dim3(pb), dim3(256), 0, stream, first_key, first_pair, P);
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}
