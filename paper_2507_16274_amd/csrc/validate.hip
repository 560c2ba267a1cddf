// stalloc_validate: pairwise check of the planning constraint of Sec. 5.1 -- no two
// allocation decisions may conflict in lifespan and in address range at once.
//
// Two forms of the same count.  val_tile tests all n(n-1)/2 unordered pairs of every plan: the
// pair space is cut into 256 x 256 tiles (upper triangle only); one workgroup owns one tile of
// one plan: each thread keeps its own request i in registers and walks the 256 requests j of the
// tile, which sit in LDS and are read as broadcasts.  val_near puts the requests into buckets of
// like lifetime and allocation time first and leaves out what cannot meet in time (see there); in
// traces whose requests live for a fifth of the time on average there is little to leave out, and
// the launch for one plan takes the first form (the trace check has found out, see kAccCrowded).
// Per plan both accumulate the number of conflicting pairs and the smallest key (i << 32 | j),
// i < j, which is the lexicographically first conflicting pair.
#include "host_util.h"
#include "wave.h"

namespace stalloc {

constexpr int kValTile = 256;

// val_near is part of calls of at least this many requests^2 x plans: its five preparing launches cost 20 to 30 us
// (10 in a crowded trace, where they return at once), against 210 us and more that all pairs take from here on.
// Lifetimes of all lengths, all pairs / val_near: 40 000 requests, one plan 219 / 97 us; 6144 requests, 40 plans
// 213 / 110; 100 000 requests, 16 plans 18.9 / 2.2 ms.  Lifetimes a third of the time long: 220 / 217, 328 / 300,
// 18.9 / 10.1.  From 3.5e8 on, where they would pay in sparse traces, crowded ones took up to twice as long.
#ifndef STALLOC_VAL_NEAR_FROM
#define STALLOC_VAL_NEAR_FROM (1500ull * 1000 * 1000)
#endif
constexpr uint64_t kVnFrom = STALLOC_VAL_NEAR_FROM;
// Below these a wave takes one plan and looks whether the trace is crowded (four plans share a look at the lifetimes
// otherwise, and are as fast as all pairs in a crowded trace, but need enough waves: 20 000 requests, 4
// plans, crowded: 260 us all pairs, 295 four together; 40 000 requests, 4 plans 790 / 640).
constexpr uint64_t kVnTogether = 3000ull * 1000 * 1000, kVnThree = 10000ull * 1000 * 1000;

__global__ void val_init(uint64_t* conflicts, uint64_t* first_key, uint32_t P)
{
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < P; p += gridDim.x * blockDim.x) {
        conflicts[p] = 0;
        first_key[p] = ~0ull;
    }
}

// One tile of one plan; called by a workgroup of 256 threads.
__device__ __forceinline__ void val_tile(uint64_t (&j_lo)[kValTile], uint64_t (&j_hi)[kValTile], uint32_t (&j_ta)[kValTile],
                                         uint32_t (&j_tf)[kValTile], const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta,
                                         const uint32_t* __restrict__ tf, const uint64_t* __restrict__ offsets, uint32_t n, uint32_t tiles,
                                         uint32_t lin, uint32_t p, uint64_t* conflicts, uint64_t* first_key, uint32_t* status)
{
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

__global__ void __launch_bounds__(kValTile)
val_pairs(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf,
          const uint64_t* __restrict__ offsets, uint32_t n, uint32_t tiles, uint32_t plan0,
          uint64_t* conflicts, uint64_t* first_key, uint32_t* status)
{
    __shared__ uint64_t j_lo[kValTile];
    __shared__ uint64_t j_hi[kValTile];
    __shared__ uint32_t j_ta[kValTile];
    __shared__ uint32_t j_tf[kValTile];
    val_tile(j_lo, j_hi, j_ta, j_tf, size, ta, tf, offsets, n, tiles, blockIdx.x, plan0 + blockIdx.y, conflicts, first_key, status);
}

// ------------------------------------------------------------------------------------------
// Pairs that can meet in time.  A training trace holds few pairs with overlapping lifetimes
// (3.5e8 of 2.0e10 for the 200k requests of an interleaved schedule), and which ones they are does
// not depend on the plan.  The requests are put, once per call, into buckets of (lifetime class,
// allocation time); 64 neighbours of that sequence make a tile with a span [first allocation, last
// release).  Short-lived requests fill tiles of short spans, long-lived ones tiles of their own at
// the end of the sequence, so that a tile of the first kind meets its neighbours and the tiles of
// the second kind, and nothing else is looked at.  Which request of a bucket comes first does not
// matter: the results are a sum and a minimum over the request numbers.
//   Bound by the integer rate on many plans (6144 requests x 1024 plans: 1.16 ms, all pairs 4.76 ms) and by
// the chain load -> address gather -> LDS of a wave's tiles on one (199 748 requests: 0.23 ms, of which 0.19
// ms val_one_plan, all pairs 4.73 ms; an integer floor of 0.07 ms for its 3.5e8 pairs).
constexpr uint32_t kVnTile = 64;
constexpr uint32_t kVnWaves = 4;
constexpr uint32_t kVnRow = kVnTile + 4;         // (the walk over a tile's requests takes four at a time)

// Lifetimes below 2^base (about the time in which 64 requests are allocated) form class 0, whose
// buckets are 2^base wide; class k holds the lifetimes of [2^(base+k-1), 2^(base+k)) in buckets of a
// half of the smallest of them.
struct VnBuckets {
    uint32_t base, t_end, count;
    uint32_t apart;              // counters lie 2^apart words apart: on a coarse clock there are few, and atomics on one line of memory queue up
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
};

static VnBuckets vn_buckets(uint32_t n, uint32_t t_end)
{
    VnBuckets b = {0, t_end, 0, 0};
    while (b.base < 31 && ((uint64_t)n << b.base) < (uint64_t)t_end * kVnTile) ++b.base;
    for (uint32_t k = 0; k <= 32 - b.base; ++k) b.count += b.in_class(k);
    while (b.apart < 5 && b.count << b.apart < 4096) ++b.apart;
    return b;
}

// Tiles of second requests per wave: few, so that a small trace still gives the chip enough waves (6144
// requests, 4 plans: 62 us with 4 tiles a wave, 136 us with 16, 241 us with 64), but on long traces nearly
// all (wave, chunk) pairs have nothing to do and cost a workgroup's start each (199 748 requests, one
// plan: 332 us with 4, 245 us with 16, 294 us with 64; 49 920: 131 us with 4, 166 us with 16).
static uint32_t vn_chunk(uint32_t tiles) { return tiles <= 1024 ? 4u : 16u; }

struct VnSorted {
    uint32_t* bucket;        // [buckets.words()] requests per bucket, then where the next one of the bucket goes
    uint2* life;             // [n] in bucket order: lifetime,
    uint64_t* size;          //     size
    uint32_t* id;            //     and number of the request
    uint2* span;             // [tiles] first allocation, last release
};

// acc: nullptr when the all-pairs form is not part of the launch that follows.
__device__ __forceinline__ bool left_to_all_pairs(const uint64_t* acc) { return acc && acc[kAccCrowded]; }

__global__ void __launch_bounds__(256) vn_clear(uint32_t* bucket, uint32_t buckets, uint64_t* conflicts, uint64_t* first_key, uint32_t P)
{
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < buckets || k < P; k += gridDim.x * blockDim.x) {
        if (k < buckets) bucket[k] = 0;
        if (k < P) { conflicts[k] = 0; first_key[k] = ~0ull; }
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

__global__ void __launch_bounds__(256)
vn_count(const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n, VnBuckets b, uint32_t* bucket, const uint64_t* acc)
{
    if (left_to_all_pairs(acc)) return;
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {        // (uniform trip count)
        const uint32_t i = i0 + threadIdx.x;
        vn_take(bucket, i < n ? b.of(ta[i], tf[i]) : 0u, i < n);
    }
}

// Exclusive sums of the bucket sizes, in place; one workgroup, four buckets a thread and step.
__global__ void __launch_bounds__(1024) vn_starts(uint32_t* bucket, uint32_t buckets, uint32_t apart, const uint64_t* acc)
{
    __shared__ uint32_t part[16];
    if (left_to_all_pairs(acc)) return;
    uint32_t carry = 0;
    for (uint32_t k0 = 0; k0 < buckets; k0 += 4096) {
        const uint32_t k = k0 + 4 * threadIdx.x;
        uint32_t v[4], mine = 0;
        for (int u = 0; u < 4; ++u) { v[u] = k + u < buckets ? bucket[(k + u) << apart] : 0u; mine += v[u]; }
        const uint32_t incl = wave_scan_add(mine);
        __syncthreads();                                              // (the step before has read part[])
        if (lane_id() == kWave - 1) part[wave_id()] = incl;
        __syncthreads();
        uint32_t before = carry + incl - mine;
        for (int w = 0; w < 16; ++w) { if (w < wave_id()) before += part[w]; carry += part[w]; }
        for (int u = 0; u < 4; ++u) { if (k + u < buckets) bucket[(k + u) << apart] = before; before += v[u]; }
    }
}

__global__ void __launch_bounds__(256)
vn_scatter(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n,
           VnBuckets b, VnSorted s, const uint64_t* acc)
{
    if (left_to_all_pairs(acc)) return;
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {        // (uniform trip count)
        const uint32_t i = i0 + threadIdx.x;
        const bool valid = i < n;
        const uint32_t a = valid ? ta[i] : 0u, f = valid ? tf[i] : 0u;
        const uint32_t at = vn_take(s.bucket, b.of(a, f), valid);      // < n: the buckets hold every request once
        if (!valid) continue;
        s.life[at] = make_uint2(a, f);
        s.size[at] = size[i];
        s.id[at] = i;
    }
}

// One wave: the span of tile t.
__device__ __forceinline__ void vn_span(const VnSorted& s, uint32_t n, uint32_t t)
{
    const uint32_t k = t * kVnTile + lane_id();
    const uint2 l = k < n ? s.life[k] : make_uint2(0xffffffffu, 0u);
    const uint32_t first = ~read_lane(wave_scan_max(~l.x), kWave - 1), last = read_lane(wave_scan_max(l.y), kWave - 1);
    if (lane_id() == 0) s.span[t] = make_uint2(first, last);
}

__global__ void __launch_bounds__(256) vn_spans(VnSorted s, uint32_t n, uint32_t tiles, const uint64_t* acc)
{
    const uint32_t t = blockIdx.x * kVnWaves + (uint32_t)wave_id();
    if (t >= tiles || left_to_all_pairs(acc)) return;                       // (uniform)
    vn_span(s, n, t);
}

// One wave = one tile of first requests (a lane each) x up to `chunk` tiles of second requests at or
// behind it, for kPlans plans.  Tiles whose spans do not meet drop out together, requests of the
// others that do not meet the first tile's span 64 at a time; what is left is put into LDS and
// taken one by one as broadcasts: two lifetime compares for all plans, two address compares a plan.
// The records of the next tile but one and the addresses of the next are on their way meanwhile.
// A group of plans beyond the last plan repeats that one, and leaves out its results.
struct Range { uint64_t lo, hi; };
template <int kPlans>
struct ValNearLds {
    uint4 who[kVnWaves][kVnRow];                                      // t_alloc, t_free, number, place in the tile
    Range range[kVnWaves][kPlans][kVnRow];
};

template <int kPlans>
__device__ __forceinline__ void val_near(ValNearLds<kPlans>& sh, const VnSorted& s, const uint64_t* __restrict__ offsets, uint32_t n,
                                         uint32_t tiles, uint32_t chunk, uint32_t p0, uint32_t plan_end, uint64_t* conflicts,
                                         uint64_t* first_key, uint32_t* status)
{
    auto& sh_who = sh.who;
    auto& sh_range = sh.range;
    const int lane = lane_id(), wave = wave_id();
    // workgroup -> (chunk c of second requests, four tiles g of first requests): with r = chunk / 4 chunk c has
    // r (c + 1) groups of four tiles at or in front of it, numbered from r c (c + 1) / 2 on
    const uint64_t r = chunk / kVnWaves;
    uint32_t c = (uint32_t)((sqrt(1.0 + 8.0 * (double)blockIdx.x / (double)r) - 1.0) * 0.5);
    while (r * c * (c + 1) / 2 > blockIdx.x) --c;
    while (r * (c + 1) * (c + 2) / 2 <= blockIdx.x) ++c;
    const uint32_t it = uniform((uint32_t)(blockIdx.x - r * c * (c + 1) / 2) * kVnWaves + (uint32_t)wave);
    if (it >= tiles) return;                                          // (uniform; the waves do not meet)
    const uint2 span = s.span[it];
    const uint32_t first_jt = uniform(c * chunk);
    uint64_t near = 0;
    {
        const uint32_t jt = first_jt + lane;
        const bool is = (uint32_t)lane < chunk && jt < tiles && jt >= it;
        const uint2 other = s.span[is ? jt : it];
        near = __builtin_amdgcn_ballot_w64(is && other.x < span.y && span.x < other.y);
    }
    // the requests with a malformed lifetime meet nothing, but an address range that would wrap is looked for in all
    const bool own_chunk = it / chunk == c;
    if (near == 0 && !own_chunk) return;
    const uint32_t at_i = it * kVnTile + lane;
    const bool i_ok = at_i < n;
    const uint2 life_i = i_ok ? s.life[at_i] : make_uint2(0xffffffffu, 0u);
    const uint32_t id_i = i_ok ? s.id[at_i] : 0u;
    // the second request of this lane: record of tile jt, then its addresses
    struct Record { uint2 life; uint64_t size; uint32_t id; };
    auto record_of = [&](uint64_t tiles_left) -> Record {
        const uint32_t at = (first_jt + (tiles_left ? (uint32_t)__builtin_ctzll(tiles_left) : 0u)) * kVnTile + lane;
        const bool ok = tiles_left != 0 && at < n;
        const uint32_t k = ok ? at : 0u;
        Record q = {s.life[k], s.size[k], s.id[k]};
        if (!ok) q.life = make_uint2(0xffffffffu, 0u);
        return q;
    };
    auto addresses_of = [&](const Record& q, uint64_t (&lo)[kPlans]) {
#pragma unroll
        for (int p = 0; p < kPlans; ++p) lo[p] = offsets[(size_t)umin(p0 + p, plan_end - 1) * n + q.id];
    };
    uint64_t ahead = near & (near - 1);
    Record now = record_of(near), next = record_of(ahead);
    uint64_t now_lo[kPlans], next_lo[kPlans];
    addresses_of(now, now_lo);
    Range mine[kPlans];
    {
        const uint64_t size_i = i_ok ? s.size[at_i] : 0u;
#pragma unroll
        for (int p = 0; p < kPlans; ++p) {
            const uint64_t lo = i_ok ? offsets[(size_t)umin(p0 + p, plan_end - 1) * n + id_i] : 0u;
            // an address range that would run past 2^64 is reported, and kept from wrapping so that what
            // it covers still counts
            const bool wraps = lo + size_i < lo;
            if (own_chunk && wraps) atomicMax(status, (uint32_t)STALLOC_ERR_OVERFLOW);
            mine[p] = Range{lo, wraps ? ~0ull : lo + size_i};
        }
    }
    uint32_t count[kPlans];
    uint64_t key[kPlans];
#pragma unroll
    for (int p = 0; p < kPlans; ++p) { count[p] = 0; key[p] = ~0ull; }

    for (; near; near &= near - 1) {
        const uint32_t jt = first_jt + (uint32_t)__builtin_ctzll(near);
        ahead &= ahead - 1;
        const Record after = record_of(ahead);
        addresses_of(next, next_lo);
        const bool meets = now.life.x < span.y && span.x < now.life.y;
        const uint64_t left = __builtin_amdgcn_ballot_w64(meets);
        const uint32_t many = (uint32_t)__builtin_popcountll(left);
        __builtin_amdgcn_wave_barrier();                              // (the wave's own LDS: its accesses complete in order)
        if (meets) {
            const uint32_t to = lanes_below(left);
            sh_who[wave][to] = make_uint4(now.life.x, now.life.y, now.id, (uint32_t)lane);
#pragma unroll
            for (int p = 0; p < kPlans; ++p)
                sh_range[wave][p][to] = Range{now_lo[p], now_lo[p] + now.size < now_lo[p] ? ~0ull : now_lo[p] + now.size};
        }
        now = next;
        next = after;
#pragma unroll
        for (int p = 0; p < kPlans; ++p) now_lo[p] = next_lo[p];
        if (lane < 4) sh_who[wave][many + lane] = make_uint4(0xffffffffu, 0u, 0u, 0u);      // up to a multiple of four
        __builtin_amdgcn_wave_barrier();
        for (uint32_t k = 0; k < many; k += 4) {
            uint64_t hit[4][kPlans], any = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint4 who = sh_who[wave][k + u];
                const uint64_t together = lanes_lt(who.x, life_i.y) & lanes_lt(life_i.x, who.y);
#pragma unroll
                for (int p = 0; p < kPlans; ++p) {
                    const Range r = sh_range[wave][p][k + u];
                    hit[u][p] = together & lanes_lt(r.lo, mine[p].hi) & lanes_lt(mine[p].lo, r.hi);
                    any |= hit[u][p];
                }
            }
            if (any == 0) continue;                                   // (uniform) the usual case
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint4 who = sh_who[wave][k + u];
                const uint32_t j = who.z, place = uniform(who.w);
                const uint64_t once = jt == it ? (1ull << place) - 1 : ~0ull;     // inside one tile: the first one lies in front
#pragma unroll
                for (int p = 0; p < kPlans; ++p) {
                    const uint64_t h = hit[u][p] & once;
                    count[p] += (uint32_t)__builtin_popcountll(h);
                    if ((h >> lane) & 1) {
                        const uint64_t pair = id_i < j ? ((uint64_t)id_i << 32) | j : ((uint64_t)j << 32) | id_i;
                        key[p] = umin64(key[p], pair);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < kPlans; ++p) {
        if (count[p] == 0 || p0 + p >= plan_end) continue;            // (uniform)
        const uint64_t wave_key = wave_min64(key[p]);
        if (lane == 0) {
            atomicAdd((unsigned long long*)&conflicts[p0 + p], (unsigned long long)count[p]);
            atomicMin((unsigned long long*)&first_key[p0 + p], (unsigned long long)wave_key);
        }
    }
}

// Four plans a wave.
__global__ void __launch_bounds__(kVnWaves * kWave)
val_near_plans(VnSorted s, const uint64_t* __restrict__ offsets, uint32_t n, uint32_t tiles, uint32_t chunk, uint32_t plan0,
               uint32_t plan_end, uint64_t* conflicts, uint64_t* first_key, uint32_t* status)
{
    __shared__ ValNearLds<4> sh;
    val_near<4>(sh, s, offsets, n, tiles, chunk, plan0 + blockIdx.y * 4, plan_end, conflicts, first_key, status);
}

// One plan a wave; or, in a crowded trace, all of its pairs, the 256 x 256 tiles dealt out grid by grid.  (At most 64
// registers: with 70, seven waves a SIMD, all pairs of one plan took 4 % longer than in val_pairs.)
__global__ void __launch_bounds__(kVnWaves * kWave, 8)
val_one_plan(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, VnSorted s,
             const uint64_t* __restrict__ offsets, uint32_t n, uint32_t near_tiles, uint32_t chunk, uint32_t tiles, uint64_t* conflicts,
             uint64_t* first_key, const uint64_t* acc, uint32_t* status)
{
    static_assert(kVnWaves * kWave == kValTile, "both forms run in workgroups of one size");
    __shared__ uint64_t j_lo[kValTile];
    __shared__ uint64_t j_hi[kValTile];
    __shared__ uint32_t j_ta[kValTile];
    __shared__ uint32_t j_tf[kValTile];
    __shared__ ValNearLds<1> near;
    const uint32_t p = blockIdx.y;
    if (left_to_all_pairs(acc)) {                                     // (uniform)
        const uint32_t tri = (uint32_t)((uint64_t)tiles * (tiles + 1) / 2);
        for (uint32_t lin = blockIdx.x; lin < tri; lin += gridDim.x) {
            __syncthreads();                                          // (the tile before has been read)
            val_tile(j_lo, j_hi, j_ta, j_tf, size, ta, tf, offsets, n, tiles, lin, p, conflicts, first_key, status);
        }
        return;
    }
    val_near<1>(near, s, offsets, n, near_tiles, chunk, p, p + 1, conflicts, first_key, status);
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
    VnBuckets buckets = {0, 0, 0, 0};
    VnSorted sorted = {};
    const uint32_t near_tiles = (tr->n + kVnTile - 1) / kVnTile;
    const size_t all_pairs = cv.used;
    if (near) {
        buckets = vn_buckets(tr->n, tr->t_end);
        sorted.bucket = cv.take<uint32_t>(buckets.words());
        sorted.life = cv.take<uint2>(tr->n);
        sorted.size = cv.take<uint64_t>(tr->n);
        sorted.id = cv.take<uint32_t>(tr->n);
        sorted.span = cv.take<uint2>(near_tiles);
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
        const uint64_t work = (uint64_t)tr->n * tr->n * P;
        const bool by_plan = P < 3 || (P == 3 && work < kVnThree) || (P < 8 && work < kVnTogether);
        const uint64_t* crowded = by_plan ? acc : nullptr;
        uint32_t blocks = (tr->n + 255) / 256;
        if (blocks > 1024) blocks = 1024;
        uint32_t cb = ((buckets.words() > P ? buckets.words() : P) + 255) / 256;
        if (cb > 1024) cb = 1024;
        hipLaunchKernelGGL(vn_clear, dim3(cb), dim3(256), 0, stream, sorted.bucket, buckets.words(), conflicts, first_key, P);
        hipLaunchKernelGGL(vn_count, dim3(blocks), dim3(256), 0, stream, tr->t_alloc, tr->t_free, tr->n, buckets, sorted.bucket, crowded);
        hipLaunchKernelGGL(vn_starts, dim3(1), dim3(1024), 0, stream, sorted.bucket, buckets.count, buckets.apart, crowded);
        hipLaunchKernelGGL(vn_scatter, dim3(blocks), dim3(256), 0, stream, tr->size, tr->t_alloc, tr->t_free, tr->n, buckets, sorted, crowded);
        hipLaunchKernelGGL(vn_spans, dim3((near_tiles + kVnWaves - 1) / kVnWaves), dim3(256), 0, stream, sorted, tr->n, near_tiles, crowded);
        // (chunk, group of first tiles) workgroups: the last chunk only has the groups that exist
        const uint32_t chunk = vn_chunk(near_tiles);
        const uint64_t chunks = (near_tiles + chunk - 1) / chunk;
        const uint32_t grid = (uint32_t)(chunk / kVnWaves * ((chunks - 1) * chunks / 2) + (near_tiles + kVnWaves - 1) / kVnWaves);
        if (by_plan)
            hipLaunchKernelGGL(val_one_plan, dim3(grid, P), dim3(kVnWaves * kWave), 0, stream, tr->size, tr->t_alloc, tr->t_free, sorted,
                               offsets, tr->n, near_tiles, chunk, (uint32_t)tiles, conflicts, first_key, crowded, device_status);
        else
            for (uint32_t p0 = 0; p0 < P;) {                  // four plans share a look at the lifetimes; grid.y is limited to 65535
                const uint32_t plans = P - p0 < 131072 ? P - p0 : 131072;
                hipLaunchKernelGGL(val_near_plans, dim3(grid, (plans + 3) / 4), dim3(kVnWaves * kWave), 0, stream, sorted, offsets, tr->n,
                                   near_tiles, chunk, p0, p0 + plans, conflicts, first_key, device_status);
                p0 += plans;
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
