// stalloc_reusable_space: the dynamic reusable space of a plan (Sec. 5.2).
//
// For a time window T the occupied addresses A_o are the union of the address ranges R_s(d) of
// the decisions d whose lifespan R_t(d) meets T; the pool A runs from the lowest start address to
// the highest end address of the whole plan; the reusable space is A_i = A \ A_o.  It is returned
// as its maximal intervals in ascending address order.  Windows are half-open like lifespans.
//
//   sort     The decisions are sorted by (start address, request number) once per call: tiles of
//            1024 keys are sorted in LDS (bitonic network) and merged four runs at a time,
//            an element's place being its place in its own run plus the numbers of elements
//            of the partner runs that sort before it (binary search); nothing depends on how
//            the addresses are distributed.
//   gather   (start, end, lifespan) of the decisions in that order; the unit of the pool's
//            addresses (largest power of two dividing every start and end relative to the
//            pool's start): when 32-bit counts of it cover the pool, the sweep below runs on
//            such counts.
//   sweep    One workgroup per window over the address-sorted decisions, each wave a contiguous
//            part, 64 decisions a step.  A decision counts if its lifespan meets the window; a
//            wave64 running maximum (DPP) of the ends of those before it is "covered so far", and a
//            counting decision that starts above it closes an idle interval [covered, start).  Three
//            walks, a barrier between them: (1) the maximum end per wave, which gives every wave the
//            "covered" it starts from; (2) the number of intervals per wave, which gives every wave
//            its place in the output; (3) the intervals themselves.  What lies between the last
//            covered address and the end of the pool is the final interval.
//            With thousands of windows the roles are exchanged: a wave takes 64 windows, one
//            per lane, and a contiguous part of the sorted decisions.  The windows are sorted so
//            that those of a wave are neighbours of like length (window_key); of 64 decisions
//            two compares and a ballot leave those that meet the span of all of them, which
//            are taken one at a time as wave-uniform values -- two compares per decision tell
//            for all 64 windows whether it counts, and "covered so far" is a per-lane maximum
//            without any cross-lane step.  The same three walks (one launch each, a wave per group
//            of windows and part of the plan; what lies in front of a part is summed up by a small
//            launch in between), at a fraction of the instructions per decision and window.
#include "host_util.h"
#include "sort_keys.h"
#include "wave.h"

namespace stalloc {

constexpr int kRsTile = kSortTile;
constexpr int kRsThreads = 256;
constexpr int kRsWaves = kRsThreads / kWave;

// A = [lo, hi); bits = all bits set in any start or end address relative to lo.
struct RsPool { uint64_t lo, hi, bits; };

// Every start and end address, taken relative to the pool's start, is a multiple of 2^shift (the largest
// such power); `narrow`: the pool counted in those units fits 32 bits.
struct RsUnits { uint32_t shift; bool narrow; };
__device__ __forceinline__ RsUnits units_of(const RsPool* pool)
{
    const uint64_t span = pool->hi - pool->lo;                  // > 0: sizes are
    const uint32_t shift = (uint32_t)__builtin_ctzll(pool->bits | span);
    return {shift, (span >> shift) <= 0xffffffffull};
}

__global__ void rs_init(RsPool* pool)
{
    if (threadIdx.x == 0) { pool->lo = ~0ull; pool->hi = 0; pool->bits = 0; }
}

// Windows that are swept together, a lane each, should lie close together and be of like length: the sweep
// then leaves out what meets none of them 64 decisions at a time.  Order: windows up to the time in which
// 64 of them begin (`near`), by start; then the longer ones, doubling by doubling, by start.
__device__ __forceinline__ ulonglong2 window_key(const uint32_t* __restrict__ windows, uint32_t w, uint32_t near)
{
    const uint32_t lo = windows[2 * w], hi = windows[2 * w + 1];
    const uint32_t length = hi > lo ? hi - lo : 0u, times = length / near;
    const uint32_t cls = times ? 32u - (uint32_t)__builtin_clz(times) : 0u;
    return make_ulonglong2(((uint64_t)cls << 32) | lo, w);
}

// One tile of 1024 decisions per workgroup, sorted in LDS; slot e past the end holds a key behind
// every real one, (~0, ~0 << 32 | e).  Also the pool's bounds.
__global__ void __launch_bounds__(kSortThreads)
rs_sort_tiles(const uint64_t* __restrict__ size, const uint64_t* __restrict__ offsets, uint32_t n, ulonglong2* keys,
              RsPool* pool, const uint32_t* __restrict__ windows, uint32_t windows_k, uint32_t near, ulonglong2* window_keys,
              const uint32_t* status)
{
    __shared__ ulonglong2 k[kRsTile];
    if (*status != STALLOC_OK) return;
    const uint32_t tiles = (n + kRsTile - 1) / kRsTile;
    if (blockIdx.x >= tiles) {                                  // (uniform) the windows' tiles follow the decisions'
        const uint32_t w0 = (blockIdx.x - tiles) * kRsTile;
        for (uint32_t t = threadIdx.x; t < (uint32_t)kRsTile; t += kSortThreads)
            k[t] = w0 + t < windows_k ? window_key(windows, w0 + t, near) : filler_key(w0 + t);
        sort_tile(k, keys_of_tile(w0, windows_k));
        for (uint32_t t = threadIdx.x; t < (uint32_t)kRsTile; t += kSortThreads) window_keys[w0 + t] = k[t];
        return;
    }
    __shared__ uint64_t lowest[kSortThreads / kWave], highest[kSortThreads / kWave];
    uint64_t lo = ~0ull, hi = 0;
    for (uint32_t t = threadIdx.x; t < (uint32_t)kRsTile; t += kSortThreads) {
        const uint32_t i = blockIdx.x * kRsTile + t;
        const bool ok = i < n;
        const uint64_t a = ok ? offsets[i] : ~0ull;
        k[t] = ok ? make_ulonglong2(a, i) : filler_key(i);      // keys (address, request number)
        lo = umin64(lo, a);                                     // (slots past n hold ~0)
        hi = umax64(hi, ok ? a + size[i] : 0ull);
    }
    lo = wave_min64(lo);
    hi = wave_max64(hi);
    if (lane_id() == 0) { lowest[wave_id()] = lo; highest[wave_id()] = hi; }
    sort_tile(k, keys_of_tile(blockIdx.x * kRsTile, n));
    // one pair of atomics per workgroup: a wave each would queue up on the two words
    if (threadIdx.x == 0) {
        for (int w = 1; w < kSortThreads / kWave; ++w) { lo = umin64(lo, lowest[w]); hi = umax64(hi, highest[w]); }
        atomicMin((unsigned long long*)&pool->lo, (unsigned long long)lo);
        atomicMax((unsigned long long*)&pool->hi, (unsigned long long)hi);
    }
    for (uint32_t t = threadIdx.x; t < (uint32_t)kRsTile; t += kSortThreads) keys[blockIdx.x * kRsTile + t] = k[t];
}

// (start, end, lifespan) of the decisions in address order; the bits set in any start or end
// address relative to the pool's start.
__global__ void __launch_bounds__(256)
rs_gather(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf,
          const uint64_t* __restrict__ offsets, const ulonglong2* __restrict__ sorted, uint32_t n,
          uint64_t* s_lo, uint64_t* s_hi, uint2* s_life, RsPool* pool, const uint32_t* status)
{
    __shared__ uint64_t part[4];
    if (*status != STALLOC_OK) return;
    const uint64_t pool_lo = pool->lo;
    uint64_t bits = 0;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
        uint32_t i = (uint32_t)sorted[r].y;
        if (i >= n) i = 0;                                   // (cannot happen: the first n sorted keys are the real ones)
        const uint64_t lo = offsets[i], hi = lo + size[i];
        s_lo[r] = lo;
        s_hi[r] = hi;
        s_life[r] = make_uint2(ta[i], tf[i]);
        bits |= (lo - pool_lo) | (hi - pool_lo);
    }
    bits = wave_or64(bits);
    if (lane_id() == 0) part[wave_id()] = bits;
    __syncthreads();
    if (threadIdx.x == 0) {
        bits = part[0] | part[1] | part[2] | part[3];
        if (bits) atomicOr((unsigned long long*)&pool->bits, (unsigned long long)bits);
    }
}

// Start and end of every sorted decision in units of the pool, relative to its start.
__global__ void __launch_bounds__(256)
rs_compress(const uint64_t* __restrict__ s_lo, const uint64_t* __restrict__ s_hi, uint32_t n, const RsPool* pool,
            uint32_t* c_lo, uint32_t* c_hi, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    const RsUnits units = units_of(pool);
    if (!units.narrow) return;
    const uint64_t pool_lo = pool->lo;
    const uint32_t shift = units.shift;
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x) {
        c_lo[r] = (uint32_t)((s_lo[r] - pool_lo) >> shift);
        c_hi[r] = (uint32_t)((s_hi[r] - pool_lo) >> shift);
    }
}

struct RsArgs {
    const uint32_t* c_lo;        // sorted decisions in 32-bit units of the pool (valid when the pool is narrow)
    const uint32_t* c_hi;
    const uint64_t* s_lo;
    const uint64_t* s_hi;
    const uint2* s_life;
    const RsPool* pool;
    const uint32_t* windows;     // [k][2]
    const ulonglong2* window_order;      // [k] window-per-lane sweep: second word = the window at this place (see window_key)
    uint64_t* ranges;            // [k][max_ranges][2] or nullptr
    uint32_t* counts;            // [k]
    uint64_t* idle_bytes;        // [k] or nullptr
    uint32_t* status;
    uint32_t n, k, max_ranges;
};

__global__ void __launch_bounds__(kRsThreads) rs_sweep(RsArgs g)
{
    __shared__ uint64_t wave_reach[kRsWaves];
    __shared__ uint32_t wave_found[kRsWaves];
    __shared__ uint64_t wave_idle[kRsWaves];
    if (status_of_workgroup(read_status(g.status), wave_found) != STALLOC_OK) return;
    const int lane = lane_id(), wave = wave_id();
    const uint64_t pool_lo = g.pool->lo, pool_hi = g.pool->hi;
    const uint32_t steps = (g.n + kRsThreads - 1) / kRsThreads;           // 64-decision steps per wave
    const uint32_t first = (uint32_t)wave * steps * kWave;

    for (uint32_t w = blockIdx.x; w < g.k; w += gridDim.x) {
        const uint32_t w_lo = g.windows[2 * w], w_hi = g.windows[2 * w + 1];
        if (w_lo >= w_hi) {                                               // (uniform) not a window
            if (threadIdx.x == 0) atomicMax(g.status, (uint32_t)STALLOC_ERR_BAD_WINDOW);
            continue;
        }
        // per step: `ends` = end address where the decision counts, else 0
        auto ends_of = [&](uint32_t s, uint64_t& lo) -> uint64_t {
            const uint32_t at = first + s * kWave + lane;
            lo = 0;
            if (at >= g.n) return 0;
            const uint2 life = g.s_life[at];
            if (!(life.x < w_hi && w_lo < life.y)) return 0;
            lo = g.s_lo[at];
            return g.s_hi[at];
        };

        // walk 1: how far the decisions of each wave reach
        uint64_t reach = 0, lo;
        for (uint32_t s = 0; s < steps; ++s) reach = umax64(reach, ends_of(s, lo));
        reach = wave_max64(reach);
        __syncthreads();                                                  // (previous window's reads done)
        if (lane == 0) wave_reach[wave] = reach;
        __syncthreads();
        uint64_t covered0 = pool_lo, covered_all = pool_lo;               // covered before this wave's part / at the end
        for (int v = 0; v < kRsWaves; ++v) {
            if (v < wave) covered0 = umax64(covered0, wave_reach[v]);
            covered_all = umax64(covered_all, wave_reach[v]);
        }

        // walk 2: idle intervals closed inside each wave's part
        uint32_t found = 0;
        uint64_t run = covered0;
        for (uint32_t s = 0; s < steps; ++s) {
            const uint64_t end = ends_of(s, lo);
            const uint64_t incl = wave_scan_max64(end);
            const uint64_t covered = umax64(run, wave_shift_up64(incl, 0));
            found += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(end != 0 && lo > covered));
            run = umax64(run, readlane64(incl, kWave - 1));
        }
        if (lane == 0) wave_found[wave] = found;
        __syncthreads();
        uint32_t place = 0, total = 0;
        for (int v = 0; v < kRsWaves; ++v) {
            if (v < wave) place += wave_found[v];
            total += wave_found[v];
        }

        // walk 3: write them
        uint64_t* out = g.ranges ? g.ranges + (size_t)w * g.max_ranges * 2 : nullptr;
        uint64_t idle = 0;
        run = covered0;
        for (uint32_t s = 0; s < steps; ++s) {
            const uint64_t end = ends_of(s, lo);
            const uint64_t incl = wave_scan_max64(end);
            const uint64_t covered = umax64(run, wave_shift_up64(incl, 0));
            const bool closes = end != 0 && lo > covered;
            const uint64_t closers = __builtin_amdgcn_ballot_w64(closes);
            if (closes) {
                const uint32_t at = place + lanes_below(closers);
                if (out && at < g.max_ranges) { out[2 * at] = covered; out[2 * at + 1] = lo; }
                idle += lo - covered;
            }
            place += (uint32_t)__builtin_popcountll(closers);
            run = umax64(run, readlane64(incl, kWave - 1));
        }
        idle = wave_sum64(idle);
        if (lane == 0) wave_idle[wave] = idle;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t sum = 0;
            for (int v = 0; v < kRsWaves; ++v) sum += wave_idle[v];
            if (covered_all < pool_hi) {                                  // from the last covered address to the end of the pool
                if (out && total < g.max_ranges) { out[2 * total] = covered_all; out[2 * total + 1] = pool_hi; }
                sum += pool_hi - covered_all;
                ++total;
            }
            g.counts[w] = total;
            if (g.idle_bytes) g.idle_bytes[w] = sum;
        }
    }
}

#ifndef STALLOC_RS_WIDE_FROM
#define STALLOC_RS_WIDE_FROM (1ull << 23)
#endif
// A lane takes a window from this many decisions x windows on (three launches and per-part
// prefixes cost more than they save below it), given at least half a wave of windows.
constexpr uint64_t kRsWideFrom = STALLOC_RS_WIDE_FROM;
__host__ inline bool rs_window_per_lane(uint32_t n, uint32_t k) { return k >= 32 && (uint64_t)n * k >= kRsWideFrom; }
// Waves per CU that the window-per-lane sweep is cut into: more than are resident, since the groups of long
// windows have ten times the work of the others (199 748 decisions, 4096 windows: 0.75 ms a call with 16
// waves per CU, 0.47 with 32, 0.39 with 64; 1.23 ms when every window looked at every decision).
constexpr uint32_t kRsWavesPerCu = 64;
constexpr uint32_t kRsMaxParts = 256;                    // parts the sorted plan is cut into, at most

// Intervals that the second walk keeps of a part and window.  Of a plan worth having little is idle, ten intervals a window
// in 256 parts, so that the third walk mostly has nothing to do.  Not where nobody asks for intervals (199 748 decisions, 512 windows:
// 190 us, 199 when they are kept all the same), and not for more (part, window) pairs than this, 128 MiB of intervals: from two million
// windows on a part is the whole plan and has more of them.
constexpr uint32_t kRsGaps = 4;
constexpr size_t kRsGapCells = (size_t)1 << 21;

// Scratch of the window-per-lane sweep, [group of 64 windows][part][lane].
struct RsParts {
    uint64_t* reach;        // walk 1: maximum end of the counting decisions of the part; then what is covered in front of it
    uint64_t* reach_all;    // [group][lane] ... of all parts
    uint64_t* idle;         // walk 2: bytes of the idle intervals closed inside the part
    uint32_t* found;        //         and their number; then the number in front of the part
    uint32_t* found_all;    // [group][lane] ... in all parts
    uint64_t* gap;          // walk 2: [group][part][kRsGaps][lane] the first of them, as the walk has addresses (room for bytes)
    uint32_t parts;         // parts per group; one wave each
    uint32_t steps;         // 64-decision steps per part
};

// The window of this lane in group grp: lanes without a window, and malformed windows, get bounds that no
// lifespan meets.
struct RsWindow { uint32_t w, lo, hi; bool live, malformed; };
__device__ __forceinline__ RsWindow window_of_lane(const RsArgs& g, uint32_t grp)
{
    const uint32_t at = grp * kWave + (uint32_t)lane_id();
    RsWindow r = {0u, 1u, 0u, false, false};
    if (at < g.k) {
        r.w = (uint32_t)g.window_order[at].y;
        const uint32_t lo = g.windows[2 * (size_t)r.w], hi = g.windows[2 * (size_t)r.w + 1];
        if (lo < hi) { r.lo = lo; r.hi = hi; r.live = true; }
        else r.malformed = true;
    }
    return r;
}

// One wave = 64 windows (one per lane) x one part of the sorted plan.  kWalk = 1, 2, 3: the
// three walks, one launch each (a part needs the results of all lower parts of the walk before).
// Addr = uint32_t: addresses in units of the pool relative to its start (a narrow pool: half the
// registers, single-instruction compares and maxima); Addr = uint64_t: byte addresses.
// The decisions that meet the span of the group's windows are put into LDS and taken from there as
// broadcasts, once 64 have come together: reading them lane by lane (four lane reads and the search
// for the next lane per decision) made a walk twice as long.  Bound by the integer rate and the longest
// units: 2.0 million of 12.8 million (group, decision) pairs are left, 63 + 74 + 7 us for the three walks
// of 199 748 decisions and 4096 windows (63 + 89 + 101 us while the third walked every part again for the few intervals there are).
template <typename Addr> struct RsKept { uint32_t ts, te; Addr lo, hi; };
template <typename Addr> struct RsGap { Addr lo, hi; };
constexpr uint32_t kRsKept = 2 * kWave + 4;                     // (the walk over them takes four at a time)

template <int kWalk, bool kKeeps, typename Addr>
__device__ __forceinline__ void sweep_by_window(const RsArgs& g, const RsParts& sc, uint32_t shift, RsKept<Addr>* kept)
{
    constexpr bool kNarrow = sizeof(Addr) == 4;
    const int lane = lane_id();
    const uint64_t pool_lo = g.pool->lo;
    if (!kNarrow) shift = 0;
    auto bytes = [&](Addr v) -> uint64_t { return kNarrow ? pool_lo + ((uint64_t)v << shift) : (uint64_t)v; };
    const uint32_t groups = (g.k + kWave - 1) / kWave;
    const uint32_t waves = groups * sc.parts;
    for (uint32_t unit = blockIdx.x * kRsWaves + (uint32_t)wave_id(); unit < waves; unit += gridDim.x * kRsWaves) {
        const uint32_t grp = groups - 1 - unit / sc.parts, part = unit % sc.parts;      // (the longest windows first)
        const RsWindow win = window_of_lane(g, grp);
        if (kWalk == 1 && part == 0 && win.malformed) atomicMax(g.status, (uint32_t)STALLOC_ERR_BAD_WINDOW);
        const size_t cell = ((size_t)grp * sc.parts + part) * kWave + lane;
        const uint32_t first = part * sc.steps * kWave;
        // what all windows of the group lie in
        const uint32_t all_lo = ~read_lane(wave_scan_max(win.live ? ~win.lo : 0u), kWave - 1);
        const uint32_t all_hi = read_lane(wave_scan_max(win.hi), kWave - 1);
        Addr covered = 0;
        uint32_t place = 0;                                               // walk 2: intervals closed; walk 3: where the next one goes
        Addr idle = 0;                                                    // (disjoint intervals of the pool: fits the address type)
        uint64_t* out = nullptr;
        RsGap<Addr>* const gaps = reinterpret_cast<RsGap<Addr>*>(sc.gap) + (cell - lane) * kRsGaps + lane;
        if constexpr (kWalk > 1) covered = (Addr)sc.reach[cell];
        if constexpr (kWalk == 2) {
            // No interval is closed in a part whose last decision starts where all windows are covered already.
            const uint32_t last = umin(first + sc.steps * kWave, g.n) - 1;
            const Addr last_lo = kNarrow ? (Addr)g.c_lo[last] : (Addr)g.s_lo[last];
            if (__builtin_amdgcn_ballot_w64(win.live && last_lo > covered) == 0) {          // (uniform)
                sc.found[cell] = 0;
                sc.idle[cell] = 0;
                continue;
            }
        }
        if constexpr (kWalk == 3) {
            place = sc.found[cell];
            const uint32_t behind = part + 1 < sc.parts ? sc.found[cell + kWave] : sc.found_all[(size_t)grp * kWave + lane], mine = behind - place;
            out = win.live ? g.ranges + (size_t)win.w * g.max_ranges * 2 : nullptr;
            const bool wanted = win.live && mine != 0 && place < g.max_ranges;
            if (__builtin_amdgcn_ballot_w64(wanted && mine > (kKeeps ? kRsGaps : 0u)) == 0) {          // (uniform) the second walk has kept them all
                if (wanted) {
                    for (uint32_t k = 0; k < mine && place + k < g.max_ranges; ++k) {
                        const RsGap<Addr> gap = gaps[k * kWave];
                        out[2 * (size_t)(place + k)] = bytes(gap.lo);
                        out[2 * (size_t)(place + k) + 1] = bytes(gap.hi);
                    }
                }
                continue;
            }
        }
        // the next decision in address order, the same for all lanes
        auto take = [&](const RsKept<Addr>& d) {
            const bool counts = d.ts < win.hi && win.lo < d.te;
            if constexpr (kWalk == 2) {
                const bool closes = counts && d.lo > covered;
                if (kKeeps && closes && place < kRsGaps) gaps[place * kWave] = RsGap<Addr>{covered, d.lo};
                place += closes ? 1u : 0u;
                idle += closes ? d.lo - covered : (Addr)0;
            }
            if constexpr (kWalk == 3) {
                if (counts && d.lo > covered) {
                    if (place < g.max_ranges) { out[2 * (size_t)place] = bytes(covered); out[2 * (size_t)place + 1] = bytes(d.lo); }
                    ++place;
                }
            }
            covered = counts ? umax(covered, d.hi) : covered;
        };
        uint32_t many = 0;                                                // decisions in kept[]
        auto take_kept = [&]() {
            if (lane < 4) kept[many + lane] = RsKept<Addr>{0xffffffffu, 0u, 0, 0};       // (meets no window) up to a multiple of four
            __builtin_amdgcn_wave_barrier();                              // (the wave's own LDS: its accesses complete in order)
            for (uint32_t k = 0; k < many; k += 4) {
                RsKept<Addr> d[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) d[u] = kept[k + u];
#pragma unroll
                for (int u = 0; u < 4; ++u) take(d[u]);
            }
            __builtin_amdgcn_wave_barrier();
            many = 0;
        };
        // (the decisions of the next step are on their way while this step's are looked at)
        auto load = [&](uint32_t s) -> RsKept<Addr> {
            const uint32_t at = first + s * kWave + lane;
            RsKept<Addr> d = {0xffffffffu, 0u, 0, 0};                     // past the end: meets no window
            if (s < sc.steps && at < g.n) {
                const uint2 life = g.s_life[at];
                d.ts = life.x; d.te = life.y;
                if constexpr (kNarrow) { d.lo = g.c_lo[at]; d.hi = g.c_hi[at]; }
                else { d.lo = g.s_lo[at]; d.hi = g.s_hi[at]; }
            }
            return d;
        };
        RsKept<Addr> next = load(0);
        for (uint32_t s = 0; s < sc.steps && first + s * kWave < g.n; ++s) {
            const RsKept<Addr> d = next;
            next = load(s + 1);
            const bool meets = d.ts < all_hi && all_lo < d.te;
            const uint64_t left = __builtin_amdgcn_ballot_w64(meets);
            if (meets) kept[many + lanes_below(left)] = d;
            many += (uint32_t)__builtin_popcountll(left);
            if (many >= (uint32_t)kWave) take_kept();                     // (uniform)
        }
        take_kept();
        if constexpr (kWalk == 1) sc.reach[cell] = covered;
        if constexpr (kWalk == 2) { sc.found[cell] = place; sc.idle[cell] = idle; }
    }
}

template <int kWalk, bool kKeeps>
__global__ void __launch_bounds__(kRsThreads) rs_sweep_by_window(RsArgs g, RsParts sc)
{
    __shared__ RsKept<uint64_t> kept[kRsWaves][kRsKept];
    if (*g.status != STALLOC_OK) return;
    const RsUnits units = units_of(g.pool);
    if (units.narrow) sweep_by_window<kWalk, kKeeps, uint32_t>(g, sc, units.shift, reinterpret_cast<RsKept<uint32_t>*>(kept[wave_id()]));   // (uniform)
    else sweep_by_window<kWalk, kKeeps, uint64_t>(g, sc, units.shift, kept[wave_id()]);
}

// What lies in front of every part, one workgroup per group of windows, an equal run of parts per wave.
// kWalk = 1: highest ends -> what is covered in front of a part (at first the pool's start).  kWalk = 2:
// numbers of intervals -> the number in front of a part; and with the totals, and the interval from the last
// covered address to the end of the pool, the answers for the windows.
constexpr int kRsPrefixWaves = 16;
template <int kWalk>
__global__ void __launch_bounds__(kRsPrefixWaves * kWave) rs_prefix(RsArgs g, RsParts sc)
{
    constexpr uint32_t kPer = kRsMaxParts / kRsPrefixWaves;
    __shared__ uint64_t sums[kRsPrefixWaves][kWave], idles[kRsPrefixWaves][kWave];
    if (*g.status != STALLOC_OK) return;
    const int lane = lane_id(), wave = wave_id();
    const RsUnits units = units_of(g.pool);
    const uint32_t per = (sc.parts + kRsPrefixWaves - 1) / kRsPrefixWaves, p0 = umin((uint32_t)wave * per, sc.parts), p1 = umin(p0 + per, sc.parts);
    const size_t row = (size_t)blockIdx.x * sc.parts * kWave + lane;
    uint64_t v[kPer], idle = 0, sum = 0;
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
        v[u] = 0;
        if (p0 + u < p1) {
            const size_t cell = row + (size_t)(p0 + u) * kWave;
            v[u] = kWalk == 1 ? sc.reach[cell] : (uint64_t)sc.found[cell];
            if (kWalk == 2) idle += sc.idle[cell];
        }
    }
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) sum = kWalk == 1 ? umax64(sum, v[u]) : sum + v[u];
    sums[wave][lane] = sum;
    idles[wave][lane] = idle;
    __syncthreads();
    uint64_t run = kWalk == 1 && !units.narrow ? g.pool->lo : 0ull, all = run;
    for (int w = 0; w < kRsPrefixWaves; ++w) {
        const uint64_t other = sums[w][lane];
        if (w < wave) run = kWalk == 1 ? umax64(run, other) : run + other;
        all = kWalk == 1 ? umax64(all, other) : all + other;
    }
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
        if (p0 + u >= p1) continue;
        const size_t cell = row + (size_t)(p0 + u) * kWave;
        if (kWalk == 1) { sc.reach[cell] = run; run = umax64(run, v[u]); }
        else { sc.found[cell] = (uint32_t)run; run += v[u]; }
    }
    if (wave != 0) return;
    if (kWalk == 1) {
        sc.reach_all[(size_t)blockIdx.x * kWave + lane] = all;
        return;
    }
    sc.found_all[(size_t)blockIdx.x * kWave + lane] = (uint32_t)all;
    const RsWindow win = window_of_lane(g, blockIdx.x);
    if (!win.live) return;
    for (int w = 1; w < kRsPrefixWaves; ++w) idle += idles[w][lane];
    if (units.narrow) idle <<= units.shift;                               // units of the pool -> bytes
    const uint64_t reach = sc.reach_all[(size_t)blockIdx.x * kWave + lane], pool_hi = g.pool->hi;
    const uint64_t covered = units.narrow ? g.pool->lo + (reach << units.shift) : reach;
    uint32_t total = (uint32_t)all;
    if (covered < pool_hi) {                                              // from the last covered address to the end of the pool
        if (g.ranges && total < g.max_ranges) {
            uint64_t* out = g.ranges + ((size_t)win.w * g.max_ranges + total) * 2;
            out[0] = covered;
            out[1] = pool_hi;
        }
        idle += pool_hi - covered;
        ++total;
    }
    g.counts[win.w] = total;
    if (g.idle_bytes) g.idle_bytes[win.w] = idle;
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_reusable_space(const stalloc_trace* tr, const uint64_t* offsets, const uint32_t* windows,
                                      uint32_t k, uint32_t max_ranges, uint64_t* ranges, uint32_t* counts,
                                      uint64_t* idle_bytes, uint32_t* device_status, void* workspace,
                                      size_t* workspace_bytes, void* hip_stream)
{
    if (!trace_args_ok(tr) || k == 0 || !workspace_bytes) return STALLOC_ERR_INVALID_ARG;
    DeviceInfo di;
    if (!device_info(&di)) return STALLOC_ERR_DEVICE;
    const uint32_t n = tr->n;

    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    RsPool* pool = cv.take<RsPool>(1);
    const uint32_t tiles = (n + kRsTile - 1) / kRsTile;
    ulonglong2* keys = cv.take<ulonglong2>((size_t)tiles * kRsTile);
    ulonglong2* spare = cv.take<ulonglong2>((size_t)tiles * kRsTile);
    uint64_t* s_lo = cv.take<uint64_t>(n);
    uint64_t* s_hi = cv.take<uint64_t>(n);
    uint2* s_life = cv.take<uint2>(n);
    uint32_t* c_lo = cv.take<uint32_t>(n);
    uint32_t* c_hi = cv.take<uint32_t>(n);
    // window-per-lane sweep: enough (group of 64 windows) x (part of the plan) waves to fill the chip
    RsParts sc = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0};
    ulonglong2 *window_keys = nullptr, *window_spare = nullptr;
    const uint32_t window_tiles = rs_window_per_lane(n, k) ? (k + kRsTile - 1) / kRsTile : 0u;
    const uint32_t groups = (k + kWave - 1) / kWave;
    if (rs_window_per_lane(n, k)) {
        const uint32_t all_steps = (n + kWave - 1) / kWave;
        uint32_t parts = ((uint32_t)di.cus * kRsWavesPerCu + groups - 1) / groups;
        if (parts > kRsMaxParts) parts = kRsMaxParts;
        if (parts > (all_steps + 1) / 2) parts = (all_steps + 1) / 2;     // at least two steps to a part
        sc.steps = (all_steps + parts - 1) / parts;
        sc.parts = (all_steps + sc.steps - 1) / sc.steps;
        const size_t cells = (size_t)groups * sc.parts * kWave;
        window_keys = cv.take<ulonglong2>((size_t)window_tiles * kRsTile);
        window_spare = cv.take<ulonglong2>((size_t)window_tiles * kRsTile);
        sc.reach = cv.take<uint64_t>(cells);
        sc.idle = cv.take<uint64_t>(cells);
        sc.reach_all = cv.take<uint64_t>((size_t)groups * kWave);
        sc.found = cv.take<uint32_t>(cells);
        sc.found_all = cv.take<uint32_t>((size_t)groups * kWave);
        if (cells <= kRsGapCells) sc.gap = cv.take<uint64_t>(2 * kRsGaps * cells);
    }
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    if (!offsets || !windows || !counts || !device_status || (max_ranges != 0 && !ranges) ||
        *workspace_bytes < cv.used || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    launch_trace_check(*tr, acc, device_status, stream);

    uint32_t blocks = (n + 255) / 256;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(rs_init, dim3(1), dim3(64), 0, stream, pool);
    const uint64_t near = (uint64_t)tr->t_end * kWave / k + 1;
    hipLaunchKernelGGL(rs_sort_tiles, dim3(tiles + window_tiles), dim3(kSortThreads), 0, stream, tr->size, offsets, n, keys, pool, windows, k,
                       near < 0x80000000ull ? (uint32_t)near : 0x80000000u, window_keys, device_status);
    const ulonglong2* sorted = launch_merge_tiles(keys, spare, tiles * kRsTile, 1, device_status, stream);
    hipLaunchKernelGGL(rs_gather, dim3(blocks), dim3(256), 0, stream, tr->size, tr->t_alloc, tr->t_free, offsets, sorted, n,
                       s_lo, s_hi, s_life, pool, device_status);
    RsArgs g;
    g.c_lo = c_lo; g.c_hi = c_hi;
    g.s_lo = s_lo; g.s_hi = s_hi; g.s_life = s_life; g.pool = pool; g.windows = windows;
    g.ranges = max_ranges ? ranges : nullptr; g.counts = counts; g.idle_bytes = idle_bytes; g.status = device_status;
    g.n = n; g.k = k; g.max_ranges = max_ranges; g.window_order = nullptr;
    if (rs_window_per_lane(n, k)) {
        g.window_order = launch_merge_tiles(window_keys, window_spare, window_tiles * kRsTile, 1, device_status, stream);
        hipLaunchKernelGGL(rs_compress, dim3(blocks), dim3(256), 0, stream, s_lo, s_hi, n, pool, c_lo,
                           c_hi, device_status);
        const uint64_t waves = (uint64_t)groups * sc.parts;
        // (a wave per unit as far as that goes: the hardware hands out the next one when one is done)
        uint32_t grid = (uint32_t)di.cus * 256;
        if (grid > (waves + kRsWaves - 1) / kRsWaves) grid = (uint32_t)((waves + kRsWaves - 1) / kRsWaves);
        const bool keeps = sc.gap && g.ranges;
        hipLaunchKernelGGL((rs_sweep_by_window<1, false>), dim3(grid), dim3(kRsThreads), 0, stream, g, sc);
        hipLaunchKernelGGL(rs_prefix<1>, dim3(groups), dim3(kRsPrefixWaves * kWave), 0, stream, g, sc);
        hipLaunchKernelGGL((keeps ? rs_sweep_by_window<2, true> : rs_sweep_by_window<2, false>), dim3(grid), dim3(kRsThreads), 0, stream, g, sc);
        hipLaunchKernelGGL(rs_prefix<2>, dim3(groups), dim3(kRsPrefixWaves * kWave), 0, stream, g, sc);
        if (g.ranges)
            hipLaunchKernelGGL((keeps ? rs_sweep_by_window<3, true> : rs_sweep_by_window<3, false>), dim3(grid), dim3(kRsThreads), 0, stream, g, sc);
    } else {
        uint32_t grid = (uint32_t)di.cus * 8;
        if (grid > k) grid = k;
        hipLaunchKernelGGL(rs_sweep, dim3(grid), dim3(kRsThreads), 0, stream, g);
    }
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}
