// stalloc_fuse_groups: candidate fusions of HomoPhase groups (Sec. 5.1, HomoPhase Group Planning),
// many at once, one workgroup per candidate pair of groups.
//
// A HomoPhase group holds the requests allocated in one computation phase and released in one
// (other) phase; its local plan packs them contiguously.  Two plans are fused by inserting the
// smaller into the larger: the larger plan is packed from 0 in descending order of release time;
// an address pointer starts at its lowest start address; the requests of the smaller plan are
// tried in order of allocation time, the first that conflicts with nothing when put at the
// pointer is placed there and the pointer moves up by its size; if none fits the pointer moves to
// the next higher start address of the larger plan; what is left when those run out is packed on
// top.  The fusion is accepted if its time-memory product (Eq. 2) exceeds the average of the two
// plans' products weighted by the memory-time each reserves, i.e. if the fused plan reserves less
// memory-time (extent x span) than the two together.
//
// Per pair everything lives in LDS.  Both plans are sorted by bitonic networks over 64-bit keys.  The
// insertion is a chain that one wave follows without barriers, and what makes its steps short is
// what is known of a request k of the smaller plan beforehand.  The larger plan is contiguous, its
// release times descend with the address, and the pointer only rises:
//   clear[k]   from this block of the larger plan on, k conflicts with no block: either all of them are
//              released by k's allocation, or all are allocated from k's release on.
//   wake[k]    k need not be tried before the pointer has reached this block.  Below clear[k] every block is
//              released after k's allocation, so it conflicts with k if it was allocated before k's
//              release; if all of them were, wake[k] = clear[k] from the start.  A request that
//              was tried and met a conflicting block sleeps until the pointer has passed the last such
//              block of the range it was tried at: as long as it has not, a higher start still reaches it.
// The lowest wake of every 64 requests sits in a register, so a step looks at the first requests that
// are awake only, and when none is the pointer goes straight to the block that wakes the next one.
//   330 pairs of up to 3262 requests: 11.3 -> 0.30 ms.  The longest chain sets the time.
//   A step at which more than four chunks are awake is shared by all waves (two barriers).
#include "host_util.h"
#include "wave.h"

namespace stalloc {

// A pair has a workgroup of 512, so that many waves can help at once where a step has many requests to look at; small
// pairs one of 128, of which a CU holds more (5000 pairs of 16 requests: 119 -> 49 us; a workgroup of 512 is mostly idle).
constexpr uint32_t kFuSmall = 256;               // requests of a pair

struct FuseParams {
    const uint64_t* size;
    const uint32_t* ta;
    const uint32_t* tf;
    const uint32_t* members;
    const uint32_t* pair_begin;
    const uint32_t* count1;
    uint32_t* order;
    uint64_t* addr;
    uint64_t* extents;
    uint32_t* accepted;
    uint32_t* status;
    uint32_t n;
    uint32_t entries;        // length of members / order / addr
    uint32_t cap;            // requests of one pair that fit the LDS arrays
};

// Sums over the workgroup, three at once.
template <int kFuThreads>
__device__ __forceinline__ void block_sums64(uint64_t (&v)[3], uint64_t (*scratch)[3])
{
    for (int u = 0; u < 3; ++u) v[u] = wave_sum64(v[u]);
    __syncthreads();
    if (lane_id() == 0)
        for (int u = 0; u < 3; ++u) scratch[wave_id()][u] = v[u];
    __syncthreads();
    for (int u = 0; u < 3; ++u) {
        v[u] = 0;
        for (int k = 0; k < kFuThreads / kWave; ++k) v[u] += scratch[k][u];
    }
}

// a * b as a 96-bit number {high 32 bits, low 64 bits}
__device__ __forceinline__ void mul_64_32(uint64_t a, uint32_t b, uint64_t& hi, uint64_t& lo)
{
    lo = a * (uint64_t)b;
    hi = __umul64hi(a, (uint64_t)b);
}

constexpr uint32_t kPlaced = 0xffffffffu;        // in wake[]: the request has an address
constexpr int kNear = 8;                         // blocks that all requests of a chunk are held against together
// The first kAlone of a chunk's requests that need a look get one each, against their whole range, the rest are held
// against the first blocks together.  One by one they sleep as long as they can, and the first that fits ends the
// search, which pays where ranges go on (an interleaved schedule: 0.30 ms, 0.49 without); together is what pays
// when lifetimes are so mixed that many are awake and few fit (200 pairs of 600 + 600, the smaller group earlier: 2.84
// ms with four looks always, 2.00 now).  So when the last kProbes chunks put nobody to sleep beyond what
// holding them together shows, only every eighth chunk still has its single looks.
constexpr int kAlone = 4, kProbes = 16;
constexpr uint32_t kDone = 0, kHelp = 1;

// Sorts keys[0..m) in LDS, ascending; called by the whole workgroup.  A bitonic network whose merges
// begin by comparing mirrored places, so that every exchange goes the same way and places past
// the end, which would hold the largest keys, need not exist.
template <int kFuThreads>
__device__ __forceinline__ void sort_keys(uint64_t* keys, uint32_t m)
{
    for (uint32_t span = 2; span < 2 * m; span <<= 1) {
        for (uint32_t gap = span >> 1; gap > 0; gap >>= 1) {
            const bool mirrored = gap == span >> 1;
            for (uint32_t e = threadIdx.x; 2 * (e - e % gap) < m; e += kFuThreads) {       // pair e: the e-th place whose bit `gap` is clear
                const uint32_t x = 2 * e - e % gap, y = mirrored ? x ^ (span - 1) : x ^ gap;
                if (y < m) {
                    const uint64_t a = keys[x], b = keys[y];
                    if (b < a) { keys[x] = b; keys[y] = a; }
                }
            }
            __syncthreads();
        }
    }
}

template <int kFuThreads>
__global__ void __launch_bounds__(kFuThreads) fuse_pairs(FuseParams prm)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint64_t scratch[kFuThreads / kWave][3];
    __shared__ uint32_t t_lo[2], t_hi[2];
    __shared__ uint32_t low_of[80];                                   // lowest wake of every 64 requests of the smaller plan
    __shared__ struct { uint64_t addr; uint32_t order, holder, fit; } help;
    if (status_of_workgroup(read_status(prm.status), t_lo) != STALLOC_OK) return;
    const uint32_t p = blockIdx.x, tid = threadIdx.x;
    const uint32_t m0 = prm.pair_begin[p], m1 = prm.pair_begin[p + 1], m = m1 - m0, c1 = prm.count1[p];
    const bool outside = m1 < m0 || m1 > prm.entries;               // (nothing is read or written beyond the arrays)
    if (outside || m > prm.cap || c1 == 0 || c1 >= m) {             // (uniform) nothing sensible to do
        if (tid == 0) atomicMax(prm.status, (uint32_t)(!outside && m > prm.cap ? STALLOC_ERR_TOO_LARGE : STALLOC_ERR_INVALID_ARG));
        return;
    }
    uint32_t* id = reinterpret_cast<uint32_t*>(smem);                 // [cap] request numbers, as given
    uint32_t* srt = id + prm.cap;                                     // [cap] the fused plan's order
    uint64_t* sz = reinterpret_cast<uint64_t*>(srt + prm.cap);        // [cap] in the fused plan's order:
    uint64_t* at = sz + prm.cap;                                      //       size, address,
    uint32_t* ts = reinterpret_cast<uint32_t*>(at + prm.cap);         //       lifetime
    uint32_t* te = ts + prm.cap;
    if (tid < 2) { t_lo[tid] = 0xffffffffu; t_hi[tid] = 0u; }
    __syncthreads();
    // the two local plans: extent = sum of sizes, span = first allocation .. last release
    uint64_t sums[3] = {0, 0, 0};                                     // sizes of the first group, of the second, upper halves of all
    int unknown = 0;
    uint32_t lo_of[2] = {0xffffffffu, 0xffffffffu}, hi_of[2] = {0u, 0u};
    for (uint32_t k = tid; k < m; k += kFuThreads) {
        uint32_t i = prm.members[m0 + k];
        if (i >= prm.n) { unknown = 1; i = 0; }
        id[k] = i;
        const int g = k < c1 ? 0 : 1;
        const uint64_t s = prm.size[i];
        (g ? sums[1] : sums[0]) += s;
        sums[2] += s >> 32;
        const uint32_t a = prm.ta[i], f = prm.tf[i];
        ts[k] = a; te[k] = f;                                         // (as given, for the sort)
        lo_of[g] = umin(lo_of[g], a);
        hi_of[g] = umax(hi_of[g], f);
    }
    for (int g = 0; g < 2; ++g) {
        const uint32_t lo = ~read_lane(wave_scan_max(~lo_of[g]), kWave - 1), hi = read_lane(wave_scan_max(hi_of[g]), kWave - 1);
        if (lane_id() == 0) { atomicMin(&t_lo[g], lo); atomicMax(&t_hi[g], hi); }
    }
    block_sums64<kFuThreads>(sums, scratch);
    // The chain below counts on starts that ascend with the block, that is on addresses that do not wrap.  Distinct
    // requests stay below 2^63 together (the trace check); requests listed twice need not, and neither would a
    // stand-in for an unknown one.  (The lower halves of fewer than 2^13 sizes add up to less than 2^45.)
    if (__syncthreads_or(unknown)) {
        if (tid == 0) atomicMax(prm.status, (uint32_t)STALLOC_ERR_BAD_ORDER);
        return;
    }
    if (sums[2] >= (1ull << 32) - (1u << 13)) {                       // (uniform)
        if (tid == 0) atomicMax(prm.status, (uint32_t)STALLOC_ERR_OVERFLOW);
        return;
    }
    const uint64_t ext1 = sums[0], ext2 = sums[1];
    const bool first_larger = ext1 >= ext2;
    const uint32_t nl = first_larger ? c1 : m - c1, ns = m - nl;
    const uint32_t l0 = first_larger ? 0 : c1, s0 = first_larger ? c1 : 0;     // where the two groups start in id[]
    // larger plan: by release time, latest first (request number among equals); smaller plan: by
    // allocation time (request number among equals)
    for (uint32_t k = tid; k < m; k += kFuThreads) {
        const bool in_larger = k >= l0 && k < l0 + nl;
        const uint64_t key = in_larger ? ((uint64_t)~te[k] << 32) | id[k] : ((uint64_t)ts[k] << 32) | id[k];
        at[in_larger ? k - l0 : nl + (k - s0)] = key;
    }
    __syncthreads();
    sort_keys<kFuThreads>(at, nl);
    sort_keys<kFuThreads>(at + nl, ns);
    for (uint32_t k = tid; k < m; k += kFuThreads) {
        const uint32_t i = (uint32_t)at[k];
        srt[k] = i;
        sz[k] = prm.size[i]; ts[k] = prm.ta[i]; te[k] = prm.tf[i];
    }
    __syncthreads();
    // the larger plan, packed from 0; over its blocks, the latest allocation up to a block (in id[], no longer needed)
    // and the earliest from a block on (in sz[], the addresses tell the sizes)
    const uint64_t larger_top = first_larger ? ext1 : ext2;
    uint32_t* const latest_upto = id;
    uint32_t* const wake = id + nl;
    if (wave_id() == 0) {
        uint64_t top = 0;
        uint32_t latest = 0;
        for (uint32_t k0 = 0; k0 < nl; k0 += kWave) {
            const uint32_t k = k0 + lane_id();
            const uint64_t mine = k < nl ? sz[k] : 0ull;
            const uint64_t incl = wave_scan_add64(mine);
            const uint32_t most = umax(latest, wave_scan_max(k < nl ? ts[k] : 0u));
            if (k < nl) { at[k] = top + incl - mine; latest_upto[k] = most; }
            top += read_lane(incl, kWave - 1);
            latest = read_lane(most, kWave - 1);
        }
        uint32_t least = 0xffffffffu;                                 // (from the last block down, lane 0 the highest)
        for (uint32_t done = 0; done < nl; done += kWave) {
            const uint32_t back = done + lane_id();
            const uint32_t low = umin(least, ~wave_scan_max(back < nl ? ~ts[nl - 1 - back] : 0u));
            if (back < nl) sz[nl - 1 - back] = low;
            least = read_lane(low, kWave - 1);
        }
    }
    __syncthreads();
    for (uint32_t k = tid; k < ns; k += kFuThreads) {
        const uint32_t from = ts[nl + k], till = te[nl + k];
        uint32_t lo = 0, hi = nl;                                     // first block released by k's allocation (and so are all behind it)
        while (lo < hi) { const uint32_t mid = (lo + hi) >> 1; if (te[mid] > from) lo = mid + 1; else hi = mid; }
        uint32_t clear = lo;
        lo = 0;                                                       // first block from which on all are allocated from k's release on
        hi = clear;
        while (lo < hi) { const uint32_t mid = (lo + hi) >> 1; if ((uint32_t)sz[mid] < till) lo = mid + 1; else hi = mid; }
        clear = lo;
        at[nl + k] = clear;                                           // (until k has an address)
        wake[k] = clear != 0 && latest_upto[clear - 1] < till ? clear : 0u;
    }
    __syncthreads();
    const int lane = lane_id();
    const uint32_t chunks = (ns + kWave - 1) / kWave;                 // <= 80: the LDS holds fewer than 5120 requests
    auto lowest_wake = [&](uint32_t w) -> uint32_t { return ~read_lane(wave_scan_max(~w), kWave - 1); };
    // The 64 requests of a chunk as the lanes of a wave hold them, tried at the pointer in turn: `fit` is the
    // first that fits (-1: none), those that were found not to are put to sleep.
    struct Chunk { uint64_t size; uint32_t wake; bool open; uint64_t awake, for_good; int fit; };
    auto try_chunk = [&](uint32_t c, uint64_t addr, uint32_t holder, int alone) -> Chunk {
        const uint32_t k = c * kWave + lane;
        Chunk ch;
        ch.wake = k < ns ? wake[k] : kPlaced;
        ch.open = ch.wake != kPlaced;
        ch.size = ch.open ? sz[nl + k] : 0ull;
        const uint32_t clear = ch.open ? (uint32_t)at[nl + k] : 0u, till = ch.open ? te[nl + k] : 0u;
        ch.awake = lanes_ge(holder, ch.wake);
        ch.for_good = ch.awake & lanes_ge(holder, clear);             // conflict with nothing any more
        ch.fit = -1;
        uint64_t fits = ch.for_good;
        int looks = 0;
        for (uint64_t left = ch.awake; left; left &= left - 1) {
            const int f = __builtin_ctzll(left);
            if (((fits >> f) & 1) == 0) {
                if (looks++ == alone) {
                    // many need a look: all of them at once, at the first blocks from the pointer's on that [addr, addr + size)
                    // meets; those below clear are all released after the request's allocation
                    const uint64_t end = addr + ch.size;
                    const uint32_t qc = umin(holder + (uint32_t)(lane < kNear ? lane : 0), nl - 1);
                    const uint64_t start_of = at[qc];
                    const uint32_t from_of = ts[qc];
                    const bool looked = ((left & ~fits) >> lane) & 1;
                    uint32_t past = 0;                                // one behind the last block that conflicts
                    bool meets = looked;
#pragma unroll
                    for (int u = 0; u < kNear; ++u) {
                        meets = meets && holder + u < clear && (u == 0 || read_lane(start_of, u) < end);
                        if (meets && read_lane(from_of, u) < till) past = holder + u + 1;
                    }
                    if (past != 0) ch.wake = past;
                    const uint64_t clash = __builtin_amdgcn_ballot_w64(past != 0);
                    fits |= __builtin_amdgcn_ballot_w64(looked && past == 0 && !meets);           // (meets is still set: the range goes on)
                    left = (left & ~clash) | (1ull << f);             // (f is dealt with here)
                    if ((clash >> f) & 1) continue;
                }
                if (((fits >> f) & 1) == 0) {
                    // all blocks of one request's range, 64 at a time
                    const uint64_t end = addr + read_lane(ch.size, f);
                    const uint32_t up_to = read_lane(clear, f), released = read_lane(till, f);
                    uint32_t past = 0;
                    for (uint32_t q0 = holder;; q0 += kWave) {
                        const uint32_t q = q0 + lane, qc = umin(q, nl - 1);
                        const bool meets = q < up_to && (q == holder || at[qc] < end);
                        const uint64_t hit = __builtin_amdgcn_ballot_w64(meets && ts[qc] < released);
                        if (hit) past = q0 + kWave - (uint32_t)__builtin_clzll(hit);
                        if (__builtin_amdgcn_ballot_w64(meets) != ~0ull) break;       // (uniform)
                    }
                    if (past != 0) {
                        if (lane == f) ch.wake = past;
                        continue;
                    }
                }
            }
            ch.fit = f;
            break;
        }
        return ch;
    };
    if (wave_id() == 0)
        for (uint32_t c = 0; c < chunks; ++c) {
            const uint32_t k = c * kWave + lane, low = lowest_wake(k < ns ? wake[k] : kPlaced);
            if (lane == 0) low_of[c] = low;
        }
    uint64_t addr = 0;                                                // lowest start address of the larger plan
    uint32_t holder = 0;                                              // block of the larger plan that holds addr (nl: behind its end)
    uint32_t left = ns;
    int near_chunks = 0;                                              // tried since one that put a request to sleep for long
    for (;;) {
        if (wave_id() == 0) {
            // lowest wake of chunk `lane` and of chunk 64 + `lane`
            uint32_t low0 = (uint32_t)lane < chunks ? low_of[lane] : kPlaced;
            uint32_t low1 = (uint32_t)lane + kWave < chunks ? low_of[lane + kWave] : kPlaced;
            uint32_t order = kDone;
            while (left) {                                            // (every pass raises the holder or places a request)
                for (;;) {                                            // blocks up to the one that holds addr, 64 at a time
                    const uint32_t q = holder + 1 + lane;
                    const uint64_t start = q < nl ? at[q] : (q == nl ? larger_top : ~0ull);
                    const uint32_t passed = (uint32_t)__builtin_popcountll(lanes_ge(addr, start));
                    holder += passed;
                    if (passed < (uint32_t)kWave) break;              // (uniform)
                }
                uint64_t awake0 = lanes_ge(holder, low0), awake1 = lanes_ge(holder, low1);
                bool found = false;
                for (int tried = 0; awake0 | awake1; ++tried) {
                    if (tried == 2 && __builtin_popcountll(awake0) + __builtin_popcountll(awake1) > 2) { order = kHelp; break; }
                    const uint32_t c = awake0 ? (uint32_t)__builtin_ctzll(awake0) : kWave + (uint32_t)__builtin_ctzll(awake1);
                    if (awake0) awake0 &= awake0 - 1; else awake1 &= awake1 - 1;
                    const uint32_t k = c * kWave + lane;
                    Chunk ch = try_chunk(c, addr, holder, near_chunks < kProbes || (near_chunks & 7) == 0 ? kAlone : 0);
                    const bool far = (ch.awake & lanes_ge(ch.wake, holder + kNear + 1)) != 0;        // (uniform) put to sleep for long
                    near_chunks = far ? 0 : near_chunks + 1;
                    if (ch.fit >= 0) {
                        uint64_t placed = 1ull << ch.fit;
                        uint64_t to = addr;
                        uint64_t grown = read_lane(ch.size, ch.fit);
                        if ((ch.for_good >> ch.fit) & 1) {
                            // Those behind it that conflict with nothing any more fit as well, one on top of the other, up
                            // to a request that needs a look -- as long as the pointer does not reach a block that wakes
                            // an earlier one.
                            const uint64_t behind = ~0ull << ch.fit, look = ch.awake & ~ch.for_good & behind;
                            const uint64_t run = ch.for_good & behind & (look ? (look & (0 - look)) - 1 : ~0ull);
                            const bool mine = (run >> lane) & 1;
                            const uint64_t incl = wave_scan_add64(mine ? ch.size : 0ull);
                            to = addr + incl - ch.size;
                            const uint32_t earlier = lowest_wake(umin((uint32_t)lane < c ? low0 : kPlaced,
                                                                      (uint32_t)lane + kWave < c ? low1 : kPlaced));
                            const uint32_t asleep = (ch.open && ch.wake > holder) ? ch.wake : kPlaced;
                            const uint32_t wakes = umin(earlier, ~wave_shift_up(wave_scan_max(~asleep), 0u));
                            const uint64_t wakes_at = wakes < nl ? at[umin(wakes, nl - 1)] : (wakes == nl ? larger_top : ~0ull);
                            const uint64_t stop = __builtin_amdgcn_ballot_w64(mine && to >= wakes_at);
                            placed = run & (stop ? (stop & (0 - stop)) - 1 : ~0ull);   // (the first is: nothing earlier is awake)
                            grown = read_lane(incl, kWave - 1 - __builtin_clzll(placed));
                        }
                        if ((placed >> lane) & 1) { at[nl + k] = to; ch.wake = kPlaced; }
                        addr += grown;
                        left -= (uint32_t)__builtin_popcountll(placed);
                        found = true;
                    }
                    if (ch.open) wake[k] = ch.wake;
                    const uint32_t low = lowest_wake(ch.wake);
                    if (c < (uint32_t)kWave) low0 = write_lane(low0, low, (int)c); else low1 = write_lane(low1, low, (int)(c - kWave));
                    if (found) break;
                }
                if (order == kHelp) break;
                if (!found) {
                    // nothing fits up to the block that wakes the next request; a pointer behind the last start ends it
                    const uint32_t next = lowest_wake(umin(low0, low1));
                    if (next >= nl) break;
                    addr = at[next];
                    holder = next;
                }
            }
            if ((uint32_t)lane < chunks) low_of[lane] = low0;
            if ((uint32_t)lane + kWave < chunks) low_of[lane + kWave] = low1;
            if (lane == 0) { help.order = order; help.holder = holder; help.addr = addr; help.fit = kPlaced; }
        }
        __syncthreads();
        if (help.order == kDone) break;                               // (uniform)
        // many chunks are awake at once: the waves take one each
        for (uint32_t c = (uint32_t)wave_id(); c < chunks; c += kFuThreads / kWave) {
            if (low_of[c] > help.holder) continue;                    // (uniform)
            const Chunk ch = try_chunk(c, help.addr, help.holder, 0);
            if (ch.open) wake[c * kWave + lane] = ch.wake;
            const uint32_t low = lowest_wake(ch.wake);
            if (lane == 0) {
                low_of[c] = low;
                if (ch.fit >= 0) atomicMin(&help.fit, c * kWave + (uint32_t)ch.fit);
            }
            if (ch.fit >= 0) break;                                   // (the wave's later chunks hold later requests only)
        }
        __syncthreads();
        if (wave_id() == 0) {
            const uint32_t k = help.fit;
            if (k != kPlaced) {
                if (lane == 0) { at[nl + k] = addr; wake[k] = kPlaced; }
                const uint32_t at_chunk = (k / kWave) * kWave + lane;
                const uint32_t low = lowest_wake(at_chunk < ns && at_chunk != k ? wake[at_chunk] : kPlaced);
                if (lane == 0) low_of[k / kWave] = low;
                addr += sz[nl + k];
                --left;
            }
        }
    }
    if (wave_id() == 0) {
        // what is left goes on top of everything placed
        uint64_t top = larger_top;
        for (uint32_t k = lane; k < ns; k += kWave)
            if (wake[k] == kPlaced) top = umax(top, at[nl + k] + sz[nl + k]);
        top = wave_max64(top);
        for (uint32_t k0 = 0; left && k0 < ns; k0 += kWave) {
            const uint32_t k = k0 + lane;
            const bool open = k < ns && wake[k] != kPlaced;
            const uint64_t mine = open ? sz[nl + k] : 0ull;
            const uint64_t incl = wave_scan_add64(mine);
            if (open) at[nl + k] = top + incl - mine;
            top += read_lane(incl, kWave - 1);
        }
        if (lane == 0) {
            const uint32_t lo_f = t_lo[0] < t_lo[1] ? t_lo[0] : t_lo[1], hi_f = t_hi[0] > t_hi[1] ? t_hi[0] : t_hi[1];
            uint64_t h1, l1, h2, l2, hf, lf;
            mul_64_32(ext1, t_hi[0] - t_lo[0], h1, l1);
            mul_64_32(ext2, t_hi[1] - t_lo[1], h2, l2);
            mul_64_32(top, hi_f - lo_f, hf, lf);
            const uint64_t ls = l1 + l2, hs = h1 + h2 + (ls < l1 ? 1 : 0);
            prm.extents[3 * (size_t)p] = ext1;
            prm.extents[3 * (size_t)p + 1] = ext2;
            prm.extents[3 * (size_t)p + 2] = top;
            prm.accepted[p] = (hf < hs || (hf == hs && lf < ls)) ? 1u : 0u;
        }
    }
    __syncthreads();
    for (uint32_t k = tid; k < m; k += kFuThreads) {
        prm.order[m0 + k] = srt[k];
        prm.addr[m0 + k] = at[k];
    }
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_fuse_groups(const stalloc_trace* tr, const uint32_t* members, const uint32_t* pair_begin,
                                   const uint32_t* count1, uint32_t k, uint32_t m, uint32_t largest_pair, uint32_t* order,
                                   uint64_t* addr, uint64_t* extents, uint32_t* accepted, uint32_t* device_status,
                                   void* workspace, size_t* workspace_bytes, void* hip_stream)
{
    if (!trace_args_ok(tr) || k == 0 || largest_pair < 2 || m < 2 || !workspace_bytes) return STALLOC_ERR_INVALID_ARG;
    DeviceInfo di;
    if (!device_info(&di)) return STALLOC_ERR_DEVICE;
    const size_t per_request = 2 * sizeof(uint32_t) + 2 * sizeof(uint64_t) + 2 * sizeof(uint32_t);
    const size_t lds_budget = di.lds_per_block - 1024;
    if ((size_t)largest_pair * per_request > lds_budget) return STALLOC_ERR_TOO_LARGE;
    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    if (!members || !pair_begin || !count1 || !order || !addr || !extents || !accepted || !device_status ||
        *workspace_bytes < cv.used || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    launch_trace_check(*tr, acc, device_status, stream);
    FuseParams prm;
    prm.size = tr->size; prm.ta = tr->t_alloc; prm.tf = tr->t_free; prm.members = members; prm.pair_begin = pair_begin;
    prm.count1 = count1; prm.order = order; prm.addr = addr; prm.extents = extents; prm.accepted = accepted;
    prm.status = device_status; prm.n = tr->n; prm.entries = m;
    prm.cap = (largest_pair + 1) & ~1u;                               // (keeps the 64-bit arrays aligned)
    if (prm.cap <= kFuSmall) {
        hipLaunchKernelGGL(fuse_pairs<128>, dim3(k), dim3(128), (size_t)prm.cap * per_request, stream, prm);
        return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
    }
    static std::atomic<bool> attr_set[64] = {};        // (set twice at worst when threads race)
    if (!attr_set[di.device]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&fuse_pairs<512>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds_budget) != hipSuccess)     // (the kernel's static LDS takes the rest)
            return STALLOC_ERR_DEVICE;
        attr_set[di.device] = true;
    }
    hipLaunchKernelGGL(fuse_pairs<512>, dim3(k), dim3(512), (size_t)prm.cap * per_request, stream, prm);
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}
