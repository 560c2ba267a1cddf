// stalloc_plan: batched greedy placement, one workgroup per candidate placement order; the
// entry point, and the placement kernel for traces the occupancy-bitmap kernel does not take.
//
// Rule (Sec. 5.1): requests are taken in the given order; each gets the lowest address at
// which it conflicts with no earlier request of the same plan in lifespan and address
// range at once.  Extent of a plan = max(a + s) (Eq. 2).
//
// Per plan the workgroup keeps the list of placed blocks SORTED BY ADDRESS, so that no
// sorting is needed when a request is placed.  Requests are handled in batches of 64:
//
//   scan     One pass over the sorted list serves the whole batch, because the list only
//            changes between batches.  The list is cut into chunks of consecutive entries, two for
//            each wave: half of its lanes take a chunk each, a lane holds two requests, and every block
//            of the chunk is taken by all its lanes at once (64-bit addresses: a chunk a wave, a request
//            a lane).  Two compares tell whose lifetime it conflicts with, the running maximum of
//            the conflicting blocks' end addresses is "covered so far", and a conflicting block that
//            starts at least size_r above it closes a hole [covered, start) in which r could
//            fit.  Per (chunk, request) the chunk's maximum and its first few holes (with
//            chunk-local "covered") are published to LDS.
//   survey   After a barrier, request r's wave gathers what was published for it into its
//            64 lanes in address order; the true "covered" of a hole is the maximum of its
//            local value and the maxima of the chunks below.  The first hole that is large
//            enough is where r lies if the rest of the batch leaves it there, else the top.  If a
//            chunk had more holes than could be published and no lower one fits, it
//            is walked again for this one request, with everything below it known.  Where the chain below
//            often gets into such chunks (orders by time), more of their holes are noted here for it.
//   settle   A request clashes when an earlier one of the batch that is alive at the same time lies
//            where it would.  All waves look for clashes; wave 0 then goes through those requests in
//            order (all others stay where they are): each takes the first of its holes in which it
//            still fits when it moves up past the blocks in its way, else goes on top.
//   merge    The settled blocks are merged into the sorted list in one pass: listed block k
//            moves up by the number of new blocks at or below its start address and the new
//            blocks drop into the gaps (in place through registers when the list is in LDS,
//            ping-pong between two slabs when it is in the workspace).
//
// What bounds it: the scan spends five vector and two scalar instructions on a block and 64 requests, and four waves a SIMD do not
// issue enough of them to keep the vector units busy; an LDS broadcast per block (16 bytes, eight cycles of the CU's LDS) comes close.
// Then the chain of clashing requests in wave 0.  6144 requests of 5 sizes, 512 orders (list in LDS): 17.9 ms with batches of 16, a
// lane per block, a running maximum across lanes per request and wave 0 settling every request, 8.8 with a request per lane and lane
// masks for what conflicts (six and five instructions), 8.4 with lanes switched off by the compares; 49 920 requests, 256 orders (list
// in the workspace): 228, 153, 145, 141 with the next part of a chunk on its way while one is looked at, and 125 where the survey notes
// what the chain would look for (the order by time, which sets the launch's time: 131 -> 114 ms).
//
// Addresses are multiples of the largest power of two dividing all sizes.  When the sum of
// sizes, in those granules, stays below 2^31 the list holds 32-bit granule counts (16-byte
// entries, single-instruction max/compare/DPP), below 2^16 (and with 16-bit timestamps) 8-byte
// cells; otherwise 64-bit byte addresses.  The sum of sizes is a bound no sensible plan comes
// near, so when only the sum is too large (no single size reaches 2^30 granules) the 32-bit
// instantiation still takes every plan, as far as the extent so far plus the sizes of the next
// batch stays below 2^32 granules, and marks the plans that fail the check for the 64-bit
// instantiation enqueued behind it.  Only the device knows which case applies (the trace
// check leaves it in the mode word), so every instantiation that could apply is enqueued and
// those with nothing to do return at once.  The list lives in LDS when it fits and in the
// workspace otherwise.
#include <type_traits>

#include "host_util.h"
#include "plan_list.h"
#include "plan_params.h"
#include "wave.h"

namespace stalloc {

constexpr int kBatch = 256;          // requests fetched per refill
constexpr int kPend = kWave;         // requests per batch
constexpr int kTogether = 4;         // blocks that a scan looks at together

template <typename Addr, bool kLds, bool kCompact, int kThreads>
struct PlanLds {
    static constexpr int kWaves = kThreads / kWave;
    static constexpr bool kDirect = kLds && !kCompact;     // the scan reads the list itself
    // Lists in the workspace leave room for the spares below.  32-bit addresses only: the 64-bit kernel's registers are all in use.
    static constexpr bool kKeeps = !kLds && sizeof(Addr) == 4;
    // Blocks behind the list's last one that the scan may read (and does not use): it fetches the next group while it
    // looks at one, up to a group behind the end of a chunk, and only where it reads the list itself.
    static constexpr uint32_t kReadAhead = kDirect ? kTogether : 0;
    // A wave scans one chunk of the list with a request per lane, or two chunks at a time, half of the lanes each, with two
    // requests per lane (64-bit addresses: what is published for twice the chunks would take 17 KB more from the list)
    static constexpr int kHalves = sizeof(Addr) == 8 ? 1 : 2;
    static constexpr int kChunks = kWaves * kHalves;
    // holes published per (chunk, request), besides the one in front of the chunk's first conflicting block
    static constexpr int kSlots = sizeof(Addr) == 8 ? 2 : kWave / kChunks - 1;
    static constexpr int kCols = kSlots + 1;
    static_assert(kChunks * kCols <= kWave && kSlots > 0, "all holes of a request lie side by side in the lanes of a wave");
    // The scan takes blocks as broadcasts from LDS: from the list itself, or from here (listed in the workspace, or packed)
    static constexpr int kStaged = kDirect ? 1 : sizeof(Addr) == 8 ? kWave / 2 : kWave;
    typename BlockList<Addr, false>::Entry staged[kWaves][kStaged];
    uint64_t rq_size[kBatch];
    uint64_t rq_addr[kBatch];
    uint32_t rq_ta[kBatch];
    uint32_t rq_tf[kBatch];
    uint32_t rq_id[kBatch];
    Addr first[kChunks][kPend];                            // start of the chunk's first conflicting block, if that may close a hole
    Addr top[kChunks][kPend];                              // chunk maximum per (chunk, request)
    Addr last[kChunks];                                    // start of the chunk's last block
    uint8_t holes[kChunks][kPend];                         // holes found per (chunk, request), may exceed kSlots
    Span<Addr> hole[kChunks][kPend][kSlots];               // {hole end, chunk-local covered}
    // Orders by time and the like: for each request the holes of the lowest chunk with more than could be published
    static constexpr int kSpares = 15;
    Span<Addr> spare[kKeeps ? kPend : 0][kSpares];           // {hole end, covered}
    uint8_t spares[kKeeps ? kPend : 0];                      // how many (may exceed kSpares; 0: they were not looked for)
    uint8_t spare_chunk[kKeeps ? kPend : 0];
    uint32_t walks[kKeeps ? 1 : 0];                          // looks at such chunks in the last chain
    uint64_t usable[kPend];                                // holes that are large enough as such (lane = chunk * kCols + column)
    uint64_t crowded[kPend];                               // lanes of chunks with more holes than could be published
    Addr top_of[kPend];                                    // maximum over all chunks
    Addr at[kPend];                                        // where the requests of the batch are to lie, as far as known
    uint64_t clashes;                                      // requests that may not stay where they would lie without the rest of the batch
    Span<Addr> pend_span[kPend];                           // blocks settled in this batch, sorted
    uint2 pend_life[kPend];
    uint32_t pend_who[kPend];                              // and the request each belongs to
    uint32_t word;
    Addr extent_now;                                       // extent of the plan after the last settled batch
};

// The part of the list that is chunk `c`: chunks are equally long, a multiple of two groups of blocks; the last one that is not
// empty ends with the list and may begin inside the one before it (a block counted by two chunks changes nothing: what a
// lower chunk covers is known when holes are judged).  The list is empty or holds at least 64 blocks.
struct Chunk { uint32_t first, blocks; };
template <int kChunks>
__device__ __forceinline__ Chunk chunk_of(uint32_t count, uint32_t c)
{
    constexpr uint32_t kUnit = 2 * kTogether;
    static_assert((kUnit & (kUnit - 1)) == 0 && kUnit <= (uint32_t)kPend, "a list that is not empty holds a chunk");
    const uint32_t blocks = ((count + kChunks - 1) / kChunks + kUnit - 1) & ~(kUnit - 1);
    const uint32_t start = c * blocks;
    const uint32_t end = umin(start + blocks, count);
    return Chunk{start < count ? end - blocks : 0u, start < count ? blocks : 0u};
}

// The requests of the wave's lanes and one block of the list.  Returns the lanes whose request is alive together with the block and
// would fit in front of it, above what is covered so far (`room_end`: how far it would reach); and adds the block to what is
// covered.  A wave issues an instruction every four cycles at best, and there are four waves a SIMD: what counts is how many there are,
// scalar ones among them.  The lifetime compares switch lanes off, the rest is done by those that are left (all lanes are
// on again at the end): five vector instructions and one scalar; lane masks, combined and selected by, take six and two.
__device__ __forceinline__ uint64_t take_block(const BlockList<uint32_t, false>::Entry& block, uint32_t s, uint32_t ta, uint32_t tf,
                                               uint32_t& covered, uint32_t& room_end)
{
    uint64_t fits;
    asm volatile("v_add_u32_e32 %[end], %[covered], %[s]\n\t"
        "v_cmpx_lt_u32_e64 %[fits], %[b_ta], %[tf]\n\t"
        "v_cmpx_lt_u32_e64 %[fits], %[ta], %[b_tf]\n\t"
        "v_cmp_ge_u32_e64 %[fits], %[lo], %[end]\n\t"
        "v_max_u32_e32 %[covered], %[covered], %[hi]\n\t"
        "s_mov_b64 exec, -1"
        : [end] "=&v"(room_end), [fits] "=&s"(fits), [covered] "+&v"(covered)
        : [s] "v"(s), [ta] "v"(ta), [tf] "v"(tf), [lo] "v"(block.lo()), [hi] "v"(block.hi()), [b_ta] "v"(block.ta()), [b_tf] "v"(block.tf()));
    return fits;
}
__device__ __forceinline__ uint64_t take_block(const BlockList<uint64_t, false>::Entry& block, uint64_t s, uint32_t ta, uint32_t tf,
                                               uint64_t& covered, uint64_t& room_end)
{
    const uint64_t conflict = lanes_lt((uint32_t)block.ta(), tf) & lanes_lt(ta, (uint32_t)block.tf());
    room_end = covered + s;
    const uint64_t fits = conflict & lanes_ge(block.lo(), room_end), reach = umax(covered, block.hi());
    covered = lane_in(conflict) ? reach : covered;
    return fits;
}
// The size of a request whose further holes are not looked for: never room for it below 2^31 granules (above, they are looked at in vain).
template <typename Addr> struct Closed { static constexpr Addr value = (Addr)1 << (8 * sizeof(Addr) - 1); };

// One pass over the sorted list for the requests b0 .. b0+nb-1 of the staged batch.  A lane holds a request (or two), and
// the blocks of a chunk are taken one at a time, in address order, by all its lanes at once: two lifetime compares, an
// add, a compare and a maximum per block and 64 requests (64 bits: and selections), and nothing that crosses lanes.  The block comes
// as a broadcast from LDS (taken out of a register of a lane it costs four more vector instructions); 64 lanes reading 16 bytes keep the LDS busy for
// eight cycles whether they read one block or two, so the halves of a wave read a block each and hold all 64
// requests each, two per lane.  Blocks are looked at four together, so that their compares overlap and one branch asks
// whether any of them closes a hole.  Published per (chunk, request): the maximum of conflicting end addresses, the
// start of the first conflicting block, and the first holes behind it with chunk-local "covered".
template <typename Addr, typename List, typename Lds>
__device__ __forceinline__ void scan_batch(const List& list, uint32_t count, uint32_t b0, uint32_t nb, uint32_t shift, uint32_t& calm, Lds& sh)
{
    constexpr bool kDirect = Lds::kDirect;
    constexpr int kSlots = Lds::kSlots, kHalves = Lds::kHalves, kLanes = kWave / kHalves;
    constexpr uint32_t kPart = Lds::kStaged / kHalves;           // staged blocks per chunk
    static_assert(kDirect || kPart % (2 * kTogether) == 0, "a part is a whole number of steps, and a step ahead wraps to its start");
    typedef typename BlockList<Addr, false>::Entry Block;
    const int lane = lane_id(), wave = wave_id();
    const int half = lane / kLanes, place = lane % kLanes;
    const uint32_t c = (uint32_t)(wave * kHalves + half);
    const Chunk chunk = chunk_of<Lds::kChunks>(count, c);
    const uint32_t blocks = uniform(chunk.blocks);               // (of the wave's lowest chunk; the other may be empty)
    // requests beyond the batch, and all where there is no chunk, get an empty lifetime (conflicts with nothing)
    Addr rq_s[kHalves], covered[kHalves], first[kHalves];        // covered: maximum end of the conflicting blocks so far
    uint32_t rq_ta[kHalves], rq_tf[kHalves], found[kHalves];     // found: holes behind the chunk's first conflicting block
    uint64_t open[kHalves];                                      // lanes that have not found more holes than there are slots
#pragma unroll
    for (int u = 0; u < kHalves; ++u) {
        const int r = place + u * kLanes;
        rq_s[u] = 0; rq_ta[u] = 0; rq_tf[u] = 0;
        if (r < (int)nb && chunk.blocks > 0) {
            rq_s[u] = (Addr)(sh.rq_size[b0 + r] >> shift);
            rq_ta[u] = sh.rq_ta[b0 + r];
            rq_tf[u] = sh.rq_tf[b0 + r];
        }
        covered[u] = 0; first[u] = 0; found[u] = 0; open[u] = ~0ull;
    }
    // Where most groups of blocks concern no request of the batch at all, as in an interleaved schedule once the large requests of
    // an order by size are placed, that is asked first: four instructions per block and 64 requests if they do not, eleven if they do,
    // seven without asking.  `calm` tells from the first groups of the wave's last scans: up by one where they concerned nobody, else down by
    // two, and asked from six on.  (8944 requests of an interleaved schedule, 178 orders: 7.67 ms, 8.15 never asking, 8.06 always; 512
    // orders 12.0, 12.4, 13.0.  Traces that are never calm pay for the first groups: 600 to 6144 requests 0.2 % at the median, at most 1.4.)
    Addr last = 0;
    if (place == 0 && chunk.blocks > 0) last = list.load(chunk.first + chunk.blocks - 1).lo();
    // (the list in the workspace: the blocks of the next part are on their way while those of this one are looked at)
    auto part_of = [&](uint32_t k0) -> typename List::Entry {
        typename List::Entry en = List::none();
        if (place < (int)kPart && k0 + place < chunk.blocks) en = list.load(chunk.first + k0 + place);
        return en;
    };
    typename List::Entry next = List::none();
    if constexpr (!kDirect) next = part_of(0);
    for (uint32_t k0 = 0; k0 < blocks; k0 += kDirect ? blocks : kPart) {
        const uint32_t stop = kDirect ? blocks : umin(kPart, blocks - k0);
        if constexpr (!kDirect) {
            __builtin_amdgcn_wave_barrier();
            if (place < (int)kPart) sh.staged[wave][half * kPart + place] = BlockList<Addr, false>::make(next.lo(), next.hi(), next.ta(), next.tf());
            __builtin_amdgcn_wave_barrier();
            next = part_of(k0 + kPart);
        }
        // (reads behind the part are not looked at: one group behind a chunk of the list, or the staged part's first one again)
        auto fetch = [&](Block (&block)[kTogether], uint32_t k) {
#pragma unroll
            for (int i = 0; i < kTogether; ++i) {
                if constexpr (kDirect) block[i] = list.load(chunk.first + k + i);
                else block[i] = sh.staged[wave][half * kPart + (k & (kPart - 1)) + i];
            }
        };
        // do the blocks concern any request of the batch?
        auto concerned = [&](const Block (&block)[kTogether]) -> bool {
            uint64_t some = 0;
#pragma unroll
            for (int i = 0; i < kTogether; ++i)
#pragma unroll
                for (int u = 0; u < kHalves; ++u)
                    some |= lanes_lt((uint32_t)block[i].ta(), rq_tf[u]) & lanes_lt(rq_ta[u], (uint32_t)block[i].tf());
            return some != 0;
        };
        // room_end: what a request would reach in front of a block; holes: requests for which a block closes one
        auto look = [&](const Block (&block)[kTogether], auto ask) {
            uint64_t holes[kHalves][kTogether], any = 0;
            Addr room_end[kHalves][kTogether];
            if (decltype(ask)::value && !concerned(block)) return;       // (uniform)
#pragma unroll
            for (int i = 0; i < kTogether; ++i) {
#pragma unroll
                for (int u = 0; u < kHalves; ++u) {
                    holes[u][i] = take_block(block[i], rq_s[u], rq_ta[u], rq_tf[u], covered[u], room_end[u][i]);
                    any |= holes[u][i];
                }
            }
            if (any == 0) return;                                // (uniform)
#pragma unroll
            for (int i = 0; i < kTogether; ++i) {                // holes [before, lo) in front of some of them
#pragma unroll
                for (int u = 0; u < kHalves; ++u) {
                    uint64_t here = holes[u][i] & open[u];
                    if (here == 0) continue;
                    const Addr before = room_end[u][i] - rq_s[u];
                    const uint64_t lowest = here & ~lanes_lt((Addr)0, before);          // no conflicting block of the chunk lies lower
                    first[u] = lane_in(lowest) ? block[i].lo() : first[u];
                    here &= ~lowest;
                    if (here == 0) continue;
                    if (lane_in(here)) {
                        if (found[u] < (uint32_t)kSlots) sh.hole[c][place + u * kLanes][found[u]] = Span<Addr>{block[i].lo(), before};
                        ++found[u];
                    }
                    open[u] = lanes_lt(found[u], (uint32_t)kSlots + 1);                 // (kSlots + 1: more holes than slots)
                }
            }
#pragma unroll
            for (int u = 0; u < kHalves; ++u) rq_s[u] = lane_in(open[u]) ? rq_s[u] : Closed<Addr>::value;
        };
        Block even[kTogether], odd[kTogether];
        fetch(even, 0);
        if (k0 == 0) calm = concerned(even) ? (calm > 2 ? calm - 2 : 0u) : umin(calm + 1, 12u);
        auto look_at_all = [&](auto ask) {
            for (uint32_t k = 0; k < stop; k += 2 * kTogether) {
                fetch(odd, k + kTogether);
                look(even, ask);
                fetch(even, k + 2 * kTogether);
                look(odd, ask);
            }
        };
        if (calm >= 6) look_at_all(std::true_type());                // (uniform)
        else look_at_all(std::false_type());
    }
#pragma unroll
    for (int u = 0; u < kHalves; ++u) {
        sh.first[c][place + u * kLanes] = first[u];
        sh.top[c][place + u * kLanes] = covered[u];
        sh.holes[c][place + u * kLanes] = (uint8_t)found[u];
    }
    if (place == 0) sh.last[c] = last;
}

// What was published for request r, gathered into the 64 lanes of one wave in address order (kCols lanes a chunk;
// first the hole that ends at the chunk's first conflicting block, then those behind it).
template <typename Addr>
struct HoleView {
    Addr covered;        // per lane: covered in front of this hole (lower chunks included)
    Addr end;            // per lane: address at which the hole ends
    Addr top;            // uniform: maximum over all chunks (where the request goes if no hole fits)
    Addr below;          // per lane: maximum over the chunks below this lane's chunk
    uint64_t published;  // lanes that hold a hole
    uint64_t crowded;    // lanes of chunks with more holes than could be published
};

template <typename Addr>
struct HolesRead { Addr top, first; Span<Addr> hole; uint32_t found; Addr last; };

template <typename Addr, typename Lds>
__device__ __forceinline__ HolesRead<Addr> read_holes(const Lds& sh, uint32_t r)
{
    constexpr int kCols = Lds::kCols;
    const int w = lane_id() / kCols, c = lane_id() % kCols, wc = w < Lds::kChunks ? w : 0;
    return HolesRead<Addr>{sh.top[wc][r], sh.first[wc][r], sh.hole[wc][r][c > 0 ? c - 1 : 0], sh.holes[wc][r], sh.last[wc]};
}

template <typename Addr, typename Lds>
__device__ __forceinline__ HoleView<Addr> view_holes(const HolesRead<Addr>& read, Addr s, const Lds&)
{
    constexpr int kCols = Lds::kCols;
    const int lane = lane_id();
    const int w = lane / kCols, c = lane % kCols;
    const bool live = w < Lds::kChunks;
    const int wc = live ? w : 0;
    const Addr topv = live ? read.top : (Addr)0;
    const uint32_t found = live ? read.found : 0u;
    const Addr first = read.first;
    const Span<Addr> hl = read.hole;
    const Addr incl = wave_scan_max(topv);
    const Addr below = lane_gather(wave_shift_up(incl, (Addr)0), wc * kCols);
    HoleView<Addr> v;
    v.covered = c > 0 ? umax(below, hl.hi) : below;
    v.below = below;
    v.end = c > 0 ? hl.lo : first;
    v.top = read_lane(incl, kWave - 1);
    v.published = __builtin_amdgcn_ballot_w64(live && (c == 0 || (uint32_t)c <= found));
    // (not those that a large block below covers whole: there are no holes left; 49 920 requests, settling 52 -> 45 million cycles a plan)
    v.crowded = __builtin_amdgcn_ballot_w64(found > (uint32_t)Lds::kSlots && read.last >= (Addr)(below + s));
    return v;
}

// True if a chunk with unpublished holes lies below lane h (h < 0: the request would go on top).
template <typename Lds>
__device__ __forceinline__ bool unpublished_below(uint64_t crowded, int h)
{
    return crowded && (h < 0 || __builtin_ctzll(crowded) / Lds::kCols < h / Lds::kCols);
}

// A request of the batch and what the rest of the batch means to it.  Rivals are the blocks of the batch settled so far
// that are alive at the same time, one per lane in the order of their start addresses.
template <typename Addr>
struct Seeker {
    Addr s;
    uint32_t ta, tf;
    uint64_t rivals;
    Addr rival_lo;       // per lane: start address
    Addr reach_before;   // per lane: highest end of the rivals in lower lanes
    Addr reach;          // uniform: of all rivals

    // Lowest address >= c at which [c, c + s) clears the rivals: in front of the first of them that leaves room above
    // c and everything below, else above them all.  (One running maximum per request serves every c; moving up past one
    // rival after the other took 5 steps of some 100 cycles for a request on top of the list.)
    __device__ __forceinline__ Addr clear(Addr c) const
    {
        const Addr before = umax(c, reach_before);
        const uint64_t gaps = rivals & lanes_ge(rival_lo, (Addr)(before + s));
        return gaps ? read_lane(before, __builtin_ctzll(gaps)) : umax(c, reach);
    }
};

template <typename Addr>
__device__ __forceinline__ Seeker<Addr> seeker(Addr s, uint32_t ta, uint32_t tf, uint64_t rivals, Addr rival_lo, Addr rival_hi)
{
    const Addr incl = wave_scan_max(keep_lanes(rivals, rival_hi));
    return Seeker<Addr>{s, ta, tf, rivals, rival_lo, wave_shift_up(incl, (Addr)0), read_lane(incl, kWave - 1)};
}

// One wave walks a chunk of the list for one request, with everything
// below the chunk known (`below` = maximum end of the conflicting blocks of all lower chunks): the first hole {end, covered}
// of the chunk that takes the request once it has moved up past its rivals, to `x`.  Returns true if there is one.
// This is for chunks with more holes than slots to publish them.
template <typename Addr, typename List>
__device__ __forceinline__ bool chunk_lowest_fit(const List& list, const Chunk& chunk, Addr below, const Seeker<Addr>& rq,
                                                 Addr& x, Span<Addr>& hole)
{
    constexpr int kSteps = sizeof(Addr) == 8 ? 2 : 4;            // 64 blocks each, read together (the list may lie in memory)
    const uint32_t lane = (uint32_t)lane_id();
    Addr run = below;
    for (uint32_t k0 = 0; k0 < chunk.blocks; k0 += kSteps * kWave) {
        typename List::Entry en[kSteps];
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const uint32_t k = k0 + j * kWave + lane;
            en[j] = list.load(chunk.first + (k < chunk.blocks ? k : 0));
        }
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            if (k0 + j * kWave >= chunk.blocks) break;           // (uniform)
            const Addr e_lo = en[j].lo();
            const bool conflict = k0 + j * kWave + lane < chunk.blocks && en[j].ta() < rq.tf && rq.ta < en[j].tf();
            const Addr incl = wave_scan_max(conflict ? (Addr)en[j].hi() : (Addr)0);
            const Addr before = umax(run, wave_shift_up(incl, (Addr)0));
            uint64_t opens = __builtin_amdgcn_ballot_w64(conflict && e_lo >= (Addr)(before + rq.s));   // holes [before, e_lo) large enough as such
            while (opens) {
                const int h = __builtin_ctzll(opens);
                opens &= opens - 1;
                hole = Span<Addr>{read_lane(e_lo, h), read_lane(before, h)};
                x = rq.clear(hole.hi);
                if (x + rq.s <= hole.lo) return true;
            }
            run = umax(run, read_lane(incl, kWave - 1));
        }
    }
    return false;
}

// One wave: the holes of a chunk that are large enough for a request as such, the first `room` of them to out[]; returns how many it found
// (it stops once there are more than that).
template <typename Addr, typename List>
__device__ __forceinline__ uint32_t holes_of_chunk(const List& list, const Chunk& chunk, Addr below, Addr s, uint32_t ta, uint32_t tf,
                                                   Span<Addr>* out, uint32_t room)
{
    constexpr int kSteps = 2;                                    // 64 blocks each, read together
    const uint32_t lane = (uint32_t)lane_id();
    Addr run = below;
    uint32_t found = 0;
    for (uint32_t k0 = 0; k0 < chunk.blocks && found <= room; k0 += kSteps * kWave) {
        typename List::Entry en[kSteps];
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const uint32_t k = k0 + j * kWave + lane;
            en[j] = list.load(chunk.first + (k < chunk.blocks ? k : 0));
        }
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const Addr e_lo = en[j].lo();
            const bool conflict = k0 + j * kWave + lane < chunk.blocks && en[j].ta() < tf && ta < en[j].tf();
            const Addr incl = wave_scan_max(conflict ? (Addr)en[j].hi() : (Addr)0);
            const Addr before = umax(run, wave_shift_up(incl, (Addr)0));
            const uint64_t opens = __builtin_amdgcn_ballot_w64(conflict && e_lo >= (Addr)(before + s));
            const uint32_t at = found + lanes_below(opens);
            if (lane_in(opens) && at < room) out[at] = Span<Addr>{e_lo, before};
            found += (uint32_t)__builtin_popcountll(opens);
            run = umax(run, read_lane(incl, kWave - 1));
        }
    }
    return found;
}

// The holes published for request r, one per lane as in HoleView: {end, covered}, the latter counting lower chunks in.
template <typename Addr, typename Lds>
__device__ __forceinline__ Span<Addr> published_hole(const Lds& sh, uint32_t r)
{
    constexpr int kCols = Lds::kCols;
    const int lane = lane_id();
    const int w = lane / kCols < Lds::kChunks ? lane / kCols : 0, c = lane % kCols;
    const Span<Addr> in_front = {sh.first[w][r], sh.top[w][r]};
    const Span<Addr> behind = sh.hole[w][r][c > 0 ? c - 1 : 0];
    return Span<Addr>{c > 0 ? behind.lo : in_front.lo, c > 0 ? behind.hi : in_front.hi};
}

// Lowest fit of request r of the batch against the list and its rivals.  `hole`: what was published; `usable`: the lanes
// whose hole is large enough as such; `crowded`: the lanes of chunks with more holes than could be published (those
// that were are the lowest of the chunk); `top`: where the request goes if no hole takes it.
template <typename Addr, typename List, typename Lds>
__device__ __forceinline__ Addr lowest_fit(const List& list, uint32_t count, uint32_t r, const Seeker<Addr>& rq,
                                           const Span<Addr>& hole, uint64_t usable, uint64_t crowded, Addr top, Lds& sh)
{
    constexpr int kCols = Lds::kCols;
    while (usable | crowded) {
        const int h = usable ? __builtin_ctzll(usable) : -1;
        Addr x;
        if (unpublished_below<Lds>(crowded, h)) {
            const int w = __builtin_ctzll(crowded) / kCols;
            Span<Addr> walked;
            if constexpr (Lds::kKeeps) {
                if (lane_id() == 0) ++sh.walks[0];
                // (the survey has noted its holes)
                const uint32_t many = uniform((uint32_t)sh.spares[r]);
                if (many != 0 && uniform((uint32_t)sh.spare_chunk[r]) == (uint32_t)w) {
                    const Span<Addr> mine = sh.spare[r][lane_id() < Lds::kSpares ? lane_id() : 0];
                    for (uint32_t k = 0; k < umin(many, (uint32_t)Lds::kSpares); ++k) {
                        x = rq.clear(read_lane(mine.hi, (int)k));
                        if (x + rq.s <= read_lane(mine.lo, (int)k)) return x;
                    }
                    if (many <= (uint32_t)Lds::kSpares) { crowded &= ~(((1ull << kCols) - 1) << (w * kCols)); continue; }
                }
            }
            if (chunk_lowest_fit(list, chunk_of<Lds::kChunks>(count, (uint32_t)w), uniform(sh.top[w][r]), rq, x, walked)) return x;
            crowded &= ~(((1ull << kCols) - 1) << (w * kCols));
        } else {
            x = rq.clear(read_lane(hole.hi, h));
            if (x + rq.s <= read_lane(hole.lo, h)) return x;
            usable &= usable - 1;
        }
    }
    return rq.clear(top);                                        // on top of everything
}

// Settles the requests of the batch.  First every request gets the lowest fit against the list alone, request r from wave
// r mod #waves.  That address is the right one unless an earlier request of the batch that is alive at the same time lies
// there (15 to 40 in a hundred): those clashes are looked for by all waves, and wave 0 goes through them in order.  When it
// comes to a request all earlier ones lie where they are to lie; if the request moves, whoever it now meets
// among the later ones clashes too.
template <typename Addr, typename List, typename Lds>
__device__ __forceinline__ void settle_batch(const List& list, uint32_t count, uint32_t b0, uint32_t nb, uint32_t shift,
                                             Addr& peak, Lds& sh)
{
    constexpr int kCols = Lds::kCols, kPer = kPend / Lds::kWaves;
    static_assert(kPend % Lds::kWaves == 0, "requests are dealt out evenly");
    const int lane = lane_id(), wave = wave_id();
    // lane q holds request q of the batch
    Addr rq_s = 0;
    uint32_t rq_ta = 0, rq_tf = 0;
    if (lane < (int)nb) {
        rq_s = (Addr)(sh.rq_size[b0 + lane] >> shift);
        rq_ta = sh.rq_ta[b0 + lane];
        rq_tf = sh.rq_tf[b0 + lane];
    }
    // those alive at the same time as request r
    auto alive_with = [&](uint32_t ta, uint32_t tf) -> uint64_t { return lanes_lt(rq_ta, tf) & lanes_lt(ta, rq_tf); };
    HolesRead<Addr> read[kPer];                                  // (all reads go out before the first is used)
#pragma unroll
    for (int i = 0; i < kPer; ++i) read[i] = read_holes<Addr>(sh, (uint32_t)(wave + i * Lds::kWaves));
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t r = (uint32_t)(wave + i * Lds::kWaves);
        if (r >= nb) break;
        const Seeker<Addr> rq = {read_lane(rq_s, (int)r), read_lane(rq_ta, (int)r), read_lane(rq_tf, (int)r), 0, 0, 0, 0};
        HoleView<Addr> v = view_holes<Addr>(read[i], rq.s, sh);
        uint64_t usable = v.published & lanes_ge(v.end, (Addr)(v.covered + rq.s));
        // A chunk with unpublished holes below the first usable one is walked here, and the first hole that takes the request
        // goes where the chunk's last published one was (none of those is usable), so that it is not walked again.
        while (unpublished_below<Lds>(v.crowded, usable ? __builtin_ctzll(usable) : -1)) {
            const int w = __builtin_ctzll(v.crowded) / kCols, last = w * kCols + kCols - 1;
            Addr x;
            Span<Addr> hole;
            if (chunk_lowest_fit(list, chunk_of<Lds::kChunks>(count, (uint32_t)w), read_lane(v.below, last), rq, x, hole)) {
                v.end = write_lane(v.end, hole.lo, last);
                v.covered = write_lane(v.covered, hole.hi, last);
                usable |= 1ull << last;
                if (lane == last) sh.hole[w][r][Lds::kSlots - 1].lo = hole.lo;
            } else {
                v.crowded &= ~(((1ull << kCols) - 1) << (w * kCols));
            }
        }
        if (lane_in(v.published)) {
            if (lane % kCols > 0) sh.hole[lane / kCols][r][lane % kCols - 1].hi = v.covered;
            else sh.top[lane / kCols][r] = v.below;
        }
        if (lane == 0) { sh.usable[r] = usable; sh.crowded[r] = v.crowded; sh.top_of[r] = v.top; }
        const Addr x = usable ? read_lane(v.covered, __builtin_ctzll(usable)) : v.top;
        if (lane == 0) sh.at[r] = x;
    }
    if constexpr (Lds::kKeeps) {
        // Where the chain of the batch before went through crowded chunks, their holes are looked for here, by all waves, and not by
        // wave 0 in the middle of the chain (49 920 requests in order of time: 23 400 walks of 3600 cycles, 131 -> 114 ms).  Not
        // for every batch: orders that seldom go through them would wait for holes that nobody asks for.
        const bool often = uniform(sh.walks[0]) >= kPend / 4;    // (wave 0 counts anew behind the next two barriers)
#pragma unroll 1
        for (uint32_t r = (uint32_t)wave; r < nb; r += Lds::kWaves) {
            const uint64_t crowded = often ? uniform(sh.crowded[r]) : 0;
            uint32_t many = 0;
            if (crowded) {
                const uint32_t w = (uint32_t)__builtin_ctzll(crowded) / kCols;
                many = holes_of_chunk<Addr>(list, chunk_of<Lds::kChunks>(count, w), uniform(sh.top[w][r]), read_lane(rq_s, (int)r),
                                            read_lane(rq_ta, (int)r), read_lane(rq_tf, (int)r), sh.spare[r], (uint32_t)Lds::kSpares);
                if (lane == 0) sh.spare_chunk[r] = (uint8_t)w;
            }
            if (lane == 0) sh.spares[r] = (uint8_t)umin(many, 255u);
        }
    }
    if (threadIdx.x == 0) sh.clashes = 0;
    __syncthreads();
    {
        const Addr lo = sh.at[lane < (int)nb ? lane : 0];
        uint64_t mine = 0;
#pragma unroll 1
        for (int i = 0; i < kPer; ++i) {
            const uint32_t r = (uint32_t)(wave + i * Lds::kWaves);
            if (r >= nb) break;
            const Addr x = read_lane(lo, (int)r), s = read_lane(rq_s, (int)r);
            const uint64_t lower = (1ull << r) - 1;
            const uint64_t meets = alive_with(read_lane(rq_ta, (int)r), read_lane(rq_tf, (int)r)) & lanes_lt(lo, (Addr)(x + s)) &
                                   lanes_lt(x, (Addr)(lo + rq_s)) & lower;
            if (meets) mine |= 1ull << r;
            // sorted by address, for wave 0 below and for the merge
            const uint64_t below = (lanes_lt(lo, x) | (lanes_ge(x, lo) & lower)) & lanes_lt((uint32_t)lane, nb);
            if (lane == (int)r) {
                const int place = __builtin_popcountll(below);
                sh.pend_span[place] = Span<Addr>{x, (Addr)(x + rq_s)};
                sh.pend_life[place] = make_uint2(rq_ta, rq_tf);
                sh.pend_who[place] = r;
            }
        }
        if (mine != 0 && lane == 0) atomicOr((unsigned long long*)&sh.clashes, (unsigned long long)mine);
    }
    __syncthreads();
    if (wave == 0) {
        const int own = lane < (int)nb ? lane : 0;
        if constexpr (Lds::kKeeps) { if (lane == 0) sh.walks[0] = 0; }
        Addr lo = sh.at[own];
        const uint64_t usable = sh.usable[own], crowded = sh.crowded[own];
        const Addr top = sh.top_of[own];
        uint64_t clashes = uniform(sh.clashes);
        // lanes without a block: nobody's, behind all others
        Pending<Addr> pd = load_pending<Addr>(sh, nb);
        uint32_t who = sh.pend_who[own];
        if (lane >= (int)nb) { pd.lo = Top<Addr>::value; who = 0xffffffffu; }
        while (clashes) {
            const int r = __builtin_ctzll(clashes);
            clashes &= clashes - 1;
            const Addr s = read_lane(rq_s, r);
            const uint32_t ta = read_lane(rq_ta, r), tf = read_lane(rq_tf, r);
            const uint64_t rivals = lanes_lt(pd.ta, tf) & lanes_lt(ta, pd.tf) & lanes_lt(who, (uint32_t)r);
            const Seeker<Addr> rq = seeker(s, ta, tf, rivals, pd.lo, pd.hi);
            const uint64_t usable_r = read_lane(usable, r), crowded_r = read_lane(crowded, r);
            Addr x = read_lane(top, r);
            if ((usable_r | crowded_r) == 0) x = rq.clear(x);
            else x = lowest_fit<Addr>(list, count, (uint32_t)r, rq, published_hole<Addr>(sh, (uint32_t)r), usable_r, crowded_r, x, sh);
            // the block moves up to its place in address order
            const uint32_t from = (uint32_t)__builtin_ctzll(lanes_eq(who, (uint32_t)r));
            const uint32_t to = (uint32_t)__builtin_popcountll(lanes_ge(x, pd.lo)) - 1;
            const Pending<Addr> up = {wave_shift_down(pd.lo, (Addr)0), wave_shift_down(pd.hi, (Addr)0), wave_shift_down(pd.ta, 0u),
                                      wave_shift_down(pd.tf, 0u)};
            const uint32_t up_who = wave_shift_down(who, 0u);
            const bool down = lane_in(lanes_ge((uint32_t)lane, from) & lanes_lt((uint32_t)lane, to)), here = lane == (int)to;
            pd.lo = here ? x : down ? up.lo : pd.lo;
            pd.hi = here ? (Addr)(x + s) : down ? up.hi : pd.hi;
            pd.ta = here ? ta : down ? up.ta : pd.ta;
            pd.tf = here ? tf : down ? up.tf : pd.tf;
            who = here ? (uint32_t)r : down ? up_who : who;
            lo = write_lane(lo, x, r);
            clashes |= alive_with(ta, tf) & ~((2ull << r) - 1) & lanes_lt(lo, (Addr)(x + s)) & lanes_lt(x, (Addr)(lo + rq_s));
        }
        if (lane < (int)nb) {
            sh.pend_span[lane] = Span<Addr>{pd.lo, pd.hi};
            sh.pend_life[lane] = make_uint2(pd.ta, pd.tf);
        }
        peak = umax(peak, read_lane(wave_scan_max(lane < (int)nb ? (Addr)(lo + rq_s) : (Addr)0), kWave - 1));
        if (lane < (int)nb) sh.rq_addr[b0 + lane] = (uint64_t)lo << shift;
        if (lane == 0) sh.extent_now = peak;
    }
    __syncthreads();
}

template <typename Addr, bool kLds, bool kCompact, int kThreads>
__global__ void __launch_bounds__(kThreads, 4) plan_kernel(PlanParams prm)   // <= 128 VGPRs: 16 waves per CU
{
    using Lds = PlanLds<Addr, kLds, kCompact, kThreads>;
    using List = BlockList<Addr, kCompact>;
    extern __shared__ __align__(16) unsigned char smem[];
    Lds& sh = *reinterpret_cast<Lds*>(smem);
    const uint32_t n = prm.n;

    const uint32_t status = read_status(prm.status);
    const uint64_t mode = prm.acc[kAccMode];
    if (bitmap_shape(mode, prm.acc[kAccGranules], prm.bitmap_pool_words) >= 0) return;   // the occupancy-bitmap kernel places this trace
    // the kernel that lists only long-lived blocks places it (and leaves the plans that outgrow
    // 32-bit counts to the 64-bit instantiation here)
    if (sizeof(Addr) == 4 && (prm.acc[kAccSplit] & 1)) return;
    const bool narrow = (mode & kModeNarrow) != 0;
    // Not narrow, but no request is large: the 32-bit instantiation takes every plan as far as
    // 32-bit granule counts certainly hold its addresses and marks the plans that outgrow them;
    // the 64-bit instantiation (enqueued behind it) places those from scratch.
    const bool try32 = (mode & kModeTry32) != 0;
    if (sizeof(Addr) == 4 ? !(narrow || try32) : narrow) return;     // another instantiation handles this trace
    // of the two 32-bit instantiations the compact one runs when it was enqueued and applies
    const bool compact = prm.compact_enqueued && (mode & kModeCompact) != 0;
    if (sizeof(Addr) == 4 && compact != kCompact) return;
    if (status_of_workgroup(status, &sh.word) != STALLOC_OK) return;   // malformed trace: nothing to plan
    const uint32_t shift = sizeof(Addr) == 4 ? (uint32_t)(mode & 63) : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && !(sizeof(Addr) == 8 && try32))
        const_cast<uint64_t*>(prm.acc)[kAccKernel] = (kLds ? STALLOC_KERNEL_LIST_LDS : STALLOC_KERNEL_LIST_MEMORY) |
                                                     ((kCompact ? 16u : 8u * (uint32_t)sizeof(Addr)) << 8);

    List list, spare;
    if constexpr (kLds) {
        list.bind(smem + sizeof(Lds), n);
        spare = list;
    } else {
        unsigned char* slab = prm.slabs + (size_t)blockIdx.x * 2 * (size_t)n * entry_bytes<uint64_t>();
        list.bind(slab, n);
        spare.bind(slab + (size_t)n * entry_bytes<uint64_t>(), n);
    }

    // Beyond one per workgroup plans are handed out as workgroups get done: an order by time takes twice as long as a random
    // one, and the workgroup that places it should not have another waiting for it.
    // Plans to place again with 64-bit addresses are handed out, too, where the list lies in the workspace (7500 requests, 785 of
    // 2000 plans again: 73 -> 52 ms); with the list in LDS they are short and stay where they are.
    auto next_plan = [&](uint32_t p) -> uint32_t {
        if (kLds && sizeof(Addr) == 8 && try32) return p + gridDim.x;
        if (gridDim.x >= prm.P) return prm.P;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t* handed_out = const_cast<uint64_t*>(prm.acc) + (sizeof(Addr) == 8 ? kAccNextWide : kAccNextPlan);
            sh.word = gridDim.x + (uint32_t)atomicAdd((unsigned long long*)handed_out, 1ull);
        }
        __syncthreads();
        return uniform(sh.word);
    };
    for (uint32_t p = blockIdx.x; p < prm.P; p = next_plan(p)) {
        if (sizeof(Addr) == 8 && try32 && !prm.wide_plans[p]) continue;   // (uniform) placed with 32-bit counts already
        if (sizeof(Addr) == 8 && try32 && threadIdx.x == 0)
            atomicAdd((unsigned long long*)&const_cast<uint64_t*>(prm.acc)[kAccWidePlans], 1ull);
        const uint32_t* order = prm.orders + (size_t)p * n;
        uint64_t* out = prm.offsets ? prm.offsets + (size_t)p * n : nullptr;
        Addr peak = 0;                                        // tracked by wave 0
        uint32_t count = 0;
        uint32_t calm = 0;                                    // (of this wave's scans)
        bool outgrown = false;                                // (uniform) 32-bit counts may not hold the next batch
        __syncthreads();                                      // (every wave has taken its decisions about the plan before)
        if (threadIdx.x == 0) {
            sh.extent_now = 0;
            if constexpr (Lds::kKeeps) sh.walks[0] = 0;
            if (sizeof(Addr) == 4) prm.wide_plans[p] = 0;
        }

        for (uint32_t r0 = 0; r0 < n; r0 += kBatch) {
            const uint32_t staged = n - r0 < (uint32_t)kBatch ? n - r0 : (uint32_t)kBatch;
            __syncthreads();                                  // previous batch fully consumed
            if (threadIdx.x < staged) {
                uint32_t i = order[r0 + threadIdx.x];
                if (i >= n) { atomicMax(prm.status, (uint32_t)STALLOC_ERR_BAD_ORDER); i = 0; }
                sh.rq_id[threadIdx.x] = i;
                sh.rq_size[threadIdx.x] = prm.size[i];
                sh.rq_ta[threadIdx.x] = prm.ta[i];
                sh.rq_tf[threadIdx.x] = prm.tf[i];
            }
            __syncthreads();

            for (uint32_t b0 = 0; b0 < staged;) {
                const uint32_t nb = staged - b0 < (uint32_t)kPend ? staged - b0 : (uint32_t)kPend;
                if (sizeof(Addr) == 4 && try32) {
                    // no address of this batch exceeds the extent so far plus the sizes of the batch
                    const int lane = lane_id();
                    const uint64_t growth = wave_sum64(lane < (int)nb ? sh.rq_size[b0 + lane] >> shift : 0ull);
                    if ((uint64_t)sh.extent_now + growth > 0xffffffffull) { outgrown = true; break; }
                }
                scan_batch<Addr>(list, count, b0, nb, shift, calm, sh);
                __syncthreads();
                settle_batch<Addr>(list, count, b0, nb, shift, peak, sh);
                const bool last_of_plan = r0 + b0 + nb >= n;
                if (!last_of_plan) merge_pending<Addr, kLds, kThreads>(list, spare, count, nb, sh);
                count += nb;
                b0 += nb;
            }
            if (outgrown) break;
            // addresses of this batch -> offsets[p][request id]
            __syncthreads();
            if (out && threadIdx.x < staged) out[sh.rq_id[threadIdx.x]] = sh.rq_addr[threadIdx.x];
        }
        if (outgrown) {
            if (threadIdx.x == 0) prm.wide_plans[p] = 1;
            continue;
        }
        if (threadIdx.x == 0) prm.peaks[p] = (uint64_t)peak << shift;
    }
}

// Index of the smallest extent (lowest index among equals), in all threads of a workgroup of 256.
__device__ __forceinline__ uint32_t index_of_best(const uint64_t* __restrict__ peaks, uint32_t P)
{
    __shared__ uint64_t w_peak[4];
    __shared__ uint64_t w_idx[4];
    uint64_t best = ~0ull, idx = ~0ull;
    for (uint32_t p = threadIdx.x; p < P; p += 256) {
        uint64_t v = peaks[p];
        if (v < best) { best = v; idx = p; }       // ascending p per thread: first of equals kept
    }
    uint64_t wbest = wave_min64(best);
    uint64_t widx = wave_min64(best == wbest ? idx : ~0ull);
    if (lane_id() == 0) { w_peak[wave_id()] = wbest; w_idx[wave_id()] = widx; }
    __syncthreads();
    uint64_t b = w_peak[0], i = w_idx[0];
    for (int k = 1; k < 4; ++k)
        if (w_peak[k] < b || (w_peak[k] == b && w_idx[k] < i)) { b = w_peak[k]; i = w_idx[k]; }
    return (uint32_t)i;
}

__global__ void __launch_bounds__(256) plan_argmin(const uint64_t* __restrict__ peaks, uint32_t P, uint32_t* best_plan,
                                                   const uint32_t* status)
{
    if (*status != STALLOC_OK) { if (threadIdx.x == 0) *best_plan = 0; return; }
    const uint32_t best = index_of_best(peaks, P);
    if (threadIdx.x == 0) *best_plan = best;
}

// The same and the best plan's addresses in one launch: every workgroup looks for the best plan by itself, which
// for up to this many plans is less than a launch (4096 extents are 32 KB, read from the L2).
constexpr uint32_t kBestAlone = 4096;
__global__ void __launch_bounds__(256) plan_best(const uint64_t* __restrict__ peaks, uint32_t P, const uint64_t* __restrict__ offsets,
                                                 uint32_t n, uint32_t* best_plan, uint64_t* best_offsets, const uint32_t* status)
{
    if (*status != STALLOC_OK) { if (blockIdx.x == 0 && threadIdx.x == 0) *best_plan = 0; return; }
    const uint32_t best = index_of_best(peaks, P);
    if (blockIdx.x == 0 && threadIdx.x == 0) *best_plan = best;
    const uint64_t* src = offsets + (size_t)best * n;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) best_offsets[i] = src[i];
}

__global__ void __launch_bounds__(256) plan_copy_best(const uint64_t* __restrict__ offsets, const uint32_t* best_plan,
                                                      uint32_t n, uint64_t* best_offsets, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    const uint64_t* src = offsets + (size_t)(*best_plan) * n;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) best_offsets[i] = src[i];
}

// Tuning knobs (overridable at build time with -D).
#ifndef STALLOC_THREADS_LDS
#define STALLOC_THREADS_LDS 1024
#endif
#ifndef STALLOC_THREADS_MEM
#define STALLOC_THREADS_MEM 1024
#endif
constexpr int kThreadsLds = STALLOC_THREADS_LDS;
constexpr int kThreadsMem = STALLOC_THREADS_MEM;

#ifndef STALLOC_THREADS_COMPACT
#define STALLOC_THREADS_COMPACT 512
#endif
constexpr int kThreadsCompact = STALLOC_THREADS_COMPACT;   // two such workgroups share one CU

// Calls from this many requests on prepare the kernel for long traces with few long-lived requests and carry its tables.
// Shorter calls do without, also those whose lists do not fit LDS: their workspace does not depend on t_end, and the some
// twenty launches of the preparation cost a call that a bitmap kernel places 70 to 100 us and 28 to 34 MB (7500 requests,
// 1 order: 2.55 ms, with the preparation 2.63).  Where few requests are long-lived the sorted list is the faster there for
// few orders (8200 requests, 256 orders: 8.0 ms, the long-list kernel 11.8), as fast for two a CU (512: 12.4 and 11.8) and the
// slower beyond (768: 16.9 and 11.9; 2048: 39 and 25), which the calls of other traces would pay for.
constexpr uint32_t kLongListFrom = 9096;

// Entries the LDS-resident list may hold, for a given entry size and LDS budget.
template <typename Addr, bool kCompact, int kThreads>
inline uint32_t lds_capacity_entries(size_t lds_budget, size_t bytes_per_entry)
{
    using Lds = PlanLds<Addr, true, kCompact, kThreads>;
    const size_t fixed = sizeof(Lds) + Lds::kReadAhead * bytes_per_entry;
    if (lds_budget <= fixed) return 0;
    return (uint32_t)((lds_budget - fixed) / bytes_per_entry);
}

template <typename Addr, bool kLds, bool kCompact, int kThreads>
inline bool launch_plan(const PlanParams& prm, uint32_t grid, const DeviceInfo& di, hipStream_t stream)
{
    auto kernel = &plan_kernel<Addr, kLds, kCompact, kThreads>;
    using Lds = PlanLds<Addr, kLds, kCompact, kThreads>;
    size_t lds = sizeof(Lds) + (kLds ? ((size_t)prm.n + Lds::kReadAhead) * BlockList<Addr, kCompact>::kEntryBytes : 0);
    static std::atomic<bool> attr_set[64] = {};        // (set twice at worst when threads race)
    if (!attr_set[di.device]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)di.lds_per_block) != hipSuccess)
            return false;
        attr_set[di.device] = true;
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), lds, stream, prm);
    return true;
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_plan_report(const void* workspace, stalloc_plan_info* info, void* hip_stream)
{
    if (!workspace || !info) return STALLOC_ERR_INVALID_ARG;
    uint64_t acc[kAccWords];
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (hipMemcpyAsync(acc, workspace, sizeof(acc), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return STALLOC_ERR_DEVICE;
    info->kernel = (uint32_t)(acc[kAccKernel] & 0xffu);
    info->address_bits = (uint32_t)((acc[kAccKernel] >> 8) & 0xffu);
    info->granule_log2 = (uint32_t)(acc[kAccMode] & 63);
    info->granules = acc[kAccGranules];
    info->plans_64bit = (uint32_t)acc[kAccWidePlans];
    info->lifetime_threshold = (acc[kAccSplit] & 1) ? (uint32_t)((acc[kAccSplit] >> 8) & 0xffffffu) : 0u;
    info->long_requests = (acc[kAccSplit] & 1) ? (uint32_t)(acc[kAccSplit] >> 32) : 0u;
    const bool large = (acc[kAccSplit] & 1) && (uint32_t)acc[kAccLargeShort] != 0xffffffffu;
    info->large_size = large ? (acc[kAccLargeShort] & 0xffffffffull) << (acc[kAccMode] & 63) : 0ull;
    info->large_requests = large ? (uint32_t)(acc[kAccLargeShort] >> 32) : 0u;
    info->list_entry_bytes = (uint32_t)((acc[kAccKernel] >> 16) & 0xffu);
    return STALLOC_OK;
}

extern "C" uint32_t stalloc_plan_lds_capacity(void)
{
    DeviceInfo di;
    if (!device_info(&di)) return 0;
    return lds_capacity_entries<uint32_t, false, kThreadsLds>(di.lds_per_block, entry_bytes<uint32_t>());
}

// allow_bitmap: false when the caller has said that its sizes cannot suit the occupancy-bitmap kernel; that
// kernel and its index of lifetime-overlapping pairs are then left out of the call and of the workspace.
static int plan_call(const stalloc_trace* tr, const uint32_t* orders, uint32_t P, uint64_t* offsets, uint64_t* peaks,
                     uint64_t* best_offsets, uint32_t* best_plan, uint32_t* device_status, bool allow_bitmap,
                     void* workspace, size_t* workspace_bytes, void* hip_stream)
{
    if (!trace_args_ok(tr) || P == 0 || !workspace_bytes) return STALLOC_ERR_INVALID_ARG;
    DeviceInfo di;
    if (!device_info(&di)) return STALLOC_ERR_DEVICE;
    const uint32_t n = tr->n;
    const bool lds32 = n <= lds_capacity_entries<uint32_t, false, kThreadsLds>(di.lds_per_block, entry_bytes<uint32_t>());
    const bool lds64 = n <= lds_capacity_entries<uint64_t, false, kThreadsLds>(di.lds_per_block, entry_bytes<uint64_t>());
    // Where the lists leave the LDS follows from what the hole tables need of it.  512 orders, sizes of up to 33 KB and an
    // odd byte: 7300 requests 13.4 ms in LDS, 8000 in the workspace 16.4 (24.4 and 27.7 before); with 64-bit addresses 4200
    // 7.6, 5000 10.1 (20.1, 25.9).
    // Compact list: 8-byte entries, two workgroups per CU (half the LDS each); 1024 orders, 3600 requests 6.3 ms, 5000 with
    // 16-byte entries 13.1 (12.6, 20.2)
    const bool compact = tr->t_end < 0x10000u &&
                         n <= lds_capacity_entries<uint32_t, true, kThreadsCompact>(di.lds_per_block / 2, sizeof(uint2));
    // One workgroup per CU is resident, with the list in LDS (that takes most of it) and with the list in the workspace (of 83
    // or 91 registers five waves fit a SIMD): a second one would hold two slabs and wait.  Compact lists: two per CU.
    uint32_t grid_lds = (uint32_t)di.cus, grid_mem = (uint32_t)di.cus, grid_compact = (uint32_t)di.cus * 2;
    if (grid_lds > P) grid_lds = P;
    if (grid_mem > P) grid_mem = P;
    if (grid_compact > P) grid_compact = P;

    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    uint64_t* own_offsets = (!offsets && best_offsets) ? cv.take<uint64_t>((size_t)P * n) : nullptr;
    uint32_t* wide_plans = cv.take<uint32_t>(P);
    const bool brief = short_plan_possible(n, P);
    // occupancy-bitmap variant: lifetime-conflict index of the trace
    uint32_t pool_words[kBitmapShapes];
    const bool bitmap = bitmap_plan_shapes(n, di, pool_words) && allow_bitmap && !brief;
    uint32_t* nbr_chunks = bitmap ? cv.take<uint32_t>(n) : nullptr;
    // The index and the lists in the workspace share their room: everything that writes or reads the index is enqueued before
    // the sorted-list kernels.  (5000 requests, 512 orders: 51 MB of index, 61 MB of lists for traces of 64-bit addresses)
    const size_t index_bytes = bitmap ? bitmap_index_entries(n) * sizeof(uint16_t) : 0;
    const size_t slab_bytes = lds64 ? 0 : (size_t)grid_mem * 2 * n * entry_bytes<uint64_t>();
    unsigned char* room = cv.take<unsigned char>(index_bytes > slab_bytes ? index_bytes : slab_bytes);
    uint16_t* nbr = bitmap ? reinterpret_cast<uint16_t*>(room) : nullptr;
    unsigned char* slabs = lds64 ? nullptr : room;
    const bool tiled = bitmap && tiled_plan_possible(n, tr->t_end, P, di);
    int32_t* net = bitmap ? cv.take<int32_t>(tiled_plan_words(n)) : nullptr;
    // variant for long traces with few long-lived requests: tables in allocation-time order
    const bool split = n >= kLongListFrom;
    SplitWorkspace sw;
    if (split) split_workspace(n, tr->t_end, di, cv, &sw);
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    if (!orders || !peaks || !best_plan || !device_status || *workspace_bytes < cv.used ||
        (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    PlanParams prm;
    prm.size = tr->size; prm.ta = tr->t_alloc; prm.tf = tr->t_free; prm.orders = orders;
    prm.offsets = offsets ? offsets : own_offsets;
    prm.peaks = peaks; prm.status = device_status; prm.acc = acc; prm.slabs = slabs; prm.n = n; prm.P = P;
    prm.compact_enqueued = compact ? 1u : 0u;
    prm.nbr_chunks = nbr_chunks; prm.nbr = nbr; prm.wide_plans = wide_plans;
    for (int shape = 0; shape < kBitmapShapes; ++shape) prm.bitmap_pool_words[shape] = bitmap ? pool_words[shape] : 0u;
    if (brief) return launch_plan_short(prm, tr->t_end, best_offsets, best_plan, stream) ? STALLOC_OK : STALLOC_ERR_DEVICE;

    launch_trace_check(*tr, acc, device_status, stream);
    bool ok = true;
    if (split) ok = ok && launch_plan_split(prm, tr->t_end, sw, di, stream);
    if (tiled) ok = ok && launch_plan_tiled(prm, tr->t_end, net, di, stream);
    if (bitmap) ok = ok && launch_plan_bitmap(prm, di, stream);
    // exactly one of the launches does the work; the trace decides which (see the mode word).  (From here on the index of the
    // bitmap variants may be overwritten.)
    if (compact) ok = ok && launch_plan<uint32_t, true, true, kThreadsCompact>(prm, grid_compact, di, stream);
    if (lds32) ok = ok && launch_plan<uint32_t, true, false, kThreadsLds>(prm, grid_lds, di, stream);
    else       ok = ok && launch_plan<uint32_t, false, false, kThreadsMem>(prm, grid_mem, di, stream);
    if (lds64) ok = ok && launch_plan<uint64_t, true, false, kThreadsLds>(prm, grid_lds, di, stream);
    else       ok = ok && launch_plan<uint64_t, false, false, kThreadsMem>(prm, grid_mem, di, stream);
    if (!ok) return STALLOC_ERR_DEVICE;

    uint32_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    if (best_offsets && P <= kBestAlone) {
        if (blocks > 256) blocks = 256;
        hipLaunchKernelGGL(plan_best, dim3(blocks), dim3(256), 0, stream, peaks, P, prm.offsets, n, best_plan, best_offsets, device_status);
        return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
    }
    hipLaunchKernelGGL(plan_argmin, dim3(1), dim3(256), 0, stream, peaks, P, best_plan, device_status);
    if (best_offsets) {
        hipLaunchKernelGGL(plan_copy_best, dim3(blocks), dim3(256), 0, stream, prm.offsets, best_plan, n, best_offsets,
                           device_status);
    }
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}

extern "C" int stalloc_plan(const stalloc_trace* tr, const uint32_t* orders, uint32_t P, uint64_t* offsets,
                            uint64_t* peaks, uint64_t* best_offsets, uint32_t* best_plan, uint32_t* device_status,
                            void* workspace, size_t* workspace_bytes, void* hip_stream)
{
    return plan_call(tr, orders, P, offsets, peaks, best_offsets, best_plan, device_status, true, workspace, workspace_bytes,
                     hip_stream);
}

extern "C" int stalloc_plan_sized(const stalloc_trace* tr, const uint32_t* orders, uint32_t P, uint64_t* offsets,
                                  uint64_t* peaks, uint64_t* best_offsets, uint32_t* best_plan, uint32_t* device_status,
                                  uint64_t largest_size, uint64_t granule, void* workspace, size_t* workspace_bytes,
                                  void* hip_stream)
{
    if (granule == 0 || (granule & (granule - 1)) != 0 || largest_size == 0) return STALLOC_ERR_INVALID_ARG;
    const bool allow_bitmap = largest_size / granule <= kBitmapMaxSize;
    return plan_call(tr, orders, P, offsets, peaks, best_offsets, best_plan, device_status, allow_bitmap, workspace,
                     workspace_bytes, hip_stream);
}
