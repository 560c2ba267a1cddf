// stalloc_plan, occupancy-bitmap variant for longer traces: the rule of plan_bitmap.hip (Sec. 5.1: requests in
// the given order, each at the lowest address where it conflicts with no earlier request of the plan in
// lifespan and address range at once), with most of the conflicting blocks read from a table.
//
// plan_bitmap.hip looks up every request with an overlapping lifetime, placed or not: 737 on average for the
// 6144 requests of a pipeline stage.  Here time is cut into tiles, and the plan keeps two bitmaps of the
// address range per tile: `cover`, the blocks alive during the whole tile, and `any`, those alive at some
// time of it.  A request that lives from tile a to tile b conflicts with
//     all of cover[a], all of cover[b], all of any[a + 1] .. any[b - 1],
// and, beyond those, only with requests that are allocated or released inside tile a or b: a list that does
// not depend on the order and is worked out once per call (a few dozen to a few hundred entries).
//
//   build    A wave other than wave 0 takes a request (or two) of the batch by itself: rows of the tables ORed into
//            its bitmap, the blocks of the list marked in it (as in plan_bitmap.hip), and the first run of free
//            granules.
//   settle   Wave 0 takes the requests of the batch before, while the others build: a candidate stands unless a
//            block its bitmap may have missed (the two batches before it, and the requests settled earlier
//            in the batch) overlaps it in lifetime and address range.
//   mark     A round later, in front of its next build, the wave enters the blocks of its requests into the
//            tables, a tile per lane.
//
// What bounds it: on 6144 requests (two workgroups a CU) the vector issue of the building waves and waiting for the wave with the
// longest request of the batch; on 19 840 (one workgroup of sixteen waves) half the time is such waiting.  In orders by size and by
// time, where nearly every request meets the one before it, the chain of those in wave 0 (an order by time of 19 840 requests: 8.4 ms
// alone, a random one 4.4; it sets the time of a launch with two plans a workgroup).
// 1024 plans of 6144 requests: 6.9 ms looking up every request, 4.66 with tables read a word at a time, 4.05 four words at a time and
// with chains in registers (fit_among), 3.96 where those pay; 512 plans of 19 840: 24.0, 13.85, 12.2, 12.0 ms.
//
// The tables hold the address range up to an eighth above the largest number of live granules (which no
// plan can stay below and plans worth having stay close to), and up to two and a half times that number where the LDS has
// room.  A plan that grows beyond that is given up and placed by plan_bitmap.hip, whose kernels follow on the
// stream and otherwise return at once; when half of the plans so far did, the later ones are left to it untried.
#include "bitmap_cells.h"
#include "host_util.h"
#include "plan_params.h"
#include "wave.h"

namespace stalloc {

constexpr uint32_t kPtMostTiles = 64;            // a tile per lane when a block is marked
constexpr uint32_t kPtRefill = 256;              // requests staged at a time, at most

// acc[kAccTiles]: bit 0 set when this variant places the trace; bits 1-7 shape (0: eight waves, several workgroups
// per CU; 1: sixteen waves, all LDS of a CU); bits 8-15 tiles; bits 16-31 words of a row; bits 32-63 timestamps
// per tile.
struct PtShape {
    uint32_t shape, tiles, row, width;
    __device__ explicit PtShape(uint64_t w)
        : shape((uint32_t)(w >> 1) & 0x7fu), tiles((uint32_t)(w >> 8) & 0xffu), row((uint32_t)(w >> 16) & 0xffffu), width((uint32_t)(w >> 32)) {}
};
// Requests of a batch per building wave: two with eight waves (a wave's long and short requests even out, half
// the barriers: 4.77 ms for 1024 plans of 6144 requests, 4.89 with one, 4.75 with three), one with sixteen (the
// bitmaps of thirty requests would take the tables' room: 14.1 ms for 512 plans of 19 840, 17.0 with two).
__host__ __device__ constexpr uint32_t pt_per_wave(uint32_t waves) { return waves == 8 ? 2u : 1u; }
__host__ __device__ constexpr uint32_t pt_batch(uint32_t waves) { return (waves - 1) * pt_per_wave(waves); }
// With more clashing requests in a batch than this, what follows their candidates is fetched for all of them at once.
constexpr int kPtFew = 2;
// Where the place of more than half of them lies further up than that (sizes up to 31 granules in tall stacks), it is not looked at in
// the next batches: a look is some seventy instructions, and the bitmap is searched all the same.  (6000 requests of 1 to 31
// granules, 256 orders: 2.92 ms without fit_among, 3.06 with it in every batch, 2.69 so.)
constexpr uint32_t kPtInVain = 15;
// Rows and bitmaps begin at multiples of four words, so that a lane reads or writes four at a time (a request that lives through 25
// tiles of 400 words: 50 reads instead of 175).  An odd multiple, so that the tiles of a block that is marked, a lane each, lie in as many
// banks as that leaves (16 of 64).
__host__ __device__ inline uint32_t pt_fours(uint32_t words) { return (words + 3) / 4 * 4; }
__host__ __device__ inline uint32_t pt_stride(uint32_t row) { return pt_fours(row) | 4u; }
// A bitmap holds a row of the tables and what three batches of the longest requests can add to the extent.
__host__ __device__ inline uint32_t pt_bitmap_words(uint32_t row, uint32_t batch, uint32_t longest) { return pt_fours(row + (3 * batch * longest + 31) / 32 + 2); }

struct PtOffer { uint32_t words[2]; };           // LDS words behind TiledLds per shape; 0: not part of this call

template <int kWaves>
struct TiledLds {
    uint32_t rq_id[kPtRefill];
    uint32_t rq_s[kPtRefill];            // size in granules
    uint32_t rq_ta[kPtRefill];
    uint32_t rq_tf[kPtRefill];
    uint32_t rq_x[kPtRefill];            // address in granules
    uint32_t rq_chunks[kPtRefill];       // chunks of the request's list
    uint32_t rq_tiles[kPtRefill];        // first tile | last tile << 8 | first covered tile << 16 | one behind the last covered << 24
    uint32_t cand[2][pt_batch(kWaves)];  // lowest fits of the batch being built and of the batch being settled
    uint32_t top[2];                     // extent after the last batch and the one before, granules
    uint32_t pad[4 - (2 * pt_batch(kWaves) + 2) % 4];
};

// One workgroup: the largest number of granules alive at once, and what fits the LDS for it.
__global__ void __launch_bounds__(1024) pt_shape(PlanParams prm, uint32_t t_end, int32_t* net, PtOffer offer)
{
    __shared__ int32_t part[16], peak[16];
    uint64_t* acc = const_cast<uint64_t*>(prm.acc);
    if (*prm.status != STALLOC_OK) return;
    if (bitmap_shape(acc[kAccMode], acc[kAccGranules], prm.bitmap_pool_words) < 0) return;
    const uint32_t shift = (uint32_t)(acc[kAccMode] & 63), tid = threadIdx.x, n = prm.n;
    for (uint32_t t = tid; t <= t_end; t += 1024) __hip_atomic_store(&net[t], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (uint32_t i = tid; i < n; i += 1024) {
        const int32_t s = (int32_t)(prm.size[i] >> shift);
        atomicAdd(&net[prm.ta[i]], s);
        atomicAdd(&net[prm.tf[i]], -s);
    }
    __syncthreads();
    const uint32_t per = (t_end + 1023) / 1024, t0 = umin(tid * per, t_end), t1 = umin(t0 + per, t_end);
    int32_t sum = 0, most = 0;                                        // of the thread's timestamps, counted from their start
    for (uint32_t t = t0; t < t1; ++t) {
        sum += __hip_atomic_load(&net[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        most = sum > most ? sum : most;
    }
    const int32_t incl = (int32_t)wave_scan_add((uint32_t)sum);
    if (lane_id() == kWave - 1) part[wave_id()] = incl;
    __syncthreads();
    int32_t before = incl - sum;
    for (int w = 0; w < wave_id(); ++w) before += part[w];
    const uint32_t wave_most = read_lane(wave_scan_max((uint32_t)(before + most)), kWave - 1);       // (live granules: never negative)
    if (lane_id() == 0) peak[wave_id()] = (int32_t)wave_most;
    __syncthreads();
    if (tid != 0) return;
    uint32_t live = 0;
    for (int w = 0; w < 16; ++w) live = umax(live, (uint32_t)peak[w]);
    const uint32_t row = (live + live / 8) / 32 + 4, stride = pt_stride(row);
    for (uint32_t shape = 0; shape < 2; ++shape) {
        const uint32_t batch = pt_batch(shape == 0 ? 8u : 16u), least = shape == 0 ? 12u : 8u;
        const uint32_t fixed = pt_fours(n + 1) + 2 * batch * pt_bitmap_words(row, batch, (uint32_t)(acc[kAccMaxSize] >> shift));
        if (row > 0xffffu || offer.words[shape] < fixed) continue;
        uint32_t tiles = umin((offer.words[shape] - fixed) / (2 * stride), umin(kPtMostTiles, t_end));
        if (tiles < least) continue;
        const uint32_t width = (t_end + tiles - 1) / tiles;
        tiles = (t_end + width - 1) / width;
        // (rows are rounded up by as much as seven words and bitmaps by three)
        const uint32_t per_word = 2 * (batch + tiles), spare = offer.words[shape] - fixed - 2 * tiles * stride;
        const uint32_t more = spare / per_word > 8 ? spare / per_word - 8 : 0u;
        const uint32_t roomy = umin(umin(row + more, (2 * live + live / 2) / 32 + 4), 0xffffu);
        acc[kAccTiles] = 1ull | (shape << 1) | (tiles << 8) | (umax(row, roomy) << 16) | ((uint64_t)width << 32);
        return;
    }
}

// The list of request i: what conflicts with it in lifetime and is in none of the rows it reads.
__global__ void __launch_bounds__(256) pt_lists(PlanParams prm, uint32_t t_end)
{
    __shared__ RowLds sh;
    const uint64_t word = prm.acc[kAccTiles];
    if (*prm.status != STALLOC_OK || word == 0) return;
    const PtShape pt(word);
    const uint32_t i = blockIdx.x, n = prm.n, ta = prm.ta[i], tf = prm.tf[i];
    const uint32_t a = ta / pt.width, b = (tf - 1) / pt.width;
    const uint32_t a0 = a * pt.width, a1 = umin(a0 + pt.width, t_end), b0 = b * pt.width, b1 = umin(b0 + pt.width, t_end);
    const uint32_t room = (n - 1 + kRowPad - 1) / kRowPad * kRowPad;
    const uint32_t entries = fill_row(prm.nbr + (size_t)i * room, room, n, sh, [&](uint32_t j) {
        const uint32_t aj = prm.ta[j], fj = prm.tf[j];
        return j != i && aj < tf && ta < fj && !(aj <= a0 && fj >= a1) && !(aj <= b0 && fj >= b1) && !(b > a + 1 && aj < b0 && fj > a1);
    });
    if (threadIdx.x == 0) prm.nbr_chunks[i] = (entries + kRowPad - 1) / kRowPad;       // chunks; the row begins at i * room
}

template <int kWaves, bool kScaledEntries>
__global__ void __launch_bounds__(kWaves * kWave, kWaves == 8 ? 6 : 4) plan_tiled_kernel(PlanParams prm, uint32_t t_end)
{
    using Lds = TiledLds<kWaves>;
    constexpr int kThreads = kWaves * kWave;
    constexpr int kPend = (int)pt_batch(kWaves), kPer = (int)pt_per_wave(kWaves);     // requests of a batch, and of a building wave
    constexpr int kAhead = kWaves == 8 ? 2 : 6;                       // chunks of a list that are fetched a batch before they are used
    static_assert(3 * kPend <= kWave, "three batches lie side by side in the lanes of the settling wave");
    constexpr uint32_t kStage = kPtRefill / kPend * kPend;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t status = read_status(prm.status);
    const uint64_t word = prm.acc[kAccTiles];
    if (word == 0) return;
    const PtShape pt(word);
    if (pt.shape != (kWaves == 8 ? 0u : 1u)) return;
    Lds& sh = *reinterpret_cast<Lds*>(smem);
    if (status_of_workgroup(status, sh.top) != STALLOC_OK) return;
    const uint32_t n = prm.n, shift = (uint32_t)(prm.acc[kAccMode] & 63);
    if (blockIdx.x == 0 && threadIdx.x == 0) const_cast<uint64_t*>(prm.acc)[kAccKernel] = STALLOC_KERNEL_BITMAP | (22u << 8);
    uint32_t* const cells = reinterpret_cast<uint32_t*>(smem + sizeof(Lds));      // [n + 1] placed blocks, see make_cell
    const uint32_t longest = (uint32_t)(prm.acc[kAccMaxSize] >> shift);
    const uint32_t row = pt.row, stride = pt_stride(row), bm_words = pt_bitmap_words(row, kPend, longest);
    uint32_t* const cover = cells + pt_fours(n + 1);                  // [tiles][stride]
    uint32_t* const any = cover + pt.tiles * stride;
    uint32_t* const pool = any + pt.tiles * stride;                   // bitmaps of two batches
    const int lane = lane_id(), wave = wave_id();
    const uint32_t room = (n - 1 + kRowPad - 1) / kRowPad * kRowPad;
    const uint2* const index = reinterpret_cast<const uint2*>(prm.nbr) + lane;    // a chunk: 64 lanes x 4 entries

    for (uint32_t p = blockIdx.x; p < prm.P; p += gridDim.x) {
        if (p >= gridDim.x) {                                         // (uniform)
            // orders that leave many holes: what the first plans lost is not lost for all
            if (threadIdx.x == 0) {
                const uint64_t missed = __hip_atomic_load(&prm.acc[kAccTilesMissed], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sh.top[0] = missed > 16 && 2 * missed > p - gridDim.x ? 1u : 0u;     // (of the plans that are no longer being placed)
                if (sh.top[0]) prm.wide_plans[p] = 1;
            }
            __syncthreads();
            const bool untried = uniform(sh.top[0]) != 0;
            __syncthreads();
            if (untried) continue;
        }
        const uint32_t* order = prm.orders + (size_t)p * n;
        uint64_t* out = prm.offsets ? prm.offsets + (size_t)p * n : nullptr;
        // nothing placed; cell n pads the lists
        for (uint32_t i = threadIdx.x; i < pt_fours(n + 1) + 2 * pt.tiles * stride; i += kThreads) cells[i] = 0;
        uint32_t top = 0;                                             // extent so far, granules
        bool missed = false;                                          // the plan has outgrown the tables
        bool chained = false;                                         // (wave 0) nearly all requests of the last batch had to move
        uint32_t in_vain = 0;                                         // (wave 0) batches to come in which fit_among is not tried

        for (uint32_t r0 = 0; r0 < n; r0 += kStage) {
            const uint32_t staged = n - r0 < kStage ? n - r0 : kStage;
            __syncthreads();                                          // previous refill fully consumed
            if (threadIdx.x < staged) {
                uint32_t i = order[r0 + threadIdx.x];
                if (i >= n) { atomicMax(prm.status, (uint32_t)STALLOC_ERR_BAD_ORDER); i = 0; }
                const uint32_t ta = prm.ta[i], tf = prm.tf[i];
                const uint32_t a = ta / pt.width, b = (tf - 1) / pt.width;
                const uint32_t b1 = umin((b + 1) * pt.width, t_end);
                const uint32_t from = ta == a * pt.width ? a : a + 1, to = tf == b1 ? b + 1 : b;
                sh.rq_id[threadIdx.x] = i;
                sh.rq_s[threadIdx.x] = (uint32_t)(prm.size[i] >> shift);
                sh.rq_ta[threadIdx.x] = ta;
                sh.rq_tf[threadIdx.x] = tf;
                sh.rq_chunks[threadIdx.x] = prm.nbr_chunks[i];
                sh.rq_tiles[threadIdx.x] = a | (b << 8) | (from << 16) | (to << 24);
            }
            __syncthreads();

            // The first chunks of a list are fetched a batch before they are used.  A wave's requests are wave - 1,
            // wave - 1 + (kWaves - 1), ... of the batch.
            uint2 ahead[kPer][kAhead];
            auto place_of = [&](uint32_t batch, int u) -> uint32_t { return batch * kPend + (uint32_t)(wave - 1 + u * (kWaves - 1)); };
            auto fetch_ahead = [&](uint32_t batch) {
                if (wave == 0) return;
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const uint32_t at = place_of(batch, u);
                    if (at >= staged) continue;                       // (uniform)
                    const uint2* list = index + (size_t)uniform(sh.rq_id[at]) * (room / 4);
                    const uint32_t chunks = uniform(sh.rq_chunks[at]);
#pragma unroll
                    for (int c = 0; c < kAhead; ++c)
                        if ((uint32_t)c < chunks) ahead[u][c] = list[c * kWave];
                }
            };
            auto mark_list = [&](uint32_t* bitmap, const uint2& ids) {
                const uint32_t e[4] = {ids.x & 0xffffu, ids.x >> 16, ids.y & 0xffffu, ids.y >> 16};
                uint32_t cell[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    cell[k] = kScaledEntries ? *reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(cells) + e[k])
                                             : cells[e[k]];
                mark_cells(bitmap, cell);
            };
            // build (waves 1 ..): the bitmaps of the wave's requests of the batch, `limit` words each, and their lowest fits
            auto build = [&](uint32_t batch, uint32_t limit) {
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const uint32_t at = place_of(batch, u);
                    if (at >= staged) continue;                       // (uniform)
                    uint32_t* const bitmap = pool + ((batch & 1) * kPend + at - batch * kPend) * bm_words;
                    const uint32_t chunks = uniform(sh.rq_chunks[at]), tiles = uniform(sh.rq_tiles[at]);
                    const uint32_t a = tiles & 0xffu, b = (tiles >> 8) & 0xffu;
                    for (uint32_t w = 4 * lane; w < limit; w += 4 * kWave) {
                        const uint32_t wc = umin(w, stride - 4);      // (a row's words from `row` on are zero)
                        auto four = [&](const uint32_t* at) -> uint4 { return *reinterpret_cast<const uint4*>(at); };
                        const uint4 c0 = four(cover + a * stride + wc), c1 = four(cover + b * stride + wc);
                        uint4 bits = make_uint4(c0.x | c1.x, c0.y | c1.y, c0.z | c1.z, c0.w | c1.w);
                        const uint32_t* from = any + (a + 1) * stride + wc;
                        uint32_t t = a + 1;
                        for (; t + 3 < b; t += 4, from += 4 * stride) {
                            const uint4 r0 = four(from), r1 = four(from + stride), r2 = four(from + 2 * stride), r3 = four(from + 3 * stride);
                            bits.x |= r0.x | r1.x | r2.x | r3.x;
                            bits.y |= r0.y | r1.y | r2.y | r3.y;
                            bits.z |= r0.z | r1.z | r2.z | r3.z;
                            bits.w |= r0.w | r1.w | r2.w | r3.w;
                        }
                        for (; t < b; ++t, from += stride) {
                            const uint4 r0 = four(from);
                            bits.x |= r0.x; bits.y |= r0.y; bits.z |= r0.z; bits.w |= r0.w;
                        }
                        if (w != wc) bits = make_uint4(0u, 0u, 0u, 0u);
                        *reinterpret_cast<uint4*>(bitmap + w) = bits;
                    }
                    __builtin_amdgcn_wave_barrier();                  // (the wave's own LDS: its accesses complete in order)
#pragma unroll
                    for (int c = 0; c < kAhead; ++c)
                        if ((uint32_t)c < chunks) mark_list(bitmap, ahead[u][c]);
                    if (chunks > (uint32_t)kAhead) {
                        const uint2* list = index + (size_t)uniform(sh.rq_id[at]) * (room / 4);
                        uint2 ids = list[kAhead * kWave];
                        for (uint32_t c = kAhead; c < chunks; ++c) {
                            const uint2 now = ids;
                            if (c + 1 < chunks) ids = list[(c + 1) * kWave];
                            mark_list(bitmap, now);
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                    const uint32_t x = first_fit(bitmap, limit, uniform(sh.rq_s[at]));
                    if (lane == 0) sh.cand[batch & 1][at - batch * kPend] = x;
                }
            };
            // settle (wave 0).  Lanes 0 .. 2K-1: the two batches before (settled), lanes 2K .. 3K-1: this batch.
            auto settle = [&](uint32_t batch, uint32_t limit) {
                constexpr int kBefore = 2 * kPend;
                uint32_t* const bitmaps = pool + (batch & 1) * kPend * bm_words;
                const uint32_t first = batch * kPend, nb = umin(staged - first, (uint32_t)kPend);
                uint32_t my_s = 0, my_ta = 0xffffffffu, my_tf = 0, mine = 0;     // empty lifetime: conflicts with nothing
                const bool prev = lane < kBefore && first + (uint32_t)lane >= (uint32_t)kBefore;
                const bool cur = lane >= kBefore && (uint32_t)(lane - kBefore) < nb;
                if (prev || cur) {
                    const uint32_t at = first + (uint32_t)lane - kBefore;
                    my_s = sh.rq_s[at];
                    my_ta = sh.rq_ta[at];
                    my_tf = sh.rq_tf[at];
                    mine = prev ? sh.rq_x[at] : sh.cand[batch & 1][lane - kBefore];
                }
                // Which requests of the batch meet an earlier one in lifetime and address range, as if every candidate
                // stood: independent of one another, so written out for all K.  (Where nearly all did in the batch before,
                // as in an order by time, that is not asked.)
                uint32_t redo = nb < 32 ? (1u << nb) - 1u : ~0u;
                const uint32_t my_end = mine + my_s;
                if (!chained) {
                    redo = 0;
#pragma unroll
                    for (int r = 0; r < kPend; ++r) {
                        const int at = kBefore + r;
                        const uint32_t s = read_lane(my_s, at), ta = read_lane(my_ta, at), tf = read_lane(my_tf, at), x = read_lane(mine, at);
                        const uint64_t hit = lanes_lt(my_ta, tf) & lanes_lt(ta, my_tf) & lanes_lt(mine, x + s) & lanes_lt(x, my_end);
                        if (hit & ((1ull << at) - 1)) redo |= 1u << r;
                    }
                }
                // Those are searched again, in order, with the earlier ones marked in their bitmaps (blocks only remove
                // room, so from the old candidate on); whatever meets the new address is searched again after them.
                // (One that met an old address only is searched for nothing and finds its candidate.)
                uint32_t moved = 0;
                uint64_t view = 0;                                    // 64 granules from the candidate's word on, as the bitmap has them
                const bool many = in_vain == 0 && __builtin_popcount(redo) > kPtFew;
                uint32_t tried = 0, missed_view = 0;
                if (many && cur) {
                    const uint32_t* at = bitmaps + (lane - kBefore) * bm_words;
                    const uint32_t w = mine / 32;
                    view = (w < limit ? at[w] : 0u) | ((uint64_t)(w + 1 < limit ? at[w + 1] : 0u) << 32);
                }
                const uint32_t ones = (1u << my_s) - 1u;              // (sizes are below 32)
                while (redo) {
                    const uint32_t r = (uint32_t)__builtin_ctz(redo);
                    const int at = kBefore + (int)r;
                    const uint32_t s = read_lane(my_s, at), ta = read_lane(my_ta, at), tf = read_lane(my_tf, at), from = read_lane(mine, at);
                    const uint64_t together = lanes_lt(my_ta, tf) & lanes_lt(ta, my_tf), behind = ~1ull << at;
                    const uint64_t earlier = together & ~behind & ~(1ull << at);
                    uint32_t x = many ? fit_among(read_lane(view, at), s, from, earlier, mine, ones) : kNoFit;
                    ++tried;
                    if (x == kNoFit) {
                        ++missed_view;
                        if (lane_in(earlier)) mark_cell(bitmaps + r * bm_words, make_cell(mine, my_s));
                        x = first_fit(bitmaps + r * bm_words, limit, s, from / 32);
                    }
                    mine = set_lane(mine, x, at);
                    moved += x != from ? 1u : 0u;
                    redo &= redo - 1;
                    if (!chained) redo |= (uint32_t)((together & behind & lanes_lt(mine, x + s) & lanes_lt(x, mine + my_s)) >> kBefore);
                }
                chained = 4 * moved >= 3 * (uint32_t)kPend;
                if (many) in_vain = 2 * missed_view > tried ? kPtInVain : 0u;
                else if (in_vain != 0) --in_vain;
                if (cur) {
                    cells[sh.rq_id[first + lane - kBefore]] = make_cell(mine, my_s);
                    sh.rq_x[first + lane - kBefore] = mine;
                }
                const uint32_t reach = umax(top, read_lane(wave_scan_max(cur ? mine + my_s : 0u), kWave - 1));
                if (lane == 0) sh.top[batch & 1] = reach;
            };
            // mark (waves 1 ..): the blocks of the wave's requests of the batch into the tables, a tile per lane
            auto mark = [&](uint32_t batch) {
                if (wave == 0) return;
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const uint32_t at = place_of(batch, u);
                    if (at >= staged) continue;                       // (uniform)
                    const uint32_t tiles = uniform(sh.rq_tiles[at]), cell = make_cell(uniform(sh.rq_x[at]), uniform(sh.rq_s[at]));
                    const uint32_t a = tiles & 0xffu, b = (tiles >> 8) & 0xffu, from = (tiles >> 16) & 0xffu, to = tiles >> 24;
                    if ((uint32_t)lane >= a && (uint32_t)lane <= b) mark_cell(any + (uint32_t)lane * stride, cell);
                    if ((uint32_t)lane >= from && (uint32_t)lane < to) mark_cell(cover + (uint32_t)lane * stride, cell);
                }
            };
            // every block that can get into a bitmap while it is in use ends below the extent known when it is
            // built plus three batches of the longest requests
            auto limit_for = [&](uint32_t top) -> uint32_t { return (top + 3 * kPend * longest) / 32 + 2; };

            // One barrier a batch: while wave 0 settles batch B the others mark batch B - 1 and build batch B + 1.  A
            // bitmap may or may not have seen the blocks of the batch being marked, and has not seen those of the
            // batch being settled: the two batches that `settle` holds its candidates against.
            const uint32_t batches = (staged + kPend - 1) / kPend;
            uint32_t limit = limit_for(top);
            fetch_ahead(0);
            if (wave != 0) build(0, limit);
            fetch_ahead(1);
            __syncthreads();
            for (uint32_t batch = 0; batch <= batches; ++batch) {     // (the last round marks only)
                const uint32_t next_limit = limit_for(top);           // (the extent after batch B - 1)
                if (wave == 0) {
                    if (batch < batches) {
                        __builtin_amdgcn_s_setprio(3);                // (the others wait for it in the end)
                        settle(batch, limit);
                        __builtin_amdgcn_s_setprio(0);
                    }
                } else {
                    if (batch > 0) mark(batch - 1);
                    if (batch + 1 < batches) build(batch + 1, next_limit);
                    fetch_ahead(batch + 2);
                }
                __syncthreads();
                if (batch < batches) top = uniform(sh.top[batch & 1]);
                if (top > 32 * row) { missed = true; break; }         // (uniform)
                limit = next_limit;
            }
            if (missed) break;
            if (out && threadIdx.x < staged) out[sh.rq_id[threadIdx.x]] = (uint64_t)sh.rq_x[threadIdx.x] << shift;
        }
        if (missed) {
            if (threadIdx.x == 0) {
                prm.wide_plans[p] = 1;
                atomicAdd((unsigned long long*)&const_cast<uint64_t*>(prm.acc)[kAccTilesMissed], 1ull);
            }
        } else if (threadIdx.x == 0) {
            prm.wide_plans[p] = 0;
            prm.peaks[p] = (uint64_t)top << shift;
        }
        __syncthreads();                                              // sh read before the next plan clears it
    }
}

// The share of a CU's LDS that a workgroup of the eight-wave shape gets for a trace of n requests.  (Below kPtShort no
// more than two ever run on a CU; the smaller share is what sets a number of tiles that suits short traces: with
// half the LDS, and more tiles, 1500 requests took 545 us instead of 505, 2304 took 870 instead of 800.)
constexpr uint32_t kPtShort = 3072;
static uint32_t pt_workgroups(uint32_t n) { return n <= 2048 ? 4u : n <= 4096 ? 3u : 2u; }

template <int kWaves>
static uint32_t pt_words(size_t lds)
{
    return lds > sizeof(TiledLds<kWaves>) ? (uint32_t)((lds / 512 * 512 - sizeof(TiledLds<kWaves>)) / sizeof(uint32_t)) : 0u;
}

template <int kWaves>
static bool launch_tiled(const PlanParams& prm, uint32_t t_end, uint32_t wgs_per_cu, uint32_t words, const DeviceInfo& di, hipStream_t stream)
{
    auto kernel = entry_shift(prm.n) ? &plan_tiled_kernel<kWaves, true> : &plan_tiled_kernel<kWaves, false>;
    static std::atomic<bool> attr_set[64][2] = {};     // (set twice at worst when threads race)
    if (!attr_set[di.device][entry_shift(prm.n) ? 1 : 0]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)di.lds_per_block) != hipSuccess)
            return false;
        attr_set[di.device][entry_shift(prm.n) ? 1 : 0] = true;
    }
    uint32_t grid = (uint32_t)di.cus * wgs_per_cu;
    if (grid > prm.P) grid = prm.P;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kWaves * kWave), sizeof(TiledLds<kWaves>) + (size_t)words * sizeof(uint32_t), stream, prm,
                       t_end);
    return true;
}

// The variant is part of a call from 3072 requests on, and from 1024 on as long as no more plans are asked for
// than two per CU: with more, the other kernel has twice the waves on a CU for lists that are short already
// (this one / the other: 1152 requests, 64 plans 0.57 / 0.61 ms, 2048 plans 1.38 / 1.33; 2304 requests, 64 plans
// 1.11 / 1.29, 1024 plans 1.70 / 1.61; 4608 requests, 512 plans 2.20 / 3.11).  The timestamps must not be far
// apart (the preparation counts per timestamp).
constexpr uint32_t kPtFrom = 1024;
static uint32_t pt_most_times(uint32_t n) { return 4 * n + 4096; }

bool tiled_plan_possible(uint32_t n, uint32_t t_end, uint32_t P, const DeviceInfo& di)
{
    return n >= kPtFrom && n <= kBmMaxRequests && t_end <= pt_most_times(n) && (n >= kPtShort || P <= 2 * (uint32_t)di.cus);
}

size_t tiled_plan_words(uint32_t n) { return n >= kPtFrom && n <= kBmMaxRequests ? (size_t)pt_most_times(n) + 1 : 0; }

bool launch_plan_tiled(const PlanParams& prm, uint32_t t_end, int32_t* net, const DeviceInfo& di, hipStream_t stream)
{
    const uint32_t wgs = pt_workgroups(prm.n);
    // (shorter traces have few live granules as a rule, and go to plan_bitmap.hip if they do not; a launch less)
    const bool large = prm.n >= kPtShort;
    PtOffer offer = {{pt_words<8>(di.lds_per_block / wgs), large ? pt_words<16>(di.lds_per_block) : 0u}};
    hipLaunchKernelGGL(pt_shape, dim3(1), dim3(1024), 0, stream, prm, t_end, net, offer);
    hipLaunchKernelGGL(pt_lists, dim3(prm.n), dim3(256), 0, stream, prm, t_end);
    return launch_tiled<8>(prm, t_end, wgs, offer.words[0], di, stream) &&
           (!large || launch_tiled<16>(prm, t_end, 1, offer.words[1], di, stream));
}

}  // namespace stalloc
