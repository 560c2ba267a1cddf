// stalloc_plan, occupancy-bitmap variant: the same rule as the sorted-list kernel (Sec. 5.1:
// requests in the given order, each at the lowest address where it conflicts with no earlier
// request of the plan in lifespan and address range at once; extent = max(a + s), Eq. 2), for
// traces whose requests are short when counted in granules.
//
// With g the largest power of two dividing all sizes, every address is a multiple of g and lies
// below the sum of sizes.  When no request is longer than 31 granules and a bitmap of one bit per
// granule of that whole range fits the LDS left over by the plan's table of placed blocks, "which
// addresses are blocked for request r" is such a bitmap, which a single wave searches in a few steps:
//
//   index    Once per call: for every request the list of requests whose lifetime overlaps its
//            own (the potential conflicts of Sec. 5.1 do not depend on the order), rows padded
//            to 256 entries with a dummy request that is never placed.
//   build    One workgroup per plan, K requests per batch, one bitmap per request.  The rows of
//            the K requests are cut into chunks of 256 entries which are dealt out to the waves,
//            so that every wave has the same amount of work whatever the row lengths.  A wave
//            looks every neighbour of its chunk up in the plan's table of placed blocks (LDS,
//            4 bytes per request: address and the two word masks in a compressed form, 0 = not
//            placed yet) and ORs the neighbour's granules into the bitmap of the request the
//            chunk belongs to (LDS atomics: any wave may add to any bitmap).
//   search   Wave r finds the first run of size_r zero bits in bitmap r: the lowest fit against
//            what the bitmap holds.
//   settle   Wave 0 takes the K requests in order.  A candidate stands unless a block the bitmap
//            may have missed -- one of the batch before, or one settled earlier in the same
//            batch -- overlaps it in lifetime and in address range; only then are those blocks
//            ORed into the request's bitmap and the search repeated.  Adding blocks can only
//            remove free runs, so an untouched candidate is still the lowest.
//
// Batches are software-pipelined over two halves of the bitmap pool: batch B is settled while
// batch B + 1 is built.  Nothing is sorted or merged and no placement needs a second pass.
#include "bitmap_cells.h"
#include "host_util.h"
#include "plan_params.h"
#include "wave.h"

namespace stalloc {

#ifndef STALLOC_BITMAP_REFILL
#define STALLOC_BITMAP_REFILL 16      // requests fetched per refill, per wave of the workgroup
#endif
#ifndef STALLOC_BITMAP_SHARES
#define STALLOC_BITMAP_SHARES 2
#endif
constexpr int kRefillPerWave = STALLOC_BITMAP_REFILL;   // (the pipeline of batches drains at every refill)
constexpr uint32_t kShares = STALLOC_BITMAP_SHARES; // chunks a building wave takes for every one wave 0 takes
constexpr int kBmWords = 1056;           // a pool of twice this many words is asked for before workgroups share a CU
template <int kWaves>
struct BitmapLds {
    static constexpr int kBmBatch = kRefillPerWave * kWaves;     // 128 requests with eight waves, 256 with sixteen
    uint32_t rq_id[kBmBatch];
    uint32_t rq_s[kBmBatch];             // size in granules
    uint32_t rq_ta[kBmBatch];
    uint32_t rq_tf[kBmBatch];
    uint32_t rq_x[kBmBatch];             // address in granules
    uint32_t rq_row[kBmBatch];           // first chunk of the request's row of the index
    uint32_t rq_chunks[kBmBatch];        // chunks in that row
    uint32_t cand[kWaves];               // lowest fit of each request of the batch against what its bitmap holds
    uint32_t top;                        // extent so far, granules
    uint32_t pad[3];
};
// Behind it in LDS: the plan's table of placed blocks (n + 1 words) and the pool the bitmaps are
// carved from, one half per batch in flight.  A bitmap is only as long as the plan's extent
// needs, so a half holds a full batch of them as long as the extent is moderate, and fewer
// (smaller batches) beyond that; the rule that admits a trace makes sure it always holds one.

// ---------------------------------------------------------------------------------------------
// Lifetime-conflict index.  Row i holds nbr_chunks[i] chunks of 256 entries; an entry is j for a request
// j != i with t_alloc_j < t_free_i and t_alloc_i < t_free_j, or n (a dummy that is never placed) -- stored as
// 4 * j, the byte offset into the plan's table, while 4 * n fits 16 bits (the build phase then needs one
// instruction less per lookup).
__device__ __forceinline__ bool plans_wanted(const PlanParams& prm)
{
    return bitmap_shape(prm.acc[kAccMode], prm.acc[kAccGranules], prm.bitmap_pool_words) >= 0 &&
           (prm.acc[kAccTiles] == 0 || prm.acc[kAccTilesMissed] != 0);      // (nothing left to place, see plan_tiled.hip)
}
__device__ __forceinline__ bool index_wanted(const PlanParams& prm) { return *prm.status == STALLOC_OK && plans_wanted(prm); }

// (Rows have the room of the longest one possible, so that nobody has to count them first: two launches less.)
__host__ __device__ inline uint32_t row_chunks(uint32_t n) { return (n - 1 + kRowPad - 1) / kRowPad; }

__global__ void __launch_bounds__(256) nbr_fill(PlanParams prm)
{
    __shared__ RowLds sh;
    if (!index_wanted(prm)) return;
    const uint32_t i = blockIdx.x, ta = prm.ta[i], tf = prm.tf[i], room = row_chunks(prm.n) * kRowPad;
    const uint32_t entries = fill_row(prm.nbr + (size_t)i * room, room, prm.n, sh,
                                      [&](uint32_t j) { return j != i && prm.ta[j] < tf && ta < prm.tf[j]; });
    if (threadIdx.x == 0) prm.nbr_chunks[i] = (entries + kRowPad - 1) / kRowPad;
}

// ---------------------------------------------------------------------------------------------

// Inclusive prefix sum inside each row of 16 lanes.
__device__ __forceinline__ uint32_t row_scan_add(uint32_t v)
{
    v += __builtin_amdgcn_update_dpp(0u, v, kDppRowShr1, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, kDppRowShr2, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, kDppRowShr4, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, kDppRowShr8, 0xf, 0xf, false);
    return v;
}

// (eight-wave shape: 8 waves per SIMD = 64 VGPRs at most, so that four workgroups share a CU)
template <int kWaves, bool kScaledEntries>
__global__ void __launch_bounds__(kWaves * kWave, kWaves == 8 ? 8 : 4) plan_bitmap_kernel(PlanParams prm)
{
    using Lds = BitmapLds<kWaves>;
    constexpr int kThreads = kWaves * kWave;
    constexpr int kShape = kWaves == 8 ? 0 : 1;
    constexpr int kAhead = kWaves == 8 ? 8 : 12;      // chunks per wave and batch whose index entries are fetched ahead
    static_assert(bitmap_shape_waves(kShape) == (uint32_t)kWaves, "shape table and instantiation disagree");
    extern __shared__ __align__(16) unsigned char smem[];
    Lds& sh = *reinterpret_cast<Lds*>(smem);
    uint32_t* cells = reinterpret_cast<uint32_t*>(smem + sizeof(Lds));     // [n + 1] placed blocks, see make_cell
    uint32_t* pool = cells + (prm.n + 1);
    const uint32_t n = prm.n;

    const uint32_t status = read_status(prm.status);
    if (!plans_wanted(prm)) return;
    if (bitmap_shape(prm.acc[kAccMode], prm.acc[kAccGranules], prm.bitmap_pool_words) != kShape) return;
    if (status_of_workgroup(status, &sh.top) != STALLOC_OK) return;
    const bool some = prm.acc[kAccTiles] != 0;         // only the plans that outgrew the tables of the tiled variant
    const uint32_t shift = (uint32_t)(prm.acc[kAccMode] & 63);
    if (blockIdx.x == 0 && threadIdx.x == 0) const_cast<uint64_t*>(prm.acc)[kAccKernel] = STALLOC_KERNEL_BITMAP | (22u << 8);
    const uint32_t pool_words = prm.bitmap_pool_words[kShape];
    const uint32_t half_words = pool_words / 2;        // two batches are in flight, each in its half of the pool
    // the rule above keeps every address of a well-formed plan at or below `highest`; a malformed
    // order row (repeated requests) is clamped to it so that a bitmap never outgrows its half
    const uint32_t highest = 32u * (half_words - 2 * kWaves - 5) + 31u;
    const int lane = lane_id(), wave = (int)uniform((uint32_t)wave_id());
    const uint2* index = reinterpret_cast<const uint2*>(prm.nbr) + lane;   // a chunk: 64 lanes x 4 entries

    for (uint32_t p = blockIdx.x; p < prm.P; p += gridDim.x) {
        if (some && !prm.wide_plans[p]) continue;             // (uniform)
        const uint32_t* order = prm.orders + (size_t)p * n;
        uint64_t* out = prm.offsets ? prm.offsets + (size_t)p * n : nullptr;
        for (uint32_t i = threadIdx.x; i <= n; i += kThreads) cells[i] = 0;     // nothing placed; cell n pads the rows
        if (threadIdx.x == 0) sh.top = 0;

        for (uint32_t r0 = 0; r0 < n; r0 += Lds::kBmBatch) {
            const uint32_t staged = n - r0 < (uint32_t)Lds::kBmBatch ? n - r0 : (uint32_t)Lds::kBmBatch;
            __syncthreads();                                  // previous refill fully consumed
            if (threadIdx.x < staged) {
                uint32_t i = order[r0 + threadIdx.x];
                if (i >= n) { atomicMax(prm.status, (uint32_t)STALLOC_ERR_BAD_ORDER); i = 0; }
                sh.rq_id[threadIdx.x] = i;
                sh.rq_s[threadIdx.x] = (uint32_t)(prm.size[i] >> shift);
                sh.rq_ta[threadIdx.x] = prm.ta[i];
                sh.rq_tf[threadIdx.x] = prm.tf[i];
                sh.rq_row[threadIdx.x] = i * row_chunks(n);
                sh.rq_chunks[threadIdx.x] = prm.nbr_chunks[i];
            }
            __syncthreads();

            // A batch: requests first .. first + nb - 1 of the refill, their bitmaps `stride` words apart
            // and `limit` words long in one half of the pool.  A batch is sized when its half is cleared:
            // two batches are in flight, so every block that can exist while it is in use ends below
            // the extent at that moment plus 2 * kWaves of the longest requests.
            struct Batch { uint32_t first, nb, limit, stride; };
            auto size_batch = [&](uint32_t first) -> Batch {
                Batch b;
                b.first = first;
                b.limit = uniform(sh.top) / 32 + 2 * kWaves + 2;
                b.stride = b.limit | 1u;
                uint32_t fit = half_words / b.stride;             // >= 1
                if (fit > (uint32_t)kWaves) fit = kWaves;
                b.nb = first >= staged ? 0u : (staged - first < fit ? staged - first : fit);
                return b;
            };
            // Which chunks a wave takes: wave 0 settles the previous batch while the others already
            // build, so it gets a smaller share -- of every kShares * (kWaves - 1) + 1 chunks, kShares
            // go to each of the waves 1 .. kWaves - 1 and the last one to wave 0.
            constexpr uint32_t kPeriod = kShares * (kWaves - 1) + 1;
            auto chunk_of = [&](uint32_t j) -> uint32_t {          // the wave's j-th chunk (ascending in j)
                return wave == 0 ? j * kPeriod + (kPeriod - 1)
                                 : (j / kShares) * kPeriod + (j % kShares) * (kWaves - 1) + (uint32_t)(wave - 1);
            };
            auto chunks_of_wave = [&](uint32_t total) -> uint32_t { // how many of `total` chunks are the wave's
                const uint32_t full = total / kPeriod, rest = total % kPeriod;
                if (wave == 0) return full;
                uint32_t c = full * kShares;
                for (uint32_t k = 0; k < kShares; ++k) c += k * (kWaves - 1) + (uint32_t)(wave - 1) < rest ? 1u : 0u;
                return c;
            };
            // The rows of a batch, cut into chunks and numbered through.  Lane q < 16 describes the row
            // of request q of the batch; `mine` = how many of the chunks are this wave's.
            struct Rows { uint32_t row, chunks, end, total, mine; };
            auto rows_of = [&](const Batch& b) -> Rows {
                Rows r = {0, 0, 0, 0, 0};
                if (lane < (int)b.nb) { r.row = sh.rq_row[b.first + lane]; r.chunks = sh.rq_chunks[b.first + lane]; }
                r.end = row_scan_add(r.chunks);                   // (nb <= 16: one DPP row)
                r.total = read_lane(r.end, 15);
                r.mine = chunks_of_wave(r.total);
                return r;
            };
            // chunk f belongs to request q = number of rows that end at or before f
            auto locate = [&](const Rows& r, uint32_t f, uint32_t& q) -> const uint2* {
                q = (uint32_t)__builtin_popcountll(lanes_ge(f, r.end) & 0xffffull);
                const uint32_t at = read_lane(r.row, (int)q) + f - (read_lane(r.end, (int)q) - read_lane(r.chunks, (int)q));
                return index + (size_t)at * (kRowPad / 4);
            };
            // The index entries of a wave's first kAhead chunks of a batch are fetched when the batch is
            // sized, a whole batch before they are used: the index is far larger than the L2 and a
            // fetch takes about as long as a chunk takes to process.
            uint2 ahead[kAhead];
            uint32_t ahead_q[kAhead];
            auto fetch_ahead = [&](const Rows& r) {
#pragma unroll
                for (int j = 0; j < kAhead; ++j) {
                    ahead_q[j] = 0;
                    if ((uint32_t)j < r.mine) ahead[j] = *locate(r, chunk_of((uint32_t)j), ahead_q[j]);
                }
            };
            auto lookup = [&](const uint2& ids, uint32_t (&cell)[4]) {
                const uint32_t e[4] = {ids.x & 0xffffu, ids.x >> 16, ids.y & 0xffffu, ids.y >> 16};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    cell[k] = kScaledEntries ? *reinterpret_cast<const uint32_t*>(reinterpret_cast<const unsigned char*>(cells) + e[k])
                                             : cells[e[k]];
            };
            auto clear = [&](uint32_t* bitmaps, const Batch& b) {
                if ((uint32_t)wave < b.nb)
                    for (uint32_t w = lane; w < b.limit; w += kWave) bitmaps[(uint32_t)wave * b.stride + w] = 0;
            };
            // build: table lookups of one chunk are in flight while the previous one is marked
            auto build = [&](uint32_t* bitmaps, const Batch& b, const Rows& rows) {
                uint32_t cell[4] = {0, 0, 0, 0}, looked[4] = {0, 0, 0, 0};
                if (rows.mine) lookup(ahead[0], cell);
#pragma unroll
                for (int j = 0; j < kAhead; ++j) {
                    if ((uint32_t)j < rows.mine) {
                        if (j + 1 < kAhead && (uint32_t)j + 1 < rows.mine) lookup(ahead[j + 1 < kAhead ? j + 1 : j], looked);
                        mark_cells(bitmaps + ahead_q[j] * b.stride, cell);
#pragma unroll
                        for (int k = 0; k < 4; ++k) cell[k] = looked[k];
                    }
                }
                for (uint32_t j = kAhead; j < rows.mine; ++j) {                           // (long rows only)
                    uint32_t q;
                    const uint2 ids = *locate(rows, chunk_of(j), q);
                    lookup(ids, cell);
                    mark_cells(bitmaps + q * b.stride, cell);
                }
            };
            // search: lowest fit of request q of the batch against what its bitmap holds
            auto search = [&](uint32_t* bitmaps, const Batch& b) {
                if ((uint32_t)wave < b.nb) {
                    const uint32_t x = first_fit(bitmaps + (uint32_t)wave * b.stride, b.limit, uniform(sh.rq_s[b.first + wave]));
                    if (lane == 0) sh.cand[wave] = x;
                }
            };
            // settle (one wave): the requests of the batch in order.  The bitmaps hold every block
            // placed before the batch except possibly those of the batch just before it (they were
            // being settled while these bitmaps were built).  A candidate stands unless one of those,
            // or a request settled earlier in this batch, overlaps it in lifetime and in address
            // range; only then are those blocks ORed into the request's bitmap and the search
            // repeated (adding blocks only removes free runs; ORing a block twice changes nothing).
            // Lanes 0 .. kWaves-1: the batch before (settled); lanes kWaves .. : this batch.
            auto settle = [&](uint32_t* bitmaps, const Batch& b, uint32_t nb_prev) {
                uint32_t my_s = 0, my_ta = 0xffffffffu, my_tf = 0, mine = 0;     // empty lifetime: conflicts with nothing
                const bool prev = lane < kWaves && (uint32_t)(kWaves - lane) <= nb_prev;    // request first - (kWaves - lane)
                const bool cur = lane >= kWaves && (uint32_t)(lane - kWaves) < b.nb;
                if (prev || cur) {
                    const uint32_t at = b.first + (uint32_t)lane - kWaves;
                    my_s = sh.rq_s[at];
                    my_ta = sh.rq_ta[at];
                    my_tf = sh.rq_tf[at];
                    mine = prev ? sh.rq_x[at] : sh.cand[lane - kWaves];
                }
                uint32_t top = sh.top;
                for (uint32_t r = 0; r < b.nb; ++r) {
                    const int at = kWaves + (int)r;
                    const uint32_t s = read_lane(my_s, at), ta = read_lane(my_ta, at), tf = read_lane(my_tf, at);
                    uint32_t x = read_lane(mine, at);
                    const bool rival = lane < at && my_ta < tf && ta < my_tf;
                    if (__builtin_amdgcn_ballot_w64(rival && mine < x + s && x < mine + my_s)) {
                        if (rival) mark_cell(bitmaps + r * b.stride, make_cell(mine, my_s));
                        x = first_fit(bitmaps + r * b.stride, b.limit, s);
                    }
                    if (x > highest) x = highest;                          // only reachable with a malformed order row
                    if (lane == at) mine = x;
                    top = umax(top, x + s);
                }
                if (cur) {
                    cells[sh.rq_id[b.first + lane - kWaves]] = make_cell(mine, my_s);
                    sh.rq_x[b.first + lane - kWaves] = mine;
                }
                if (lane == 0) sh.top = top;
            };

            // Software pipeline over the batches of the refill: while wave 0 settles batch B in one
            // half of the pool, all waves (wave 0 once it is done) build the bitmaps of batch B + 1 in
            // the other half; then B + 1 is searched, and the half of B is cleared for B + 2.
            uint32_t* half[2] = {pool, pool + half_words};
            int h = 0;
            Batch cur = size_batch(0);
            Rows rows = rows_of(cur);
            fetch_ahead(rows);
            clear(half[0], cur);
            __syncthreads();
            build(half[0], cur, rows);
            Batch nxt = size_batch(cur.nb);
            if (nxt.nb) {
                rows = rows_of(nxt);
                fetch_ahead(rows);
                clear(half[1], nxt);
            }
            __syncthreads();
            search(half[0], cur);
            __syncthreads();
            uint32_t nb_prev = 0;
            while (cur.nb) {
                if (wave == 0) settle(half[h], cur, nb_prev);
                if (nxt.nb) build(half[h ^ 1], nxt, rows);
                __syncthreads();
                Batch after = {0, 0, 0, 0};
                if (nxt.nb) {
                    search(half[h ^ 1], nxt);
                    after = size_batch(nxt.first + nxt.nb);
                    if (after.nb) {
                        rows = rows_of(after);
                        fetch_ahead(rows);
                        clear(half[h], after);
                    }
                    __syncthreads();
                }
                nb_prev = cur.nb;
                cur = nxt;
                nxt = after;
                h ^= 1;
            }
            if (out && threadIdx.x < staged) out[sh.rq_id[threadIdx.x]] = (uint64_t)sh.rq_x[threadIdx.x] << shift;
        }
        if (threadIdx.x == 0) prm.peaks[p] = (uint64_t)sh.top << shift;
        __syncthreads();                                      // sh.top read before the next plan clears it
    }
}

// Workgroups per CU of the eight-wave shape for a trace of n requests, and the words of its
// bitmap pool: as many workgroups as leave each a pool of 2 * kBmWords words.  0 = none.
static uint32_t shared_cu_residency(uint32_t n, const DeviceInfo& di, uint32_t* pool_words)
{
    const size_t fixed = sizeof(BitmapLds<8>) + ((size_t)n + 1) * sizeof(uint32_t);
    for (uint32_t wgs = 4; wgs >= 2; --wgs) {
        const size_t budget = di.lds_per_block / wgs / 512 * 512;       // LDS is handed out in 512-byte pieces
        if (budget < fixed + 2 * (size_t)kBmWords * sizeof(uint32_t)) continue;
        *pool_words = (uint32_t)((budget - fixed) / sizeof(uint32_t));
        return wgs;
    }
    return 0;
}

bool bitmap_plan_shapes(uint32_t n, const DeviceInfo& di, uint32_t (&pool_words)[kBitmapShapes])
{
    pool_words[0] = pool_words[1] = 0;
    if (n > kBmMaxRequests) return false;
    shared_cu_residency(n, di, &pool_words[0]);
    const size_t fixed = sizeof(BitmapLds<16>) + ((size_t)n + 1) * sizeof(uint32_t);
    if (di.lds_per_block >= fixed + (size_t)kBmWords * sizeof(uint32_t))
        pool_words[1] = (uint32_t)((di.lds_per_block - fixed) / sizeof(uint32_t));
    return pool_words[0] != 0 || pool_words[1] != 0;
}

size_t bitmap_index_entries(uint32_t n)
{
    return (size_t)n * row_chunks(n) * kRowPad;
}

template <int kWaves>
static bool launch_shape(const PlanParams& prm, uint32_t wgs_per_cu, uint32_t pool_words, const DeviceInfo& di,
                         hipStream_t stream)
{
    auto kernel = entry_shift(prm.n) ? &plan_bitmap_kernel<kWaves, true> : &plan_bitmap_kernel<kWaves, false>;
    const size_t lds = sizeof(BitmapLds<kWaves>) + ((size_t)prm.n + 1 + pool_words) * sizeof(uint32_t);
    static std::atomic<bool> attr_set[64][2] = {};     // (set twice at worst when threads race)
    if (!attr_set[di.device][entry_shift(prm.n) ? 1 : 0]) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)di.lds_per_block) != hipSuccess)
            return false;
        attr_set[di.device][entry_shift(prm.n) ? 1 : 0] = true;
    }
    uint32_t grid = (uint32_t)di.cus * wgs_per_cu;
    if (grid > prm.P) grid = prm.P;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kWaves * kWave), lds, stream, prm);
    return true;
}

// Enqueues the index build and every shape of the placement kernel that prm.bitmap_pool_words names.
bool launch_plan_bitmap(const PlanParams& prm, const DeviceInfo& di, hipStream_t stream)
{
    hipLaunchKernelGGL(nbr_fill, dim3(prm.n), dim3(256), 0, stream, prm);
    bool ok = true;
    if (prm.bitmap_pool_words[0]) {
        uint32_t pool_words = 0;
        const uint32_t wgs = shared_cu_residency(prm.n, di, &pool_words);
        ok = ok && wgs != 0 && pool_words == prm.bitmap_pool_words[0] && launch_shape<8>(prm, wgs, pool_words, di, stream);
    }
    if (prm.bitmap_pool_words[1]) ok = ok && launch_shape<16>(prm, 1, prm.bitmap_pool_words[1], di, stream);
    return ok;
}

}  // namespace stalloc
