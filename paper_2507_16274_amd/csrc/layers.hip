// stalloc_memory_layers: memory-layer construction for the HomoSize groups of a trace
// (Sec. 5.1, HomoSize Group Planning, Algorithm 1), and stalloc_expand_layers.
//
// A HomoSize group holds the requests of one size; requests of a group whose lifetimes do not
// overlap share one range of that size, a memory-layer.  The group's requests are taken by
// allocation time; each goes to the free layer whose last request ended latest (lifetimes are
// half-open: a layer released at t is free at t), the one opened first among equals; if none is
// free a new layer is opened.  Layers are numbered group by group in descending size, inside
// a group in the order in which they were opened.
//
//   sort     Requests are sorted by (size descending, allocation time, request number): tiles
//            of 1024 keys sorted in LDS (bitonic network), merged four runs at a time (an
//            element's place is its place in its own run plus the numbers of elements of the
//            partner runs that sort before it, found by binary search).
//   groups   A group starts where the size changes in the sorted sequence; exclusive sums of
//            the start flags number the groups.
//   match    Groups of 256 requests or more: the construction as a matching of releases and
//            allocations, all requests at once (see ly_match).
//   build    The other groups: one wave per group walks its requests in order -- the construction is
//            sequential by nature, the groups are what runs in parallel.  The ends of the
//            first 1024 layers of the group live in registers (lane = layer mod 64); finding
//            the free layer with the latest end is a 32-bit wave maximum (DPP) and a ballot,
//            in code chosen once per 64 requests for the registers they can come to use.
//            Further layers, if a group ever needs them, are kept in memory.
//   number   Exclusive sums of the groups' layer counts give every group its first layer.
//   emit     layer_of per request; size, first allocation and last release per layer.
#include "host_util.h"
#include "sort_keys.h"
#include "wave.h"

namespace stalloc {

constexpr int kLyTile = kSortTile;
constexpr int kLyRegs = 16;                      // 64 layers per register: 1024 layers of a group in registers
static_assert(kLyRegs == 16, "ly_build dispatches on one to sixteen registers in use");

// One tile of 1024 requests per workgroup, sorted in LDS; slot e past the end holds a key behind
// every real one, (~0, ~0 << 32 | e) (sizes are > 0, so no real key starts with ~0).
__global__ void __launch_bounds__(kSortThreads)
ly_sort_tiles(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, uint32_t n, ulonglong2* keys,
              const uint32_t* status)
{
    __shared__ ulonglong2 k[kLyTile];
    if (*status != STALLOC_OK) return;
    for (uint32_t t = threadIdx.x; t < (uint32_t)kLyTile; t += kSortThreads) {
        const uint32_t i = blockIdx.x * kLyTile + t;
        // (size descending, allocation time, request number) as two ascending 64-bit words
        k[t] = i < n ? make_ulonglong2(~size[i], ((uint64_t)ta[i] << 32) | i) : filler_key(i);
    }
    sort_tile(k, keys_of_tile(blockIdx.x * kLyTile, n));
    for (uint32_t t = threadIdx.x; t < (uint32_t)kLyTile; t += kSortThreads) keys[blockIdx.x * kLyTile + t] = k[t];
}

// sorted[k] = request at sorted position k; flag[k] = 1 where a group starts; no layers in any group yet.
__global__ void __launch_bounds__(256)
ly_ids(const ulonglong2* __restrict__ keys, uint32_t n, uint32_t* sorted, uint32_t* flag, uint32_t* group_layers, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        const uint32_t i = (uint32_t)keys[k].y;
        sorted[k] = i < n ? i : 0u;                           // (the first n sorted keys are the real ones)
        flag[k] = (k == 0 || keys[k].x != keys[k - 1].x) ? 1u : 0u;
        group_layers[k] = 0;
    }
}

// Exclusive sums of m 32-bit values; total[0] receives the sum of all.  Up to kScanSmall values in one launch of one
// workgroup, four values a thread and step; beyond, in three: sums of 1024-value chunks, their exclusive
// sums (one workgroup), and the values' own.
constexpr int kScanChunk = 1024;
constexpr uint32_t kScanSmall = 16384;

__global__ void __launch_bounds__(1024)
scan_small(const uint32_t* __restrict__ in, uint32_t m, uint32_t* out, uint32_t* total, const uint32_t* status)
{
    __shared__ uint32_t part[16];
    if (*status != STALLOC_OK) return;
    uint32_t carry = 0;
    for (uint32_t k0 = 0; k0 < m; k0 += 4096) {
        const uint32_t k = k0 + 4 * threadIdx.x;
        uint32_t v[4], mine = 0;
        for (int u = 0; u < 4; ++u) { v[u] = k + u < m ? in[k + u] : 0u; mine += v[u]; }
        const uint32_t incl = wave_scan_add(mine);
        __syncthreads();                                      // (the step before has read part[])
        if (lane_id() == kWave - 1) part[wave_id()] = incl;
        __syncthreads();
        uint32_t before = carry + incl - mine;
        for (int w = 0; w < 16; ++w) { if (w < wave_id()) before += part[w]; carry += part[w]; }
        for (int u = 0; u < 4; ++u) { if (k + u < m) out[k + u] = before; before += v[u]; }
    }
    if (threadIdx.x == 0) total[0] = carry;
}

__global__ void __launch_bounds__(256)
scan_chunk_sums(const uint32_t* __restrict__ in, uint32_t m, uint32_t* chunk_sum, const uint32_t* status)
{
    __shared__ uint32_t part[4];
    if (*status != STALLOC_OK) return;
    const uint32_t base = blockIdx.x * kScanChunk;
    uint32_t s = 0;
    for (uint32_t j = threadIdx.x; j < (uint32_t)kScanChunk; j += 256)
        if (base + j < m) s += in[base + j];
    s = wave_sum32(s);
    if (lane_id() == 0) part[wave_id()] = s;
    __syncthreads();
    if (threadIdx.x == 0) chunk_sum[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

__global__ void __launch_bounds__(256)
scan_of_chunk_sums(uint32_t* chunk_sum, uint32_t chunks, uint32_t* total, const uint32_t* status)
{
    __shared__ uint32_t part[4];
    __shared__ uint32_t carry;
    if (*status != STALLOC_OK) return;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (uint32_t c0 = 0; c0 < chunks; c0 += 256) {
        const uint32_t c = c0 + threadIdx.x;
        const uint32_t v = c < chunks ? chunk_sum[c] : 0u;
        // inclusive sums inside the wave, then across the four waves
        uint32_t incl = v;
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr1, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr2, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr4, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr8, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowBcast15, 0xa, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowBcast31, 0xc, 0xf, false);
        if (lane_id() == kWave - 1) part[wave_id()] = incl;
        __syncthreads();
        uint32_t before_wave = carry;
        for (int w = 0; w < wave_id(); ++w) before_wave += part[w];
        if (c < chunks) chunk_sum[c] = before_wave + incl - v;
        __syncthreads();
        if (threadIdx.x == 0) carry += part[0] + part[1] + part[2] + part[3];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

__global__ void __launch_bounds__(256)
scan_apply(const uint32_t* __restrict__ in, uint32_t m, const uint32_t* __restrict__ chunk_sum, uint32_t* out,
           const uint32_t* status)
{
    __shared__ uint32_t part[4];
    if (*status != STALLOC_OK) return;
    const uint32_t base = blockIdx.x * kScanChunk;
    uint32_t run = chunk_sum[blockIdx.x];
    for (uint32_t j0 = 0; j0 < (uint32_t)kScanChunk; j0 += 256) {                 // (uniform trip count)
        const uint32_t j = base + j0 + threadIdx.x;
        const uint32_t v = j < m ? in[j] : 0u;
        uint32_t incl = v;
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr1, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr2, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr4, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowShr8, 0xf, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowBcast15, 0xa, 0xf, false);
        incl += __builtin_amdgcn_update_dpp(0u, incl, kDppRowBcast31, 0xc, 0xf, false);
        __syncthreads();                                                        // (part[] of the previous round consumed)
        if (lane_id() == kWave - 1) part[wave_id()] = incl;
        __syncthreads();
        uint32_t before_wave = run;
        for (int w = 0; w < wave_id(); ++w) before_wave += part[w];
        if (j < m) out[j] = before_wave + incl - v;
        run += part[0] + part[1] + part[2] + part[3];
    }
}

// group_start[g] = sorted position at which group g starts (g = number of flags before k).
__global__ void __launch_bounds__(256)
ly_group_starts(const uint32_t* __restrict__ flag, const uint32_t* __restrict__ flags_before, uint32_t n,
                uint32_t* group_start, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
        if (flag[k]) group_start[flags_before[k]] = k;
}

struct LyBuild {
    const uint32_t* ta;
    const uint32_t* tf;
    const uint32_t* sorted;          // [n] request numbers by (size descending, allocation time, number)
    const uint32_t* group_start;     // [groups]
    const uint32_t* n_groups;        // [1]
    uint32_t* local;                 // [n] by sorted position: the request's layer inside its group
    uint32_t* first_ts;              // [n] slot group_start + l: allocation time of layer l's first request
    uint32_t* ends;                  // [n] slot group_start + l: free time of layer l's last request
    uint32_t* group_layers;          // [groups] layers of the group
    const uint32_t* status;
    uint32_t n;
};

// Groups with at most this many registers of layers are tested for being idle: the groups of small
// transient tensors, a few layers each, are idle between most of their requests; those with hundreds
// of layers hardly ever (and the number of registers in use only grows, so once a group is past
// the limit the record below is no longer needed).
constexpr int kLyIdleRegs = 2;

// The group's layer that was released last (the lowest-numbered of several released together): when a
// request starts at or after that release, every layer of the group is free and this is the one it
// takes -- no search.  Kept up to date as requests are appended to layers.
struct LastReleased {
    uint32_t end, layer;             // (uniform)
    __device__ __forceinline__ void appended(uint32_t te, uint32_t to_layer)
    {
        if (te > end) { end = te; layer = to_layer; }
        else if (te == end && to_layer < layer) layer = to_layer;
    }
};

// One request of a group whose layers all sit in the first kRegs registers (a layer it opens
// included): returns its layer and makes the request the layer's last one.  `layers` is uniform.
template <int kRegs>
__device__ __forceinline__ uint32_t take_layer(uint32_t (&end_of)[kLyRegs], uint32_t ts, uint32_t te, uint32_t layers,
                                               const LastReleased& last)
{
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t layer = layers;                                              // a new one unless a free layer is found
    if (kRegs <= kLyIdleRegs && layers != 0 && ts >= last.end) {
        layer = last.layer;                                               // the whole group is idle
    } else {
        // latest end among the free layers (an end is a free time, hence >= 1; 0 = not opened)
        uint32_t latest = 0;
#pragma unroll
        for (int r = 0; r < kRegs; ++r) latest = umax(latest, end_of[r] <= ts ? end_of[r] : 0u);
        const uint32_t best = __builtin_amdgcn_readlane(wave_scan_max(latest), kWave - 1);
        if (best != 0) {
            bool found = false;
#pragma unroll
            for (int r = 0; r < kRegs; ++r) {
                const uint64_t hit = __builtin_amdgcn_ballot_w64(end_of[r] == best);
                if (!found && hit) { layer = (uint32_t)r * kWave + (uint32_t)__builtin_ctzll(hit); found = true; }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kRegs; ++r) end_of[r] = ((uint32_t)r == layer / kWave && lane == layer % kWave) ? te : end_of[r];
    return layer;
}

// The (up to 64) requests a wave has loaded, lane q holding request q, taken one by one while all
// layers the group can have by the end of the block sit in the first kRegs registers.  Returns the
// layer of the request this lane loaded; `layers` and `last` are kept up to date.
template <int kRegs>
__device__ __forceinline__ uint32_t take_block(uint32_t (&end_of)[kLyRegs], uint32_t ts_k, uint32_t te_k, int members,
                                               uint32_t& layers, LastReleased& last, uint32_t* first_ts)
{
    const int lane = lane_id();
    uint32_t mine = 0;
    uint32_t opened = layers;                                             // (uniform)
    LastReleased lr = last;
    for (int q = 0; q < members; ++q) {
        const uint32_t ts = __builtin_amdgcn_readlane(ts_k, q), te = __builtin_amdgcn_readlane(te_k, q);
        const uint32_t layer = take_layer<kRegs>(end_of, ts, te, opened, lr);
        if (layer == opened) {
            if (lane == 0) first_ts[opened] = ts;
            ++opened;
        }
        if (kRegs <= kLyIdleRegs) lr.appended(te, layer);
        if (lane == q) mine = layer;
    }
    layers = opened;
    last = lr;
    return mine;
}

__global__ void __launch_bounds__(256) ly_build(LyBuild g)
{
    if (*g.status != STALLOC_OK) return;
    const int lane = lane_id();
    const uint32_t groups = *g.n_groups;
    // (the wave's number, the same in all its lanes, as a scalar: the loops below then run on scalar
    // counters and branches instead of lane masks)
    const uint32_t first_group = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (uint32_t)wave_id());
    for (uint32_t grp = first_group; grp < groups; grp += gridDim.x * 4) {
        if (g.group_layers[grp] != 0) continue;                       // ly_match has built it
        const uint32_t s = g.group_start[grp];
        const uint32_t e = grp + 1 < groups ? g.group_start[grp + 1] : g.n;
        uint32_t end_of[kLyRegs];        // lane holds the ends of layers lane, 64 + lane, ...; 0 = not opened
#pragma unroll
        for (int r = 0; r < kLyRegs; ++r) end_of[r] = 0;
        uint32_t layers = 0;             // (uniform) layers opened so far
        LastReleased last = {0, 0};
        uint32_t regs = 0;               // (uniform) registers of end_of in use
        // the lifetimes of the next 64 requests are on their way while these 64 are taken one by one
        uint32_t ts_next = 0, te_next = 0;
        if (s + lane < e) {
            const uint32_t i = g.sorted[s + lane];
            ts_next = g.ta[i];
            te_next = g.tf[i];
        }
        for (uint32_t base = s; base < e; base += kWave) {
            const uint32_t k = base + lane;
            const uint32_t ts_k = ts_next, te_k = te_next;
            if (k + kWave < e) {
                const uint32_t i = g.sorted[k + kWave];
                ts_next = g.ta[i];
                te_next = g.tf[i];
            }
            uint32_t mine = 0;           // layer of the request this lane loaded
            const int members = e - base < (uint32_t)kWave ? (int)(e - base) : kWave;
            layers = __builtin_amdgcn_readfirstlane(layers);
            // registers that hold every layer the group can have once these requests are placed (never
            // fewer than for an earlier block, a short last one included: see kLyIdleRegs)
            regs = umax(regs, (layers + (uint32_t)members + kWave - 1) / kWave);
            if (regs <= (uint32_t)kLyRegs) {
                // the usual case: everything in registers, code specialised for the registers in use
                uint32_t* const first_ts = g.first_ts + s;
                switch (regs) {
                    case 1: mine = take_block<1>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 2: mine = take_block<2>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 3: mine = take_block<3>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 4: mine = take_block<4>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 5: mine = take_block<5>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 6: mine = take_block<6>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 7: mine = take_block<7>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 8: mine = take_block<8>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 9: mine = take_block<9>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 10: mine = take_block<10>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 11: mine = take_block<11>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 12: mine = take_block<12>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 13: mine = take_block<13>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 14: mine = take_block<14>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    case 15: mine = take_block<15>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                    default: mine = take_block<16>(end_of, ts_k, te_k, members, layers, last, first_ts); break;
                }
                if (k < e) g.local[k] = mine;
                continue;
            }
            // a group that may pass 1024 layers: the further ones are kept in memory
            for (int q = 0; q < members; ++q) {
                const uint32_t ts = __builtin_amdgcn_readlane(ts_k, q), te = __builtin_amdgcn_readlane(te_k, q);
                layers = __builtin_amdgcn_readfirstlane(layers);
                uint32_t latest = 0;
#pragma unroll
                for (int r = 0; r < kLyRegs; ++r)
                    if ((uint32_t)r * kWave < layers) latest = umax(latest, end_of[r] <= ts ? end_of[r] : 0u);   // (uniform)
                const uint32_t in_regs = __builtin_amdgcn_readlane(wave_scan_max(latest), kWave - 1);
                uint32_t in_mem = 0;
                for (uint32_t l0 = kLyRegs * kWave; l0 < layers; l0 += kWave) {
                    const uint32_t l = l0 + lane;
                    const uint32_t v = l < layers ? __hip_atomic_load(&g.ends[s + l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
                    in_mem = umax(in_mem, __builtin_amdgcn_readlane(wave_scan_max(v <= ts ? v : 0u), kWave - 1));
                }
                const uint32_t best = umax(in_regs, in_mem);
                uint32_t layer = layers;                                          // a new one unless a free layer is found
                if (best != 0) {
                    bool found = false;
                    if (in_regs == best) {
#pragma unroll
                        for (int r = 0; r < kLyRegs; ++r) {
                            if (found || (uint32_t)r * kWave >= layers) continue;                      // (uniform)
                            const uint64_t hit = __builtin_amdgcn_ballot_w64(end_of[r] == best);
                            if (hit) { layer = (uint32_t)r * kWave + (uint32_t)__builtin_ctzll(hit); found = true; }
                        }
                    }
                    for (uint32_t l0 = kLyRegs * kWave; !found && l0 < layers; l0 += kWave) {
                        const uint32_t l = l0 + lane;
                        const uint32_t v = l < layers ? __hip_atomic_load(&g.ends[s + l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
                        const uint64_t hit = __builtin_amdgcn_ballot_w64(v == best);
                        if (hit) { layer = l0 + (uint32_t)__builtin_ctzll(hit); found = true; }
                    }
                } else {
                    if (lane == 0) g.first_ts[s + layers] = ts;
                    ++layers;
                }
                // the request becomes the layer's last one
                if (layer < (uint32_t)(kLyRegs * kWave)) {
#pragma unroll
                    for (int r = 0; r < kLyRegs; ++r)
                        if ((uint32_t)r == layer / kWave) end_of[r] = (uint32_t)lane == layer % kWave ? te : end_of[r];   // (uniform test)
                } else if (lane == 0) {
                    __hip_atomic_store(&g.ends[s + layer], te, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (lane == q) mine = layer;
            }
            if (k < e) g.local[k] = mine;
        }
#pragma unroll
        for (int r = 0; r < kLyRegs; ++r) {
            const uint32_t l = (uint32_t)r * kWave + lane;
            if (l < layers) g.ends[s + l] = end_of[r];
        }
        if (lane == 0) g.group_layers[grp] = layers;
    }
}

// ------------------------------------------------------------------------------------------
// Groups of many requests in parallel.  The layer a request takes is the one released last, and a
// released layer is not released again before it was taken: the free layers are a stack.  In the
// sequence of the group's releases and allocations (a release in front of an allocation at the same
// time) a release pushes and an allocation pops, so which release an allocation follows is the
// matching of brackets, found without walking the sequence:
//   gap      releases between two neighbouring allocations, by binary search; in order of time inside a gap
//            by comparing them to one another
//   height   of the stack in front of every gap: h <- max(0, h + releases of the gap - 1), a scan over
//            functions x -> max(b, x + a)
//   match    the allocation behind gap g takes height h = height[g] + releases of g.  If that is 0 it opens a
//            layer; else the release that was pushed to height h last, in the last gap g' <= g with
//            height[g'] < h (a look back, over the lowest height of every 64 gaps where it goes far)
//   layer    by pointer jumping to the request that opened it; layers are numbered in the order of opening
// Two releases at one time would be told apart by their layers' numbers: such groups (and those that do not
// fit LDS, or have thousands of releases in one gap) are left to ly_build, one request after another.
//   One workgroup per group, everything but the release times in LDS, 12 bytes a request.  A group of 11 900
// requests: 1.6 ms in ly_build -> 0.115 ms for it and the 21 others.
constexpr int kLyMatchThreads = 1024;
constexpr uint32_t kLyMatchFrom = 256;           // smaller groups: ly_build, a wave each (0.13 us a request), four to a workgroup
constexpr uint32_t kLyMostInGap = 2048;
constexpr uint32_t kLyMatchBytes = 12;
constexpr uint16_t kLyTaken = 0xffff;

// x -> max(b, x + a)
struct LyRise {
    int a, b;
    __device__ __forceinline__ LyRise then(const LyRise& next) const { return {a + next.a, b + next.a > next.b ? b + next.a : next.b}; }
};

__global__ void __launch_bounds__(kLyMatchThreads)
ly_match(LyBuild g, const uint32_t* __restrict__ flag, const uint32_t* __restrict__ flags_before, uint32_t cap)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t sh_start, sh_count, sh_group, sh_give_up;
    __shared__ int rise_a[16], rise_b[16];
    __shared__ uint32_t part[16];
    __shared__ uint16_t low_of[1024];
    if (*g.status != STALLOC_OK) return;
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id(), wave = wave_id();
    if (tid == 0) { sh_count = 0; sh_give_up = 0; }
    __syncthreads();
    // at most one group of 256 requests or more begins among 256 sorted positions
    if (tid < 256) {
        const uint32_t k = blockIdx.x * 256 + tid;
        if (k < g.n && flag[k]) {
            const uint32_t grp = flags_before[k], e = grp + 1 < *g.n_groups ? g.group_start[grp + 1] : g.n;
            if (e - k >= kLyMatchFrom && e - k <= cap) { sh_start = k; sh_count = e - k; sh_group = grp; }
        }
    }
    __syncthreads();
    const uint32_t s = sh_start, m = sh_count;
    if (m == 0) return;                                               // (uniform)
    uint32_t* cnt = reinterpret_cast<uint32_t*>(smem);                // [cap + 1] allocation times, then releases per gap, their sums
    uint16_t* gap = reinterpret_cast<uint16_t*>(cnt + cap + 1);       // [cap] per request: its release's gap; then kLyTaken when followed
    uint16_t* height = gap + cap;                                     // [cap] per gap; then per opening request its layer
    uint16_t* rel = height + cap;                                     // [cap] requests in order of release
    uint16_t* prev = rel + cap;                                       // [cap] the same, unsorted inside gaps; then the request followed
    uint32_t* te = g.local + s;                                       // (release times wait where the layers will be written)
    for (uint32_t k = tid; k < m; k += kLyMatchThreads) {
        const uint32_t i = g.sorted[s + k];
        cnt[k] = g.ta[i];
        te[k] = g.tf[i];
    }
    __syncthreads();
    for (uint32_t k = tid; k < m; k += kLyMatchThreads) {
        const uint32_t t = te[k];
        uint32_t lo = k + 1, hi = m;                                  // (it is released after its own allocation)
        while (lo < hi) { const uint32_t mid = (lo + hi) >> 1; if (cnt[mid] < t) lo = mid + 1; else hi = mid; }
        gap[k] = (uint16_t)lo;                                        // m: behind the last allocation
    }
    __syncthreads();
    for (uint32_t k = tid; k <= m; k += kLyMatchThreads) cnt[k] = 0;
    __syncthreads();
    for (uint32_t k = tid; k < m; k += kLyMatchThreads) atomicAdd(&cnt[gap[k]], 1u);
    __syncthreads();
    // a run of gaps per thread: releases in front of it, height of the stack in front of it, layers opened in front of it
    const uint32_t per = (m + kLyMatchThreads - 1) / kLyMatchThreads, k_lo = umin(tid * per, m), k_hi = umin(k_lo + per, m);
    uint32_t released = 0;
    LyRise mine = {0, -0x40000000};
    for (uint32_t k = k_lo; k < k_hi; ++k) {
        const uint32_t c = cnt[k];
        released += c;
        mine = mine.then(LyRise{(int)c - 1, 0});
        if (c > kLyMostInGap) sh_give_up = 1;
    }
    uint32_t released_incl = wave_scan_add(released);
    LyRise incl = mine;
    for (int d = 1; d < kWave; d <<= 1) {
        const LyRise below = {(int)lane_gather((uint32_t)incl.a, lane - d), (int)lane_gather((uint32_t)incl.b, lane - d)};
        if (lane >= d) incl = below.then(incl);
    }
    if (lane == kWave - 1) { rise_a[wave] = incl.a; rise_b[wave] = incl.b; part[wave] = released_incl; }
    LyRise before = {(int)lane_gather((uint32_t)incl.a, lane - 1), (int)lane_gather((uint32_t)incl.b, lane - 1)};
    if (lane == 0) before = LyRise{0, -0x40000000};
    __syncthreads();
    int h = 0;                                                        // height in front of this thread's first gap
    uint32_t start = released_incl - released;
    for (int w = 0; w < wave; ++w) {
        h = h + rise_a[w] > rise_b[w] ? h + rise_a[w] : rise_b[w];
        start += part[w];
    }
    h = h + before.a > before.b ? h + before.a : before.b;
    uint32_t opened = 0;
    for (uint32_t k = k_lo; k < k_hi; ++k) {
        const uint32_t c = cnt[k];
        cnt[k] = start;
        start += c;
        height[k] = (uint16_t)h;
        opened += h + (int)c == 0 ? 1u : 0u;
        h = h + (int)c - 1 > 0 ? h + (int)c - 1 : 0;
    }
    if (k_hi == m && k_lo < m) cnt[m] = start;                        // releases behind the last allocation follow
    const uint32_t opened_incl = wave_scan_add(opened);
    __syncthreads();                                                  // (part[] has been read)
    if (lane == kWave - 1) part[wave] = opened_incl;
    __syncthreads();
    uint32_t first_layer = opened_incl - opened, layers = 0;
    for (int w = 0; w < kLyMatchThreads / kWave; ++w) { if (w < wave) first_layer += part[w]; layers += part[w]; }
    if (sh_give_up) return;                                           // (uniform; no layers are noted, so ly_build takes the group)
    // requests by gap; afterwards cnt[k] = end of gap k = start of gap k + 1
    for (uint32_t k = tid; k < m; k += kLyMatchThreads) prev[atomicAdd(&cnt[gap[k]], 1u)] = (uint16_t)k;
    for (uint32_t b = tid; b * 64 < m; b += kLyMatchThreads) {        // lowest height of 64 gaps
        uint32_t low = 0xffff;
        for (uint32_t k = b * 64; k < umin(b * 64 + 64, m); ++k) low = umin(low, (uint32_t)height[k]);
        low_of[b] = (uint16_t)low;
    }
    __syncthreads();
    for (uint32_t p = tid; p < m; p += kLyMatchThreads) {
        const uint32_t k = prev[p], at = gap[k], lo = at ? cnt[at - 1] : 0u, hi = cnt[at];
        uint32_t place = p;
        if (at < m && hi - lo > 1) {
            const uint32_t t = te[k];
            place = lo;
            for (uint32_t q = lo; q < hi; ++q) {
                const uint32_t other = prev[q], t_other = te[other];
                place += t_other < t ? 1u : 0u;
                if (t_other == t && other != k) sh_give_up = 1;
            }
        }
        rel[place] = (uint16_t)k;
    }
    __syncthreads();
    if (sh_give_up) return;                                           // (uniform)
    for (uint32_t k = tid; k < m; k += kLyMatchThreads) {
        const uint32_t lo = k ? cnt[k - 1] : 0u, c = cnt[k] - lo, top = (uint32_t)height[k] + c;
        uint32_t follows = k;                                         // opens a layer
        if (top != 0) {
            uint32_t at = k;                                          // the last gap that began below `top`
            if (c == 0) {
                while (height[at] >= top && at % 64 != 0) --at;
                if (height[at] >= top) {
                    uint32_t b = at / 64 - 1;                         // (gap 0 begins at height 0: there is one)
                    while (low_of[b] >= top) --b;
                    at = b * 64 + 63;
                    while (height[at] >= top) --at;
                }
            }
            follows = rel[(at ? cnt[at - 1] : 0u) + (top - height[at]) - 1];
            gap[follows] = kLyTaken;
        }
        prev[k] = (uint16_t)follows;
    }
    __syncthreads();
    {
        uint32_t layer = first_layer;                                 // (heights are no longer needed)
        for (uint32_t k = k_lo; k < k_hi; ++k)
            if (prev[k] == k) height[k] = (uint16_t)layer++;
    }
    for (;;) {
        int moved = 0;
        for (uint32_t k = tid; k < m; k += kLyMatchThreads) {
            const uint16_t p = prev[k], q = prev[p];                  // (either is a request of the same layer in front of k)
            if (p != q) { prev[k] = q; moved = 1; }
        }
        if (!__syncthreads_or(moved)) break;
    }
    for (uint32_t k = tid; k < m; k += kLyMatchThreads) {
        const uint32_t layer = height[prev[k]];
        if (prev[k] == k) g.first_ts[s + layer] = g.ta[g.sorted[s + k]];
        if (gap[k] != kLyTaken) g.ends[s + layer] = te[k];            // nobody follows: the layer's last request
        te[k] = layer;                                                // (the request's place in g.local)
    }
    if (tid == 0) g.group_layers[sh_group] = layers;
}

struct LyEmit {
    const uint64_t* size;
    const uint32_t* sorted;
    const uint32_t* flag;            // [n] 1 where a group starts
    const uint32_t* flags_before;    // [n] exclusive sums of flag
    const uint32_t* group_start;
    const uint32_t* group_layers;
    const uint32_t* group_base;      // [groups] exclusive sums of group_layers
    const uint32_t* local;
    const uint32_t* first_ts;
    const uint32_t* ends;
    uint32_t* layer_of;
    uint64_t* layer_size;
    uint32_t* layer_ta;
    uint32_t* layer_tf;
    const uint32_t* status;
    uint32_t n;
};

__global__ void __launch_bounds__(256) ly_emit(LyEmit g)
{
    if (*g.status != STALLOC_OK) return;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < g.n; k += gridDim.x * blockDim.x) {
        const uint32_t i = g.sorted[k];
        const uint32_t grp = g.flags_before[k] + g.flag[k] - 1;
        const uint32_t s = g.group_start[grp], base = g.group_base[grp];
        g.layer_of[i] = base + g.local[k];
        const uint32_t l = k - s;                    // slot of the group: a layer if the group has that many
        if (l < g.group_layers[grp]) {
            g.layer_size[base + l] = g.size[i];
            g.layer_ta[base + l] = g.first_ts[k];
            g.layer_tf[base + l] = g.ends[k];
        }
    }
}

__global__ void ly_expand_init(uint32_t* status)
{
    if (threadIdx.x == 0) *status = STALLOC_OK;
}

// offsets[p][i] = layer_offsets[p][layer_of[i]]; a layer number that does not exist is reported.
__global__ void __launch_bounds__(256)
ly_expand(const uint32_t* __restrict__ layer_of, const uint64_t* __restrict__ layer_offsets, uint32_t n_layers,
          uint32_t n, uint64_t* offsets, uint32_t* status)
{
    const uint64_t* row = layer_offsets + (size_t)blockIdx.y * n_layers;
    uint64_t* out = offsets + (size_t)blockIdx.y * n;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint32_t l = layer_of[i];
        if (l < n_layers) out[i] = row[l];
        else atomicMax(status, (uint32_t)STALLOC_ERR_BAD_LAYER);
    }
}

// Exclusive sums of in[0..m) into out; total[0] = sum.  chunk_sum: (m + 1023) / 1024 words.
void launch_scan(const uint32_t* in, uint32_t m, uint32_t* out, uint32_t* chunk_sum, uint32_t* total,
                 const uint32_t* status, hipStream_t stream)
{
    const uint32_t chunks = (m + kScanChunk - 1) / kScanChunk;
    if (m <= kScanSmall) {
        hipLaunchKernelGGL(scan_small, dim3(1), dim3(1024), 0, stream, in, m, out, total, status);
        return;
    }
    hipLaunchKernelGGL(scan_chunk_sums, dim3(chunks), dim3(256), 0, stream, in, m, chunk_sum, status);
    hipLaunchKernelGGL(scan_of_chunk_sums, dim3(1), dim3(256), 0, stream, chunk_sum, chunks, total, status);
    hipLaunchKernelGGL(scan_apply, dim3(chunks), dim3(256), 0, stream, in, m, chunk_sum, out, status);
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_memory_layers(const stalloc_trace* tr, uint32_t* layer_of, uint32_t* n_layers,
                                     uint64_t* layer_size, uint32_t* layer_t_alloc, uint32_t* layer_t_free,
                                     uint32_t* device_status, void* workspace, size_t* workspace_bytes,
                                     void* hip_stream)
{
    if (!trace_args_ok(tr) || !workspace_bytes) return STALLOC_ERR_INVALID_ARG;
    DeviceInfo di;
    if (!device_info(&di)) return STALLOC_ERR_DEVICE;
    const uint32_t n = tr->n;
    const uint32_t tiles = (n + kLyTile - 1) / kLyTile;
    const uint32_t chunks = (n + kScanChunk - 1) / kScanChunk;

    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    ulonglong2* keys = cv.take<ulonglong2>((size_t)tiles * kLyTile);
    ulonglong2* spare = cv.take<ulonglong2>((size_t)tiles * kLyTile);
    uint32_t* sorted = cv.take<uint32_t>(n);
    uint32_t* flag = cv.take<uint32_t>(n);
    uint32_t* flags_before = cv.take<uint32_t>(n);
    uint32_t* group_start = cv.take<uint32_t>(n);
    uint32_t* group_layers = cv.take<uint32_t>(n);
    uint32_t* group_base = cv.take<uint32_t>(n);
    uint32_t* local = cv.take<uint32_t>(n);
    uint32_t* first_ts = cv.take<uint32_t>(n);
    uint32_t* ends = cv.take<uint32_t>(n);
    uint32_t* chunk_sum = cv.take<uint32_t>(chunks);
    uint32_t* n_groups = cv.take<uint32_t>(1);
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    if (!layer_of || !n_layers || !layer_size || !layer_t_alloc || !layer_t_free || !device_status ||
        *workspace_bytes < cv.used || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    launch_trace_check(*tr, acc, device_status, stream);

    uint32_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(ly_sort_tiles, dim3(tiles), dim3(kSortThreads), 0, stream, tr->size, tr->t_alloc, n, keys, device_status);
    const ulonglong2* by_key = launch_merge_tiles(keys, spare, tiles * kLyTile, 1, device_status, stream);
    hipLaunchKernelGGL(ly_ids, dim3(blocks), dim3(256), 0, stream, by_key, n, sorted, flag, group_layers, device_status);
    launch_scan(flag, n, flags_before, chunk_sum, n_groups, device_status, stream);
    hipLaunchKernelGGL(ly_group_starts, dim3(blocks), dim3(256), 0, stream, flag, flags_before, n, group_start,
                       device_status);

    LyBuild b;
    b.ta = tr->t_alloc; b.tf = tr->t_free; b.sorted = sorted; b.group_start = group_start; b.n_groups = n_groups;
    b.local = local; b.first_ts = first_ts; b.ends = ends; b.group_layers = group_layers; b.status = device_status;
    b.n = n;
    // (With fewer timestamps than requests the clock is coarse: a large group has tied releases and ly_match would
    // give up on it, for about 10 us a call.)
    if (n >= kLyMatchFrom && tr->t_end >= n) {
        const size_t lds_budget = di.lds_per_block - 4096;            // (static LDS takes the rest)
        uint32_t cap = (uint32_t)((lds_budget - 16) / kLyMatchBytes) & ~3u;
        if (cap > n) cap = (n + 3) & ~3u;
        static std::atomic<bool> attr_set[64] = {};        // (set twice at worst when threads race)
        if (!attr_set[di.device]) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(&ly_match), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds_budget) != hipSuccess)
                return STALLOC_ERR_DEVICE;
            attr_set[di.device] = true;
        }
        hipLaunchKernelGGL(ly_match, dim3((n + 255) / 256), dim3(kLyMatchThreads), (size_t)cap * kLyMatchBytes + 16, stream, b, flag,
                           flags_before, cap);
    }
    uint32_t build_blocks = (n + 3) / 4;                  // at most n groups, four waves to a workgroup
    if (build_blocks > (uint32_t)di.cus * 8) build_blocks = (uint32_t)di.cus * 8;
    hipLaunchKernelGGL(ly_build, dim3(build_blocks), dim3(256), 0, stream, b);
    // (only the device knows how many groups there are: the slots past the last group hold no layers)
    launch_scan(group_layers, n, group_base, chunk_sum, n_layers, device_status, stream);

    LyEmit e;
    e.size = tr->size; e.sorted = sorted; e.flag = flag; e.flags_before = flags_before; e.group_start = group_start;
    e.group_layers = group_layers; e.group_base = group_base; e.local = local; e.first_ts = first_ts; e.ends = ends;
    e.layer_of = layer_of; e.layer_size = layer_size; e.layer_ta = layer_t_alloc; e.layer_tf = layer_t_free;
    e.status = device_status; e.n = n;
    hipLaunchKernelGGL(ly_emit, dim3(blocks), dim3(256), 0, stream, e);
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}

extern "C" int stalloc_expand_layers(uint32_t n, uint32_t P, const uint32_t* layer_of, const uint64_t* layer_offsets,
                                     uint32_t n_layers, uint64_t* offsets, uint32_t* device_status, void* hip_stream)
{
    if (n == 0 || n >= 0x80000000u || P == 0 || n_layers == 0 || !layer_of || !layer_offsets || !offsets || !device_status)
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    uint32_t blocks = (n + 255) / 256;
    if (blocks > 64) blocks = 64;
    hipLaunchKernelGGL(ly_expand_init, dim3(1), dim3(64), 0, stream, device_status);
    for (uint32_t p0 = 0; p0 < P; p0 += 32768) {           // grid.y is limited to 65535
        const uint32_t py = P - p0 < 32768 ? P - p0 : 32768;
        hipLaunchKernelGGL(ly_expand, dim3(blocks, py), dim3(256), 0, stream, layer_of, layer_offsets + (size_t)p0 * n_layers,
                           n_layers, n, offsets + (size_t)p0 * n, device_status);
    }
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}
