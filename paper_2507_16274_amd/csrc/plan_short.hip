// stalloc_plan for short traces (up to 512 requests): one wave per candidate placement order, the rule of Sec. 5.1 (every
// request gets the lowest address at which it conflicts with no earlier request of the plan in lifespan and address range
// at once), the list of placed blocks sorted by address in the registers of that wave.
//
// A plan is a chain: each request needs the address of the one before it.  What a short trace costs is the length
// of one link of that chain, and launches.  A workgroup that shares a request out among its waves pays barriers and LDS round
// trips for every link; here a link is some sixty instructions of one wave that never leave its registers: the list
// lies in the lanes in address order, J blocks a lane.  Two compares keep the blocks alive together with
// the request, a running maximum of their ends over the lanes (DPP) is "covered so far", the first of them that starts at
// least `size` above it closes the hole that the request takes (else it goes on top), and the blocks above move up by one.
// The first 64 requests of an order see one block per lane, the next 64 two, and so on.
// A wave also checks the trace by itself (512 requests are eight loads per lane): a call is two launches.
//   Bound by the instructions of a lone wave, one after another: about 60 per request with one block per lane, some 16 more for each
// further one (75 and 25 while the place in the list was counted out and written to by a branch per block of a lane).  The
// workgroup kernels / this one with such branches / now: 96 requests, 64 orders 64 / 28 / 24 us, 384 requests, 64 orders 190 / 152 / 108,
// 480 requests in 32-bit counts, 64 orders 340 / 229 / 163, 4096 orders 3502 / 397 / 323; one order by size of 512 requests of an
// interleaved schedule 178 / 251 / 177.
#include <utility>

#include "host_util.h"
#include "plan_params.h"
#include "trace_sums.h"
#include "wave.h"

namespace stalloc {

// How a placed block is kept in kFields registers of a lane.  Key: what the running maximum is taken over.  none: a block
// behind all others that conflicts with nothing.
struct ShortCompact {                        // 16-bit counts and times: start | end << 16, allocation | release << 16
    typedef uint32_t Addr;
    typedef uint32_t Key;
    static constexpr int kFields = 2;
    static constexpr uint32_t kBits = 16;
    static __device__ __forceinline__ uint32_t none(int f) { return f == 0 || f == 1 ? 0xffffu : 0u; }
    static __device__ __forceinline__ uint32_t field(int f, Addr x, Addr end, uint32_t ta, uint32_t tf)
    {
        return f == 0 ? x | (end << 16) : ta | (tf << 16);
    }
    static __device__ __forceinline__ uint64_t alive(const uint32_t (&b)[kFields], uint32_t ta, uint32_t tf)
    {
        return lanes_lt(b[1] & 0xffffu, tf) & lanes_ge(b[1], (ta + 1) << 16);     // (release > t_alloc, in the upper half)
    }
    static __device__ __forceinline__ Addr lo(const uint32_t (&b)[kFields]) { return b[0] & 0xffffu; }
    static __device__ __forceinline__ Key end(const uint32_t (&b)[kFields]) { return b[0]; }     // (the larger end is the larger word)
    static __device__ __forceinline__ Addr covered(Key k) { return k >> 16; }
};
struct ShortBrief {                          // 32-bit granule counts, 16-bit times
    typedef uint32_t Addr;
    typedef uint32_t Key;
    static constexpr int kFields = 3;
    static constexpr uint32_t kBits = 32;
    static __device__ __forceinline__ uint32_t none(int f) { return f == 0 ? 0xffffffffu : f == 2 ? 0xffffu : 0u; }
    static __device__ __forceinline__ uint32_t field(int f, Addr x, Addr end, uint32_t ta, uint32_t tf)
    {
        return f == 0 ? x : f == 1 ? end : ta | (tf << 16);
    }
    static __device__ __forceinline__ uint64_t alive(const uint32_t (&b)[kFields], uint32_t ta, uint32_t tf)
    {
        return lanes_lt(b[2] & 0xffffu, tf) & lanes_ge(b[2], (ta + 1) << 16);
    }
    static __device__ __forceinline__ Addr lo(const uint32_t (&b)[kFields]) { return b[0]; }
    static __device__ __forceinline__ Key end(const uint32_t (&b)[kFields]) { return b[1]; }
    static __device__ __forceinline__ Addr covered(Key k) { return k; }
};
struct ShortNarrow {                         // 32-bit granule counts
    typedef uint32_t Addr;
    typedef uint32_t Key;
    static constexpr int kFields = 4;
    static constexpr uint32_t kBits = 32;
    static __device__ __forceinline__ uint32_t none(int f) { return f == 0 || f == 2 ? 0xffffffffu : 0u; }
    static __device__ __forceinline__ uint32_t field(int f, Addr x, Addr end, uint32_t ta, uint32_t tf)
    {
        return f == 0 ? x : f == 1 ? end : f == 2 ? ta : tf;
    }
    static __device__ __forceinline__ uint64_t alive(const uint32_t (&b)[kFields], uint32_t ta, uint32_t tf)
    {
        return lanes_lt(b[2], tf) & lanes_lt(ta, b[3]);
    }
    static __device__ __forceinline__ Addr lo(const uint32_t (&b)[kFields]) { return b[0]; }
    static __device__ __forceinline__ Key end(const uint32_t (&b)[kFields]) { return b[1]; }
    static __device__ __forceinline__ Addr covered(Key k) { return k; }
};
struct ShortWide {                           // 64-bit addresses
    typedef uint64_t Addr;
    typedef uint64_t Key;
    static constexpr int kFields = 6;
    static constexpr uint32_t kBits = 64;
    static __device__ __forceinline__ uint32_t none(int f) { return f <= 1 || f == 4 ? 0xffffffffu : 0u; }
    static __device__ __forceinline__ uint32_t field(int f, Addr x, Addr end, uint32_t ta, uint32_t tf)
    {
        return f == 0 ? (uint32_t)x : f == 1 ? (uint32_t)(x >> 32) : f == 2 ? (uint32_t)end : f == 3 ? (uint32_t)(end >> 32) : f == 4 ? ta : tf;
    }
    static __device__ __forceinline__ uint64_t alive(const uint32_t (&b)[kFields], uint32_t ta, uint32_t tf)
    {
        return lanes_lt(b[4], tf) & lanes_lt(ta, b[5]);
    }
    static __device__ __forceinline__ Addr lo(const uint32_t (&b)[kFields]) { return ((uint64_t)b[1] << 32) | b[0]; }
    static __device__ __forceinline__ Key end(const uint32_t (&b)[kFields]) { return ((uint64_t)b[3] << 32) | b[2]; }
    static __device__ __forceinline__ Addr covered(Key k) { return k; }
};

// Requests of a plan in the order they are placed: number 64 j + lane in set j.
template <int kSets>
struct ShortOrder {
    uint64_t size[kSets];
    uint32_t ta[kSets], tf[kSets], id[kSets];
};

// Places the requests of set J - 1 on top of the 64 (J - 1) blocks listed so far; block k of the list is block k mod J of lane
// k / J.  Returns false when a plan that is tried with 32-bit counts may outgrow them.
template <typename Cells, int J, int kSets>
__device__ __forceinline__ bool place_set(uint32_t (&block)[kSets][Cells::kFields], const ShortOrder<kSets>& rq, uint32_t many, uint32_t shift,
                                          bool try32, typename Cells::Addr& peak, typename Cells::Addr& mine)
{
    typedef typename Cells::Addr Addr;
    typedef typename Cells::Key Key;
    constexpr int kFields = Cells::kFields;
    const Addr granules = (Addr)(rq.size[J - 1] >> shift);
    const uint32_t rq_ta = rq.ta[J - 1], rq_tf = rq.tf[J - 1];
    for (uint32_t q = 0; q < many; ++q) {
        const Addr s = read_lane(granules, (int)q);
        const uint32_t ta = read_lane(rq_ta, (int)q), tf = read_lane(rq_tf, (int)q);
        if (sizeof(Addr) == 4 && try32 && s > (Addr)~peak) return false;       // (uniform) peak + s may not fit
        // covered so far in front of each block, and the first hole that is large enough
        uint64_t alive[J], some = 0;
        Key before[J], run = 0;
#pragma unroll
        for (int u = 0; u < J; ++u) {
            alive[u] = Cells::alive(block[u], ta, tf);
            before[u] = run;
            run = umax(run, lane_in(alive[u]) ? Cells::end(block[u]) : (Key)0);
        }
        const Key incl = wave_scan_max(run), below = wave_shift_up(incl, (Key)0);
        Addr covered = 0;                                             // in front of the lane's first such hole
#pragma unroll
        for (int u = J - 1; u >= 0; --u) {
            const Addr here = Cells::covered(umax(before[u], below));
            const uint64_t holes = alive[u] & lanes_ge(Cells::lo(block[u]), (Addr)(here + s));
            covered = lane_in(holes) ? here : covered;
            some |= holes;
        }
        const Addr x = some ? read_lane(covered, __builtin_ctzll(some)) : Cells::covered(read_lane(incl, kWave - 1));
        peak = umax(peak, (Addr)(x + s));
        mine = set_lane(mine, x, (int)q);
        // The blocks that start above it move up by one, and it takes the place of the first of them: block k is one of them if it starts
        // above, and gets the one before if that does, too.  (Counting them for the place and writing the block there, a branch per block
        // of a lane, took twice as many instructions.)
        uint32_t field[kFields], last[kFields];
#pragma unroll
        for (int f = 0; f < kFields; ++f) {
            field[f] = Cells::field(f, x, (Addr)(x + s), ta, tf);
            last[f] = wave_shift_up(block[J - 1][f], 0u);
        }
        uint64_t above[J];
#pragma unroll
        for (int u = 0; u < J; ++u) above[u] = lanes_lt(x, Cells::lo(block[u]));
#pragma unroll
        for (int u = J - 1; u >= 0; --u) {
            const uint64_t further = u > 0 ? above[u > 0 ? u - 1 : 0] : above[J - 1] << 1;
#pragma unroll
            for (int f = 0; f < kFields; ++f) {
                const uint32_t here = lane_in(above[u]) ? field[f] : block[u][f];
                block[u][f] = lane_in(further) ? (u > 0 ? block[u > 0 ? u - 1 : 0][f] : last[f]) : here;
            }
        }
    }
    return true;
}

// A full list of J blocks per lane becomes one of J + 1, with 64 blocks that conflict with nothing behind it.
template <typename Cells, int J, int kSets>
__device__ __forceinline__ void widen_list(uint32_t (&block)[kSets][Cells::kFields], uint32_t* swap)
{
    const int lane = lane_id();
#pragma unroll
    for (int f = 0; f < Cells::kFields; ++f) {
        __builtin_amdgcn_wave_barrier();                              // (the wave's own LDS: its accesses complete in order)
#pragma unroll
        for (int u = 0; u < J; ++u) swap[lane * J + u] = block[u][f];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u <= J; ++u) {
            const int k = lane * (J + 1) + u;
            block[u][f] = k < J * kWave ? swap[k] : Cells::none(f);
        }
    }
}

// One plan; returns false when it has to be placed again with 64-bit addresses.
template <typename Cells, int kSets, int... kBefore>
__device__ __forceinline__ bool place_plan(const ShortOrder<kSets>& rq, uint32_t n, uint32_t shift, bool try32, uint64_t& peak, uint64_t* out,
                                           uint32_t* swap, std::integer_sequence<int, kBefore...>)
{
    typedef typename Cells::Addr Addr;
    uint32_t block[kSets][Cells::kFields];
#pragma unroll
    for (int f = 0; f < Cells::kFields; ++f) block[0][f] = Cells::none(f);
    Addr top = 0, at[kSets];
    bool fits = true;
    auto next = [&](auto before) {
        constexpr int j = decltype(before)::value;
        at[j] = 0;
        if (!fits || (uint32_t)j * kWave >= n) return;                // (uniform)
        if constexpr (j > 0) widen_list<Cells, j, kSets>(block, swap);
        const uint32_t many = umin(n - (uint32_t)j * kWave, (uint32_t)kWave);
        fits = place_set<Cells, j + 1, kSets>(block, rq, many, shift, try32, top, at[j]);
    };
    (next(std::integral_constant<int, kBefore>()), ...);
    if (!fits) return false;
    if (out) {
#pragma unroll
        for (int j = 0; j < kSets; ++j)
            if ((uint32_t)(j * kWave + lane_id()) < n) out[rq.id[j]] = (uint64_t)at[j] << shift;
    }
    peak = (uint64_t)top << shift;
    return true;
}

constexpr uint32_t kShortAgain = 0x100u;     // in a plan's flags, beside its status: placed again with 64-bit addresses

template <int kSets>
__global__ void __launch_bounds__(kWave)
plan_short(PlanParams prm, uint32_t t_end, uint64_t* acc, uint32_t* flags)
{
    __shared__ uint64_t sh_size[kSets * kWave];
    __shared__ uint32_t sh_ta[kSets * kWave], sh_tf[kSets * kWave];
    const uint32_t n = prm.n, p = blockIdx.x, lane = (uint32_t)lane_id();
    const uint32_t* order = prm.orders + (size_t)p * n;
    // the trace and the order of the plan; the trace is checked by every wave for itself
    ShortOrder<kSets> rq;
    uint64_t size[kSets];
    uint32_t ta[kSets], tf[kSets];
#pragma unroll
    for (int j = 0; j < kSets; ++j) {
        const uint32_t k = umin(j * kWave + lane, n - 1);
        rq.id[j] = order[k];
        size[j] = prm.size[k]; ta[j] = prm.ta[k]; tf[j] = prm.tf[k];
    }
    TraceSums sums = TraceSums::none();
#pragma unroll
    for (int j = 0; j < kSets; ++j) {
        const uint32_t k = j * kWave + lane;
        sh_size[k] = size[j]; sh_ta[k] = ta[j]; sh_tf[k] = tf[j];
        if (k < n) sums.add(size[j], ta[j], tf[j], t_end);
    }
    sums.over_wave();
    uint64_t words[kAccWords];
    const uint32_t code = verdict(sums, n, t_end, words);
    const uint64_t mode = words[kAccMode];
    const bool compact = t_end < 0x10000u && (mode & kModeCompact) != 0, try32 = (mode & kModeTry32) != 0;
    const bool wide = !(mode & (kModeNarrow | kModeTry32));
    if (p == 0 && lane == 0) {
        if (code == STALLOC_OK)
            words[kAccKernel] = STALLOC_KERNEL_LIST_LDS | ((compact ? ShortCompact::kBits : wide ? ShortWide::kBits : ShortNarrow::kBits) << 8);
        for (int k = 0; k < kAccWords; ++k) acc[k] = words[k];
    }
    __builtin_amdgcn_wave_barrier();                                  // (the wave's own LDS: its accesses complete in order)
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kSets; ++j) {
        if (rq.id[j] >= n) { bad = bad || j * kWave + lane < n; rq.id[j] = 0; }
        const uint32_t i = rq.id[j];
        rq.size[j] = sh_size[i]; rq.ta[j] = sh_ta[i]; rq.tf[j] = sh_tf[i];
    }
    const uint32_t status = code != STALLOC_OK ? code : __builtin_amdgcn_ballot_w64(bad) ? (uint32_t)STALLOC_ERR_BAD_ORDER : (uint32_t)STALLOC_OK;
    uint32_t flag = status;
    if (code == STALLOC_OK) {                                         // (uniform)
        const uint32_t shift = (uint32_t)(mode & 63);
        uint64_t* out = prm.offsets ? prm.offsets + (size_t)p * n : nullptr;
        uint64_t peak = 0;
        constexpr auto sets = std::make_integer_sequence<int, kSets>();
        bool placed = false;
        if (compact) placed = place_plan<ShortCompact, kSets>(rq, n, shift, false, peak, out, sh_ta, sets);
        else if (!wide && t_end < 0x10000u) placed = place_plan<ShortBrief, kSets>(rq, n, shift, try32, peak, out, sh_ta, sets);
        else if (!wide) placed = place_plan<ShortNarrow, kSets>(rq, n, shift, try32, peak, out, sh_ta, sets);
        if (!placed) {
            place_plan<ShortWide, kSets>(rq, n, 0, false, peak, out, sh_ta, sets);
            if (!wide) flag |= kShortAgain;
        }
        if (lane == 0) prm.peaks[p] = peak;
    }
    if (lane == 0) flags[p] = flag;
}

// The status of the call, the best plan and its addresses; one workgroup.
__global__ void __launch_bounds__(1024)
plan_short_best(const uint32_t* __restrict__ flags, const uint64_t* __restrict__ peaks, uint32_t P, const uint64_t* __restrict__ offsets, uint32_t n,
                uint32_t* best_plan, uint64_t* best_offsets, uint64_t* acc, uint32_t* status)
{
    __shared__ uint64_t w_peak[16], w_idx[16];
    __shared__ uint32_t w_status[16], w_again[16];
    uint64_t best = ~0ull, idx = ~0ull;
    uint32_t worst = 0, again = 0;
    for (uint32_t p = threadIdx.x; p < P; p += 1024) {
        const uint32_t f = flags[p];
        const uint64_t v = peaks[p];
        worst = umax(worst, f & (kShortAgain - 1));
        again += f / kShortAgain;
        if (v < best) { best = v; idx = p; }                          // ascending p per thread: first of equals kept
    }
    const uint64_t wbest = wave_min64(best), widx = wave_min64(best == wbest ? idx : ~0ull);
    worst = read_lane(wave_scan_max(worst), kWave - 1);
    again = wave_sum32(again);
    if (lane_id() == 0) { w_peak[wave_id()] = wbest; w_idx[wave_id()] = widx; w_status[wave_id()] = worst; w_again[wave_id()] = again; }
    __syncthreads();
    uint64_t b = ~0ull, i = ~0ull;
    worst = 0; again = 0;
    for (int k = 0; k < 16; ++k) {
        if (w_peak[k] < b || (w_peak[k] == b && w_idx[k] < i)) { b = w_peak[k]; i = w_idx[k]; }
        worst = umax(worst, w_status[k]);
        again += w_again[k];
    }
    const bool ok = worst == STALLOC_OK;
    if (threadIdx.x == 0) {
        *status = worst;
        *best_plan = ok ? (uint32_t)i : 0u;
        acc[kAccWidePlans] = again;
    }
    if (!ok || !best_offsets) return;
    for (uint32_t k = threadIdx.x; k < n; k += 1024) best_offsets[k] = offsets[(size_t)i * n + k];
}

bool short_plan_possible(uint32_t n, uint32_t P) { return n <= kShortMost && P <= kShortPlans; }

bool launch_plan_short(const PlanParams& prm, uint32_t t_end, uint64_t* best_offsets, uint32_t* best_plan, hipStream_t stream)
{
    uint64_t* acc = const_cast<uint64_t*>(prm.acc);
    auto kernel = prm.n <= 64 ? &plan_short<1> : prm.n <= 128 ? &plan_short<2> : prm.n <= 256 ? &plan_short<4> : &plan_short<8>;
    hipLaunchKernelGGL(kernel, dim3(prm.P), dim3(kWave), 0, stream, prm, t_end, acc, prm.wide_plans);
    hipLaunchKernelGGL(plan_short_best, dim3(1), dim3(1024), 0, stream, prm.wide_plans, prm.peaks, prm.P, prm.offsets, prm.n, best_plan,
                       best_offsets, acc, prm.status);
    return hipGetLastError() == hipSuccess;
}

}  // namespace stalloc
