// Device-side sanity pass over a trace: sizes > 0, t_alloc < t_free <= t_end, and the
// sum of sizes below 2^63 so that no address can wrap (requests are the events
// m = (s, t_s, t_e) of Sec. 4).  The verdict lands in the caller's device status word.
// The pass also derives the address granule: every address a plan can produce is a sum of
// request sizes, hence a multiple of the largest power of two dividing all sizes; when the
// sum of sizes counted in granules stays below 2^31 the placement kernel may keep
// addresses as 32-bit granule counts without any loss.
#include "host_util.h"
#include "trace_sums.h"
#include "wave.h"

namespace stalloc {

// Of the requests that the calling threads take, `step` apart; valid in thread 0 of the workgroup.
template <int kThreads>
__device__ __forceinline__ TraceSums sum_requests(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta,
                                                  const uint32_t* __restrict__ tf, uint32_t n, uint32_t t_end, uint32_t first, uint32_t step)
{
    __shared__ TraceSums part[kThreads / kWave];
    TraceSums t = TraceSums::none();
#pragma unroll 4
    for (uint32_t i = first; i < n; i += step) t.add(size[i], ta[i], tf[i], t_end);
    t.over_wave();
    if (lane_id() == 0) part[wave_id()] = t;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kThreads / kWave; ++w) t.add(part[w]);
    return t;
}

// The accumulators (the other words are zero) and the status, from the sums over all requests; one thread.
__device__ __forceinline__ void write_verdict(const TraceSums& t, uint32_t n, uint32_t t_end, uint64_t* acc, uint32_t* status)
{
    uint64_t words[kAccWords];
    *status = verdict(t, n, t_end, words);
    for (int k = 0; k < kAccWords; ++k) acc[k] = words[k];
}

__global__ void __launch_bounds__(1024)
trace_check_small(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n,
                  uint32_t t_end, uint64_t* acc, uint32_t* status)
{
    const TraceSums t = sum_requests<1024>(size, ta, tf, n, t_end, threadIdx.x, 1024);
    if (threadIdx.x == 0) write_verdict(t, n, t_end, acc, status);
}

__global__ void __launch_bounds__(256)
trace_check_scan(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta,
                 const uint32_t* __restrict__ tf, uint32_t n, uint32_t t_end, TraceSums* part)
{
    const TraceSums t = sum_requests<256>(size, ta, tf, n, t_end, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ void __launch_bounds__(kTraceCheckBlocks) trace_check_finish(const TraceSums* part, uint32_t parts, uint32_t n, uint32_t t_end, uint64_t* acc,
                                                                        uint32_t* status)
{
    __shared__ TraceSums of[kTraceCheckBlocks / kWave];
    TraceSums t = TraceSums::none();
    if (threadIdx.x < parts) t = part[threadIdx.x];
    t.over_wave();
    if (lane_id() == 0) of[wave_id()] = t;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kTraceCheckBlocks / kWave; ++w) t.add(of[w]);
    write_verdict(t, n, t_end, acc, status);
}

// One launch for short traces (up to this many requests a single workgroup needs no longer than a launch
// takes), else two, the workgroups' sums in the workspace in between: 256 workgroups adding to five words
// with atomics took 14 us on 199 748 requests, and clearing those words was a launch of its own.
constexpr uint32_t kTraceCheckSmall = 8192;

void launch_trace_check(const stalloc_trace& tr, uint64_t* acc, uint32_t* device_status, hipStream_t stream)
{
    if (tr.n <= kTraceCheckSmall) {
        hipLaunchKernelGGL(trace_check_small, dim3(1), dim3(1024), 0, stream, tr.size, tr.t_alloc, tr.t_free, tr.n, tr.t_end, acc,
                           device_status);
        return;
    }
    uint32_t blocks = (tr.n + 255) / 256;
    if (blocks > kTraceCheckBlocks) blocks = kTraceCheckBlocks;
    TraceSums* part = reinterpret_cast<TraceSums*>(acc + kAccWords);
    hipLaunchKernelGGL(trace_check_scan, dim3(blocks), dim3(256), 0, stream, tr.size, tr.t_alloc, tr.t_free,
                       tr.n, tr.t_end, part);
    hipLaunchKernelGGL(trace_check_finish, dim3(1), dim3(kTraceCheckBlocks), 0, stream, part, blocks, tr.n, tr.t_end, acc, device_status);
}

}  // namespace stalloc

extern "C" const char* stalloc_status_string(int status)
{
    switch (status) {
        case STALLOC_OK: return "STALLOC_OK";
        case STALLOC_ERR_INVALID_ARG: return "STALLOC_ERR_INVALID_ARG";
        case STALLOC_ERR_BAD_TRACE: return "STALLOC_ERR_BAD_TRACE";
        case STALLOC_ERR_OVERFLOW: return "STALLOC_ERR_OVERFLOW";
        case STALLOC_ERR_NOMEM: return "STALLOC_ERR_NOMEM";
        case STALLOC_ERR_DEVICE: return "STALLOC_ERR_DEVICE";
        case STALLOC_ERR_BAD_ORDER: return "STALLOC_ERR_BAD_ORDER";
        case STALLOC_ERR_BAD_WINDOW: return "STALLOC_ERR_BAD_WINDOW";
        case STALLOC_ERR_BAD_LAYER: return "STALLOC_ERR_BAD_LAYER";
        case STALLOC_ERR_TOO_LARGE: return "STALLOC_ERR_TOO_LARGE";
        default: return "STALLOC_UNKNOWN_STATUS";
    }
}
