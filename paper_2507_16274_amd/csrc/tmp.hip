// stalloc_tmp: the time-memory product of Eq. 2 for P plans of one trace, with the whole
// plan as the group D_g:
//
//     TMP = sum_i s_i (t_e,i - t_s,i)  /  ( extent * (max t_e - min t_s) ),   extent = max(a + s).
//
// The numerator and the span belong to the trace; the extent is what differs between plans
// (stalloc_plan returns it per plan).  A higher value means fewer spatio-temporal bubbles.
//
// The numerator is summed exactly: every product s * (t_e - t_s) has up to 96 bits and is cut
// into three 32-bit limbs, each limb summed in a 64-bit word (fewer than 2^31 terms: no
// wrap).  The limbs are combined in double precision and divided once per plan: at most eight
// roundings, a relative error below 10 * 2^-53.
#include "host_util.h"
#include "wave.h"

namespace stalloc {

struct TmpAcc {
    uint64_t limb[3];      // sums of bits 0-31, 32-63, 64-95 of the products
    uint32_t t_first;      // min t_alloc
    uint32_t t_last;       // max t_free
};

__global__ void tmp_init(TmpAcc* acc)
{
    if (threadIdx.x == 0) { acc->limb[0] = acc->limb[1] = acc->limb[2] = 0; acc->t_first = 0xffffffffu; acc->t_last = 0; }
}

// Sums over the requests that the calling threads take, `step` apart; valid in thread 0 of the workgroup.
template <int kThreads>
__device__ __forceinline__ TmpAcc tmp_sum(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta,
                                          const uint32_t* __restrict__ tf, uint32_t n, uint32_t from, uint32_t step)
{
    __shared__ TmpAcc part[kThreads / kWave];
    TmpAcc t = {{0, 0, 0}, 0xffffffffu, 0};
    for (uint32_t i = from; i < n; i += step) {
        const uint64_t s = size[i];
        const uint32_t a = ta[i], f = tf[i];
        const uint64_t life = f - a;
        const uint64_t low = (s & 0xffffffffull) * life;           // < 2^64
        const uint64_t high = (s >> 32) * life + (low >> 32);       // bits 32.. of the product; < 2^64
        t.limb[0] += low & 0xffffffffull;
        t.limb[1] += high & 0xffffffffull;
        t.limb[2] += high >> 32;
        t.t_first = umin(t.t_first, a);
        t.t_last = umax(t.t_last, f);
    }
    for (int k = 0; k < 3; ++k) t.limb[k] = wave_sum64(t.limb[k]);
    t.t_first = ~read_lane(wave_scan_max(~t.t_first), kWave - 1);
    t.t_last = read_lane(wave_scan_max(t.t_last), kWave - 1);
    if (lane_id() == 0) part[wave_id()] = t;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kThreads / kWave; ++w) {
            for (int k = 0; k < 3; ++k) t.limb[k] += part[w].limb[k];
            t.t_first = umin(t.t_first, part[w].t_first);
            t.t_last = umax(t.t_last, part[w].t_last);
        }
    return t;
}

__global__ void __launch_bounds__(256)
tmp_used(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n,
         TmpAcc* acc, const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    const TmpAcc t = tmp_sum<256>(size, ta, tf, n, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
    if (threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) atomicAdd((unsigned long long*)&acc->limb[k], (unsigned long long)t.limb[k]);
        atomicMin(&acc->t_first, t.t_first);
        atomicMax(&acc->t_last, t.t_last);
    }
}

__device__ __forceinline__ void tmp_of_plans(const TmpAcc& t, const uint64_t* __restrict__ extents, uint32_t P, double* tmp, uint32_t from,
                                             uint32_t step)
{
    const double used = ((double)t.limb[2] * 4294967296.0 + (double)t.limb[1]) * 4294967296.0 + (double)t.limb[0];
    const double span = (double)(t.t_last - t.t_first);
    for (uint32_t p = from; p < P; p += step) tmp[p] = used / ((double)extents[p] * span);
}

__global__ void __launch_bounds__(256)
tmp_per_plan(const TmpAcc* __restrict__ acc, const uint64_t* __restrict__ extents, uint32_t P, double* tmp,
             const uint32_t* status)
{
    if (*status != STALLOC_OK) return;
    tmp_of_plans(*acc, extents, P, tmp, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// Few requests and plans: sums and ratios in one workgroup instead of three launches.
constexpr uint32_t kTmpSmallRequests = 8192, kTmpSmallPlans = 8192;
__global__ void __launch_bounds__(1024)
tmp_small(const uint64_t* __restrict__ size, const uint32_t* __restrict__ ta, const uint32_t* __restrict__ tf, uint32_t n,
          const uint64_t* __restrict__ extents, uint32_t P, double* tmp, const uint32_t* status)
{
    __shared__ TmpAcc all;
    if (*status != STALLOC_OK) return;
    const TmpAcc t = tmp_sum<1024>(size, ta, tf, n, threadIdx.x, 1024);
    if (threadIdx.x == 0) all = t;
    __syncthreads();
    tmp_of_plans(all, extents, P, tmp, threadIdx.x, 1024);
}

}  // namespace stalloc

using namespace stalloc;

extern "C" int stalloc_tmp(const stalloc_trace* tr, const uint64_t* extents, uint32_t P, double* tmp,
                           uint32_t* device_status, void* workspace, size_t* workspace_bytes, void* hip_stream)
{
    if (!trace_args_ok(tr) || P == 0 || !workspace_bytes) return STALLOC_ERR_INVALID_ARG;
    Carver cv(workspace);
    uint64_t* acc = cv.take<uint64_t>(kAccSpace);
    TmpAcc* sums = cv.take<TmpAcc>(1);
    if (!workspace) { *workspace_bytes = cv.used; return STALLOC_OK; }
    if (!extents || !tmp || !device_status || *workspace_bytes < cv.used ||
        (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return STALLOC_ERR_INVALID_ARG;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    launch_trace_check(*tr, acc, device_status, stream);
    if (tr->n <= kTmpSmallRequests && P <= kTmpSmallPlans) {
        hipLaunchKernelGGL(tmp_small, dim3(1), dim3(1024), 0, stream, tr->size, tr->t_alloc, tr->t_free, tr->n, extents, P, tmp,
                           device_status);
        return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
    }
    hipLaunchKernelGGL(tmp_init, dim3(1), dim3(64), 0, stream, sums);
    uint32_t blocks = (tr->n + 255) / 256;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(tmp_used, dim3(blocks), dim3(256), 0, stream, tr->size, tr->t_alloc, tr->t_free, tr->n, sums,
                       device_status);
    uint32_t pb = (P + 255) / 256;
    if (pb > 1024) pb = 1024;
    hipLaunchKernelGGL(tmp_per_plan, dim3(pb), dim3(256), 0, stream, sums, extents, P, tmp, device_status);
    return hipGetLastError() == hipSuccess ? STALLOC_OK : STALLOC_ERR_DEVICE;
}
