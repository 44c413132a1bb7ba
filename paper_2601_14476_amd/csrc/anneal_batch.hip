// anneal_batch.hip -- the sweeps of many runs in one launch.
#include <hip/hip_runtime.h>

#include "ell_sweep.hpp"
#include "engine.hpp"
#include "sweep.hpp"

namespace psa {
namespace {

// ---------------------------------------------------------------------------
// Batched launch: one grid over the work items of many runs.  Work item b is
// (run jobs[work[b].x], trial group work[b].y); each run carries its own
// graph, factors, spins and step range, and names its kernel variant.  All
// variants share one launch (dynamic LDS = the largest any item needs).
// ---------------------------------------------------------------------------
template <int BLOCK>
__global__ __launch_bounds__(BLOCK, 4) void anneal_batch_kernel(const BatchJob *__restrict__ jobs,
                                                             const int2 *__restrict__ work) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 w = work[blockIdx.x];
    if (w.x < 0) return;  // padding slot of the XCD-aware work list
    const BatchJob &job = jobs[w.x];
    const AnnealArgs a = job.a;
    switch (job.variant) {
        case kBatchUnitLds2: anneal_body<1, 2, kCsrUnit, true, BLOCK, false>(a, w.y, smem); break;
        case kBatchUnitGlb2: anneal_body<1, 2, kCsrUnit, false, BLOCK, false>(a, w.y, smem); break;
        case kBatchUnitLds4: anneal_body<1, 4, kCsrUnit, true, BLOCK, false>(a, w.y, smem); break;
        case kBatchUnitGlb4: anneal_body<1, 4, kCsrUnit, false, BLOCK, false>(a, w.y, smem); break;
        case kBatchP32Lds2: anneal_body<1, 2, kCsrPack32, true, BLOCK, false>(a, w.y, smem); break;
        case kBatchP32Glb2: anneal_body<1, 2, kCsrPack32, false, BLOCK, false>(a, w.y, smem); break;
        case kBatchPairGlb2: anneal_body<1, 2, kCsrPair, false, BLOCK, false>(a, w.y, smem); break;
        case kBatchP32Lds4T: anneal_body<4, 1, kCsrPack32, true, BLOCK, false>(a, w.y, smem); break;
        case kBatchP32Glb4T: anneal_body<4, 1, kCsrPack32, false, BLOCK, false>(a, w.y, smem); break;
        case kBatchPairGlb4T: anneal_body<4, 1, kCsrPair, false, BLOCK, false>(a, w.y, smem); break;
        case kBatchEll1Unit: ell1_body<false>(a, w.y, smem); break;
        case kBatchEll1: ell1_body<true>(a, w.y, smem); break;
        case kBatchEll4 + kEllUnit: ell4_body<kEllUnit>(a, w.y, smem); break;
        case kBatchEll4 + kEllByte: ell4_body<kEllByte>(a, w.y, smem); break;
        case kBatchEll4 + kEllHalf: ell4_body<kEllHalf>(a, w.y, smem); break;
        default: break;
    }
}

}  // namespace

hipError_t launch_anneal_batch(hipStream_t stream, const BatchJob *jobs, const int2 *work,
                               int32_t nwork, int32_t block, size_t lds_bytes) {
    if (nwork <= 0) return hipSuccess;
    const void *kern;
    switch (block) {
        case 256: kern = reinterpret_cast<const void *>(anneal_batch_kernel<256>); break;
        case 512: kern = reinterpret_cast<const void *>(anneal_batch_kernel<512>); break;
        case 1024: kern = reinterpret_cast<const void *>(anneal_batch_kernel<1024>); break;
        default: return hipErrorInvalidValue;
    }
    hipError_t err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         static_cast<int>(lds_bytes));
    if (err != hipSuccess) return err;
    switch (block) {
        case 256:
            hipLaunchKernelGGL(anneal_batch_kernel<256>, dim3(nwork), dim3(256), lds_bytes, stream, jobs, work);
            break;
        case 512:
            hipLaunchKernelGGL(anneal_batch_kernel<512>, dim3(nwork), dim3(512), lds_bytes, stream, jobs, work);
            break;
        default:
            hipLaunchKernelGGL(anneal_batch_kernel<1024>, dim3(nwork), dim3(1024), lds_bytes, stream, jobs, work);
            break;
    }
    return hipGetLastError();
}

}  // namespace psa
