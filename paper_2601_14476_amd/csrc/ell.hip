// ell.hip -- launches of the streaming sweeps (ell_sweep.hpp) and the kernel
// that lays a graph's rows out for them.
#include <hip/hip_runtime.h>

#include "ell_sweep.hpp"
#include "engine.hpp"

namespace psa {
namespace {

template <bool WEIGHTS>
__global__ __launch_bounds__(1024) void ell1_kernel(AnnealArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    ell1_body<WEIGHTS>(a, static_cast<int32_t>(blockIdx.x), smem);
}

template <int MODE>
__global__ __launch_bounds__(1024) void ell4_kernel(AnnealArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    ell4_body<MODE>(a, static_cast<int32_t>(blockIdx.x), smem);
}

// Workgroup (w, c) writes kBuildGroups pairs of entries of wavefront w's 64
// tasks: thread (lane, row p of the lane's task) walks its part of the row and
// pads it to the wavefront's length.  Bound by the latency of its gathers, so
// rows are cut into parts.
constexpr int32_t kBuildGroups = 4;
__global__ __launch_bounds__(256) void build_ell_kernel(int32_t tasks, int32_t n4, const int32_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const int32_t *__restrict__ val,
                                                        const int32_t *__restrict__ gorder,
                                                        const int32_t *__restrict__ wofs, uint32_t *__restrict__ e4,
                                                        uint32_t *__restrict__ e1, uint32_t *__restrict__ e1j) {
    const int32_t w = static_cast<int32_t>(blockIdx.x);
    const int32_t p = static_cast<int32_t>(threadIdx.x) & 3, lane = static_cast<int32_t>(threadIdx.x) >> 2;
    const int32_t slot = 64 * w + lane;
    const int32_t i = slot < tasks ? 4 * gorder[slot] + p : 0;
    const int32_t b = slot < tasks ? row_ptr[i] : 0, e = slot < tasks ? row_ptr[i + 1] : 0;
    const int32_t g0 = wofs[w] + static_cast<int32_t>(blockIdx.y) * kBuildGroups, g1 = min(g0 + kBuildGroups, wofs[w + 1]);
    for (int32_t g = g0; g < g1; ++g) {
        uint32_t idx[2], mag[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int32_t x = b + 2 * (g - wofs[w]) + h;
            const int32_t j = x < e ? col[x] : 0, J = x < e ? val[x] : 0;
            const uint32_t neg = J < 0 ? 1u : 0u;
            mag[h] = static_cast<uint32_t>(neg ? -J : J);
            idx[h] = static_cast<uint32_t>(x < e ? j + (neg ? n4 : 0) : 2 * n4);
            if (e4)
                e4[(static_cast<size_t>(2 * g + h) * 64 + lane) * 4 + p] =
                    x < e ? 8u * static_cast<uint32_t>(j) | mag[h] << 18 | neg << 31 : 8u * static_cast<uint32_t>(n4);
        }
        const size_t at = (static_cast<size_t>(g) * 64 + lane) * 4 + p;
        e1[at] = idx[0] | idx[1] << 16;
        if (e1j) e1j[at] = mag[0] | mag[1] << 16;
    }
}

}  // namespace

hipError_t launch_ell(hipStream_t stream, const AnnealArgs &args, const AnnealPlan &plan, int32_t e4_mode) {
    void (*kern)(AnnealArgs);
    if (plan.tpw == 4)
        kern = e4_mode == kEllUnit ? ell4_kernel<kEllUnit>
                                   : (e4_mode == kEllByte ? ell4_kernel<kEllByte> : ell4_kernel<kEllHalf>);
    else
        kern = args.e1j ? ell1_kernel<true> : ell1_kernel<false>;
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               static_cast<int>(plan.lds_bytes));
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(plan.grid), dim3(plan.block), plan.lds_bytes, stream, args);
    return hipGetLastError();
}

hipError_t launch_build_ell(hipStream_t stream, int32_t waves, int32_t most, int32_t tasks, int32_t n4, const int32_t *row_ptr,
                            const int32_t *col, const int32_t *val, const int32_t *gorder, const int32_t *wofs,
                            uint32_t *e4, uint32_t *e1, uint32_t *e1j) {
    if (waves <= 0 || most <= 0) return hipSuccess;
    hipLaunchKernelGGL(build_ell_kernel, dim3(waves, (most + kBuildGroups - 1) / kBuildGroups), dim3(256),
                       0, stream, tasks, n4, row_ptr, col, val, gorder, wofs,
                       e4, e1, e1j);
    return hipGetLastError();
}

}  // namespace psa
