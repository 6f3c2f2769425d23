// Patch kernels for fabrics of one patch (no exchange), and the launcher of all patch kernels.
#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

PatchKernel multi_kernel_sum(const PatchShape &s);
PatchKernel multi_kernel_max(const PatchShape &s);

namespace {

// every word of the exchange starts with the sign of an exchange that has not happened yet
__global__ __launch_bounds__(256) void k_patch_clear(unsigned long long *parts, int64_t n_parts,
                                                     unsigned long long *maxima, int64_t n_maxima,
                                                     uint32_t *abort_word, double *lambda,
                                                     int plans)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < n_parts; i += stride) parts[i] = kSign;
    for (int64_t i = i0; i < n_maxima; i += stride) maxima[i] = kSign;
    for (int64_t i = i0; i < plans; i += stride) lambda[i] = 0.0;
    if (i0 == 0) *abort_word = 0u;
}

PatchKernel kernel_of(const DevicePatches &p, bool cost_max)
{
    if (p.n_patches > 1) return cost_max ? multi_kernel_max(p.shape) : multi_kernel_sum(p.shape);
    return cost_max ? kernel_for<true, false>(p.shape) : kernel_for<false, false>(p.shape);
}

}  // namespace

}  // namespace patch

size_t patch_lds_bytes(const DevicePatches &p)
{
    return static_cast<size_t>(patch::lds_layout(p.max_local, p.max_groups, p.max_comm,
                                                 p.shape.lanes * p.shape.quads)
                                   .bytes);
}

int patch_blocks_per_cu(const DevicePatches &p, bool cost_max)
{
    const patch::PatchKernel k = patch::kernel_of(p, cost_max);
    const size_t lds = patch_lds_bytes(p);
    if (k == nullptr || lds > 160 * 1024) return 0;
    const void *f = reinterpret_cast<const void *>(k);
    int n = 0;
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) !=
            hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, p.shape.threads, lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

hipError_t launch_patches(const DeviceTopo &t, const DevicePatches &p, int32_t plans,
                          const double *demand, const double *len_in, double *len_out, double eps,
                          int32_t iters, uint32_t spin_limit, double *splits, double *lambda,
                          hipStream_t s)
{
    const patch::PatchKernel k = patch::kernel_of(p, t.cost_max);
    if (k == nullptr) return hipErrorInvalidValue;
    PatchArgs a;
    a.desc = p.desc;
    a.loc_link = p.loc_link;
    a.comm = p.comm;
    a.group = p.group;
    a.words = p.words;
    a.first = p.first;
    a.comm_ptr = t.comm_ptr;
    a.invcap = t.invcap;
    a.demand = demand;
    a.len_in = len_in;
    a.len_out = len_out;
    a.splits = splits;
    a.lambda = lambda;
    a.parts = p.parts;
    a.maxima = p.maxima;
    a.abort_word = p.abort_word;
    a.n_parts = p.n_parts;
    a.K = t.K;
    a.P = t.P;
    a.n_patches = p.n_patches;
    a.plans = plans;
    a.teams = plans < p.max_teams ? plans : p.max_teams;
    a.iters = iters;
    a.spin_limit = spin_limit;
    a.eps = eps;
    const size_t lds = patch_lds_bytes(p);
    const void *f = reinterpret_cast<const void *>(k);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    void *args[] = {&a};
    if (p.n_patches == 1)
        return hipLaunchKernel(f, dim3(plans), dim3(p.shape.threads), args, lds, s);
    const int64_t words = a.teams * 2 * p.n_parts;
    int64_t grid = (words + 255) / 256;
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(patch::k_patch_clear, dim3(static_cast<unsigned>(grid)), dim3(256), 0, s,
                       reinterpret_cast<unsigned long long *>(p.parts), words,
                       reinterpret_cast<unsigned long long *>(p.maxima),
                       static_cast<int64_t>(a.teams) * 2 * p.n_patches, p.abort_word, lambda,
                       plans);
    // patches wait for each other, so all of them have to be resident at once: a cooperative
    // launch is refused otherwise
    return hipLaunchCooperativeKernel(f, dim3(a.teams * p.n_patches), dim3(p.shape.threads), args,
                                      static_cast<unsigned>(lds), s);
}

}  // namespace nimble
