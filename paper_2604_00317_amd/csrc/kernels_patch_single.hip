// Patch kernels for fabrics of one patch (no exchange), and the launcher of all patch kernels.
#include <algorithm>

#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

PatchKernel multi_kernel_sum(const PatchShape &s);
PatchKernel multi_kernel_max(const PatchShape &s);
PatchKernel adaptive_kernel(const PatchShape &s, bool multi);
PatchKernel block_kernel_sum(const PatchShape &s);
PatchKernel block_kernel_max(const PatchShape &s);

namespace {

// Every word of the exchange starts with the sign of an exchange that has not happened yet.
__global__ __launch_bounds__(256) void k_patch_clear(unsigned long long *parts, int64_t n_parts,
                                                     unsigned long long *maxima, int64_t n_maxima,
                                                     unsigned long long *terms, int64_t n_terms,
                                                     uint32_t *abort_word, uint32_t given_up,
                                                     int32_t *ad_flags, double *lambda, int plans,
                                                     const double *len, double *len_start, int E)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < n_parts; i += stride) parts[i] = kSign;
    for (int64_t i = i0; i < n_maxima; i += stride) maxima[i] = kSign;
    for (int64_t i = i0; i < n_terms; i += stride) terms[i] = kSign;
    for (int64_t i = i0; i < plans; i += stride) lambda[i] = 0.0;
    if (len != nullptr)
        for (int64_t i = i0; i < E; i += stride) len_start[i] = len[i];
    if (i0 == 0) {
        *abort_word = given_up;
        if (ad_flags != nullptr) ad_flags[0] = 0;
    }
}

PatchKernel kernel_of(const DevicePatches &p, bool cost_max, bool adaptive)
{
    if (p.shape.blocks) {
        if (adaptive || p.n_patches == 1) return nullptr;
        return cost_max ? block_kernel_max(p.shape) : block_kernel_sum(p.shape);
    }
    if (adaptive) return cost_max ? nullptr : adaptive_kernel(p.shape, p.n_patches > 1);
    if (p.n_patches > 1) return cost_max ? multi_kernel_max(p.shape) : multi_kernel_sum(p.shape);
    return cost_max ? kernel_for<true, false, false>(p.shape)
                    : kernel_for<false, false, false>(p.shape);
}

}  // namespace

}  // namespace patch

size_t patch_lds_bytes(const DevicePatches &p, bool adaptive)
{
    if (p.shape.blocks)
        return static_cast<size_t>(block_lds(p.max_local, p.max_heads, p.max_tails, p.max_comm, p.max_at,
                                             p.shape, 8).bytes);
    return static_cast<size_t>(patch::lds_layout(p.max_local, p.max_groups, p.max_at, p.max_comm,
                                                 p.shape.lanes * p.shape.quads, adaptive ? 32 : 8)
                                   .bytes);
}

int patch_blocks_per_cu(const DevicePatches &p, bool cost_max, bool adaptive)
{
    const patch::PatchKernel k = patch::kernel_of(p, cost_max, adaptive);
    const size_t lds = patch_lds_bytes(p, adaptive);
    if (k == nullptr || lds > kPatchLdsBytes) return 0;
    const void *f = reinterpret_cast<const void *>(k);
    int n = 0;
    // (the limit belongs to the kernel, which topologies with patches of other sizes share: it is
    // always set to all there is)
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                            kPatchLdsBytes) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, p.shape.threads, lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

hipError_t launch_patches(const DeviceTopo &t, const DevicePatches &p, int32_t plans,
                          const double *demand, double *len_io, double eps,
                          int32_t iters, uint32_t spin_limit, double *splits, double *lambda,
                          hipStream_t s, const PatchAdaptive *adaptive)
{
    const patch::PatchKernel k = patch::kernel_of(p, t.cost_max, adaptive != nullptr);
    if (k == nullptr) return hipErrorInvalidValue;
    PatchArgs a = {};
    a.desc = p.desc;
    a.loc_link = p.loc_link;
    a.comm = p.comm;
    a.group = p.group;
    a.words = p.words;
    a.first = p.first;
    a.heads = p.heads;
    a.tails = p.tails;
    a.comm_ptr = t.comm_ptr;
    a.invcap = t.invcap;
    a.demand = demand;
    // several patches start from a copy of the lengths: a solve that is given up half way has
    // overwritten some of the caller's, and some patches may not have started by then
    const bool warm = len_io != nullptr;
    a.len_in = warm && p.n_patches > 1 ? p.len_start : len_io;
    a.len_out = len_io;
    a.splits = splits;
    a.lambda = lambda;
    a.parts = p.parts;
    a.maxima = p.maxima;
    a.abort_word = p.abort_word;
    a.n_parts = p.n_parts;
    a.K = t.K;
    a.P = t.P;
    a.E = t.E;
    a.n_patches = p.n_patches;
    a.plans = plans;
    // The words of a team that keeps to one XCD go from patch to patch through that XCD's L2 (sixteen
    // plans of the 16-node fabric, 16 patches each: 4.56 -> 3.87 ms; patches of a team spread over the
    // XCDs, neighbours side by side on one, were slower than dealt out in turn: 16 nodes, variable step
    // 5.9 -> 7.5 ms).
    const bool near = teams_keep_near(p.teams, plans);
    a.teams = std::min(plans, near ? p.teams.near : p.teams.spread);
    a.near_xcds = near ? p.xcds : 1;
    a.by_xcd = a.teams == 1 && p.xcds == kPatchXcds && p.n_patches >= kPatchXcds &&
               p.n_patches <= kPatchXcds * kPatchXcdPatches;
    a.row = p.row;
    a.max_users = p.max_users;
    a.at = p.at;
    const int32_t blocks = a.near_xcds * p.n_patches * ((a.teams + a.near_xcds - 1) / a.near_xcds);
    a.iters = iters;
    a.spin_limit = spin_limit;
    a.eps = eps;
    int64_t n_terms = 0;
    if (adaptive != nullptr) {
        a.terms = adaptive->terms;
        a.idle = adaptive->idle;
        a.n_idle = adaptive->n_idle;
        a.check_every = adaptive->check_every;
        a.ad_flags = adaptive->flags;
        a.ad_scalars = adaptive->scalars;
        a.abort_word = adaptive->abort_word;
        n_terms = patch_adaptive_words(t.K, t.E);
    }
    const size_t lds = patch_lds_bytes(p, adaptive != nullptr);
    const void *f = reinterpret_cast<const void *>(k);
    void *args[] = {&a};
    if (p.n_patches == 1 && adaptive == nullptr)
        return hipLaunchKernel(f, dim3(plans), dim3(p.shape.threads), args, lds, s);
    const int64_t words = p.n_patches > 1 ? a.teams * 2 * p.n_parts : 0;
    const int64_t maxima =
        p.n_patches > 1 ? static_cast<int64_t>(a.teams) * patch_meeting_words(p.n_patches)
                         : 0;
    // (patches that share no link have no parts, but maxima, an abort word and a lambda all the same)
    int64_t grid = (std::max({words, maxima, n_terms, static_cast<int64_t>(plans),
                             static_cast<int64_t>(warm ? t.E : 0)}) + 255) / 256;
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(patch::k_patch_clear, dim3(static_cast<unsigned>(grid)), dim3(256), 0, s,
                       reinterpret_cast<unsigned long long *>(p.parts), words,
                       reinterpret_cast<unsigned long long *>(p.maxima), maxima,
                       reinterpret_cast<unsigned long long *>(a.terms), n_terms, a.abort_word,
                       spin_limit == 0 ? 1u : 0u, a.ad_flags, lambda, plans, len_io, p.len_start, t.E);
    const hipError_t cleared = hipGetLastError();
    if (cleared != hipSuccess) return cleared;
    if (p.n_patches == 1) return hipLaunchKernel(f, dim3(1), dim3(p.shape.threads), args, lds, s);
    // patches wait for each other, so all of them have to be resident at once: a cooperative
    // launch is refused otherwise
    return hipLaunchCooperativeKernel(f, dim3(blocks), dim3(p.shape.threads), args, static_cast<unsigned>(lds), s);
}

}  // namespace nimble
