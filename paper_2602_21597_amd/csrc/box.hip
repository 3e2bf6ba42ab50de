// Box-embedding operator family (the paper's Sec. 5.1 lists the box model among the
// backbones trained on the framework): the two operator pieces that are not MLPs.
// Projections translate the centre and widen the offset by the relation's rows, and
// the offset of an intersection is the smallest input offset shrunk by a gate
// computed from all inputs (pool.h).  Both are memory bound: one thread per (member, 4
// coordinates), rows read and written once.
#include "pool.h"

namespace ngdb {
namespace {

template <bool BWD>
__device__ __forceinline__ void proj_body(const BoxProjArgs& a, size_t t) {
    const int d4 = a.d >> 2;
    if (t >= (size_t)a.n * d4) return;
    const int i = (int)(t / d4), c = (int)(t % d4);
    const size_t out = ((size_t)(a.out_base + i) * a.d >> 2) + c;
    if (BWD) {
        const size_t in = ((size_t)a.gslot[i] * a.d >> 2) + c;
        reinterpret_cast<float4*>(a.dact_c)[in] = reinterpret_cast<const float4*>(a.dact_c)[out];
        reinterpret_cast<float4*>(a.dact_o)[in] = reinterpret_cast<const float4*>(a.dact_o)[out];
        return;
    }
    const int32_t ref = a.ref[i];
    const size_t r = ((size_t)a.rel[i] * a.d >> 2) + c;
    float4 x, o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ref >= 0) {
        const size_t in = ((size_t)ref * a.d >> 2) + c;
        x = reinterpret_cast<const float4*>(a.act_c)[in];
        o = reinterpret_cast<const float4*>(a.act_o)[in];
    } else {
        x = reinterpret_cast<const float4*>(a.E)[((size_t)(-1 - ref) * a.d >> 2) + c];
    }
    const float4 rc = reinterpret_cast<const float4*>(a.Rc)[r];
    const float4 ro = reinterpret_cast<const float4*>(a.Ro)[r];
    x.x += rc.x; x.y += rc.y; x.z += rc.z; x.w += rc.w;
    o.x += fmaxf(ro.x, 0.f); o.y += fmaxf(ro.y, 0.f); o.z += fmaxf(ro.z, 0.f); o.w += fmaxf(ro.w, 0.f);
    reinterpret_cast<float4*>(a.act_c)[out] = x;
    reinterpret_cast<float4*>(a.act_o)[out] = o;
}

template <bool BWD>
__global__ __launch_bounds__(256) void box_proj_kernel(const BoxProjArgs a) {
    proj_body<BWD>(a, (size_t)blockIdx.x * blockDim.x + threadIdx.x);
}

template <bool BWD>
__global__ __launch_bounds__(pool::THREADS) void box_offset_kernel(const InterJobs jobs) {
    pool::member<BWD, true>(jobs.job[blockIdx.y], jobs.d, (size_t)blockIdx.x * pool::THREADS + threadIdx.x);
}

// centre and offset jobs of one level in one launch (the job kind is uniform per workgroup)
template <bool BWD>
__global__ __launch_bounds__(pool::THREADS) void box_pool_kernel(const BoxPoolJobs bj) {
    const size_t t = (size_t)blockIdx.x * pool::THREADS + threadIdx.x;
    if ((int)blockIdx.y == bj.jobs.count) {     // the projections riding along
        proj_body<BWD>(bj.proj, t);
        return;
    }
    const InterJob jb = bj.jobs.job[blockIdx.y];
    if ((bj.gate_mask >> blockIdx.y) & 1u) pool::member<BWD, true>(jb, bj.jobs.d, t);
    else pool::member<BWD, false>(jb, bj.jobs.d, t);
}

}  // namespace

hipError_t launch_box_proj(const BoxProjArgs& a, bool backward, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    if (a.d & 3) return hipErrorInvalidValue;
    const size_t work = (size_t)a.n * (a.d >> 2);
    const dim3 grid((unsigned)((work + 255) / 256));
    if (backward) hipLaunchKernelGGL((box_proj_kernel<true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((box_proj_kernel<false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_box_offset(const InterJobs& jobs, bool backward, hipStream_t s) {
    if (jobs.count <= 0) return hipSuccess;
    if (jobs.count > INTER_MAX_JOBS) return hipErrorInvalidValue;
    size_t most = 0;
    for (int i = 0; i < jobs.count; ++i) {
        if (jobs.job[i].n <= 0 || jobs.job[i].k < 1 || jobs.job[i].k > NGDB_MAX_CARD) return hipErrorInvalidValue;
        most = std::max(most, (size_t)jobs.job[i].n * (jobs.d >> 2));
    }
    if (jobs.d & 3) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((most + pool::THREADS - 1) / pool::THREADS), jobs.count), block(pool::THREADS);
    if (backward) hipLaunchKernelGGL((box_offset_kernel<true>), grid, block, 0, s, jobs);
    else hipLaunchKernelGGL((box_offset_kernel<false>), grid, block, 0, s, jobs);
    return hipGetLastError();
}

hipError_t launch_box_pool(const BoxPoolJobs& bj, bool backward, hipStream_t s) {
    const InterJobs& jobs = bj.jobs;
    if (jobs.count <= 0) return hipSuccess;
    if (jobs.count > INTER_MAX_JOBS) return hipErrorInvalidValue;
    size_t most = 0;
    for (int i = 0; i < jobs.count; ++i) {
        if (jobs.job[i].n <= 0 || jobs.job[i].k < 1 || jobs.job[i].k > NGDB_MAX_CARD) return hipErrorInvalidValue;
        most = std::max(most, (size_t)jobs.job[i].n * (jobs.d >> 2));
    }
    if (bj.has_proj) {
        if (bj.proj.n <= 0 || (bj.proj.d & 3)) return hipErrorInvalidValue;
        most = std::max(most, (size_t)bj.proj.n * (bj.proj.d >> 2));
    }
    if (jobs.d & 3) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((most + pool::THREADS - 1) / pool::THREADS), jobs.count + (bj.has_proj ? 1 : 0)), block(pool::THREADS);
    if (backward) hipLaunchKernelGGL((box_pool_kernel<true>), grid, block, 0, s, bj);
    else hipLaunchKernelGGL((box_pool_kernel<false>), grid, block, 0, s, bj);
    return hipGetLastError();
}

}  // namespace ngdb
