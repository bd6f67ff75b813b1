// A host stand-in for the HIP runtime and for the kernel launchers, so that the host interface
// (lbdem_api.cpp) runs without a device: device memory is host memory, every queued operation
// completes at once, and a launcher writes recognisable values instead of running a kernel.
// Test switches: host_hold(ms) makes the first read launch wait until another one follows or
// the time is over; host_fail_new(bytes) makes operator new fail from that size on.
#include <chrono>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

#include "../paper_1808_08921_amd/csrc/lbdem_internal.hpp"

static size_t g_fail_new = 0;

void *operator new(size_t n)
{
    void *p = (g_fail_new && n >= g_fail_new) ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new[](size_t n, const std::nothrow_t &) noexcept
{
    return (g_fail_new && n >= g_fail_new) ? nullptr : std::malloc(n ? n : 1);
}
void operator delete[](void *p) noexcept { std::free(p); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

namespace {

std::mutex g_mu;
std::condition_variable g_cv;
int g_hold_ms = 0, g_launches = 0;

// called at the end of a read's launch, its values written
void hold()
{
    std::unique_lock<std::mutex> lk(g_mu);
    const int mine = ++g_launches;
    g_cv.notify_all();
    if (mine == 1 && g_hold_ms > 0)
        g_cv.wait_for(lk, std::chrono::milliseconds(g_hold_ms), [] { return g_launches > 1; });
}

} // namespace

extern "C" {
void host_hold(int ms)
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_hold_ms = ms;
    g_launches = 0;
}
int host_launches() { return g_launches; }
void host_fail_new(size_t n) { g_fail_new = n; }

hipError_t hipMalloc(void **p, size_t n) { return (*p = std::aligned_alloc(256, (n + 255) / 256 * 256)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "host stand-in"; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t *, unsigned int) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphAddKernelNode(hipGraphNode_t *, hipGraph_t, const hipGraphNode_t *, size_t, const hipKernelNodeParams *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
}

namespace lbdem {

hipError_t launch_particles_out(const DevSet &, int p0, int n, double *out, hipStream_t)
{
    for (int k = 0; k < 15 * n; ++k) out[k] = 1000.0 * p0 + k;
    hold();
    return hipSuccess;
}
hipError_t launch_fields(int, const DevSet &, int m, long long ncell, double *out, hipStream_t)
{
    for (long long k = 0; k < 4 * ncell; ++k) out[k] = m + 1.0;
    hold();
    return hipSuccess;
}

hipError_t launch_refresh(int, const DevSet &, hipStream_t) { return hipSuccess; }
hipError_t launch_links(int, const DevSet &, hipStream_t) { return hipSuccess; }
hipError_t launch_motion(const DevSet &, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_fluid(int, const DevSet &, hipStream_t) { return hipSuccess; }
hipError_t launch_remap(int, const DevSet &, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_init_pops(int, const DevSet &, long long, hipStream_t) { return hipSuccess; }
hipError_t launch_expand(int, const DevSet &, hipStream_t) { return hipSuccess; }
void *refresh_kernel_ptr(int) { return nullptr; }
bool links_fused(const DevSet &) { return true; }
void *links_kernel_ptr(int, const DevSet &) { return nullptr; }
void *motion_kernel_ptr(const DevSet &) { return nullptr; }
void *fluid_kernel_ptr(int, int, int) { return nullptr; }
void *remap_kernel_ptr(int, const DevSet &) { return nullptr; }
int refresh_grid(const DevSet &) { return 1; }
dim3 links_grid(const DevSet &) { return dim3(1); }
int links_block(const DevSet &) { return 64; }
int motion_grid(const DevSet &) { return 1; }
int remap_grid(const DevSet &) { return 1; }
hipError_t launch_adj_geometry(const AdjDev &, const int *, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_start(int, const AdjDev &, const void *, void *, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_wall(int, const AdjDev &, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_step(int, const AdjDev &, const void *, void *, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_signal(const AdjDev &, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_back(int, const AdjDev &, const void *, const void *, void *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_adj_vgrad(const AdjDev &, hipStream_t) { return hipSuccess; }
int adj_blocks(const AdjDev &a) { return (a.ns + 255) / 256; }
DftPlan dft_plan(long long, int, int, int) { return DftPlan{}; }
hipError_t launch_st_dft(const DftPlan &, const double *, long long, int, const double *, double, double, double, int,
                         double, double, int, double *, int *, void *, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_wave_fit(const double *, long long, int, const double *, double, double, double *, void *,
                           hipStream_t) { return hipErrorNotSupported; }
hipError_t noalloc_scratch(void **) { return hipErrorNotSupported; }
hipError_t launch_particle_signal(const double *, int, int, int, long long, long long, const int *, const int *, int,
                                  int, double *, hipStream_t) { return hipErrorNotSupported; }
hipError_t launch_probe_signal(const double *, int, int, long long, long long, int, double *, hipStream_t)
{
    return hipErrorNotSupported;
}

} // namespace lbdem
