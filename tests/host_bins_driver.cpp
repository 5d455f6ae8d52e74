// Host-only model of what the library's calls do to the bin counts, built with g++
// by tests/host_model.py: pm_api.cpp as it is, over launchers that only
// track whether a context's counts are zero, counted or unknown on the device.  A
// kernel that counts must find them zero and a sort must find them counted exactly
// once; anything else would write the order out of range on a GPU.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <vector>

#include "host_cosmo.h"
#include "kernels.h"
#include "pm.h"

namespace {

enum State { kUnknown, kZero, kPresent, kOrdered };   // kOrdered: sorted, not yet cleared
std::map<const void*, State> counts;
bool executing = true;   // false: calls are captured, and never replayed
int copies_until_failure = -1;
bool scatter_fails = false;   // its launch
hipError_t last_error = hipSuccess;
const char* where = "";

long checks = 0;
std::map<void*, size_t> pinned;
bool memory_is_short = false;   // ordinary allocations throw

void need(const void* p, State want, const char* what) {
    ++checks;
    if (!executing || counts[p] == want) return;
    std::printf("%s: %s with counts in state %d\n", where, what, (int)counts[p]);
    std::exit(1);
}
void set(const void* p, State s) {
    if (executing) counts[p] = s;
}
void count(const pmx::Bins& b, const char* what) {
    need(b.counts, kZero, what);
    set(b.counts, kPresent);
}

}  // namespace

void* operator new(size_t n) {
    void* p = memory_is_short ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// ------------------------------------------------------------------ HIP runtime
extern "C" {
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
    if (copies_until_failure >= 0 && copies_until_failure-- == 0) return hipErrorUnknown;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = executing ? hipStreamCaptureStatusNone : hipStreamCaptureStatusActive;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0.f;
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::calloc(n, 1);
    pinned[*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    pinned.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
}

// ------------------------------------------------------------------ launchers
namespace pmx {

void fill_stage_twiddles(float2*) {}
int device_cus() { return 256; }
int choose_tile(int ng) { return ng >= 256 ? 16 : (ng >= 16 ? 8 : 4); }
long scan_tmp_elems(long nkeys) { return nkeys / 4096 + 2; }
long gather_partials(int, int ng) { return (long)ng * ng; }
int particle_blocks(long P) { return (int)((P + 255) / 256); }
long mlp_backward_scratch(int) { return 4417; }

void launch_zero(void* p, size_t, hipStream_t) { set(p, kZero); }
void launch_bin(const uint32_t*, const Lattice&, Bins& b, Counted counted, hipStream_t s) {
    if (counted == kNotCounted) {
        launch_bin_zero(b, s);
        count(b, "count");
    }
    need(b.counts, kPresent, "sort");
    set(b.counts, b.nkeys() <= 4096 ? kOrdered : kZero);
}
void launch_scatter_density(const uint32_t*, const Lattice&, const Bins& b, float*, float*,
                            hipStream_t) {
    if (scatter_fails) {
        last_error = hipErrorUnknown;
        return;
    }
    if (counts[b.counts] == kOrdered) set(b.counts, kZero);
}
void launch_to_fixed_count(const float*, uint32_t*, const Lattice&, Bins& b, hipStream_t s) {
    launch_bin_zero(b, s);
    count(b, "positions");
}
void launch_gather_kick_drift(uint32_t*, int32_t*, const uint32_t*, const float*, long,
                              const Lattice&, const Bins& b, float, float, int drift, uint32_t*,
                              int32_t*, unsigned*, bool count_bins, hipStream_t) {
    if (drift && count_bins) count(b, "drift");
}
void launch_wgrad(const float*, long, float, uint32_t*, const int32_t*, float*, float*,
                  const Lattice&, const Bins& b, float, int mode, double*, hipStream_t, bool,
                  bool count_bins, float*) {
    if (mode == 1 && count_bins) count(b, "un-drift");
}
void launch_undrift(uint32_t*, const int32_t*, const float*, float*, const Lattice&, const Bins& b,
                    float, double*, float*, int, hipStream_t) {
    count(b, "first un-drift");
}

}  // namespace pmx

// the other launchers, doing nothing: generated from kernels.h by the test
#include "no_work.inc"

namespace {

struct Run {
    std::vector<char> memory;
    pm_ctx* ctx = nullptr;
    pm_config cfg;
    float x[8];

    explicit Run(const pm_config& c) : cfg(c) {
        const pm_cosmology co{0.3, 0.05, 0.7, 0.8, 0.96, 2.7255};
        const size_t n = pm_workspace_bytes(&c, nullptr);
        memory.resize(n + 256);
        char* p = memory.data() + (256 - reinterpret_cast<uintptr_t>(memory.data()) % 256);
        counts.clear();   // memory of any contents
        if (pm_init(&c, &co, p, n, nullptr, &ctx) != PM_OK) std::exit(2);
        if (c.filter && pm_set_filter(ctx, x) != PM_OK) std::exit(2);
    }
    ~Run() { pm_destroy(ctx); }
    int forward() { return pm_forward(ctx, x, x, x, x); }
    int adjoint(bool mom) { return pm_adjoint(ctx, x, x, mom ? x : nullptr, x, nullptr, nullptr); }
    void blocks() {
        pm_density(ctx, x, x);
        pm_force(ctx, x, 0.5, x);
        pm_force_vjp(ctx, x, 0.5, x, x);
    }
    void everything() {
        if (forward() != PM_OK) std::exit(3);
        for (bool mom : {false, true}) {
            if (adjoint(mom) != PM_OK) std::exit(3);
            blocks();
        }
        if (forward() != PM_OK || forward() != PM_OK || adjoint(true) != PM_OK) std::exit(3);
    }
};

}  // namespace

// kernel_bytes of one step and its adjoint: family, bytes
int print_bytes(int mesh, int filter, bool density, bool displacement, bool momentum) {
    const pm_config c{8, mesh, 32.0, 1.0 / 64, 0.5, 1, 0, filter, PM_F_TIMING};
    Run r(c);
    if (r.forward() != PM_OK || pm_stats_reset(r.ctx) != PM_OK) return 1;
    float* x = r.x;
    if (pm_adjoint(r.ctx, density ? x : nullptr, displacement ? x : nullptr,
                   momentum ? x : nullptr, x, nullptr, nullptr) != PM_OK)
        return 1;
    pm_stats s;
    if (pm_stats_get(r.ctx, &s) != PM_OK) return 1;
    for (int k = 0; k < PM_NKERNELS; ++k) std::printf("%.0f\n", s.kernel_bytes[k]);
    return 0;
}

int main(int argc, char** argv) {
    if (argc == 6)
        return print_bytes(std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]),
                           std::atoi(argv[4]), std::atoi(argv[5]));
    for (int ng : {8, 128})
        for (int steps : {1, 5})
            for (int ckpt : {0, 1, 2})
                for (int mode : {0, 3}) {
                    static char name[80];
                    std::snprintf(name, sizeof(name), "mesh %d steps %d checkpoint %d mode %d", ng,
                                  steps, ckpt, mode);
                    where = name;
                    const pm_config c{8, ng, 32.0, 1.0 / 64, 0.5, steps, ckpt, mode & 1,
                                      mode & 2 ? (uint64_t)PM_F_2LPT : 0};
                    {
                        Run r(c);
                        r.everything();
                        // calls without a host result need no host memory: an
                        // exception must not leave a C entry
                        memory_is_short = true;
                        r.blocks();
                        if (r.forward() != PM_OK) return 10;
                        memory_is_short = false;
                    }
                    {   // calls that are captured, and the captures dropped
                        Run r(c);
                        executing = false;
                        r.blocks();
                        r.forward();
                        executing = true;
                        r.blocks();
                        r.everything();
                    }
                    // every copy of an adjoint fails in turn, with calls of every kind next
                    for (int k = 0; ckpt == 1 && k < 12; ++k) {
                        Run r(c);
                        if (r.forward() != PM_OK) return 3;
                        copies_until_failure = k;
                        const int rc = r.adjoint(k & 1);
                        const bool failed = copies_until_failure < 0;
                        copies_until_failure = -1;
                        if ((rc == PM_EHIP) != failed) return 4;
                        if (k % 3 == 0) r.blocks();
                        if (k % 3 == 1) {
                            executing = false;
                            r.blocks();
                            executing = true;
                            r.blocks();
                        }
                        r.everything();
                    }
                    {   // a launch fails
                        Run r(c);
                        scatter_fails = true;
                        const int rc = pm_density(r.ctx, r.x, r.x);
                        scatter_fails = false;
                        if (rc != PM_EHIP) return 5;
                        r.everything();
                    }
                }
    // pinned memory kept from many contexts at a time: bounded, and used again
    pm_config c{8, 8, 32.0, 1.0 / 64, 0.5, 1, 0, 0, 0};
    for (int turn = 0; turn < 2; ++turn) {
        std::vector<Run*> runs;
        for (int k = 0; k < 40; ++k) {
            c.mesh = k % 2 ? 8 : 256;
            runs.push_back(new Run(c));
        }
        if (pinned.size() != 40) return 6;
        for (Run* r : runs) delete r;
        size_t bytes = 0;
        for (auto& b : pinned) bytes += b.second;
        if (pinned.size() > 32 || bytes > (1u << 20)) return 7;
    }
    // a block that a failed call may still write to is not kept
    const size_t before = pinned.size();
    {
        Run r(c);
        if (pinned.size() != before) return 8;
        last_error = hipErrorUnknown;
        if (pm_density(r.ctx, r.x, r.x) != PM_EHIP) return 8;
    }
    if (pinned.size() != before - 1) return 9;
    std::printf("ok %ld\n", checks);
    return 0;
}
