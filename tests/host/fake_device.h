// A device that is the host: the HIP calls and kernel launches that the library's
// host code makes, for checks of its host paths on the CPU.  Device memory is host
// memory, a launch does nothing but leave a line in the log, and any call can be
// made to fail.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <thread>
#include <vector>

#include "da_runtime.h"

namespace fake {

struct Call {
    std::string name;
    const void *stream = nullptr;   // of the call, if it has one
    const void *event = nullptr;
    std::thread::id thread;
};
struct State {
    std::recursive_mutex mu;
    std::vector<Call> log;
    std::map<std::string, int> fail_from;    // name -> calls left before it fails
    size_t memory = SIZE_MAX, used = 0;      // device memory, and what is allocated
    std::map<void *, size_t> live;
    hipError_t last = hipSuccess;            // as hipGetLastError keeps it
    std::vector<int> mix_blocks;             // workgroups of each mixed launch
    std::vector<dapt::JobDesc> mix_jobs;     // the jobs they ran
    std::vector<dapt::JobDesc> runs;         // launches of the table-driven step kernel
    uintptr_t handles = 0x1000;
};
inline State &st() {
    static State s;
    return s;
}
inline bool fails(const char *name) {
    auto it = st().fail_from.find(name);
    return it != st().fail_from.end() && it->second-- <= 0;
}
inline hipError_t note(const char *name, const void *stream = nullptr, const void *event = nullptr,
                       hipError_t error = hipErrorUnknown) {
    std::lock_guard<std::recursive_mutex> lock(st().mu);
    st().log.push_back(Call{name, stream, event, std::this_thread::get_id()});
    if (!fails(name)) return hipSuccess;
    return st().last = error;
}
// A launch reports, and clears, the error left by the calls before it.
inline int launched(const char *name, const void *stream) {
    std::lock_guard<std::recursive_mutex> lock(st().mu);
    hipError_t e = note(name, stream, nullptr, hipErrorLaunchFailure);
    if (e == hipSuccess) e = st().last;
    st().last = hipSuccess;
    return (int)e;
}
template <typename H>
void handle(H *h) {
    std::lock_guard<std::recursive_mutex> lock(st().mu);
    *h = reinterpret_cast<H>(st().handles += 16);
}
inline void reset() {
    std::lock_guard<std::recursive_mutex> lock(st().mu);
    st().log.clear();
    st().fail_from.clear();
    st().mix_blocks.clear();
    st().mix_jobs.clear();
    st().runs.clear();
    st().memory = SIZE_MAX;
    st().last = hipSuccess;
}
inline int count(const char *name) {
    std::lock_guard<std::recursive_mutex> lock(st().mu);
    return (int)std::count_if(st().log.begin(), st().log.end(),
                              [&](const Call &c) { return c.name == name; });
}

}  // namespace fake

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    std::lock_guard<std::recursive_mutex> lock(fake::st().mu);
    hipError_t e = fake::note("hipMalloc", nullptr, nullptr, hipErrorOutOfMemory);
    if (e == hipSuccess && n > fake::st().memory - std::min(fake::st().memory, fake::st().used))
        e = fake::st().last = hipErrorOutOfMemory;
    if (e != hipSuccess) return e;
    *p = std::malloc(n ? n : 1);
    fake::st().live[*p] = n;
    fake::st().used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::recursive_mutex> lock(fake::st().mu);
    (void)fake::note("hipFree");
    auto it = fake::st().live.find(p);
    if (it == fake::st().live.end()) return p ? hipErrorInvalidValue : hipSuccess;
    fake::st().used -= it->second;
    fake::st().live.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipFreeAsync(void *p, hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lock(fake::st().mu);
    const hipError_t e = hipFree(p);
    fake::st().log.back().name = "hipFreeAsync";
    fake::st().log.back().stream = s;
    return e;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    const hipError_t e = fake::note("hipHostMalloc", nullptr, nullptr, hipErrorOutOfMemory);
    if (e == hipSuccess) *p = std::malloc(n);
    return e;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return fake::note("hipMemcpy");
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t q) {
    std::memcpy(d, s, n);
    return fake::note("hipMemcpyAsync", q);
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h,
                            hipMemcpyKind, hipStream_t q) {
    for (size_t r = 0; r < h; ++r)
        std::memcpy(static_cast<char *>(d) + r * dp, static_cast<const char *>(s) + r * sp, w);
    return fake::note("hipMemcpy2DAsync", q);
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t q) {
    std::memset(d, v, n);
    return fake::note("hipMemsetAsync", q);
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    p->sharedMemPerBlock = 163840;
    return hipSuccess;
}
hipError_t hipGetLastError(void) {
    std::lock_guard<std::recursive_mutex> lock(fake::st().mu);
    const hipError_t e = fake::st().last;
    fake::st().last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipDeviceSynchronize(void) { return fake::note("hipDeviceSynchronize"); }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { fake::handle(s); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return fake::note("hipStreamSynchronize", s); }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    return fake::note("hipStreamWaitEvent", s, e);
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { fake::handle(g); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    fake::handle(x);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return fake::note("hipGraphLaunch", s); }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { fake::handle(e); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { fake::handle(e); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return fake::note("hipEventRecord", s, e); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
}

namespace dapt {

using fake::launched;
int launch_state_zero(const JobDesc &, void *s) { return launched("state_zero", s); }
int launch_rand_bits(uint8_t *, int32_t, int32_t, int32_t, uint32_t, uint64_t, void *s) {
    return launched("rand_bits", s);
}
int coupling_planes(int dtype, int64_t, int32_t) { return dtype; }
int launch_fields(const JobDesc &, int, const uint8_t *, int32_t, int32_t *, void *s) {
    return launched("fields", s);
}
int64_t energy_scratch_elems(const JobDesc &, int, int32_t) { return 0; }
int launch_energy(const JobDesc &, int, const uint8_t *, int32_t, int64_t *, int64_t *, void *s) {
    return launched("energy", s);
}
int launch_finish_start(const JobDesc &, void *s) { return launched("finish_start", s); }
int launch_run(const JobDesc &J, int, bool, const TraceDesc *, int, int, size_t, void *s) {
    {
        std::lock_guard<std::recursive_mutex> lock(fake::st().mu);
        fake::st().runs.push_back(J);
    }
    return launched("run", s);
}
size_t wave_lds_bytes(int, int, int, int, int, int64_t w) { return (size_t)w; }
int launch_wave(const JobDesc &J, int, int, int, size_t, void *s) {
    for (int32_t r = 0; r < J.R; ++r) {   // some state
        J.E[r] = 3 * r;
        J.bE[r] = -r;
        J.nacc[r] = 7 * r;
        for (int32_t i = 0; i < J.N; ++i) {
            J.x[(size_t)r * J.ld + i] = (uint8_t)((r + i) % 3);
            J.bx[(size_t)r * J.ld + i] = (uint8_t)((r ^ i) % 5);
        }
    }
    return launched("wave", s);
}
int launch_mix(const JobDesc *jobs, const BatchItem *items, int, int, int blocks, size_t, void *s) {
    {
        std::lock_guard<std::recursive_mutex> lock(fake::st().mu);
        fake::st().mix_blocks.push_back(blocks);
        for (int q = 0; q < blocks; ++q)
            if (q == 0 || items[q].job != items[q - 1].job)
                fake::st().mix_jobs.push_back(jobs[items[q].job]);
    }
    return launched("mix", s);
}
int launch_log_error(const double *, float *out, void *s) {
    *out = 1e-6f;
    return launched("log_error", s);
}
int launch_batch(const JobDesc *, const BatchItem *, const int32_t *, int32_t *, int, int, size_t,
                 void *s, bool) {
    return launched("batch", s);
}
int launch_pt_exchange(int64_t *, int32_t *, int32_t *, const double *, const double *, int32_t,
                       int32_t, uint64_t, uint32_t *, int64_t *, int64_t *, void *s) {
    return launched("pt_exchange", s);
}
int launch_pt_setup(int32_t *, int32_t *, int64_t *, int64_t *, uint32_t *, int32_t, int32_t,
                    void *s) {
    return launched("pt_setup", s);
}
size_t derive_scratch_bytes(int N) { return 24 + 8 * (size_t)N; }
int launch_derive(const int32_t *Q, int N, uint64_t *scratch, uint64_t **out, void *s) {
    uint64_t row = 0, maxw = 0, g = 0;
    for (int i = 0; i < N; ++i) {
        uint64_t sum = (uint64_t)std::llabs((long long)Q[(size_t)i * N + i]);
        for (int j = 0; j < N; ++j) {
            if (i == j) continue;
            uint64_t w = (uint64_t)std::llabs((long long)Q[(size_t)i * N + j] + Q[(size_t)j * N + i]);
            sum += w;
            maxw = std::max(maxw, w);
            g = std::gcd(g, w);
        }
        row = std::max(row, sum);
    }
    scratch[0] = row;
    scratch[1] = maxw;
    scratch[2] = g;
    *out = scratch;
    return launched("derive", s);
}
int launch_image(const int32_t *, int, int, int, int64_t, void *, int32_t *, void *s) {
    return launched("image", s);
}
int launch_outputs(const JobDesc &J, const da_result &o, void *s) {
    for (int32_t r = 0; r < J.R; ++r) {
        if (o.best_E) o.best_E[r] = J.bE[r];
        if (o.final_E) o.final_E[r] = J.E[r];
        if (o.n_accept) o.n_accept[r] = J.nacc[r];
        for (int32_t i = 0; i < J.N; ++i) {
            if (o.best_x) o.best_x[(size_t)r * J.N + i] = J.bx[(size_t)r * J.ld + i];
            if (o.final_x) o.final_x[(size_t)r * J.N + i] = J.x[(size_t)r * J.ld + i];
        }
    }
    return launched("outputs", s);
}
int launch_fill_i32(int32_t *, int32_t, int64_t, void *s) { return launched("fill", s); }
int launch_gen_calibrate(LevelHdr *, const int32_t *, int, void *s) {
    return launched("calibrate", s);
}
size_t run_lds_bytes(int, int, int, int, int, int, bool, bool, bool) { return 1024; }

}  // namespace dapt
