// A stand-in for the HIP runtime: loaded before the library, it takes the
// library's calls, so that its host code runs where there is no GPU.  Kernels
// do nothing, but a launch that the device's limits do not allow fails; the
// step kernel takes steps from a script and publishes their schedules, late:
// a queued kernel runs when the host asks about the stream.
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <string>
#include <vector>

#include "internal.h"

namespace {

std::map<const void *, std::string> g_names;   // kernels by the address of their host stub
hipError_t g_last = hipSuccess;
struct Launch {
    std::string name;
    dim3 grid, block;
};
std::vector<Launch> g_launches;
struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
std::vector<Config> g_config;

// The step kernel's schedules: after k steps, time (k + 1) ticks and g_n_act
// active particles.
int64_t g_n_act = 1, g_steps = 0;
std::deque<nb::StepArgs> g_queue;
int g_fail_at = 0;   // the launch, counted from the next one, that fails (0: none)

void run_step(const nb::StepArgs &a)
{
    nb::DevScalars *sc = a.sc;
    if (a.mode == nb::kStepSmall) {
        const int64_t na = sc->n_act;
        if (na < 1 || na > nb::kSmallMax || sc->t_next > a.t_limit || a.tab.n_split[na - 1] <= 0) return;
    }
    if (a.mode != nb::kStepSchedule) ++g_steps;
    sc->seq = a.mode == nb::kStepSchedule ? a.seq : sc->seq + 1;
    sc->t_next = g_steps + 1;
    sc->n_act = g_n_act;
    nb::HostScalars *p = a.pub + (sc->seq & (nb::kPubSlots - 1));
    p->t_next = sc->t_next;
    p->n_act = sc->n_act;
    p->underflow = p->nonfinite = 0;
    p->seq = sc->seq;
}

hipError_t give(hipError_t e)
{
    if (e != hipSuccess) g_last = e;
    return e;
}

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    g_names[stub] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    g_config.push_back({grid, block, shared, stream});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    const Config c = g_config.back();
    g_config.pop_back();
    *grid = c.grid;
    *block = c.block;
    *shared = c.shared;
    *stream = c.stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *stub, dim3 grid, dim3 block, void **args, size_t, hipStream_t)
{
    if (g_fail_at > 0 && --g_fail_at == 0) return give(hipErrorLaunchFailure);
    const std::string &name = g_names[stub];
    g_launches.push_back({name, grid, block});
    if (name.find("k_step") != std::string::npos && name.find("k_step_gather") == std::string::npos)
        g_queue.push_back(*static_cast<const nb::StepArgs *>(args[0]));
    const bool in_limits = grid.x > 0 && grid.y > 0 && grid.z > 0 && block.x > 0 && block.x * block.y * block.z <= 1024 &&
                           uint64_t(grid.x) * block.x < (uint64_t(1) << 32) && grid.y <= 65535 && grid.z <= 65535;
    return give(in_limits ? hipSuccess : hipErrorInvalidConfiguration);
}

hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "an error of the stand-in"; }
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned)
{
    *p = calloc(1, bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned)
{
    *d = h;
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind, hipStream_t s)
{
    (void)hipStreamSynchronize(s);
    memcpy(dst, src, bytes);
    return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t)
{
    if (g_queue.empty()) return hipSuccess;
    run_step(g_queue.front());
    g_queue.pop_front();
    return hipErrorNotReady;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    for (; !g_queue.empty(); g_queue.pop_front()) run_step(g_queue.front());
    return hipSuccess;
}

// For the test: the active particles of every schedule from the next step on, and
// the launch that fails.
void fake_script(int64_t n_act, int fail_at)
{
    g_n_act = n_act;
    g_fail_at = fail_at;
}
int64_t fake_steps() { return g_steps; }   // steps taken by the device
int fake_queued() { return int(g_queue.size()); }
// For the test: the launches since the last call, "name gx gy gz bx" a line.
const char *fake_launches()
{
    static std::string s;
    s.clear();
    for (const Launch &l : g_launches)
        s += l.name + " " + std::to_string(l.grid.x) + " " + std::to_string(l.grid.y) + " " + std::to_string(l.grid.z) +
             " " + std::to_string(l.block.x) + "\n";
    g_launches.clear();
    return s.c_str();
}

}  // extern "C"
