// The host half of the low-rank launchers (csrc/cf_lowrank.hip compiled for the host alone) against a runtime that refuses one
// launch and, like some, forgets the refusal at the next success: the launcher has to report it.
#include <cstdio>
#include <cstring>

#include "cf_internal.h"

static int g_launches, g_refused;           // launches so far; which of them is refused
static hipError_t g_last = hipSuccess;

extern "C" {
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t)
{
    g_last = g_launches++ == g_refused ? hipErrorLaunchOutOfResources : hipSuccess;
    return g_last;
}
hipError_t hipGetLastError(void) { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = dim3(1); *block = dim3(1); *shared = 0; *stream = nullptr;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
}

int main()
{
    using namespace cf;
    BatchView v;
    std::memset(static_cast<void *>(&v), 0, sizeof v);
    TensorPtrs sets[kDirectTensors];
    std::memset(static_cast<void *>(sets), 0, sizeof sets);
    LaunchRange r;
    std::memset(static_cast<void *>(&r), 0, sizeof r);
    r.count = 2;
    r.dts = 2;              // both storage types
    r.lr_wires = 3;         // and both kinds of factors
    r.lr_max_channels = 512;
    r.lr_max_tokens = 100;
    r.lr_project_blocks = 4;
    r.lr_split = 1;
    int failed = 0;
    for (int what = 0; what < 5; ++what)
        for (int direct = 0; direct < (what == 1 ? 2 : 1); ++direct) {
            r.direct = direct ? sets : nullptr;
            auto call = [&](int refused) {
                g_launches = 0;
                g_refused = refused;
                g_last = hipSuccess;
                switch (what) {
                case 0: return launch_lr_encode(v, r, 0, true, nullptr);
                case 1: return launch_lr_decode(v, r, nullptr);
                case 2: return launch_lr_project(v, r, true, 0, nullptr);
                case 3: return launch_lr_backproject(v, r, 0, nullptr);
                default: return launch_lr_orth(v, r, true, 0, nullptr);
                }
            };
            if (call(-1) != hipSuccess || g_launches < 2) { std::printf("launcher %d: %d launches\n", what, g_launches); ++failed; }
            const int n = g_launches;
            for (int k = 0; k < n; ++k)
                if (call(k) == hipSuccess) { std::printf("launcher %d, pointers in arguments %d: the refusal of launch %d is lost\n", what, direct, k); ++failed; }
        }
    if (failed) return 1;
    std::printf("every refused launch is reported\n");
    return 0;
}
