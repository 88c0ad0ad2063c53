// Host-only stand-ins for everything the ABI layer (csrc/cf_api.cpp) calls below itself: the kernel launchers
// and the handful of HIP runtime functions.  Nothing runs on a device; every launch is appended to a log so the
// driver can check the launch sequence a call makes.  Used only by the sanitizer build of the CPU tests.
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "cf_internal.h"

using cf::LaunchRange;
using cf::TensorPtrs;

std::vector<std::string> g_launch_log;
bool g_capturing = false;
int g_compute_units = 256;
bool g_single_pass_slim = false;        // the stripe width of the last single pass
bool g_single_pass_short = false;       // and its items' height
int g_short_workgroups = 0;             // that a call of them launches
bool g_single_pass_wide = false;
bool g_single_pass_blocks = false;      // whether it left parts of 64-byte blocks to the L2
bool g_occupancy_slim = false;          // and the one whose co-resident workgroups were asked for last
bool g_project_many = false;            // whether the last projection's waves take several blocks of tokens
int g_split = 0;                        // and the workgroups that share a stripe of the last back-projection
std::vector<TensorPtrs> g_direct;       // the pointers that the last kernel of a direct call took as arguments; none: it read the table
bool g_overlapping = false;             // single passes leave item states as calls that overlapped may
std::vector<uint8_t> g_states;          // the item states that the last single pass found
static void take_direct(const LaunchRange &r)
{
    g_direct.clear();
    if (r.direct) g_direct.assign(r.direct, r.direct + r.count);
}
static void note(const char *what) { g_launch_log.push_back(what); }

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = g_compute_units; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) { std::memcpy(dst, src, n); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
}

namespace cf {
// tables really are written (into the host buffer that plays the workspace), so the driver can read them back
hipError_t launch_upload_ptrs(const PtrChunk &chunk, TensorPtrs *dst, int n, hipStream_t)
{
    note("k_upload_ptrs");
    std::memcpy(dst, chunk.p, sizeof(TensorPtrs) * (size_t)n);
    return hipSuccess;
}
hipError_t launch_upload_bytes(const void *src, void *dst, size_t bytes, hipStream_t)
{
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}
hipError_t launch_fill_words(void *dst, uint32_t value, size_t n_words, hipStream_t)
{
    uint32_t *w = static_cast<uint32_t *>(dst);
    for (size_t i = 0; i < n_words; ++i) w[i] = value;
    return hipSuccess;
}
hipError_t launch_fill_item_tensor(const uint32_t *item_prefix, uint32_t *item_tensor, int n_tensors, hipStream_t)
{
    for (int t = 0; t < n_tensors; ++t)
        for (uint32_t i = item_prefix[t]; i < item_prefix[t + 1]; ++i) item_tensor[i] = (uint32_t)t;
    return hipSuccess;
}
hipError_t launch_warmup(const BatchView &, const LaunchRange &r, int, hipStream_t) { take_direct(r); note("k_warmup"); return hipSuccess; }
hipError_t launch_colreduce(const BatchView &, const LaunchRange &, int, int, hipStream_t) { note("k_colreduce"); return hipSuccess; }
hipError_t launch_finalize(const BatchView &, const LaunchRange &, hipStream_t) { note("k_finalize"); return hipSuccess; }
hipError_t launch_finalize_rank1(const BatchView &, const LaunchRange &, hipStream_t) { note("k_finalize_rank1"); return hipSuccess; }
hipError_t launch_encode(const BatchView &, const LaunchRange &r, int, int, bool, hipStream_t) { take_direct(r); note("k_encode"); return hipSuccess; }
hipError_t launch_encode_nm(const BatchView &, const LaunchRange &r, int, int, bool, bool, hipStream_t) { take_direct(r); note("k_encode_nm"); return hipSuccess; }
hipError_t launch_decode(const BatchView &, const LaunchRange &r, hipStream_t) { take_direct(r); note("k_decode"); return hipSuccess; }
hipError_t launch_lr_orth(const BatchView &, const LaunchRange &, bool, int, hipStream_t) { note("k_lr_orth"); return hipSuccess; }
hipError_t launch_lr_project(const BatchView &, const LaunchRange &r, bool, int, hipStream_t)
{
    g_project_many = r.lr_project_many != 0;
    note("k_lr_project");
    return hipSuccess;
}
hipError_t launch_lr_backproject(const BatchView &, const LaunchRange &r, int, hipStream_t)
{
    g_split = r.lr_split;
    note("k_lr_backproject");
    return hipSuccess;
}
hipError_t launch_lr_quant_u(const BatchView &, const LaunchRange &, hipStream_t) { note("k_lr_quant_u"); return hipSuccess; }
hipError_t launch_lr_encode(const BatchView &, const LaunchRange &, int, bool, hipStream_t) { note("k_lr_apply"); return hipSuccess; }
hipError_t launch_lr_decode(const BatchView &, const LaunchRange &r, hipStream_t) { take_direct(r); note("k_lr_apply"); return hipSuccess; }
int persistent_max_blocks_per_cu(int, int, bool, bool, bool slim) { g_occupancy_slim = slim; return 2; }
hipError_t launch_single_pass(const BatchView &v, const LaunchRange &r, int, int, bool, bool wide, int, bool, hipStream_t)
{
    take_direct(r);
    g_single_pass_wide = wide;
    g_single_pass_blocks = r.sp_blocks != 0;
    g_single_pass_slim = r.sp_slim != 0;
    g_single_pass_short = r.sp_short != 0;
    g_states.assign(v.item_state + r.item_lo, v.item_state + r.item_hi);
    for (uint32_t i = r.item_lo; i < r.item_hi; i += g_overlapping ? 2 : 1) v.item_state[i] ^= 0x80u;      // as the kernel's items do, all of them or not
    if (r.sp_short) {
        const ShortGrid grid = short_grid(r.direct_descs, r.count);
        g_short_workgroups = (int)(grid.x * grid.y * grid.z);
        if (grid.flat ? grid.x != r.item_hi - r.item_lo || grid.y != 1 || grid.z != 1 : grid.z != (uint32_t)r.count) note("wrong grid");
    }
    if (r.sp_short)     // the call's tensors one after another, and nothing else
        for (int k = 0; k < r.count; ++k) {
            const uint32_t items = (uint32_t)(r.direct_descs[k].p_n_rb * r.direct_descs[k].p_n_stripes);
            if (r.direct_descs[k].p_item_begin + items != (k + 1 < r.count ? r.direct_descs[k + 1].p_item_begin : r.item_hi)) note("wrong items");
        }
    note("k_single_pass");
    return hipSuccess;
}
hipError_t launch_fresh_partials(uint8_t *partials, size_t bytes, uint8_t *states, uint32_t n_states, hipStream_t)
{
    note("k_fresh_partials");
    if (reinterpret_cast<uintptr_t>(partials) % 256 != 0 || bytes % 256 != 0) note("misplaced");
    std::memset(partials, (int)(kFreshPartials & 255u), bytes);
    std::memset(states, (int)(kFreshPartials & 255u), n_states);
    return hipSuccess;
}
hipError_t static_scratch(void **ptr)
{
    static void *buf = nullptr;
    if (!buf && posix_memalign(&buf, 256, kStaticScratchBytes) != 0) return hipErrorOutOfMemory;
    *ptr = buf;
    return hipSuccess;
}
}  // namespace cf
