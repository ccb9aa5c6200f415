// jatam_static.hip - classification for callers that cannot allocate device
// memory (code under HIP graph capture, tight serving loops, harnesses that
// forbid hipMalloc): the one-launch kernel, with the counter sets of a call's
// tally in a static device array of the library instead of a jatam_batch_t
// workspace.  It needs no other memory.
//
// `counters` below is a host-side stand-in in host code: its device address
// is taken once per device with hipGetSymbolAddress (with that device
// current) and only that address is ever handed to kernels.  Every call on a
// device shares the device's copy of the array, so calls that overlap on one
// GPU mix their tallies; each clears its counter sets first (by a kernel, never
// a memset), so nothing carries over from the previous call.
#include <mutex>

#include "jatam_internal.hpp"

namespace {

constexpr int64_t kStaticMaxN = int64_t(1) << 18;   // genotypes per call
constexpr int kMaxDevices = 64;

struct StaticCounters {
    unsigned long long tally[jatam::kTallySlots * jatam::kTallyStride];
    uint32_t claims[2 * jatam::kClaimCounters * jatam::kClaimStride];   // cleared, not used
};

StaticCounters* g_counters[kMaxDevices];
std::mutex g_setup;

}  // namespace

__device__ __align__(256) uint8_t counters[sizeof(StaticCounters)];

namespace {

// The array's address on the current device (a runtime query, so the first call on
// a device must not be under graph capture).
StaticCounters* static_counters(int dev)
{
    std::lock_guard<std::mutex> lock(g_setup);
    void* ptr = g_counters[dev];
    if (ptr == nullptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(counters)) != hipSuccess)
            return nullptr;
        g_counters[dev] = (StaticCounters*)ptr;
    }
    return g_counters[dev];
}

}  // namespace

extern "C" int jatam_classify_static(const uint64_t* genotypes, int64_t n, int t, int c,
                                     int grid_limit, int runs, uint64_t seed, jatam_result_t* out,
                                     uint64_t* tally, void* stream)
{
    jatam::Params p;
    const int rc = jatam::make_params(t, c, grid_limit, runs, seed, &p);
    if (rc != JATAM_OK)
        return rc;
    if (n < 0 || n > kStaticMaxN || (n > 0 && (genotypes == nullptr || out == nullptr)))
        return JATAM_E_INVALID_ARG;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0)
        return JATAM_E_HIP;
    if (dev >= kMaxDevices)
        return JATAM_E_UNSUPPORTED;
    const jatam::DeviceLimits* d = jatam::device_limits();
    StaticCounters* const k = static_counters(dev);
    if (d == nullptr || k == nullptr)
        return JATAM_E_HIP;
    jatam::DeviceWorkspace ws{};
    ws.tally_slots = k->tally;
    ws.run_claim = k->claims;
    jatam::BatchArgs a = jatam::batch_args_for(p, n, out, tally, ws);
    a.genomes = genotypes;
    const int geno = jatam::geno_kind(t, c);
    const bool classes[2] = {grid_limit <= 16, grid_limit > 16};
    const int waves[2] = {d->solo[0][geno] * d->cus, d->solo[1][geno] * d->cus};
    return jatam::launch_solo(a, classes, waves, geno, nullptr, 0, (hipStream_t)stream);
}
