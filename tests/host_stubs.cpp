// The HIP runtime and the launch functions of the kernels as stand-ins that only
// count, for tests of the library's host code (jatam_api.cpp) on a machine without
// a GPU: which kernels a call would launch with which arguments, and what it leaves
// behind when one of them fails.
//
// Time is a counter that launches add to, so that measurements have known results.
#include <hip/hip_runtime.h>

#include <stdlib.h>
#include <string.h>

#include "../paper_2205_15311_amd/csrc/jatam_internal.hpp"

extern "C" {
// what the test sets
int fail_attribute = 0;      // hipDeviceGetAttribute calls that fail
int fail_train = 0;          // training launches that fail
double solo_ms = 1.0;        // cost of the one launch and of the pipeline
double pipeline_ms = 2.0;
int fast_refill = 0;         // a first-run refill at which the pipeline takes half
// what the stand-ins count
int solo_launches = 0, pipeline_launches = 0, shape_hists = 0, graph_launches = 0;
int last_step = -1, last_refill = -1, last_mapping = -1;
long long last_n = 0;
double now_ms = 0.0;
}

static int event_slot = 0;
static double events[1 << 16];

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    if (fail_attribute > 0) {
        --fail_attribute;
        return hipErrorInvalidValue;
    }
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    strcpy(p->gcnArchName, "none");
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    *g = (hipGraph_t)1;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t)
{
    *e = (hipGraphExec_t)1;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { ++graph_launches; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes)
{
    *p = malloc(bytes);
    return *p != nullptr ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void*, size_t bytes, hipMemcpyKind kind, hipStream_t)
{
    if (kind == hipMemcpyDeviceToHost)
        memset(dst, 0, bytes);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)&events[event_slot++ & 0xFFFF]; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *(double*)e = now_ms; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(*(double*)b - *(double*)a);
    return hipSuccess;
}
}

namespace jatam {

void solo_occupancy(int solo[2][kGenoKinds])
{
    for (int k = 0; k < 2; ++k)
        for (int i = 0; i < kGenoKinds; ++i)
            solo[k][i] = k == 0 ? 11 : 3;
}

void batch_occupancy(BatchOccupancy& occ)
{
    for (int k = 0; k < 2; ++k)
        for (int i = 0; i < kGenoKinds; ++i)
            for (int j = 0; j < 3; ++j)
                occ.blocks[k][i][j] = k == 0 ? 14 : 4;
    solo_occupancy(occ.solo);
}

int launch_solo(const BatchArgs& a, const bool*, const int*, int, jatam_shape_count_t*, int,
                hipStream_t)
{
    ++solo_launches;
    last_n = a.n;
    now_ms += solo_ms;
    return JATAM_OK;
}

int launch_batched(const BatchArgs& a, const bool classes[2], const StageLaunch launch[2], int,
                   hipStream_t, hipEvent_t*, uint8_t*)
{
    const StageLaunch& l = launch[classes[1] ? 1 : 0];
    ++pipeline_launches;
    last_n = a.n;
    last_refill = l.refill;
    last_mapping = l.repeat_mapping;
    const bool fast = (classes[0] && launch[0].refill == fast_refill) ||
                      (classes[1] && launch[1].refill == fast_refill);
    now_ms += fast ? 0.5 * pipeline_ms : pipeline_ms;
    return JATAM_OK;
}

int launch_shape_hist(const jatam_result_t*, uint64_t, jatam_shape_count_t*, int, uint64_t*, int,
                      const uint32_t*, hipStream_t)
{
    ++shape_hists;
    return JATAM_OK;
}

int mlp_launch_train(const MlpArgs&, const uint64_t*, const uint8_t*, int, const jatam_result_t*,
                     uint32_t, uint32_t, float, int step, float*, hipStream_t)
{
    last_step = step;
    if (fail_train > 0) {
        --fail_train;
        return JATAM_E_HIP;
    }
    return JATAM_OK;
}

int launch_gather(const uint64_t*, const uint32_t*, uint32_t, uint64_t*, hipStream_t) { return JATAM_OK; }
int launch_variant(const uint64_t*, uint64_t, int64_t, const Params&, int, jatam_result_t*, hipStream_t) { return JATAM_OK; }
int mlp_launch_init(const MlpArgs&, uint64_t, hipStream_t) { return JATAM_OK; }
int mlp_launch_score(const MlpArgs&, const uint64_t*, const uint8_t*, int, uint32_t, float*, int, hipStream_t) { return JATAM_OK; }
int mlp_launch_refresh(const MlpArgs&, hipStream_t) { return JATAM_OK; }
int mlp_launch_forward(const MlpArgs&, const uint64_t*, const uint8_t*, int, uint32_t, float*, hipStream_t) { return JATAM_OK; }
size_t mlp_partial_floats(size_t) { return 1; }
uint64_t order_work_words(uint64_t n) { return n; }
int launch_order_by_cost(const float*, uint32_t, uint32_t*, uint32_t*, hipStream_t) { return JATAM_OK; }
int launch_ga_fitness(const jatam_result_t*, uint32_t, int32_t*, hipStream_t) { return JATAM_OK; }
int launch_ga_offspring(const uint64_t*, const int32_t*, uint32_t, const GaArgs&, uint32_t, uint64_t*, hipStream_t) { return JATAM_OK; }
int launch_select_top(const float*, uint32_t, uint32_t, uint32_t*, uint32_t*, hipStream_t) { return JATAM_OK; }
int launch_slice_reset(uint32_t*, hipStream_t) { return JATAM_OK; }
int launch_slice_advance(uint32_t*, hipStream_t) { return JATAM_OK; }
int launch_records_differ(const jatam_result_t*, const jatam_result_t*, uint64_t, uint32_t*, hipStream_t) { return JATAM_OK; }

}  // namespace jatam
