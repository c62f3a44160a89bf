// pd_video on a pretended runtime: host calls only record what a device would
// still have to do, and the n-th call inside a push can be made to fail.
// Nothing may touch a slot's buffers while work enqueued by a failed push is
// outstanding: its graph must not be launched on another stream, and its pinned
// frame must not be written, before the earlier launch or copy was waited for.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <vector>

#include "pd_internal.h"

namespace {

struct Work {
    hipStream_t stream;
    const void* what;  // a graph, or the host side of an upload
};
std::vector<Work> outstanding;
int calls = 0, fail_at = 0, violations = 0;

bool fails() { return ++calls == fail_at; }

void finish(hipStream_t s) {
    std::vector<Work> rest;
    for (const Work& w : outstanding)
        if (s && w.stream != s) rest.push_back(w);
    outstanding.swap(rest);
}

void enqueue(hipStream_t s, const void* what, bool same_stream_is_ordered) {
    for (const Work& w : outstanding)
        if (w.what == what && !(same_stream_is_ordered && w.stream == s)) {
            ++violations;
            std::printf("work on %p enqueued while an earlier one is outstanding (call %d failed)\n", what, fail_at);
        }
    outstanding.push_back(Work{s, what});
}

}  // namespace

struct pd_graph {
    int dummy;
};

int pd::fail(int code, const char*, ...) { return code; }
int pd::hip_status(hipError_t e, const char*) { return e == hipSuccess ? PD_OK : PD_E_HIP; }

extern "C" {

int64_t pd_detect_workspace_bytes(const pd_frame*, int, const pd_params*, int) { return 4096; }
int pd_graph_create(const pd_frame*, int, const float*, const float*, int, const pd_params*, const double*, void*,
                    int64_t, pd_box*, int, pd_counts*, void*, pd_graph** out) {
    *out = new pd_graph();
    return PD_OK;
}
int pd_graph_destroy(pd_graph* g) {
    delete g;
    return PD_OK;
}
int pd_graph_launch(pd_graph* g, void* stream) {
    if (fails()) return PD_E_HIP;
    enqueue((hipStream_t)stream, g, true);
    return PD_OK;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = (hipStream_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    finish(s);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    *p = std::calloc(n, 1);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = (hipEvent_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return fails() ? hipErrorUnknown : hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return fails() ? hipErrorUnknown : hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void* src, size_t, hipMemcpyKind kind, hipStream_t s) {
    if (fails()) return hipErrorUnknown;
    if (kind == hipMemcpyHostToDevice) enqueue(s, src, false);  // the host has written the buffer by now
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) {  // the slot's last event: everything before it is done
    finish(nullptr);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0.0f;
    return hipSuccess;
}

}  // extern "C"

int main() {
    const float weight = 0.0f;
    std::vector<uint8_t> frame(64 * 128);
    int failed = 0;
    for (int depth = 1; depth <= 3; ++depth)
        for (int n = 1; n <= 12; ++n) {
            outstanding.clear();
            fail_at = 0;
            pd_params params{};
            pd_video* v = nullptr;
            if (pd_video_create(64, 128, &params, &weight, &weight, 1, 4, depth, &v) != PD_OK) return 2;
            pd_counts counts{};
            pd_box boxes[4];
            // some good frames first, so that the failing push meets every slot and stream
            for (int k = 0; k < n % 4; ++k)
                if (pd_video_push(v, frame.data(), 64, 0.0) || pd_video_pop(v, boxes, 4, &counts, nullptr)) return 3;
            calls = 0;
            fail_at = n;
            const int rc = pd_video_push(v, frame.data(), 64, 0.0);
            fail_at = 0;
            failed += rc != PD_OK;
            if (rc == PD_OK && pd_video_pop(v, boxes, 4, &counts, nullptr)) return 4;
            fail_at = -n;  // (named in the message)
            for (int k = 0; k < 2; ++k)
                if (pd_video_push(v, frame.data(), 64, 0.0) || pd_video_pop(v, boxes, 4, &counts, nullptr)) return 5;
            pd_video_destroy(v);
        }
    std::printf("%d failed pushes, %d violations\n", failed, violations);
    return violations ? 1 : failed < 20 ? 6 : 0;
}
