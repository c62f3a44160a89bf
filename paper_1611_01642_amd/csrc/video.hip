// Streaming video mode: frames arrive one at a time in host memory (Section
// 4.1 step 1 copies each to the GPU, step 5 brings the detections back), and
// the copies of one frame overlap the detection of its neighbours.
//
// A ring of `depth` slots; each owns a device frame, a pd_detect workspace,
// device and pinned-host result buffers, and the pd_detect kernel sequence
// captured once as a graph on its own buffers.  A push copies the frame into
// the slot's pinned buffer (host), then enqueues the upload on the upload
// stream, the graph on a compute stream (after the upload's event) and
// the download of counts and boxes on the download stream (after the graph's
// event).  Streams at default priority, so the upload of frame n+1 and the
// download of frame n-1 run while frame n is detected; two compute streams,
// taken in turn (the slots share nothing but the weights), because one frame's
// kernels leave most of the chip idle.  A frame and its threshold go up in one
// copy, its counts and boxes come down in one.  8 frames of 1242x375, three in
// flight: 804 us; on one compute stream with two copies each way 949.  A pop waits
// for its slot's last event and hands the results to the caller; the slot is
// then free for a new push.
#include <cstring>
#include <vector>

#include "pd_internal.h"

using namespace pd;

struct pd_video {
    int w = 0, h = 0, pitch = 0, cap = 0, depth = 0;
    hipStream_t up = nullptr, compute[2] = {nullptr, nullptr}, down = nullptr;
    struct Slot {
        uint8_t* d_frame = nullptr;
        double* d_thr = nullptr;      // after the frame
        void* ws = nullptr;
        uint8_t* d_down = nullptr;    // counts, then boxes
        pd_box* d_boxes = nullptr;
        pd_counts* d_counts = nullptr;
        uint8_t* h_frame = nullptr;
        double* h_thr = nullptr;
        uint8_t* h_down = nullptr;
        pd_box* h_boxes = nullptr;
        pd_counts* h_counts = nullptr;
        hipEvent_t ev_start = nullptr, ev_up = nullptr, ev_det = nullptr, ev_done = nullptr;
        pd_graph* graph = nullptr;
    };
    std::vector<Slot> slots;
    unsigned pushed = 0;  // frames so far: the next one's compute stream
    int head = 0, n_busy = 0;  // oldest pushed slot, slots pushed and not popped
};

namespace {

void release(pd_video* v) {
    for (auto s : {v->up, v->compute[0], v->compute[1], v->down})
        if (s) (void)hipStreamSynchronize(s);
    for (pd_video::Slot& s : v->slots) {
        (void)pd_graph_destroy(s.graph);
        for (hipEvent_t e : {s.ev_start, s.ev_up, s.ev_det, s.ev_done})
            if (e) (void)hipEventDestroy(e);
        for (void* p : {(void*)s.d_frame, s.ws, (void*)s.d_down})
            if (p) (void)hipFree(p);
        for (void* p : {(void*)s.h_frame, (void*)s.h_down})
            if (p) (void)hipHostFree(p);
    }
    for (auto s : {v->up, v->compute[0], v->compute[1], v->down})
        if (s) (void)hipStreamDestroy(s);
    delete v;
}

}  // namespace

extern "C" {

int pd_video_create(int w, int h, const pd_params* params, const float* weights, const float* bias, int n_models,
                    int cap, int depth, pd_video** out) {
    if (!out) return fail(PD_E_ARG, "out is NULL");
    *out = nullptr;
    if (depth < 1 || depth > PD_VIDEO_MAX_DEPTH) return fail(PD_E_SIZE, "depth %d outside [1, %d]", depth, PD_VIDEO_MAX_DEPTH);
    if (cap < 1) return fail(PD_E_SIZE, "cap %d < 1", cap);
    if (w < 1 || h < 1 || w > PD_MAX_DIM || h > PD_MAX_DIM) return fail(PD_E_SIZE, "frame %dx%d", w, h);
    if (!weights || !bias) return fail(PD_E_ARG, "NULL pointer argument");
    pd_frame desc{nullptr, w, h, (w + 15) / 16 * 16, 0};
    const int64_t ws_bytes = pd_detect_workspace_bytes(&desc, 1, params, n_models);
    if (ws_bytes < 0) return (int)ws_bytes;  // message set by the size query
    pd_video* v = new pd_video();
    v->w = w;
    v->h = h;
    v->pitch = desc.pitch;
    v->cap = cap;
    v->depth = depth;
    v->slots.resize(depth);
    int rc = PD_OK;
    for (hipStream_t* s : {&v->up, &v->compute[0], &v->compute[1], &v->down})
        if (!rc) rc = hip_status(hipStreamCreateWithFlags(s, hipStreamNonBlocking), "video stream");
    const size_t frame_bytes = (size_t)v->pitch * h;  // a multiple of 16
    const size_t up_bytes = frame_bytes + sizeof(double);
    constexpr size_t BOXES = 64;  // where the boxes begin
    static_assert(sizeof(pd_counts) <= BOXES, "counts before the boxes");
    const size_t down_bytes = BOXES + sizeof(pd_box) * cap;
    for (pd_video::Slot& s : v->slots) {
        if (rc) break;
        rc = hip_status(hipMalloc(&s.d_frame, up_bytes), "video frame");
        if (!rc) rc = hip_status(hipMalloc(&s.ws, (size_t)ws_bytes), "video workspace");
        if (!rc) rc = hip_status(hipMalloc(&s.d_down, down_bytes), "video boxes");
        if (!rc) rc = hip_status(hipHostMalloc(&s.h_frame, up_bytes, hipHostMallocDefault), "video pinned frame");
        if (!rc) rc = hip_status(hipHostMalloc(&s.h_down, down_bytes, hipHostMallocDefault), "video pinned");
        if (!rc) rc = hip_status(hipEventCreate(&s.ev_start), "video event");
        if (!rc) rc = hip_status(hipEventCreate(&s.ev_done), "video event");
        if (!rc) rc = hip_status(hipEventCreateWithFlags(&s.ev_up, hipEventDisableTiming), "video event");
        if (!rc) rc = hip_status(hipEventCreateWithFlags(&s.ev_det, hipEventDisableTiming), "video event");
        if (!rc) {
            s.d_thr = reinterpret_cast<double*>(s.d_frame + frame_bytes);
            s.h_thr = reinterpret_cast<double*>(s.h_frame + frame_bytes);
            s.d_counts = reinterpret_cast<pd_counts*>(s.d_down);
            s.h_counts = reinterpret_cast<pd_counts*>(s.h_down);
            s.d_boxes = reinterpret_cast<pd_box*>(s.d_down + BOXES);
            s.h_boxes = reinterpret_cast<pd_box*>(s.h_down + BOXES);
            std::memset(s.h_frame, 0, up_bytes);
            rc = hip_status(hipMemcpyAsync(s.d_frame, s.h_frame, up_bytes, hipMemcpyHostToDevice, v->compute[0]),
                            "video frame clear");
        }
        if (!rc) {
            pd_frame f{s.d_frame, w, h, v->pitch, 0};
            rc = pd_graph_create(&f, 1, weights, bias, n_models, params, s.d_thr, s.ws, ws_bytes, s.d_boxes, cap,
                                 s.d_counts, v->compute[0], &s.graph);
        }
    }
    if (!rc) rc = hip_status(hipStreamSynchronize(v->compute[0]), "video setup");
    if (rc) {
        release(v);
        return rc;
    }
    *out = v;
    return PD_OK;
}

int pd_video_push(pd_video* v, const uint8_t* frame, int pitch, double threshold) {
    if (!v || !frame) return fail(PD_E_ARG, "NULL pointer argument");
    if (pitch < v->w) return fail(PD_E_ARG, "pitch %d < width %d", pitch, v->w);
    if (v->n_busy == v->depth) return fail(PD_E_SIZE, "all %d slots hold frames not yet popped", v->depth);
    pd_video::Slot& s = v->slots[(v->head + v->n_busy) % v->depth];
    for (int y = 0; y < v->h; ++y) std::memcpy(s.h_frame + (size_t)y * v->pitch, frame + (size_t)y * pitch, v->w);
    *s.h_thr = threshold;
    const hipStream_t compute = v->compute[v->pushed % 2];
    int rc = hip_status(hipEventRecord(s.ev_start, v->up), "video record");
    if (!rc)
        rc = hip_status(hipMemcpyAsync(s.d_frame, s.h_frame, (size_t)v->pitch * v->h + sizeof(double),
                                       hipMemcpyHostToDevice, v->up),
                        "video upload");
    if (!rc) rc = hip_status(hipEventRecord(s.ev_up, v->up), "video record");
    if (!rc) rc = hip_status(hipStreamWaitEvent(compute, s.ev_up, 0), "video wait");
    if (!rc) rc = pd_graph_launch(s.graph, compute);
    if (!rc) rc = hip_status(hipEventRecord(s.ev_det, compute), "video record");
    if (!rc) rc = hip_status(hipStreamWaitEvent(v->down, s.ev_det, 0), "video wait");
    if (!rc)
        rc = hip_status(hipMemcpyAsync(s.h_down, s.d_down,
                                       (size_t)(reinterpret_cast<uint8_t*>(s.d_boxes + v->cap) - s.d_down),
                                       hipMemcpyDeviceToHost, v->down),
                        "video download");
    if (!rc) rc = hip_status(hipEventRecord(s.ev_done, v->down), "video record");
    if (rc) {
        // The slot stays free: its next push writes the pinned frame and may
        // launch the graph on the other compute stream, so what this one has
        // enqueued must be over by then.
        for (hipStream_t q : {v->up, compute, v->down}) (void)hipStreamSynchronize(q);
        return rc;
    }
    ++v->pushed;
    ++v->n_busy;
    return PD_OK;
}

int pd_video_pop(pd_video* v, pd_box* boxes, int cap, pd_counts* counts, float* device_ms) {
    if (!v || !counts || (!boxes && cap > 0)) return fail(PD_E_ARG, "NULL pointer argument");
    if (v->n_busy == 0) return fail(PD_E_ARG, "no frame pushed and not yet popped");
    pd_video::Slot& s = v->slots[v->head];
    if (int rc = hip_status(hipEventSynchronize(s.ev_done), "video wait")) return rc;
    if (device_ms)
        if (int rc = hip_status(hipEventElapsedTime(device_ms, s.ev_start, s.ev_done), "video timing")) return rc;
    *counts = *s.h_counts;
    const int n = std::min(std::min(s.h_counts->kept, v->cap), std::max(cap, 0));
    if (n > 0) std::memcpy(boxes, s.h_boxes, sizeof(pd_box) * n);
    v->head = (v->head + 1) % v->depth;
    --v->n_busy;
    if (s.h_counts->overflow || s.h_counts->kept > cap)
        return fail(PD_E_OVERFLOW, "frame results truncated: %d candidates, %d kept, %d boxes room",
                    s.h_counts->candidates, s.h_counts->kept, cap);
    return PD_OK;
}

int pd_video_destroy(pd_video* v) {
    if (v) release(v);
    return PD_OK;
}

}  // extern "C"
