// C-ABI entry points of libadpsgd, part 1: handle life cycle, validation, per-call planning and
// the per-round launch loop of adpsgd_run_events.  See include/adpsgd.h for the contract.
#include <cmath>
#include <cstring>
#include <memory>

#include "handle.hpp"
#include "strips.hpp"

namespace adpsgd_impl {

hipError_t DevBuf::reserve(size_t bytes) {
    if (bytes <= cap) return hipSuccess;
    if (p) {
        // kernels enqueued earlier may still read the old buffer
        hipError_t e = hipDeviceSynchronize();
        if (e == hipSuccess) e = hipFree(p);
        p = nullptr;
        cap = 0;
        if (e != hipSuccess) return e;
    }
    size_t want = std::max<size_t>(bytes, 256);
    hipError_t e = hipMalloc(&p, want);
    if (e != hipSuccess) { p = nullptr; return e; }
    cap = want;
    return hipSuccess;
}
void DevBuf::release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    cap = 0;
}

namespace {
thread_local std::string g_create_error;
}  // namespace

const std::string& create_error() { return g_create_error; }

int fail(adpsgd_t* h, int code, const std::string& msg) {
    if (h) h->err = msg;
    else g_create_error = msg;
    return code;
}
int hip_fail(adpsgd_t* h, hipError_t e, const char* what) {
    return fail(h, ADPSGD_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

bool is_neighbour(const adpsgd_t* h, int32_t i, int32_t j) {
    if (j == i) return true;     // W_k = I: a gradient step without averaging
    const int32_t b = h->rowptr[i], e = h->rowptr[i + 1];
    for (int32_t t = b; t < e; ++t)
        if (h->col[t] == j) return true;
    return false;
}

void metropolis(const std::vector<int32_t>& rowptr, const std::vector<int32_t>& col, float* w_self, float* w_edge) {
    const int32_t n = static_cast<int32_t>(rowptr.size()) - 1;
    for (int32_t i = 0; i < n; ++i) {
        const int32_t di = rowptr[i + 1] - rowptr[i];
        double self = 1.0;
        for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e) {
            const int32_t j = col[e], dj = rowptr[j + 1] - rowptr[j];
            const double w = 1.0 / (1.0 + static_cast<double>(std::max(di, dj)));
            w_edge[e] = static_cast<float>(w);
            self -= w;
        }
        w_self[i] = static_cast<float>(self);
    }
}

hipEvent_t take_event(adpsgd_t* h) {
    if (!h->ev_pool.empty()) {
        hipEvent_t e = h->ev_pool.back();
        h->ev_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

int check_exchange(adpsgd_t* h) {
    const volatile int* status = static_cast<const volatile int*>(h->exchange_status.p);
    if (!status || *status == 0) return ADPSGD_OK;
    return fail(h, ADPSGD_ERR_HIP, "the blocks of a launch lost each other, the models are undefined (set_models replaces them)");
}

// Fold the timings of finished launches into the statistics (synchronises the stream).
int drain_profile(adpsgd_t* h) {
    if (h->ev_fused.empty() && h->ev_grad.empty()) return ADPSGD_OK;
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    for (int which = 0; which < 2; ++which) {
        auto& list = which == 0 ? h->ev_fused : h->ev_grad;
        double& total = which == 0 ? h->stats.fused_ms : h->stats.grad_ms;
        for (auto& pr : list) {
            float ms = 0.0f;
            HIP_TRY(h, hipEventElapsedTime(&ms, pr.first, pr.second));
            total += ms;
            h->ev_pool.push_back(pr.first);
            h->ev_pool.push_back(pr.second);
        }
        list.clear();
    }
    return ADPSGD_OK;
}

namespace {

// 17 to 32 strips, which exchange their sums directly: the slowest for its size.
bool slow_exchange(int64_t d) { return d > 16 * kStripCols && d <= kStripGroupBlocks * kStripCols; }

// Workers up to which the one-launch path of the linear models (kernels_strips.hip) is the faster one.  An iteration of the
// strip kernel evaluates as many gradients as there are teams at most (12, 6, 4 and 2 up to M = 16, 32, 64 and 128), so its time
// per event jumps with their number and does not fall with n, while the kernels of a round take its gradients side by side.
// Measured, rounds over strips for a call of 12 n or 400 events (800 set-ups on both sides of the lines: both models, momentum,
// wait-free, losses, T_max 0 ... 40):
//                        ring                                              random 4-regular graph
//   d = 300   M <= 8     n = 17 ... 28 1.3 ... 1.8, n = 30 1.14            n = 27 ... 36 1.3 ... 1.7, n = 40 0.98
//   d = 2000  M <= 8     n = 22 ... 36 1.1 ... 1.8, n = 38 0.92            n = 34 ... 46 1.1 ... 1.5 (n = 41 0.93), n = 59 0.50
//   d = 4096  M <= 8     n = 33 ... 73 1.3 ... 2.3, n = 79 1.01            n = 35 ... 77 1.4 ... 2.7
//   d = 8192  M <= 8     n = 31 ... 58 1.4 ... 2.3, n = 54 1.06            n = 38 ... 78 1.4 ... 2.0, n = 90 0.76
//   d > 8192  M <= 8     n = 30 ... 45 1.2 ... 2.5, n = 60 1.14            n = 37 ... 56 1.4 ... 2.1, n = 83 1.40, n = 100 0.92
//   d = 8192  M <= 16    n = 19, 29 1.35; T_max >= 8: n = 28 0.65          n = 25 ... 34 1.2 ... 1.3, n = 56 0.77 ... 0.86; T_max >= 8: n = 33 0.79
//   d = 4096  M <= 32    n = 21 ... 25 1.06 ... 1.3; T_max = 40: 0.7        n = 25 1.32, n = 33 0.88, n = 40 0.63
//   d = 8192  M <= 32    n = 13 1.08 ... 1.3, n = 15 0.5 ... 0.9, n = 20 0.45    n = 16 1.09, n = 22 0.66, n = 34 0.45
//   d > 8192  M <= 32    n = 22 1.1 ... 1.4, n = 25 ... 28 0.83 ... 1.37  n = 29 1.22, n = 41 0.93
//   d = 4096  M <= 64    T_max = 40: n = 15 0.66                           n = 13 1.21; T_max = 40: n = 22 0.62
//   d = 8192  M <= 64    n = 6 0.8 ... 1.3, n = 11 0.40 ... 0.84           n = 6 1.28, n = 10 0.7 ... 1.07, n = 12 0.5, n = 16 0.54
//   d = 4096  M <= 128   n = 8 1.04, n = 11 0.5 ... 0.8                    n = 8 1.22, n = 10 0.6
//   d > 8192  M <= 128   n = 5 1.2 ... 1.4, n = 10 1.08; T_max >= 8: 0.7   n = 8 1.0 ... 1.1, n = 11 0.7 ... 1.07; T_max >= 8: 0.78
// Long staleness lets a round take more gradients at once, where an iteration is held to its teams.
// 17 to 32 strips (d = 8192) have lines of their own (slow_exchange).  Ten strips and fewer keep n = 48 for
// M <= 32 on denser graphs.  Models and slots that do not fit LDS cost more than the table says.
int32_t strip_workers(int64_t d, int32_t M, int64_t T_max, bool ring, bool lds_state) {
    const bool late = T_max >= 8, slow = slow_exchange(d);
    int32_t n;
    if (M <= 8) {
        if (d < 1024) n = ring ? 28 : 36;
        else if (d <= 2048) n = ring ? 34 : 40;
        else if (slow) n = ring ? 50 : 64;
        else if (M <= 3) n = ring ? 46 : 54;
        else n = ring ? 60 : 76;
    } else if (d <= 2048) {
        const bool shorter = d < 1024;
        if (M <= 16) n = shorter ? (ring ? 16 : 24) : (ring ? 20 : 32);
        else if (M <= 32) n = shorter ? (ring ? 12 : 16) : (ring ? 16 : 24);
        else if (M <= 64) n = shorter ? 8 : 16;
        else n = shorter ? 5 : 8;
    } else if (slow) {
        n = M <= 16 ? (late ? 24 : ring ? 34 : 44) : M <= 32 ? (ring ? (late ? 10 : 14) : 16) : M <= 48 && !late ? 10 : M <= 64 ? 6 : late ? 4 : 5;
    } else if (d <= 16 * kStripCols) {
        if (M <= 16) n = ring ? 40 : 64;
        else if (M <= 32) n = ring ? (late ? 20 : 28) : d <= 10 * kStripCols ? 48 : 28;
        else n = M > 64 ? 8 : late ? (M <= 48 ? 12 : 8) : 16;
    } else {
        if (M <= 16) n = ring ? 40 : 64;
        else if (M <= 32) n = ring ? 28 : 36;
        else if (M <= 64) n = ring ? (M <= 48 ? 16 : 14) : (M <= 48 ? 22 : 20);
        else n = M > 96 ? 9 : late ? 8 : 11;
    }
    return lds_state ? n : std::min(n, 16);
}

// Gradients of a call that the strip kernel can hold in LDS beside the models of its columns.
int64_t strip_lds_slots(const adpsgd_t* h) {
    const int64_t fixed = static_cast<int64_t>(strip_lds_bytes(h->o.M, h->n, h->o.V != nullptr, 0, true));
    return (kStripLdsBytes - fixed) / (kStripCols * static_cast<int64_t>(sizeof(float)));
}

}  // namespace

// Whether the calls of a handle may take the one-launch path of the linear models is settled when it is created, with the
// memory that path needs; a handle that cannot have it goes by rounds.
void settle_strips(adpsgd_t* h) {
    const int32_t model = h->o.model;
    if ((model != ADPSGD_MODEL_LSQ && model != ADPSGD_MODEL_LOGREG) || h->d > kStripMaxD || h->o.M > kStripMaxM) return;
    const bool ring = h->rowptr[h->n] <= 3 * static_cast<int64_t>(h->n), lds_state = strip_lds_slots(h) >= static_cast<int64_t>(h->o.T_max) + 1;
    if (h->n > strip_workers(h->d, h->o.M, h->o.T_max, ring, lds_state)) return;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    int dev = 0, cus = 0, cooperative = 0;
    const size_t words = strip_exchange_bytes(model, h->o.M);
    const size_t alone = static_cast<size_t>(strip_window(h->o.T_max, true, strip_lds_slots(h), h->n_slots)) * h->o.ldx * sizeof(float);
    if (hipStreamIsCapturing(h->stream, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone && hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipDeviceGetAttribute(&cooperative, hipDeviceAttributeCooperativeLaunch, dev) == hipSuccess && cooperative != 0 &&
        strip_blocks(h->d) <= std::min(cus, kStripGroups * kStripGroupBlocks) && h->exchange.reserve(words) == hipSuccess &&
        h->exchange_status.reserve(sizeof(int)) == hipSuccess &&
        (!lds_state || h->alone_slots.reserve(alone) == hipSuccess) &&
        hipMemset(h->exchange.p, 0, h->exchange.cap) == hipSuccess &&      // no sequence number
        hipStreamSynchronize(nullptr) == hipSuccess) {
        *static_cast<int*>(h->exchange_status.p) = 0;
        h->strip_units = std::min(cus, kStripGroups * kStripGroupBlocks);
        return;
    }
    (void)hipGetLastError();
    h->exchange.release();
    h->exchange_status.release();
    h->alone_slots.release();
}

void settle_onepass(adpsgd_t* h) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    int dev = 0, cus = 0;
    if (hipStreamIsCapturing(h->stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    const OnePassShape s = onepass_shape(h->o.model, h->d, h->o.M, cus), sync = onepass_shape(h->o.model, h->d, h->o.M, cus, h->n);
    if (!s.ok() || !sync.ok()) return;
    const size_t bytes = std::max(onepass_exchange_bytes(s, h->o.M), onepass_exchange_bytes(sync, h->o.M));
    const bool has_status = h->exchange_status.p != nullptr;
    if (h->onepass_words.reserve(bytes + sizeof(unsigned long long)) == hipSuccess &&
        h->exchange_status.reserve(sizeof(int)) == hipSuccess &&
        hipMemsetAsync(h->onepass_words.p, 0, h->onepass_words.cap, h->stream) == hipSuccess) {       // before all launches of the handle
        if (!has_status) *static_cast<int*>(h->exchange_status.p) = 0;
        h->onepass = s;
        h->onepass_sync = sync;
        h->onepass_bytes = bytes;
        return;
    }
    (void)hipGetLastError();
    h->onepass_words.release();
    if (!has_status) h->exchange_status.release();
}

bool can_run_onepass(const adpsgd_t* h) {
    if (!h->onepass.ok()) return false;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return capture == hipStreamCaptureStatusNone;
}

int launch_onepass(adpsgd_t* h, const OnePassShape& shape, const LinearGradArgs& a) {
    const size_t bytes = h->onepass_bytes;
    if (h->onepass_seq > 0xFFFFFFFFu - static_cast<uint32_t>(a.n_ops)) {      // before the numbers wrap
        HIP_TRY(h, hipMemsetAsync(h->onepass_words.p, 0, bytes, h->stream));
        h->onepass_seq = 0;
    }
    const uint64_t wait_us = static_cast<uint64_t>(std::min(h->assembly_us, kOnePassWaitUs));
    const OnePassArgs o{shape, a.model, a.X, a.ld, a.d, a.ops, a.n_ops, a.M, a.batch_idx, a.slots, a.gscale, a.lambda, a.loss,
                        static_cast<unsigned long long*>(h->onepass_words.p), static_cast<unsigned long long*>(h->onepass_words.p) + bytes / sizeof(unsigned long long),
                        static_cast<int*>(h->exchange_status.p), h->onepass_seq + 1, wait_us * kClockTicksPerUs};
    HIP_TRY(h, launch_onepass_gradient(o, h->stream));
    h->onepass_seq += static_cast<uint32_t>(a.n_ops);
    return ADPSGD_OK;
}

}  // namespace adpsgd_impl

using namespace adpsgd_impl;

namespace {

// Everything a handle holds, once no work of it is under way.
void release_all(adpsgd_t* h) {
    for (auto& t : h->tables) {
        t.stage.release();
        t.dev.release();
        if (t.done) (void)hipEventDestroy(t.done);
    }
    for (auto& pr : h->ev_fused) { (void)hipEventDestroy(pr.first); (void)hipEventDestroy(pr.second); }
    for (auto& pr : h->ev_grad) { (void)hipEventDestroy(pr.first); (void)hipEventDestroy(pr.second); }
    for (auto e : h->ev_pool) (void)hipEventDestroy(e);
    h->grad_scratch.release();
    h->comp_rows.release();
    h->diag.release();
    h->sync_other.release();
    h->exchange.release();
    h->exchange_status.release();
    h->alone_slots.release();
    h->onepass_words.release();
}

}  // namespace

extern "C" const char* adpsgd_last_error(const adpsgd_t* h) { return h ? h->err.c_str() : create_error().c_str(); }

extern "C" int adpsgd_create(adpsgd_t** out, const adpsgd_graph_t* graph, int64_t d, const adpsgd_opts_t* opts) {
    if (!out) return fail(nullptr, ADPSGD_ERR_ARG, "create: out is NULL");
    *out = nullptr;
    if (!graph || !opts) return fail(nullptr, ADPSGD_ERR_ARG, "create: graph or opts is NULL");
    std::string msg;
    if (!graph_ok(graph, msg)) return fail(nullptr, ADPSGD_ERR_GRAPH, msg);
    const int32_t n = graph->n;
    if (n > 65535) return fail(nullptr, ADPSGD_ERR_ARG, "create: at most 65535 workers");
    if (d < 1) return fail(nullptr, ADPSGD_ERR_ARG, "create: d < 1");
    const adpsgd_opts_t& o = *opts;
    if (o.model < ADPSGD_MODEL_LSQ || o.model > ADPSGD_MODEL_EXTERNAL) return fail(nullptr, ADPSGD_ERR_ARG, "create: unknown model");
    const bool external = o.model == ADPSGD_MODEL_EXTERNAL;
    if (!o.X || !aligned16(o.X)) return fail(nullptr, ADPSGD_ERR_ARG, "create: X is NULL or not 16-byte aligned");
    if (o.ldx < d || (o.ldx & 3)) return fail(nullptr, ADPSGD_ERR_ARG, "create: ldx must be >= d and a multiple of 4");
    if (o.T_max < 0) return fail(nullptr, ADPSGD_ERR_ARG, "create: T_max < 0");
    if (!std::isfinite(o.gamma)) return fail(nullptr, ADPSGD_ERR_ARG, "create: gamma not finite");
    int32_t n_slots = 0;
    if (o.model != ADPSGD_MODEL_SYNTH) {
        if (!external && (o.M < 1 || o.M > 65536)) return fail(nullptr, ADPSGD_ERR_ARG, "create: minibatch size M outside [1, 65536]");
        if (!o.workspace || !aligned16(o.workspace)) return fail(nullptr, ADPSGD_ERR_ARG, "create: workspace is NULL or misaligned");
        const int64_t slot_bytes = o.ldx * 4;
        const int64_t have = o.workspace_bytes / slot_bytes;
        if (have < static_cast<int64_t>(o.T_max) + 1)
            return fail(nullptr, ADPSGD_ERR_ARG, "create: workspace smaller than (T_max + 1) gradient slots");
        n_slots = static_cast<int32_t>(std::min<int64_t>(have, kMaxSlots));
    }
    if (o.model == ADPSGD_MODEL_MLP) {
        if (o.mlp_in < 1 || o.mlp_hidden < 1 || o.mlp_out < 1 ||
            d != static_cast<int64_t>(o.mlp_in) * o.mlp_hidden + o.mlp_hidden +
                     static_cast<int64_t>(o.mlp_hidden) * o.mlp_out + o.mlp_out)
            return fail(nullptr, ADPSGD_ERR_ARG, "create: d does not match the MLP layer sizes");
        if (!o.Xbf16 || !aligned16(o.Xbf16)) return fail(nullptr, ADPSGD_ERR_ARG, "create: Xbf16 is NULL or misaligned");
        if (o.ldx & 7) return fail(nullptr, ADPSGD_ERR_ARG, "create: ldx must be a multiple of 8 for the MLP");
        if (mlp_scratch_bytes(1, o.M, o.mlp_in, o.mlp_hidden, o.mlp_out) == 0)
            return fail(nullptr, ADPSGD_ERR_ARG, "create: MLP shape not supported by the gradient kernel");
    }
    if (!std::isfinite(o.momentum) || !std::isfinite(o.weight_decay))
        return fail(nullptr, ADPSGD_ERR_ARG, "create: momentum or weight_decay not finite");
    if ((o.momentum != 0.0f || o.weight_decay != 0.0f) && (!o.V || !aligned16(o.V)))
        return fail(nullptr, ADPSGD_ERR_ARG, "create: momentum / weight decay need the buffer V (16-byte aligned)");
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count < 1)
        return fail(nullptr, ADPSGD_ERR_HIP, "create: no HIP device available");

    std::unique_ptr<adpsgd> h(new (std::nothrow) adpsgd);
    if (!h) return fail(nullptr, ADPSGD_ERR_ARG, "create: out of host memory");
    h->n = n;
    h->d = d;
    h->o = o;
    h->rowptr.assign(graph->rowptr, graph->rowptr + n + 1);
    h->col.assign(graph->col, graph->col + graph->rowptr[n]);
    h->data.resize(n);
    h->n_slots = n_slots;
    h->stream = static_cast<hipStream_t>(o.stream);
    h->streaming = static_cast<int64_t>(n) * o.ldx * 4 > kStreamingThreshold;
    h->stats.slots = n_slots;
    settle_strips(h.get());
    settle_onepass(h.get());
    for (auto& t : h->tables) {
        const hipError_t e = hipEventCreateWithFlags(&t.done, hipEventDisableTiming);
        if (e != hipSuccess) {
            release_all(h.get());
            return hip_fail(nullptr, e, "create: hipEventCreate");
        }
    }
    *out = h.release();
    return ADPSGD_OK;
}

extern "C" void adpsgd_destroy(adpsgd_t* h) {
    if (!h) return;
    (void)hipStreamSynchronize(h->stream);
    release_all(h);
    delete h;
}

extern "C" int adpsgd_load_data(adpsgd_t* h, int32_t worker, const void* features, int64_t rows, int64_t ld,
                                const void* targets) {
    if (!h) return ADPSGD_ERR_ARG;
    if (h->o.model == ADPSGD_MODEL_SYNTH || h->o.model == ADPSGD_MODEL_EXTERNAL)
        return fail(h, ADPSGD_ERR_STATE, "load_data: this model takes no data");
    if (worker < 0 || worker >= h->n) return fail(h, ADPSGD_ERR_ARG, "load_data: worker out of range");
    if (!features || !targets || rows < 1 || rows > 0x7FFFFFFF) return fail(h, ADPSGD_ERR_ARG, "load_data: null data or bad row count");
    if (!aligned16(features)) return fail(h, ADPSGD_ERR_ARG, "load_data: features not 16-byte aligned");
    if (h->o.model == ADPSGD_MODEL_MLP) {
        if (ld < h->o.mlp_in || (ld & 7)) return fail(h, ADPSGD_ERR_ARG, "load_data: ld must be >= mlp_in and a multiple of 8");
    } else {
        if (ld < h->d || (ld & 3)) return fail(h, ADPSGD_ERR_ARG, "load_data: ld must be >= d and a multiple of 4");
    }
    WorkerData& w = h->data[worker];
    w.features = features;
    w.targets = targets;
    w.rows = rows;
    w.ld = ld;
    return ADPSGD_OK;
}

extern "C" int adpsgd_set_models(adpsgd_t* h, const float* x, int64_t ld_in, int32_t on_device) {
    if (!h || !x) return h ? fail(h, ADPSGD_ERR_ARG, "set_models: x is NULL") : ADPSGD_ERR_ARG;
    if (ld_in != 0 && ld_in < h->d) return fail(h, ADPSGD_ERR_ARG, "set_models: ld_in < d");
    if (h->exchange_status.p) {                // what a launch that was given up has left is replaced; one may still be under way
        HIP_TRY(h, hipStreamSynchronize(h->stream));
        *static_cast<int*>(h->exchange_status.p) = 0;
    }
    h->pending.clear();      // gradients evaluated at the old models are dropped
    h->pending_batch.clear();
    const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    if (ld_in == 0) {
        const float* src = x;
        if (!on_device) {
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            HIP_TRY(h, h->diag.reserve(static_cast<size_t>(h->d) * 4));
            HIP_TRY(h, hipMemcpy(h->diag.p, x, static_cast<size_t>(h->d) * 4, hipMemcpyHostToDevice));
            src = static_cast<const float*>(h->diag.p);
        }
        HIP_TRY(h, launch_broadcast_rows(h->o.X, h->o.ldx, h->d, h->n, src, h->stream));
    } else {
        HIP_TRY(h, hipMemsetAsync(h->o.X, 0, static_cast<size_t>(h->n) * h->o.ldx * 4, h->stream));
        HIP_TRY(h, hipMemcpy2DAsync(h->o.X, static_cast<size_t>(h->o.ldx) * 4, x, static_cast<size_t>(ld_in) * 4,
                                    static_cast<size_t>(h->d) * 4, h->n, kind, h->stream));
    }
    if (h->o.model == ADPSGD_MODEL_MLP)
        HIP_TRY(h, launch_refresh_bf16(h->o.X, h->o.Xbf16, h->o.ldx, h->n, h->stream));
    if (h->o.V) HIP_TRY(h, hipMemsetAsync(h->o.V, 0, static_cast<size_t>(h->n) * h->o.ldx * 4, h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    return ADPSGD_OK;
}

namespace {

// Checks a schedule against the documented constraints; nothing is launched and no state changes
// when it fails.
int validate_schedule(adpsgd_t* h, const adpsgd_schedule_t* s, bool with_data, int32_t M, int64_t n_extra) {
    const int64_t K = s->K;
    const int64_t n_pending = static_cast<int64_t>(h->pending.size());
    if (s->lookahead < 0 || s->lookahead > K) return fail(h, ADPSGD_ERR_ARG, "run_events: lookahead outside [0, K]");
    if (s->lookahead > 0 && h->o.model == ADPSGD_MODEL_SYNTH)
        return fail(h, ADPSGD_ERR_ARG, "run_events: the synthetic-gradient model has no stale reads to look ahead to");
    if (K < n_pending)
        return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: the call must start with the " + std::to_string(n_pending) +
                                                " events the previous call looked ahead to");
    for (int64_t k = 0; k < n_pending; ++k) {
        const PendingEvent& e = h->pending[k];
        bool same = s->worker[k] == e.worker && s->tau[k] == e.tau;
        for (int32_t m = 0; same && m < M; ++m) same = s->batch_idx[k * static_cast<int64_t>(M) + m] == h->pending_batch[k * static_cast<int64_t>(M) + m];
        if (!same)
            return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: event " + std::to_string(k) + " differs from the event the previous call looked ahead to");
    }
    if (s->extra_ptr) {
        if (s->extra_ptr[0] != 0 || n_extra < 0 || (n_extra > 0 && (!s->extra_a || !s->extra_b)))
            return fail(h, ADPSGD_ERR_ARG, "run_events: malformed extra-pair arrays");
        std::vector<int64_t> stamp(h->n, -1);
        for (int64_t k = 0; k < K; ++k) {
            if (s->extra_ptr[k + 1] < s->extra_ptr[k] || s->extra_ptr[k + 1] > n_extra)
                return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: extra_ptr not monotone at event " + std::to_string(k));
            if (s->worker[k] >= 0 && s->worker[k] < h->n) stamp[s->worker[k]] = k;
            if (s->neighbour[k] >= 0 && s->neighbour[k] < h->n) stamp[s->neighbour[k]] = k;
            for (int64_t q = s->extra_ptr[k]; q < s->extra_ptr[k + 1]; ++q) {
                const int32_t a = s->extra_a[q], b = s->extra_b[q];
                if (a < 0 || a >= h->n || b < 0 || b >= h->n || a == b || !is_neighbour(h, a, b))
                    return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: extra pair is not an edge of the graph at event " + std::to_string(k));
                if (stamp[a] == k || stamp[b] == k)
                    return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: the pairs of one event must be disjoint (event " + std::to_string(k) + ")");
                stamp[a] = stamp[b] = k;
            }
        }
    }
    for (int64_t k = 0; k < K; ++k) {
        const int32_t i = s->worker[k], j = s->neighbour[k];
        if (i < 0 || i >= h->n || j < 0 || j >= h->n)
            return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: worker or neighbour out of range at event " + std::to_string(k));
        if (!is_neighbour(h, i, j))
            return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: neighbour is not adjacent to worker at event " + std::to_string(k));
        const bool carried = k < n_pending && h->pending[k].slot >= 0;      // read before this call began
        if (s->tau[k] < 0 || s->tau[k] > h->o.T_max || (carried ? s->tau[k] <= k : s->tau[k] > k))
            return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: tau outside [0, min(k, T_max)] at event " + std::to_string(k));
        if (s->gamma && !std::isfinite(s->gamma[k]))
            return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: gamma not finite at event " + std::to_string(k));
        if (with_data) {
            const WorkerData& w = h->data[i];
            if (!w.features) return fail(h, ADPSGD_ERR_STATE, "run_events: no data loaded for worker " + std::to_string(i));
            const int32_t* b = s->batch_idx + k * static_cast<int64_t>(M);
            for (int32_t m = 0; m < M; ++m)
                if (b[m] < 0 || b[m] >= w.rows)
                    return fail(h, ADPSGD_ERR_SCHEDULE, "run_events: batch index out of range at event " + std::to_string(k));
        }
    }
    return ADPSGD_OK;
}

// What one call of run_events works with: the paths taken, the plan sorted by round, the tables.
struct EventCall {
    const adpsgd_schedule_t* s = nullptr;
    int64_t K = 0;              // events in the arrays
    int64_t A = 0;              // of which this call applies the first A (the others are looked ahead to)
    int64_t n_extra = 0;        // extra averaging pairs of the applied events
    int32_t M = 0;
    bool external = false;      // gradients from the caller's function
    bool with_grad = false;     // the events carry gradients held in pending slots (every model but SYNTH)
    bool mlp_comp = false;      // perceptron, wait-free variant: compensated bf16 rows
    bool ext_comp = false;      // caller's function, wait-free variant: compensated fp32 rows
    bool factored = false;      // perceptron: dW1 stays in factored form until the update kernel
    int32_t chain = 1;          // updates of a round that may follow each other on a row
    bool chained() const { return chain > 1 || lin_factored; }      // the update kernel takes chains (of one, where chain is 1)
    std::vector<UpdateChain> chains;        // chained: the updates, by round ...
    std::vector<int64_t> chain_off;         // ... and where those of a round begin
    std::vector<int64_t> chain_event;       // ... and the event of every operation, -1: averaging only
    const UpdateChain* d_chains = nullptr;
    bool lin_factored = false;  // least squares on long models: the gradient stays M coefficients
    bool strips = false;        // linear models: all events in one launch (kernels_strips.hip)
    bool onepass = false;       // linear models: gradients in one pass over the rows (kernels_onepass.hip), dense
    Plan plan;
    std::vector<int64_t> u_off, r_off;      // first update / gradient operation of every round
    int32_t group = 1;                      // gradients of a round are launched in groups of this many operations
    TableSet* T = nullptr;
    PairOp* uops = nullptr;                 // pinned staging, sorted by round
    GradOp* rops = nullptr;
    const PairOp* d_uops = nullptr;         // the device copy
    const GradOp* d_rops = nullptr;
    const int32_t* d_batch = nullptr;
    int32_t* batch_r = nullptr;             // perceptron: the minibatch indices again, in the order of rops (pinned staging)
    const int32_t* d_batch_r = nullptr;
    const int32_t* d_batch_u = nullptr;
    std::vector<int32_t> carried_slot;      // per event: slot of a gradient evaluated by an earlier call, or -1; or empty
    size_t off_coef = 0;                    // linear models: offset of the coefficients in the gradient scratch
};

// Whether a call takes the one-launch path of the linear models.  Decided by the handle, so that a schedule gives the same
// bits however it is cut into calls; only a stream under capture goes by rounds (a captured call would need a cooperative
// launch in a graph), a handle whose caller has asked for them, and short calls (small_call).
bool can_run_strips(const adpsgd_t* h) {
    if (h->strip_units == 0 || h->route != ADPSGD_ROUTE_AUTO) return false;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (capture != hipStreamCaptureStatusNone) return false;
    for (const WorkerData& w : h->data)
        if (w.ld > 0xFFFFFFFFll) return false;          // the row pitch has to fit a word of a record
    return true;
}

// A call of few events: the cooperative launch, the assembly of its blocks and the first iterations take 50 us, where a call in
// rounds takes 14 and 2.8 for each round with updates, and for each with gradients 8.6 in one pass over the rows, 7 and 11.6 in two
// and three launches, or on short models, whose gradients are a block each, 3.8 and what the block takes to read the rows of one.
// Fitted to 290 such calls, each by both routes (K 1 ... 100, M 1 ... 128, d 300 ... 65 536, T_max 1 ... 40): on these and 280 others
// it takes 1.004 times as long as the better route in the mean and 1.24 at most; the estimate before it, which counted three
// launches and two reads of the rows for every gradient of a long model and no time for the single blocks, 1.026 and 2.5 (rounds
// always: 1.28, one launch always: 1.26).  Strips / rounds in us:  n = 8, d = 2000, M = 64, 64 events 166 / 412;  n = 16, d = 65 536, M = 16, 12
// events 87 / 64;  n = 8, d = 1024, M = 32: 1 event 47 / 23, 16 events 66 / 63, 32 events 84 / 116;  n = 16, d = 7395, M = 6,
// T_max = 100, where most reads of a short call precede its first update and share their launches: 23 events 83 / 48.
// Calls that are cut out of one schedule (looking ahead, or without stale reads at all) keep the handle's route, up to 25 us
// slower for a few events, so that the cut does not change the order of any sum.
bool small_call(const adpsgd_t* h, const EventCall& c) {
    if (c.K > 128 || h->o.T_max == 0 || c.s->lookahead > 0 || !h->pending.empty()) return false;
    const bool short_model = h->d <= 2048;
    const double events = static_cast<double>(c.K), gradient_mb = 4.0e-6 * c.M * static_cast<double>(h->d);
    const double per_set = short_model ? 3.8 + 17.0 * gradient_mb : c.onepass ? 8.6 : c.lin_factored ? 7.0 : 11.6;
    const double per_mb = short_model ? 0.0 : c.onepass ? 0.25 : 2.0;
    double rounds = 14.0 + per_mb * events * gradient_mb;
    for (int32_t r = 0; r < c.plan.n_rounds; ++r) rounds += (c.u_off[r + 1] > c.u_off[r] ? 2.8 : 0.0) + (c.r_off[r + 1] > c.r_off[r] ? per_set : 0.0);
    const int32_t teams = strip_teams(c.M);
    const double per_event = teams == 12 ? 0.8 : (teams == 6 ? 1.1 : teams == 4 ? 1.7 : 3.5) * (slow_exchange(h->d) ? strip_blocks(h->d) / 16.0 : 1.0);
    return rounds < 50.0 + (per_event + 0.3 * gradient_mb) * events;
}

// Validation, choice of paths, plan of rounds, counting sort of the operations by round.
int prepare_call(adpsgd_t* h, const adpsgd_schedule_t* s, EventCall& c) {
    c.s = s;
    c.K = s->K;
    if (c.K > 0x7FFFFFF0) return fail(h, ADPSGD_ERR_ARG, "run_events: at most 2^31 - 16 events per call");
    if (!s->worker || !s->neighbour || !s->tau) return fail(h, ADPSGD_ERR_ARG, "run_events: null schedule array");
    c.external = h->o.model == ADPSGD_MODEL_EXTERNAL;
    c.with_grad = h->o.model != ADPSGD_MODEL_SYNTH;
    const bool with_data = c.with_grad && !c.external;
    c.M = with_data ? h->o.M : 0;
    if (with_data && !s->batch_idx) return fail(h, ADPSGD_ERR_ARG, "run_events: batch_idx is NULL");
    const int rc_valid = validate_schedule(h, s, with_data, c.M, s->extra_ptr ? s->extra_ptr[c.K] : 0);
    if (rc_valid != ADPSGD_OK) return rc_valid;
    c.A = c.K - s->lookahead;
    c.n_extra = s->extra_ptr ? s->extra_ptr[c.A] : 0;
    bool any_carried = false;
    if (!h->pending.empty()) {
        c.carried_slot.assign(static_cast<size_t>(c.K), -1);
        for (size_t k = 0; k < h->pending.size(); ++k) {
            c.carried_slot[k] = h->pending[k].slot;
            any_carried |= h->pending[k].slot >= 0;
        }
    }
    const int32_t* carried = c.carried_slot.empty() ? nullptr : c.carried_slot.data();

    // the wait-free variant reads the pending gradient as a dense vector, so it keeps the dense form
    const bool comp = h->o.local_compensation != 0, dense = (h->o.flags & ADPSGD_FLAG_DENSE_GRADIENT) != 0;
    c.mlp_comp = h->o.model == ADPSGD_MODEL_MLP && comp;
    c.ext_comp = c.external && comp;
    c.factored = h->o.model == ADPSGD_MODEL_MLP && !dense && !comp && mlp_can_factor(h->o.mlp_in, h->o.mlp_hidden, c.M);
    c.lin_factored = with_data && !dense && !comp && linear_can_factor(h->o.model, h->d, c.M, h->o.ldx);
    // gradients pending from an earlier call come as it left them: dense vectors, or coefficients
    c.strips = with_data && can_run_strips(h) && (!any_carried || h->pending_dense);
    if (any_carried && h->pending_dense) c.lin_factored = false;
    // Chains move a row once for several updates and make fewer rounds (caller's gradients, n = 8, d = 12 M, momentum, 60 events: 31
    // rounds and 4.73 ms without, 19 and 3.91 with them; least squares, n = 32, M = 8, d = 4 Mi, 200 events: 33 and 10.75, 22 and
    // 10.31; logistic, n = 64, M = 128, d = 65 536, 500 events: 36 and 4.59, 25 and 4.45).  A caller's gradients on short models keep
    // the rounds of the synthetic model, as the interface has it (7 % in the mean of 20 such calls, which the caller's own
    // launches bind).  A handle whose calls go in one launch keeps plain rounds for its short calls (small_call was drawn with them).
    c.chain = h->o.model == ADPSGD_MODEL_MLP ? mlp_chain(h->o.V != nullptr, h->d) : (with_data && !c.strips) || (c.external && h->d > 4096) ? kChain : 1;
    c.onepass = with_data && onepass_for_events(h->onepass, h->o.model, c.M, comp) && can_run_onepass(h) && (!any_carried || h->pending_dense);
    if (c.onepass) c.lin_factored = false;

    std::string perr;
    const int rc = plan_rounds(h->n, c.K, s->worker, s->neighbour, s->tau, h->n_slots, c.with_grad, c.plan, perr,
                               s->extra_ptr, s->extra_a, s->extra_b, comp, c.A, carried, c.chain);
    if (rc != ADPSGD_OK) return fail(h, rc, perr);
    if ((h->o.flags & ADPSGD_FLAG_VERIFY_PLAN) &&
        !verify_plan(h->n, c.K, s->worker, s->neighbour, s->tau, h->n_slots, c.with_grad, c.plan, perr, s->extra_ptr, s->extra_a,
                     s->extra_b, c.A, carried, c.chain > 1))
        return fail(h, ADPSGD_ERR_STATE, perr);

    const int32_t R = c.plan.n_rounds;
    c.u_off.assign(static_cast<size_t>(R) + 1, 0);
    c.r_off.assign(static_cast<size_t>(R) + 1, 0);
    for (int64_t k = 0; k < c.K; ++k) {
        if (k < c.A) c.u_off[c.plan.u_round[k] + 1] += 1 + (s->extra_ptr ? s->extra_ptr[k + 1] - s->extra_ptr[k] : 0);
        if (c.with_grad && c.plan.r_round[k] >= 0) ++c.r_off[c.plan.r_round[k] + 1];      // not carried, not left to the next call
    }
    int64_t max_r = 0;
    for (int32_t r = 0; r < R; ++r) {
        max_r = std::max(max_r, c.r_off[r + 1]);
        c.u_off[r + 1] += c.u_off[r];
        c.r_off[r + 1] += c.r_off[r];
    }
    c.strips = c.strips && !small_call(h, c);
    if (c.with_grad)
        c.group = static_cast<int32_t>(std::min<int64_t>(std::max<int64_t>(max_r, 1), h->o.model == ADPSGD_MODEL_MLP ? 64 : 65535));
    return ADPSGD_OK;
}

// The update operations of event k (its own pair and the extra pairs of its W_k), appended to the event's round.
void fill_update(adpsgd_t* h, EventCall& c, int64_t k, std::vector<int64_t>& u_fill) {
    const adpsgd_schedule_t* s = c.s;
    const uint64_t gk = h->events_done + static_cast<uint64_t>(k);
    const int32_t ur = c.plan.u_round[k];
    PairOp& u = c.uops[u_fill[ur]++];
    u.i = s->worker[k];
    u.j = s->neighbour[k];
    u.k_lo = static_cast<uint32_t>(gk);
    u.k_hi = static_cast<uint32_t>(gk >> 32);
    u.gamma = s->gamma ? s->gamma[k] : h->o.gamma;
    u.slot = c.with_grad ? c.plan.slot[k] : 0;
    u.flags = 0;
    u.pad = 0;
    if (s->extra_ptr)
        for (int64_t q = s->extra_ptr[k]; q < s->extra_ptr[k + 1]; ++q)
            c.uops[u_fill[ur]++] = PairOp{s->extra_a[q], s->extra_b[q], 0u, 0u, 0.0f, 0, 1, 0};
}

// The updates of a call as the chains of every round.
int build_chains(adpsgd_t* h, EventCall& c) {
    const adpsgd_schedule_t* s = c.s;
    const ChainCall call{h->n, c.A, s->worker, s->neighbour, s->extra_ptr, s->extra_a, s->extra_b, s->gamma, h->o.gamma, &c.plan, h->data.data(), &c.u_off};
    ChainLayout layout;
    std::vector<ColumnPair> pairs;
    chain_pairs(call, pairs);
    chain_rounds(pairs, c.u_off, h->n, layout);
    if ((h->o.flags & ADPSGD_FLAG_VERIFY_PLAN) && !verify_chains(pairs, c.u_off, h->n, c.chain, layout))
        return fail(h, ADPSGD_ERR_STATE, "plan check: chains of updates out of order");
    if (!fill_chains(call, pairs, layout, c.chain, c.chains, c.chain_event)) return fail(h, ADPSGD_ERR_STATE, "run_events: a chain of updates is too long");
    c.chain_off = layout.round;
    return ADPSGD_OK;
}

// The stale read and gradient of event k, appended to its round.
void fill_gradient(adpsgd_t* h, EventCall& c, int64_t k, std::vector<int64_t>& r_fill) {
    const adpsgd_schedule_t* s = c.s;
    const int32_t rr = c.plan.r_round[k];
    const int64_t at = r_fill[rr]++;
    if (c.batch_r) std::memcpy(c.batch_r + at * c.M, s->batch_idx + k * static_cast<int64_t>(c.M), static_cast<size_t>(c.M) * 4);
    GradOp& g = c.rops[at];
    g.worker = s->worker[k];
    g.slot = c.plan.slot[k];
    g.event = static_cast<int32_t>(k);
    const int64_t kp = c.plan.prev[k];
    g.comp_slot = kp >= 0 ? c.plan.slot[kp] : -1;
    g.comp_gamma = kp >= 0 ? (s->gamma ? s->gamma[kp] : h->o.gamma) : 0.0f;
    g.count = 0;
    const WorkerData& w = h->data[g.worker];
    g.features = w.features;
    g.targets = w.targets;
    g.ld = w.ld;
    g.xrow_bf16 = nullptr;
    if (c.mlp_comp && kp >= 0)      // one compensated row per operation of a launch group
        g.xrow_bf16 = static_cast<uint16_t*>(h->comp_rows.p) + ((at - c.r_off[rr]) % c.group) * h->o.ldx;
}

// Tables [PairOp x (K + extra pairs), or the chains][GradOp x K][batch_idx K x M], filled in pinned memory in round
// order and uploaded with one copy; scratch memory of the gradient kernels.
int upload_tables(adpsgd_t* h, EventCall& c) {
    const adpsgd_schedule_t* s = c.s;
    const int64_t K = c.K;
    const int32_t M = c.M;
    if (c.mlp_comp) HIP_TRY(h, h->comp_rows.reserve(static_cast<size_t>(c.group) * h->o.ldx * sizeof(uint16_t)));
    if (c.ext_comp) HIP_TRY(h, h->comp_rows.reserve(static_cast<size_t>(c.group) * h->o.ldx * sizeof(float)));
    if (c.chained()) {
        const int rc = build_chains(h, c);
        if (rc != ADPSGD_OK) return rc;
    }
    const size_t bytes_u = c.chained() ? c.chains.size() * sizeof(UpdateChain) : static_cast<size_t>(c.A + c.n_extra) * sizeof(PairOp);
    const size_t bytes_r = c.with_grad ? static_cast<size_t>(K) * sizeof(GradOp) : 0;
    const size_t bytes_b = static_cast<size_t>(K) * M * sizeof(int32_t);
    const size_t off_r = bytes_u, off_b = (off_r + bytes_r + 15) & ~size_t(15);
    // the perceptron's kernels read the indices by operation instead of by event: one copy in the order of the
    // gradient operations, one in the order of the chains' operations (rows of averaging-only pairs stay zero)
    const bool by_op = h->o.model == ADPSGD_MODEL_MLP;
    const size_t bytes_br = by_op ? bytes_b : 0, bytes_bu = c.factored ? static_cast<size_t>(c.A + c.n_extra) * M * sizeof(int32_t) : 0;
    const size_t off_br = off_b + (by_op ? 0 : bytes_b), off_bu = off_br + bytes_br;
    const size_t total = off_bu + bytes_bu;

    TableSet& T = h->tables[h->next_table];
    h->next_table ^= 1;
    if (T.in_flight) {
        HIP_TRY(h, hipEventSynchronize(T.done));
        T.in_flight = false;
    }
    HIP_TRY(h, T.stage.reserve(total));
    HIP_TRY(h, T.dev.reserve(total));
    c.T = &T;
    char* stage = static_cast<char*>(T.stage.p);
    c.uops = reinterpret_cast<PairOp*>(stage);
    c.rops = reinterpret_cast<GradOp*>(stage + off_r);
    if (by_op) {
        c.batch_r = reinterpret_cast<int32_t*>(stage + off_br);
        std::memset(stage + off_br, 0, bytes_br + bytes_bu);
    }
    if (c.chained()) std::memcpy(stage, c.chains.data(), bytes_u);
    if (c.factored) {
        int32_t* batch_u = reinterpret_cast<int32_t*>(stage + off_bu);
        for (size_t q = 0; q < c.chain_event.size(); ++q)
            if (c.chain_event[q] >= 0) std::memcpy(batch_u + q * M, s->batch_idx + c.chain_event[q] * static_cast<int64_t>(M), static_cast<size_t>(M) * 4);
    }
    std::vector<int64_t> u_fill(c.u_off.begin(), c.u_off.end() - 1), r_fill(c.r_off.begin(), c.r_off.end() - 1);
    for (int64_t k = 0; k < K; ++k) {
        if (k < c.A && !c.chained()) fill_update(h, c, k, u_fill);
        if (c.with_grad && c.plan.r_round[k] >= 0) fill_gradient(h, c, k, r_fill);
    }
    if (bytes_b > 0 && !by_op) std::memcpy(stage + off_b, s->batch_idx, bytes_b);
    HIP_TRY(h, hipMemcpyAsync(T.dev.p, T.stage.p, total, hipMemcpyHostToDevice, h->stream));
    const char* dev = static_cast<const char*>(T.dev.p);
    c.d_uops = reinterpret_cast<const PairOp*>(dev);
    c.d_chains = reinterpret_cast<const UpdateChain*>(dev);
    c.d_rops = reinterpret_cast<const GradOp*>(dev + off_r);
    c.d_batch = reinterpret_cast<const int32_t*>(dev + off_b);
    c.d_batch_r = reinterpret_cast<const int32_t*>(dev + off_br);
    c.d_batch_u = reinterpret_cast<const int32_t*>(dev + off_bu);

    if (c.with_grad && !c.external) {
        if (h->o.model == ADPSGD_MODEL_MLP) {
            HIP_TRY(h, h->grad_scratch.reserve(mlp_scratch_bytes(c.group, M, h->o.mlp_in, h->o.mlp_hidden, h->o.mlp_out)));
        } else {
            // all gradients of a round go into one set of launches (measured: splitting a round so
            // that the gathered rows stay within the memory-side cache only adds launches)
            const size_t partial_bytes = static_cast<size_t>(c.group) * (M + 1) * linear_grad_chunks(h->d) * 4;
            c.off_coef = (partial_bytes + 255) & ~size_t(255);
            HIP_TRY(h, h->grad_scratch.reserve(c.off_coef + static_cast<size_t>(c.group) * M * 4));
        }
    }
    return ADPSGD_OK;
}

// A pair of HIP events around a launch when per-launch timing is on (nullptr otherwise).
int begin_timing(adpsgd_t* h, hipEvent_t& e0, hipEvent_t& e1) {
    e0 = e1 = nullptr;
    if (!(h->o.flags & ADPSGD_FLAG_PROFILE)) return ADPSGD_OK;
    e0 = take_event(h);
    e1 = take_event(h);
    if (!e0 || !e1) return fail(h, ADPSGD_ERR_HIP, "run_events: hipEventCreate failed");
    HIP_TRY(h, hipEventRecord(e0, h->stream));
    return ADPSGD_OK;
}
int end_timing(adpsgd_t* h, hipEvent_t e0, hipEvent_t e1, std::vector<std::pair<hipEvent_t, hipEvent_t>>& into) {
    if (!e0) return ADPSGD_OK;
    HIP_TRY(h, hipEventRecord(e1, h->stream));
    into.push_back({e0, e1});
    return ADPSGD_OK;
}

// The stale gradients of round r: the library's kernels, or the caller's function.
int launch_gradients(adpsgd_t* h, const EventCall& c, int32_t r, float* loss, adpsgd_gradient_fn fn, void* user,
                     std::vector<adpsgd_grad_request_t>& requests) {
    float* slots = static_cast<float*>(h->o.workspace);
    const float gscale = h->o.grad_sum ? 1.0f : 1.0f / static_cast<float>(std::max(c.M, 1));
    for (int64_t g0 = c.r_off[r]; g0 < c.r_off[r + 1]; g0 += c.group) {
        const int32_t cnt = static_cast<int32_t>(std::min<int64_t>(c.group, c.r_off[r + 1] - g0));
        hipEvent_t e0, e1;
        int rc = begin_timing(h, e0, e1);
        if (rc != ADPSGD_OK) return rc;
        int launches = 0;
        if (c.external) {
            requests.resize(static_cast<size_t>(cnt));
            bool any_comp = false;
            for (int32_t t = 0; t < cnt; ++t) {
                const GradOp& g = c.rops[g0 + t];
                const bool comp = c.ext_comp && g.comp_slot >= 0;
                any_comp |= comp;
                requests[t] = adpsgd_grad_request_t{
                    g.worker, 0, g.event,
                    comp ? static_cast<const float*>(h->comp_rows.p) + static_cast<int64_t>(t) * h->o.ldx
                         : h->o.X + static_cast<int64_t>(g.worker) * h->o.ldx,
                    slots + static_cast<int64_t>(g.slot) * h->o.ldx};
            }
            if (any_comp)
                HIP_TRY(h, launch_compensated_rows(h->o.X, h->o.ldx, c.d_rops + g0, cnt, slots, static_cast<float*>(h->comp_rows.p),
                                                   h->stream));
            if (fn(user, cnt, requests.data(), h->stream) != 0) {
                (void)hipStreamSynchronize(h->stream);      // the table upload and the rounds enqueued so far
                return fail(h, ADPSGD_ERR_CALLBACK, "run_events_with: the gradient function failed in round " + std::to_string(r));
            }
            launches = 1;
        } else if (h->o.model == ADPSGD_MODEL_MLP) {
            MlpGradArgs a{h->o.X, h->o.Xbf16, h->o.ldx, h->o.mlp_in, h->o.mlp_hidden, h->o.mlp_out, c.d_rops + g0, cnt, c.M,
                          c.d_batch_r + g0 * c.M, slots, gscale, loss, h->grad_scratch.p, c.factored, c.mlp_comp};
            HIP_TRY(h, launch_mlp_gradient(a, h->stream, &launches));
        } else {
            LinearGradArgs a{h->o.model, h->o.X, h->o.ldx, h->d, c.d_rops + g0, cnt, c.M, c.d_batch, slots, gscale, h->o.lambda,
                             static_cast<float*>(h->grad_scratch.p),
                             reinterpret_cast<float*>(static_cast<char*>(h->grad_scratch.p) + c.off_coef), loss, c.lin_factored};
            if (c.onepass) {
                rc = launch_onepass(h, h->onepass, a);
                if (rc != ADPSGD_OK) return rc;
                launches = 1;
            } else {
                HIP_TRY(h, launch_linear_gradient(a, h->stream, &launches));
            }
        }
        h->stats.grad_launches += launches;
        rc = end_timing(h, e0, e1, h->ev_grad);
        if (rc != ADPSGD_OK) return rc;
    }
    return ADPSGD_OK;
}

// The averaging and update operations of round r: one launch.
int launch_updates(adpsgd_t* h, const EventCall& c, int32_t r) {
    const int64_t nu = c.u_off[r + 1] - c.u_off[r];
    if (nu <= 0) return ADPSGD_OK;
    float* slots = static_cast<float*>(h->o.workspace);
    const PairOp* d_ops = c.d_uops + c.u_off[r];
    hipEvent_t e0, e1;
    int rc = begin_timing(h, e0, e1);
    if (rc != ADPSGD_OK) return rc;
    const UpdateChain* d_chains = c.d_chains + (c.chained() ? c.chain_off[r] : 0);
    const int32_t n_chains = c.chained() ? static_cast<int32_t>(c.chain_off[r + 1] - c.chain_off[r]) : 0;
    if (c.lin_factored) {
        LinearApplyArgs a{h->o.X, h->o.ldx, h->d, d_chains, n_chains, slots, c.d_batch, c.M,
                          h->streaming, h->o.V, h->o.momentum, h->o.weight_decay};
        HIP_TRY(h, launch_linear_apply_chains(a, h->stream));
    } else if (h->o.model == ADPSGD_MODEL_MLP) {
        MlpApplyArgs a{h->o.X, h->o.ldx, h->d, h->o.mlp_in, h->o.mlp_hidden, c.M, d_chains, n_chains, slots, h->o.Xbf16, c.d_batch_u, c.factored,
                       h->o.V, h->o.momentum, h->o.weight_decay};
        HIP_TRY(h, launch_mlp_apply_chains(a, h->stream));
    } else if (c.chained()) {
        const ChainArgs a{h->o.X, h->o.ldx, h->d, d_chains, n_chains, slots, h->streaming, h->o.V, h->o.momentum, h->o.weight_decay};
        HIP_TRY(h, launch_gossip_chains(a, h->stream));
    } else {
        bool has_solo = false;
        for (int64_t t = c.u_off[r]; t < c.u_off[r + 1] && !has_solo; ++t) has_solo = c.uops[t].i == c.uops[t].j;
        FusedArgs a{h->o.X, h->o.ldx, h->d, d_ops, static_cast<int32_t>(nu), slots,
                    h->o.synth_std, h->o.synth_seed,
                    !c.with_grad, h->streaming, has_solo, h->o.V, h->o.momentum, h->o.weight_decay};
        HIP_TRY(h, launch_fused_gossip_apply(a, h->stream));
    }
    ++h->stats.fused_launches;
    return end_timing(h, e0, e1, h->ev_fused);
}

// Synthetic gradients: how the column kernel (kernels_columns.hip) would execute the call.
struct ColumnPlan {
    std::vector<int32_t> rows;          // rows the call touches; the pairs use positions in this list
    std::vector<ColumnPair> pairs;      // the call's operations in event order
    std::vector<int64_t> place;         // position of every operation in the table
    int32_t quads = 0;                  // float4 columns per wavefront, 0: the call goes through the rounds
    int64_t batches = 0;
};

// The operations and the width of the strips.  A strip of q quads takes rows * 16 q bytes of LDS and leaves room for
// 64 / q operations in a batch: narrow strips let more wavefronts share a compute unit, wide ones lose less to batches
// that the dependences leave half empty.  The estimate below is in cycles of a SIMD: a batch costs a wavefront about 1500
// from its operands to its results, and a SIMD with several of them one per 350.  The constant stays at 420: with 350 the
// route is the same for nearly all of 250 set-ups, but some take another width, which loses more often than it
// gains (n = 6, d = 262 923, 254 events in a ring 91 -> 135 us; n = 53,
// d = 1.44 M, 72 events 199 -> 163).  The cost is compared for every width whose strips leave at least eight wavefronts to
// a compute unit.  Below that the
// rounds are the better route: 32 KB strips (n = 500, four quads) leave one wavefront per SIMD to hide that latency.
//
// The rounds are also the better route for a call that touches its rows once or twice: they move 16 (24) bytes per
// parameter and event at 6.4 TB/s, the column kernel 8 (16) per touched row, at 0.3 TB/s per wavefront of a compute unit
// (measured 2.6 with 8 to 8 with 16; half as much again where the state fits the memory-side cache), before and after it
// computes.  Measured, one launch / rounds in us:  n = 160, d = 4 M, 19 events 320 / 209, 80 events 1129 / 822, 240 events
// 1770 / 2467;  n = 320, d = 16 M, 480 events 24 800 / 19 400, 960 events 31 500 / 38 600;  n = 117 with momentum, d = 1 M,
// 29 events 199 / 128, 117 events 461 / 506.  And a launch of its own costs 4.5 us where a round costs 2.5 at least, so a call
// of a single round stays one (one event: 25 / 22), and what cannot gain is turned away before the strips are laid out.
// Of 700 set-ups measured (n 4 ... 320, d 1000 ... 16 M, up to 5 n events, with and without momentum) the line takes none to
// the slower route by more than 5 %, where all to the column kernel lost up to 2.0 times.
void plan_columns(adpsgd_t* h, const EventCall& c, ColumnPlan& out) {
    const adpsgd_schedule_t* s = c.s;
    if (h->d > (1ll << 34)) return;                 // the quad has to fit one word of the generator's counter
    if (c.plan.n_rounds < 2) return;                // one launch as it is
    std::vector<int32_t> local(h->n, -1);
    auto row = [&](int32_t r) {
        if (local[r] < 0) {
            local[r] = static_cast<int32_t>(out.rows.size());
            out.rows.push_back(r);
        }
        return local[r];
    };
    out.pairs.reserve(static_cast<size_t>(c.A + c.n_extra));
    int64_t accesses = 0;                           // rows that the rounds read or write
    for (int64_t k = 0; k < c.A; ++k) {
        const int32_t i = row(s->worker[k]), j = row(s->neighbour[k]);
        accesses += (i == j ? 2 : 4) + (h->o.V ? 2 : 0);
        out.pairs.push_back(ColumnPair{i, j, k});
        if (s->extra_ptr)
            for (int64_t q = s->extra_ptr[k]; q < s->extra_ptr[k + 1]; ++q) {
                const int32_t a = row(s->extra_a[q]), b = row(s->extra_b[q]);
                accesses += 4;
                out.pairs.push_back(ColumnPair{a, b, -1});
            }
    }
    const int64_t n_vec = (h->d + 3) / 4, n_rows = static_cast<int64_t>(out.rows.size());
    constexpr double kIssue = 420.0, kLatency = 1500.0, kSimds = 1024.0, kLdsPerCu = 160.0 * 1024.0;
    constexpr double kCycle = 1.0 / 2.4e9, kRoundRate = 6.4e12, kLaunch = 4.5e-6, kRound = 2.5e-6;
    const double state = static_cast<double>(h->n) * h->o.ldx * 4.0 * (h->o.V ? 2.0 : 1.0), row_bytes = 4.0 * static_cast<double>(h->d);
    const double moved = static_cast<double>(n_rows) * row_bytes * (h->o.V ? 4.0 : 2.0), rate = state > kStreamingThreshold ? 0.3e12 : 0.45e12;
    const double rounds = static_cast<double>(c.plan.n_rounds) * kRound + static_cast<double>(accesses) * row_bytes / kRoundRate;
    if (kLaunch + kLatency * kCycle + moved / (rate * 16.0) >= rounds) return;
    double best = 0.0, waves_per_cu = 16.0;
    std::vector<int64_t> place;
    for (int32_t quads = 4; quads <= 64; quads *= 2) {
        const double strip = static_cast<double>(n_rows) * quads * 16.0 * (h->o.V ? 2.0 : 1.0);
        const double per_cu = std::min(16.0, std::floor(kLdsPerCu / strip));
        if (per_cu < 8.0) break;
        const int64_t batches = pack_columns(out.pairs, static_cast<int32_t>(n_rows), 64 / quads, place);
        const double waves = static_cast<double>((n_vec + quads - 1) / quads) / kSimds;
        const double cost = static_cast<double>(batches) * std::max(kLatency, waves * std::max(kIssue, kLatency / (per_cu / 4.0)));
        if (out.quads == 0 || cost < best) {
            best = cost;
            waves_per_cu = per_cu;
            out.quads = quads;
            out.batches = batches;
            out.place.swap(place);
        }
    }
    if (out.batches > 0x7FFFFFF0 || kLaunch + best * kCycle + moved / (rate * waves_per_cu) >= rounds) out.quads = 0;
}

// All events of the call in one launch of the column kernel.
int run_columns(adpsgd_t* h, const EventCall& c, const ColumnPlan& plan) {
    const int32_t capacity = 64 / plan.quads;
    if ((h->o.flags & ADPSGD_FLAG_VERIFY_PLAN) && !verify_columns(plan.pairs, static_cast<int32_t>(plan.rows.size()), capacity, plan.place, plan.batches))
        return fail(h, ADPSGD_ERR_STATE, "column layout: the order of the events is not kept");
    const size_t n_ops = static_cast<size_t>(plan.batches + 2) * capacity, off_rows = n_ops * sizeof(ColumnOp);
    const size_t total = off_rows + plan.rows.size() * sizeof(int32_t);
    TableSet& T = h->tables[h->next_table];
    h->next_table ^= 1;
    if (T.in_flight) {
        HIP_TRY(h, hipEventSynchronize(T.done));
        T.in_flight = false;
    }
    HIP_TRY(h, T.stage.reserve(total));
    HIP_TRY(h, T.dev.reserve(total));
    char* stage = static_cast<char*>(T.stage.p);
    ColumnOp* ops = reinterpret_cast<ColumnOp*>(stage);
    std::memset(stage, 0, off_rows);
    for (size_t t = 0; t < plan.pairs.size(); ++t) {
        const ColumnPair& pr = plan.pairs[t];
        ColumnOp& op = ops[plan.place[t]];
        const uint32_t pitch = 16u * static_cast<uint32_t>(plan.quads);        // a strip has at most 64 KB: its places fit 16 bits
        op.rows = pitch * static_cast<uint32_t>(pr.i) | (pitch * static_cast<uint32_t>(pr.j)) << 16;
        op.flags = pr.event >= 0 ? kColumnEvent : kColumnAverage;
        if (pr.event < 0) continue;
        op.gamma = c.s->gamma ? c.s->gamma[pr.event] : h->o.gamma;
        column_words(h->events_done + static_cast<uint64_t>(pr.event), h->o.synth_seed, op);
    }
    std::memcpy(stage + off_rows, plan.rows.data(), plan.rows.size() * sizeof(int32_t));
    HIP_TRY(h, hipMemcpyAsync(T.dev.p, T.stage.p, total, hipMemcpyHostToDevice, h->stream));
    const char* dev = static_cast<const char*>(T.dev.p);
    hipEvent_t e0, e1;
    int rc = begin_timing(h, e0, e1);
    if (rc != ADPSGD_OK) return rc;
    ColumnArgs a{h->o.X, h->o.V, h->o.ldx, h->d, reinterpret_cast<const ColumnOp*>(dev), reinterpret_cast<const int32_t*>(dev + off_rows),
                 static_cast<int32_t>(plan.rows.size()), static_cast<int32_t>(plan.batches), plan.quads, h->o.synth_seed, h->o.synth_std,
                 h->o.momentum, h->o.weight_decay, c.n_extra > 0};
    HIP_TRY(h, launch_column_events(a, h->stream));
    rc = end_timing(h, e0, e1, h->ev_fused);
    if (rc != ADPSGD_OK) return rc;
    ++h->stats.fused_launches;
    HIP_TRY(h, hipEventRecord(T.done, h->stream));
    T.in_flight = true;
    return ADPSGD_OK;
}

// All events of the call in one launch of the strip kernel.  Sets `launched` when the launch was made; without memory for the
// records, which take several times that of the rounds' tables, or with a launch that the device refuses, everything is
// as it was, for the rounds.
int run_strips(adpsgd_t* h, EventCall& c, float* loss, bool& launched) {
    launched = false;
    const int32_t M = c.M, n = h->n;
    if (h->exchange_seq > 0xFFFFFFFFu - static_cast<uint64_t>(c.K)) {                  // before the numbers wrap
        HIP_TRY(h, hipMemsetAsync(h->exchange.p, 0, h->exchange.cap, h->stream));
        h->exchange_seq = 0;
    }
    const int64_t slots_fit = strip_lds_slots(h);
    const bool lds_state = slots_fit >= static_cast<int64_t>(h->o.T_max) + 1;
    const int32_t window = strip_window(h->o.T_max, lds_state, slots_fit, h->n_slots);
    StripCall sc{n, h->n_slots, window, c.K, c.A, c.s->worker, c.s->neighbour, c.s->tau, c.s->gamma, h->o.gamma, c.s->extra_ptr, c.s->extra_a, c.s->extra_b,
                 &c.plan, c.carried_slot.empty() ? nullptr : c.carried_slot.data(), h->data.data(), lds_state,
                 h->exchange_seq + 1, strip_blocks(h->d)};
    const int32_t teams = strip_teams(M);
    StripProgram prog;
    try {
        if (!build_strips(sc, 2 * teams, prog, teams)) return ADPSGD_OK;
    } catch (const std::bad_alloc&) {
        return ADPSGD_OK;
    }
    std::string verr;
    if ((h->o.flags & ADPSGD_FLAG_VERIFY_PLAN) && !verify_strips(sc, prog, verr)) return fail(h, ADPSGD_ERR_STATE, verr);
    // slots that cross the ends of the call: (slot of the call, slot of the workspace)
    std::vector<int32_t> carry;
    int32_t n_in = 0, n_out = 0;
    if (lds_state) {
        for (int64_t k = 0; k < c.K; ++k)
            if (!c.carried_slot.empty() && c.carried_slot[k] >= 0) carry.insert(carry.end(), {prog.slot[k], c.carried_slot[k]}), ++n_in;
        for (int64_t k = c.A; k < c.K; ++k)
            if (prog.slot[k] >= 0) carry.insert(carry.end(), {prog.slot[k], c.plan.slot[k]}), ++n_out;
    }
    const size_t bytes_recs = prog.recs.size() * sizeof(StripEntry), off_idx = bytes_recs;
    const size_t off_carry = off_idx + prog.order.size() * M * sizeof(int32_t);
    const size_t off_count = (off_carry + carry.size() * sizeof(int32_t) + 63) & ~size_t(63);
    const size_t off_args = off_count + kStripCounters * sizeof(uint32_t), total = off_args + sizeof(StripArgs);
    TableSet& T = h->tables[h->next_table];
    h->next_table ^= 1;
    if (T.in_flight) {
        HIP_TRY(h, hipEventSynchronize(T.done));
        T.in_flight = false;
    }
    if (T.stage.reserve(total) != hipSuccess || T.dev.reserve(total) != hipSuccess) {
        (void)hipGetLastError();
        return ADPSGD_OK;
    }
    char* stage = static_cast<char*>(T.stage.p);
    std::memset(stage + off_count, 0, kStripCounters * sizeof(uint32_t));
    std::memcpy(stage, prog.recs.data(), bytes_recs);
    int32_t* idx = reinterpret_cast<int32_t*>(stage + off_idx);
    for (size_t q = 0; q < prog.order.size(); ++q)
        std::memcpy(idx + q * M, c.s->batch_idx + prog.order[q] * static_cast<int64_t>(M), static_cast<size_t>(M) * sizeof(int32_t));
    if (!carry.empty()) std::memcpy(stage + off_carry, carry.data(), carry.size() * sizeof(int32_t));
    const char* dev = static_cast<const char*>(T.dev.p);
    StripArgs a{};
    a.X = h->o.X;
    a.V = h->o.V;
    a.ld = h->o.ldx;
    a.d = h->d;
    a.n = n;
    a.model = h->o.model;
    a.M = M;
    a.teams = teams;
    a.recs = reinterpret_cast<const StripEntry*>(dev);
    a.rec_len = prog.rec_len;
    a.iterations = static_cast<int32_t>(prog.iterations);
    a.idx = reinterpret_cast<const int32_t*>(dev + off_idx);
    a.carry = reinterpret_cast<const int32_t*>(dev + off_carry);
    a.n_in = n_in;
    a.n_out = n_out;
    a.slots = static_cast<float*>(h->o.workspace);
    a.n_lds_slots = prog.n_slots;
    a.lds_state = lds_state;
    a.words = static_cast<unsigned long long*>(h->exchange.p);
    a.counters = reinterpret_cast<unsigned int*>(static_cast<char*>(T.dev.p) + off_count);
    // as many blocks on every XCD as form a group (see the kernel); few strips: of these the blocks of one XCD stay.  A block per
    // compute unit for any number of strips took calls of 60 events 1.03 times as long in the mean, up to 1.08 (d = 200: 95 and 89 us)
    a.grid = std::min(h->strip_units, kStripGroups * strip_group_size(h->d));
    a.gscale = h->o.grad_sum ? 1.0f : 1.0f / static_cast<float>(std::max(M, 1));
    a.lambda = h->o.lambda;
    a.momentum = h->o.momentum;
    a.weight_decay = h->o.weight_decay;
    a.loss = loss;
    a.status = static_cast<int*>(h->exchange_status.p);
    a.alone_slots = static_cast<float*>(h->alone_slots.p);
    a.seq0 = h->exchange_seq + 1;
    a.wait_ticks = static_cast<uint64_t>(h->assembly_us) * kClockTicksPerUs;
    a.lose = h->lose_exchange;
    a.self = reinterpret_cast<const StripArgs*>(dev + off_args);
    std::memcpy(stage + off_args, &a, sizeof(a));
    HIP_TRY(h, hipMemcpyAsync(T.dev.p, T.stage.p, total, hipMemcpyHostToDevice, h->stream));
    hipEvent_t e0, e1;
    int rc = begin_timing(h, e0, e1);
    if (rc != ADPSGD_OK) return rc;
    const hipError_t e = launch_strips(a, h->stream);
    if (e != hipSuccess) {                     // nothing has run; the tables may still be on their way
        (void)hipGetLastError();
        if (e0) h->ev_pool.insert(h->ev_pool.end(), {e0, e1});
        HIP_TRY(h, hipEventRecord(T.done, h->stream));
        T.in_flight = true;
        return ADPSGD_OK;
    }
    launched = true;
    if (!lds_state)
        for (int64_t k = c.A; k < c.K; ++k)
            if (prog.slot[k] >= 0) c.plan.slot[k] = prog.slot[k];
    h->exchange_seq += static_cast<uint32_t>(prog.order.size());
    rc = end_timing(h, e0, e1, h->ev_fused);
    if (rc != ADPSGD_OK) return rc;
    ++h->stats.fused_launches;
    HIP_TRY(h, hipEventRecord(T.done, h->stream));
    T.in_flight = true;
    return ADPSGD_OK;
}

// The rounds of the call: tables, then per round the gradients and one update launch.
int run_rounds(adpsgd_t* h, EventCall& c, float* loss, adpsgd_gradient_fn fn, void* user) {
    int rc = upload_tables(h, c);
    if (rc != ADPSGD_OK) return rc;
    std::vector<adpsgd_grad_request_t> requests;
    for (int32_t r = 0; r < c.plan.n_rounds; ++r) {
        rc = launch_gradients(h, c, r, loss, fn, user, requests);
        if (rc != ADPSGD_OK) return rc;
        rc = launch_updates(h, c, r);
        if (rc != ADPSGD_OK) return rc;
    }
    HIP_TRY(h, hipEventRecord(c.T->done, h->stream));
    c.T->in_flight = true;
    return ADPSGD_OK;
}

// The events of one call: plan, then one launch for all of them where the model allows it, or round by round.
int run_events_impl(adpsgd_t* h, const adpsgd_schedule_t* s, float* loss, adpsgd_gradient_fn fn, void* user) {
    if (!s || s->K < 0) return fail(h, ADPSGD_ERR_ARG, "run_events: schedule is NULL or K < 0");
    if (s->K == 0) return ADPSGD_OK;
    EventCall c;
    int rc = check_exchange(h);
    if (rc != ADPSGD_OK) return rc;
    rc = prepare_call(h, s, c);
    if (rc != ADPSGD_OK) return rc;
    ColumnPlan columns;
    if (!c.with_grad && h->route == ADPSGD_ROUTE_AUTO) plan_columns(h, c, columns);
    if (c.strips) rc = run_strips(h, c, loss, c.strips);
    if (rc != ADPSGD_OK) return rc;
    if (!c.strips) rc = columns.quads > 0 ? run_columns(h, c, columns) : run_rounds(h, c, loss, fn, user);
    if (rc != ADPSGD_OK) return rc;
    h->pending_dense = c.strips || !c.lin_factored;
    h->events_done += static_cast<uint64_t>(c.A);
    h->stats.events += c.A;
    h->stats.rounds += c.plan.n_rounds;
    for (int32_t r = 0; r < c.plan.n_rounds; ++r) h->stats.max_round_pairs = std::max<int64_t>(h->stats.max_round_pairs, c.u_off[r + 1] - c.u_off[r]);
    // the events looked ahead to: the next call must start with them; some have their gradient pending already
    h->pending.clear();
    h->pending_batch.clear();
    for (int64_t k = c.A; k < c.K; ++k) h->pending.push_back(PendingEvent{s->worker[k], s->tau[k], c.with_grad ? c.plan.slot[k] : -1});
    if (c.M > 0 && c.A < c.K)
        h->pending_batch.assign(s->batch_idx + c.A * static_cast<int64_t>(c.M), s->batch_idx + c.K * static_cast<int64_t>(c.M));
    return ADPSGD_OK;
}

// No exception leaves the library: the host memory a call's plan takes is the only one there is.
int run_events_guarded(adpsgd_t* h, const adpsgd_schedule_t* s, float* loss, adpsgd_gradient_fn fn, void* user) {
    try {
        return run_events_impl(h, s, loss, fn, user);
    } catch (const std::bad_alloc&) {
        return fail(h, ADPSGD_ERR_ARG, "run_events: out of host memory");
    }
}

}  // namespace

extern "C" int adpsgd_run_events(adpsgd_t* h, const adpsgd_schedule_t* s, float* loss) {
    if (!h) return ADPSGD_ERR_ARG;
    if (h->o.model == ADPSGD_MODEL_EXTERNAL)
        return fail(h, ADPSGD_ERR_STATE, "run_events: caller-supplied gradients need adpsgd_run_events_with");
    return run_events_guarded(h, s, loss, nullptr, nullptr);
}

extern "C" int adpsgd_run_events_with(adpsgd_t* h, const adpsgd_schedule_t* s, adpsgd_gradient_fn fn, void* user) {
    if (!h) return ADPSGD_ERR_ARG;
    if (h->o.model != ADPSGD_MODEL_EXTERNAL)
        return fail(h, ADPSGD_ERR_STATE, "run_events_with: the handle was not created with ADPSGD_MODEL_EXTERNAL");
    if (!fn) return fail(h, ADPSGD_ERR_ARG, "run_events_with: fn is NULL");
    return run_events_guarded(h, s, nullptr, fn, user);
}

extern "C" int adpsgd_set_wait_limits(adpsgd_t* h, int64_t assembly_us, int32_t lose_exchange) {
    if (!h) return ADPSGD_ERR_ARG;
    if (assembly_us < 0 || assembly_us > 0x7FFFFFFF) return fail(h, ADPSGD_ERR_ARG, "set_wait_limits: assembly_us outside [0, 2^31)");
    h->assembly_us = assembly_us;
    h->lose_exchange = lose_exchange != 0;
    return ADPSGD_OK;
}

extern "C" int adpsgd_set_route(adpsgd_t* h, int32_t route) {
    if (!h) return ADPSGD_ERR_ARG;
    if (route != ADPSGD_ROUTE_AUTO && route != ADPSGD_ROUTE_ROUNDS) return fail(h, ADPSGD_ERR_ARG, "set_route: unknown route");
    h->route = route;
    return ADPSGD_OK;
}

extern "C" int adpsgd_get_late_blocks(adpsgd_t* h, int64_t* out) {
    if (!h) return ADPSGD_ERR_ARG;
    if (!out) return fail(h, ADPSGD_ERR_ARG, "get_late_blocks: out is NULL");
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    unsigned long long count = 0;
    if (h->onepass.ok())
        HIP_TRY(h, hipMemcpy(&count, static_cast<char*>(h->onepass_words.p) + h->onepass_bytes, sizeof(count), hipMemcpyDeviceToHost));
    *out = static_cast<int64_t>(count);
    return ADPSGD_OK;
}

extern "C" int adpsgd_synchronize(adpsgd_t* h) {
    if (!h) return ADPSGD_ERR_ARG;
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    return check_exchange(h);
}

extern "C" int adpsgd_get_stats(adpsgd_t* h, adpsgd_stats_t* out) {
    if (!h) return ADPSGD_ERR_ARG;
    if (!out) return fail(h, ADPSGD_ERR_ARG, "get_stats: out is NULL");
    const int rc = drain_profile(h);
    if (rc != ADPSGD_OK) return rc;
    *out = h->stats;
    return ADPSGD_OK;
}

extern "C" int adpsgd_get_event_count(adpsgd_t* h, uint64_t* out) {
    if (!h) return ADPSGD_ERR_ARG;
    if (!out) return fail(h, ADPSGD_ERR_ARG, "get_event_count: out is NULL");
    *out = h->events_done;
    return ADPSGD_OK;
}

extern "C" int adpsgd_set_event_count(adpsgd_t* h, uint64_t events) {
    if (!h) return ADPSGD_ERR_ARG;
    h->events_done = events;
    h->pending.clear();
    h->pending_batch.clear();
    return ADPSGD_OK;
}

extern "C" int adpsgd_synth_gradient(uint64_t seed, uint64_t k, float std, int64_t d, float* out_device, void* stream) {
    if (!out_device || d < 0) return ADPSGD_ERR_ARG;
    const hipError_t e = launch_synth_gradient(seed, k, std, d, out_device, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? ADPSGD_OK : ADPSGD_ERR_HIP;
}
