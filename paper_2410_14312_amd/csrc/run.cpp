// One-GPU pipeline emulator: K stages on K HIP streams, tasks issued in nF1B order, cross-stage
// dependencies as events (sections "Work Scheduling" and "Overlapping of Computation and
// Communication": what would be a message between workers is an event between streams here).
//
// Each stage has its own host thread that issues that stage's tasks in schedule order on the stage's
// stream, like a worker process would; a thread that needs another stage's result first waits until
// the producing thread has recorded the event, then makes its stream wait for it.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <shared_mutex>
#include <thread>
#include <vector>

#include "profile.h"
#include "schedule.h"
#include "stage.h"

using namespace tmps;

namespace {

// The events that stand for messages between workers are kept by the stage that records them (tmps_stage::events,
// destroyed with the stage): a second run on the same stages creates none.
int grow_events(tmps_stage* st, size_t n) {
    while (st->events.size() < n) {
        hipEvent_t e;
        TMPS_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        st->events.push_back(e);
    }
    return TMPS_OK;
}

// What a worker issues in one go: a backward pass with its update, or the forward passes of `count` consecutive
// micro-batches of one mini-batch that stand next to each other in the worker's order and read the same weights.
// Their rows are consecutive in the stash, so they are one pass over `count` times the rows: the layers' kernels then
// have the rows to fill the device and are launched once.  (The GEMMs of a GPT-2 micro-batch, 1024 rows, reach 180 to 400
// TFLOP/s, those of 8192 rows 520 to 750.  Time per mini-batch pass by pass and merged, in runs of 20: GPT-2 13.6 and 11.8 ms on
// four streams, 16.0 and 12.3 on one; ResNet-50 8.3 and 7.4, 10.1 and 7.5; VGG-16 1.30 and 1.13, 1.59 and 1.15; the tiny fp32
// MLP on one stream 76 and 46 us.  The backward passes that fall between a mini-batch's micro-batches cut its forward into
// 1.7 passes of GPT-2 on average.)
// No dependency is added that could close a circle: whatever follows from one member and precedes a later one would
// have to pass through a backward pass of this worker between the two.
struct Node {
    int stage, kind, b0, j0, count;
    int32_t t, stage_version, net_version;   // of the first task
    size_t first_task;                       // indices into the task list: first_task, and the members' own in `tasks`
    std::vector<size_t> tasks;
};

struct RunCtx {
    bool vsync = false;              // forward passes read the weight version they are tagged with
    bool one_f1b = false;            // the comparison system: a backward pass per batch, on the weights of its forward pass
    bool one_queue = false;          // all stages issue on one stream: its order stands for the events
    std::vector<tmps_stage*> updates;   // then: stages whose update is still to be issued, with those of other stages or before their next pass
    std::vector<long> base_version;  // every stage's version when the run started
    tmps_stage** stages;
    int K, N, M, mb, n_minibatches;
    const void* inputs;
    const int32_t* labels;
    void** streams;
    float* losses_out;
    int32_t* log;
    const Task* tasks;
    size_t total_micro, n_fwd_ev;
    std::vector<int> groups;
    std::vector<std::vector<Node>> nodes;     // per stage, in the worker's order
    std::vector<size_t> last_of;              // [stage * total_micro + q]: the last micro-batch of the pass that forwards q
    std::vector<std::atomic<unsigned char>> recorded;
    std::atomic<int> err{TMPS_OK};
    char err_text[512];
    std::atomic_flag err_lock = ATOMIC_FLAG_INIT;

    size_t fwd_ev(int s, size_t q) const { return (size_t)s * total_micro + q; }
    size_t bwd_ev(int s, int b0) const { return n_fwd_ev + (size_t)s * n_minibatches + b0; }
    // the event behind an index: stage s keeps its forward events first, then its backward events
    hipEvent_t event(size_t e) const {
        if (e < n_fwd_ev) return stages[e / total_micro]->events[e % total_micro];
        const size_t r = e - n_fwd_ev;
        return stages[r / n_minibatches]->events[total_micro + r % n_minibatches];
    }

    // Block until the producer thread has recorded event e (or a thread failed), then make stream s wait for it.
    int wait_for(size_t e, hipStream_t s) {
        if (one_queue) return TMPS_OK;
        while (!recorded[e].load(std::memory_order_acquire)) {
            if (err.load(std::memory_order_relaxed) != TMPS_OK) return TMPS_EINVAL;
            std::this_thread::yield();
        }
        std::shared_lock<std::shared_mutex> no_capture(capture_lock());   // (see capture_lock)
        TMPS_HIP(hipStreamWaitEvent(s, event(e), 0));
        return TMPS_OK;
    }
    int record(size_t e, hipStream_t s) {
        if (!one_queue) TMPS_HIP(hipEventRecord(event(e), s));
        recorded[e].store(1, std::memory_order_release);
        return TMPS_OK;
    }
    // The events that node n waits for.
    template <class F> void for_each_dependency(const Node& n, F&& f) const {
        if (n.kind == kFwd) {
            if (n.stage == 0) return;
            const size_t q0 = (size_t)n.b0 * N + n.j0;
            for (size_t q = q0; q < q0 + n.count;) {
                const size_t last = last_of[(size_t)(n.stage - 1) * total_micro + q];
                f(fwd_ev(n.stage - 1, last));
                q = last + 1;
            }
        } else {
            if (n.stage < K - 1) f(bwd_ev(n.stage + 1, n.b0));
            // the worker below must have consumed what the boundary-gradient buffer held two mini-batches ago
            if (n.stage > 0 && n.b0 >= 2) f(bwd_ev(n.stage - 1, n.b0 - 2));
        }
    }
    void set_error(int rc) {
        while (err_lock.test_and_set(std::memory_order_acquire)) {}
        if (err.load() == TMPS_OK) {
            strncpy(err_text, tmps_last_error(), sizeof(err_text) - 1);
            err_text[sizeof(err_text) - 1] = 0;
            err.store(rc);
        }
        err_lock.clear(std::memory_order_release);
    }
};

int issue_updates(RunCtx& c) {
    if (c.updates.empty()) return TMPS_OK;
    const int rc = update_all(c.updates.data(), (int)c.updates.size(), c.streams[0]);
    c.updates.clear();
    return rc;
}

// Issue one node on its stage's stream.
int issue(RunCtx& c, const Node& n) {
    tmps_stage* st = c.stages[n.stage];
    hipStream_t s = (hipStream_t)(c.one_queue ? c.streams[0] : c.streams[n.stage]);
    if (std::find(c.updates.begin(), c.updates.end(), st) != c.updates.end()) {
        const int rc = issue_updates(c);
        if (rc != TMPS_OK) return rc;
    }
    const int b0 = n.b0, N = c.N, K = c.K;
    if (c.log) {
        const int32_t live = (int32_t)(st->version - c.base_version[n.stage]);
        for (size_t ti : n.tasks) {
            const Task& k = c.tasks[ti];
            int32_t* o = c.log + 7 * ti;
            o[0] = k.t; o[1] = k.stage; o[2] = k.kind; o[3] = k.b; o[4] = k.j;
            if (c.one_f1b) {   // version the task reads (a backward pass: the one its forward pass read), version the worker is at
                o[5] = k.kind == kFwd ? live : k.stage_version;
                o[6] = live;
            } else {
                o[5] = live;
                o[6] = k.net_version;
            }
        }
    }
    int rc = TMPS_OK;
    c.for_each_dependency(n, [&](size_t e) {
        if (rc == TMPS_OK) rc = c.wait_for(e, s);
    });
    if (rc != TMPS_OK) return rc;
    const int group = b0 % c.groups[n.stage];
    if (n.kind == kFwd) {
        const size_t row = (size_t)b0 * c.M + (size_t)n.j0 * c.mb;
        const int slot = group * N + n.j0;
        const void* x = n.stage == 0 ? (const void*)((const char*)c.inputs + row * st->in_elems * st->in_esize)
                                     : tmps_stage_output_ptr(c.stages[n.stage - 1], (b0 % c.groups[n.stage - 1]) * N + n.j0);
        const int32_t* lab = st->cfg.is_last ? c.labels + row * st->label_rps : nullptr;
        const long version = c.vsync ? c.base_version[n.stage] + n.net_version : st->version;
        // The pass over a mini-batch's last micro-batches also forms its loss.  (Not on a stage that replays graphs: the address
        // of the loss is another one for every mini-batch.)
        const bool ends = st->cfg.is_last && n.j0 + n.count == N && c.losses_out;
        float* const loss = ends && !st->use_graphs ? c.losses_out + b0 : nullptr;
        if ((rc = forward_run_at(st, version, slot, n.count, x, nullptr, lab, loss, s, loss ? n.j0 : 0)) != TMPS_OK) return rc;
        if (n.stage < K - 1 && (rc = c.record(c.fwd_ev(n.stage, (size_t)b0 * N + n.j0 + n.count - 1), s)) != TMPS_OK) return rc;
        if (ends && !loss) {
            ProfileScope scope(kcReduce, s);
            const int rows = c.M * st->label_rps;
            TMPS_HIP(reduce_scaled_sum(stage_row_loss(st, group * N), rows, 1.0f / (float)rows, c.losses_out + b0, s));
        }
    } else {
        const void* dy = n.stage < K - 1 ? stage_dxout(c.stages[n.stage + 1], b0 & 1) : nullptr;
        void* dx = n.stage > 0 ? stage_dxout(st, b0 & 1) : nullptr;
        int slots[64];
        for (int j = 0; j < N; ++j) slots[j] = group * N + j;
        // does worker a pass a gradient down through the ReLU that ends the worker below it?
        auto masked_above = [&](int below) {
            return below >= 0 && below < K - 1 && c.stages[below]->layers.back().relu && can_mask_dx(*c.stages[below + 1]);
        };
        const int flags = (masked_above(n.stage - 1) ? kMaskDx : 0) | (masked_above(n.stage) ? kDyMasked : 0);
        if (c.one_f1b)   // horizontal weight stashing: differentiate at the weights the forward pass read
            rc = backward_between_at(st, c.base_version[n.stage] + n.stage_version, slots, N, dy, dx, s, flags);
        else
            rc = backward_between(st, slots, N, dy, dx, s, flags);
        if (rc != TMPS_OK) return rc;
        if ((rc = c.record(c.bwd_ev(n.stage, b0), s)) != TMPS_OK) return rc;
        if (c.one_queue) c.updates.push_back(st);
        else if ((rc = tmps_update(st, s)) != TMPS_OK) return rc;
    }
    return TMPS_OK;
}

// Nodes of every stage in the worker's order, and which node forwards which micro-batch.
void build_nodes(RunCtx& c, const std::vector<Task>& tasks) {
    c.nodes.assign(c.K, {});
    c.last_of.assign((size_t)c.K * c.total_micro, 0);
    for (size_t i = 0; i < tasks.size(); ++i) {
        const Task& k = tasks[i];
        std::vector<Node>& mine = c.nodes[k.stage];
        const int j = k.j < 0 ? 0 : k.j;   // (the comparison system has no micro-batches: N = 1)
        if (k.kind == kFwd && !mine.empty()) {
            Node& p = mine.back();
            if (p.kind == kFwd && p.b0 == k.b - 1 && p.j0 + p.count == j && p.count < c.stages[k.stage]->max_run &&
                (!c.vsync || p.net_version == k.net_version)) {
                ++p.count;
                p.tasks.push_back(i);
                continue;
            }
        }
        mine.push_back(Node{k.stage, k.kind, k.b - 1, j, 1, k.t, k.stage_version, k.net_version, i, {i}});
    }
    for (int s = 0; s < c.K; ++s)
        for (const Node& n : c.nodes[s])
            if (n.kind == kFwd)
                for (int j = 0; j < n.count; ++j)
                    c.last_of[(size_t)s * c.total_micro + (size_t)n.b0 * c.N + n.j0 + j] = (size_t)n.b0 * c.N + n.j0 + n.count - 1;
}

// Device time of a pass over `rows` samples, roughly: 5 us for every launch it is expected to make (a contraction one
// forward and a split now and then, two to three backward; other layers one and two), its operations at the rates that
// mid-sized contractions reach, and the update at 4 TB/s.  Whole runs take less than their estimate: two mini-batches on one
// stream 96 us of 166 (tiny fp32 MLP), 235 of 408 (bf16 MLP), 1.90 ms of 3.3 (VGG-16), 11.8 of 17.9 (ResNet-50), 21.7 of 47.8 (GPT-2).
double pass_us(const tmps_stage& st, int rows, bool backward) {
    double us = 0.0;
    for (const LayerRT& L : st.layers) {
        const int32_t* d = L.d.dims;
        double flops = 0.0;
        bool contraction = true;
        if (L.d.kind == TMPS_LINEAR) flops = 2.0 * L.rps * d[0] * d[1];
        else if (L.d.kind == TMPS_CONV2D) flops = 2.0 * L.out_elems * d[4] * d[5] * d[2];
        else contraction = false;
        us += (contraction ? (backward ? 12.5 : 6.5) : (backward ? 7.5 : 5.0)) + flops * rows * (backward ? 2.0 : 1.0) / (st.asz == 2 ? 250e6 : 60e6);
    }
    return backward ? us + 5.0 + (double)st.P * 22.0 / 4e6 : us;
}

// Whether the whole run is quicker on ONE stream, issued from one host thread.  On K streams it pays for issue threads
// (about 100 us a run) and for every hand-over from stream to stream (about 25 us in a chain of short passes) and gains
// what the workers' passes overlap: nothing within a single mini-batch, some 5 % of the work where a mini-batch's
// micro-batches are forwarded together, some 20 % where mini-batches are short against the pipeline (N <= 2) and in 1F1B
// order.  Measured on K streams and on one: two mini-batches of the tiny fp32 MLP 222 and 96 us, the bf16 MLP 464 and 235,
// the tiny fp32 transformer 455 and 303, VGG-16 1.91 and 1.90 ms, ResNet-50 11.8 and 11.8, GPT-2 21.1 and 21.7; twenty of VGG-16 19.5 and
// 19.6 ms, ResNet-50 116 and 120, GPT-2 208 and 221; eight batches in 1F1B order, VGG-16 5.1 and 6.0 ms, ResNet-50 11.9 and 17.3, GPT-2 21.7 and 26.5.
// Not in the estimate: a hand-over costs a short pass some 8 us of every run, however long; twenty mini-batches of the bf16 MLP (3.5 and 2.6 ms)
// or the tiny transformer (4.1 and 3.4) are left on K streams.  One stream wherever less than 0.35 of the estimate is operations mends these and
// loses 3 % or more on others (three mini-batches of an fp32 residual network of 9 blocks on 30 images of 99 x 99).
bool serial_is_quicker(const RunCtx& c) {
    double total = 0.0;
    size_t nodes = 0;
    for (int s = 0; s < c.K; ++s)
        for (const Node& n : c.nodes[s]) {
            total += pass_us(*c.stages[s], n.kind == kFwd ? n.count * c.mb : c.M, n.kind != kFwd);
            ++nodes;
        }
    const double overlapped = c.n_minibatches == 1 ? 1.0 : (c.one_f1b || c.N <= 2) ? 0.78 : 0.95;
    const double chain = (double)nodes / c.K * (total / nodes + 25.0);
    return total <= 100.0 + (overlapped * total > chain ? overlapped * total : chain);
}

// From one host thread: every node after the nodes it depends on, otherwise in the order of the schedule's time-points.
int issue_all(RunCtx& c) {
    std::vector<size_t> head(c.K, 0);
    for (;;) {
        const Node* best = nullptr;
        for (int s = 0; s < c.K; ++s) {
            if (head[s] == c.nodes[s].size()) continue;
            const Node& n = c.nodes[s][head[s]];
            bool ready = true;
            c.for_each_dependency(n, [&](size_t e) { ready = ready && c.recorded[e].load(std::memory_order_relaxed); });
            if (ready && (!best || n.first_task < best->first_task)) best = &n;
        }
        if (!best) {
            // nothing is ready: everything has been issued, or the order asks for a pass that never comes
            const int rc = issue_updates(c);
            for (int s = 0; s < c.K; ++s)
                if (head[s] < c.nodes[s].size())
                    return fail(TMPS_EINVAL, "the schedule's order cannot be satisfied: stage %d is left with %zu of %zu passes", s,
                                c.nodes[s].size() - head[s], c.nodes[s].size());
            return rc;
        }
        const int rc = issue(c, *best);
        if (rc != TMPS_OK) {
            (void)issue_updates(c);   // (of the passes before)
            return rc;
        }
        ++head[best->stage];
    }
}

}  // namespace

enum { kModeInPlace = 0, kModeVsync = 1, kMode1F1B = 2 };

static int schedule_run(tmps_stage** stages, int K, int N, int n_minibatches, const void* inputs, const int32_t* labels,
                        void** hip_streams, float* losses_out, int32_t* version_log_out, int mode) {
    const bool vsync = mode == kModeVsync, one_f1b = mode == kMode1F1B;
    if (!stages || !hip_streams || !inputs || !labels) return fail(TMPS_EINVAL, "null argument");
    if (K < 1 || N < 1 || n_minibatches < 1) return fail(TMPS_EINVAL, "K, N and n_minibatches must be positive");
    const int mb = stages[0] ? stages[0]->cfg.micro_batch : 0;
    for (int s = 0; s < K; ++s) {
        tmps_stage* st = stages[s];
        if (!st) return fail(TMPS_EINVAL, "stage %d is null", s);
        if (st->cfg.n_micro != N || st->cfg.micro_batch != mb)
            return fail(TMPS_EMICRO, "stage %d was created for %d micro-batches of %d, the run uses %d of %d", s,
                        st->cfg.n_micro, st->cfg.micro_batch, N, mb);
        if ((st->cfg.is_last != 0) != (s == K - 1)) return fail(TMPS_ESHAPE, "only the last stage may end in the loss");
        if (s > 0 && stages[s - 1]->out_elems != st->in_elems)
            return fail(TMPS_ESHAPE, "stage %d output (%lld) does not match stage %d input (%lld)", s - 1,
                        (long long)stages[s - 1]->out_elems, s, (long long)st->in_elems);
        if (s > 0 && stages[s - 1]->cfg.dtype != st->cfg.dtype) return fail(TMPS_ESHAPE, "stages differ in dtype");
        int need = one_f1b ? K - s : stash_groups(K, N, s);
        if (st->cfg.max_stash / N < need)
            return fail(TMPS_ESTASH, "stage %d can stash %d mini-batches, the schedule needs %d", s, st->cfg.max_stash / N, need);
        for (char u : st->slot_used)
            if (u) return fail(TMPS_ESLOT, "stage %d has a stash slot in use", s);
        if (vsync && st->shadow_n < shadow_versions(K, N, s))
            return fail(TMPS_ESTASH, "stage %d keeps %d older weight versions, vertical weight stashing needs %d", s,
                        st->shadow_n, shadow_versions(K, N, s));
        if (one_f1b && st->shadow_n < K - s - 1)
            return fail(TMPS_ESTASH, "stage %d keeps %d older weight versions, horizontal weight stashing needs %d", s,
                        st->shadow_n, K - s - 1);
    }
    const std::vector<Task> tasks = one_f1b ? plan_1f1b(K, n_minibatches) : plan_nf1b(K, N, n_minibatches);

    RunCtx c;
    c.stages = stages; c.K = K; c.N = N; c.mb = mb; c.M = mb * N; c.n_minibatches = n_minibatches;
    c.inputs = inputs; c.labels = labels; c.streams = hip_streams; c.losses_out = losses_out;
    c.log = version_log_out;
    c.vsync = vsync;
    c.one_f1b = one_f1b;
    for (int s = 0; s < K; ++s) c.base_version.push_back(stages[s]->version);
    c.total_micro = (size_t)n_minibatches * N;
    c.n_fwd_ev = (size_t)(K - 1) * c.total_micro;
    c.groups.resize(K);
    for (int s = 0; s < K; ++s) c.groups[s] = stages[s]->cfg.max_stash / N;
    const size_t n_events = c.n_fwd_ev + (size_t)K * n_minibatches;
    c.recorded = std::vector<std::atomic<unsigned char>>(n_events);
    for (auto& f : c.recorded) f.store(0, std::memory_order_relaxed);

    c.tasks = tasks.data();
    build_nodes(c, tasks);
    c.one_queue = true;
    for (int s = 1; s < K; ++s) c.one_queue = c.one_queue && hip_streams[s] == hip_streams[0];
    const char* env = getenv("TMPS_ISSUE_THREADS");   // (0: issue from the calling thread; 1: K streams, a thread for each)
    const bool ask_streams = env && env[0] == '1';
    if (!c.one_queue && !ask_streams && serial_is_quicker(c)) {
        // (what the caller has pending on the other streams comes first)
        for (int s = 1; s < K; ++s) {
            if (hip_streams[s] == hip_streams[0] || hipStreamQuery((hipStream_t)hip_streams[s]) == hipSuccess) continue;
            (void)hipGetLastError();   // ("not ready" is an answer, not an error)
            const int rc = grow_events(stages[s], 1);
            if (rc != TMPS_OK) return rc;
            TMPS_HIP(hipEventRecord(stages[s]->events[0], (hipStream_t)hip_streams[s]));
            TMPS_HIP(hipStreamWaitEvent((hipStream_t)hip_streams[0], stages[s]->events[0], 0));
        }
        c.one_queue = true;
    }
    if (!c.one_queue)
        for (int s = 0; s < K; ++s) {
            const int rc = grow_events(stages[s], c.total_micro + (size_t)n_minibatches);
            if (rc != TMPS_OK) return rc;
        }

    const bool threaded = K > 1 && !(env && env[0] == '0') && !c.one_queue;
    const bool report = getenv("TMPS_REPORT_ISSUE_TIME") != nullptr;
    const auto t0 = std::chrono::steady_clock::now();
    if (threaded) {
        int dev = 0;
        TMPS_HIP(hipGetDevice(&dev));
        std::vector<std::thread> workers;
        for (int s = 0; s < K; ++s)
            workers.emplace_back([&, s]() {
                if (hipSetDevice(dev) != hipSuccess) {
                    fail(TMPS_EHIP, "hipSetDevice failed in an issue thread");
                    c.set_error(TMPS_EHIP);
                    return;
                }
                for (const Node& n : c.nodes[s]) {
                    if (c.err.load(std::memory_order_relaxed) != TMPS_OK) return;
                    int r = issue(c, n);
                    if (r != TMPS_OK) {
                        if (c.err.load() == TMPS_OK) c.set_error(r);
                        return;
                    }
                }
            });
        for (std::thread& t : workers) t.join();
    } else {
        const int r = issue_all(c);
        if (r != TMPS_OK) c.set_error(r);
    }
    const auto t1 = std::chrono::steady_clock::now();
    for (int s = 0; s < (c.one_queue ? 1 : K); ++s) TMPS_HIP(hipStreamSynchronize((hipStream_t)hip_streams[s]));
    if (c.err.load() != TMPS_OK) {
        // the mini-batches in flight are lost: free their stash slots, so that the stages can run again
        for (int s = 0; s < K; ++s) {
            std::fill(stages[s]->slot_used.begin(), stages[s]->slot_used.end(), 0);
            std::fill(stages[s]->slot_x.begin(), stages[s]->slot_x.end(), nullptr);
        }
        return fail(c.err.load(), "%s", c.err_text);
    }
    if (report) {
        const auto t2 = std::chrono::steady_clock::now();
        fprintf(stderr, "tmps_schedule_run: %d mini-batches, host issue %.3f ms, until idle %.3f ms\n", n_minibatches,
                std::chrono::duration<double, std::milli>(t1 - t0).count(),
                std::chrono::duration<double, std::milli>(t2 - t0).count());
    }
    return TMPS_OK;
}

extern "C" int tmps_schedule_run(tmps_stage** stages, int K, int N, int n_minibatches, const void* inputs,
                                 const int32_t* labels, void** hip_streams, float* losses_out,
                                 int32_t* version_log_out) {
    return schedule_run(stages, K, N, n_minibatches, inputs, labels, hip_streams, losses_out, version_log_out, kModeInPlace);
}

extern "C" int tmps_schedule_run_vsync(tmps_stage** stages, int K, int N, int n_minibatches, const void* inputs,
                                       const int32_t* labels, void** hip_streams, float* losses_out,
                                       int32_t* version_log_out) {
    return schedule_run(stages, K, N, n_minibatches, inputs, labels, hip_streams, losses_out, version_log_out, kModeVsync);
}

extern "C" int tmps_schedule_run_1f1b(tmps_stage** stages, int K, int n_batches, const void* inputs, const int32_t* labels,
                                      void** hip_streams, float* losses_out, int32_t* version_log_out) {
    return schedule_run(stages, K, 1, n_batches, inputs, labels, hip_streams, losses_out, version_log_out, kMode1F1B);
}

extern "C" int tmps_streams_create(void** out, int n) {
    if (!out || n < 1) return fail(TMPS_EINVAL, "tmps_streams_create needs an array and a positive count");
    for (int i = 0; i < n; ++i) out[i] = nullptr;
    for (int i = 0; i < n; ++i) {
        hipStream_t s = nullptr;
        hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
        if (e != hipSuccess) {
            for (int j = 0; j < i; ++j) (void)hipStreamDestroy((hipStream_t)out[j]);
            return fail(TMPS_EHIP, "hipStreamCreateWithFlags failed: %s", hipGetErrorString(e));
        }
        out[i] = s;
    }
    return TMPS_OK;
}

extern "C" int tmps_streams_destroy(void** streams, int n) {
    if (!streams) return fail(TMPS_EINVAL, "streams is null");
    for (int i = 0; i < n; ++i)
        if (streams[i]) {
            TMPS_HIP(hipStreamDestroy((hipStream_t)streams[i]));
            streams[i] = nullptr;
        }
    return TMPS_OK;
}
