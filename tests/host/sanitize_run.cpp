// Host-only driver of the pipeline runner: which streams and events a run uses, the version log of runs on K streams with a
// host thread each under the three weight policies, failing passes, and forward passes over as many micro-batches as fit
// the convolutions' index range.
#include "kernel_stubs.h"
#include "run_stages.h"
#include "runtime_stubs.h"

static const int R = TMPS_FLAG_RELU;
static std::vector<std::vector<tmps_layer_desc>> mlp(int K, int width) {
    std::vector<std::vector<tmps_layer_desc>> s;
    for (int k = 0; k < K; ++k) s.push_back({L(TMPS_LINEAR, {width, width, 0, 1}, R)});
    s.back().push_back(L(TMPS_LINEAR, {width, 10, 0, 1}));
    s.back().push_back(L(TMPS_SOFTMAX_CE, {10, 1}));
    return s;
}

// A run so short that it is issued on the first stream alone.
static void short_run() {
    Pipe p(mlp(4, 16), TMPS_F32, 2, 4, 6, false, false);
    auto run = [&](int n) {
        return tmps_schedule_run(p.stages.data(), 4, 4, n, p.input.data(), p.labels.data(), p.streams.data(), p.losses.data(), nullptr);
    };
    stub_counters = StubCounters();
    expect(run(6) == TMPS_OK, "short run");
    expect(stub_counters.events == 0 && stub_counters.records == 0 && stub_counters.waits == 0, "one stream needs no events");
    stub_counters.busy_streams = true;
    expect(run(6) == TMPS_OK, "short run behind pending work");
    expect(stub_counters.events == 3 && stub_counters.records == 3 && stub_counters.waits == 3 && stub_counters.waits_without_record == 0,
           "the first stream waits once for each of the others");
    expect(run(2) == TMPS_OK && stub_counters.events == 3 && stub_counters.waits == 6, "events are kept");
}

enum { kInPlace, kVsync, k1F1B };
static int run(Pipe& p, int mode, int n, int32_t* log) {
    const int K = (int)p.stages.size();
    if (mode == k1F1B) return tmps_schedule_run_1f1b(p.stages.data(), K, n, p.input.data(), p.labels.data(), p.streams.data(), p.losses.data(), log);
    return (mode == kVsync ? tmps_schedule_run_vsync : tmps_schedule_run)(p.stages.data(), K, p.N, n, p.input.data(), p.labels.data(),
                                                                          p.streams.data(), p.losses.data(), log);
}

// Runs asked for on K streams (TMPS_ISSUE_THREADS=1), and the same issued by one thread: the planned log, no wait for an event
// that nobody records, events created by the first run that uses them.
static void k_streams() {
    for (int mode : {kInPlace, kVsync, k1F1B})
        for (int K : {2, 3, 5})
            for (int N : {1, 2, 4})
                for (const char* threads : {"1", "0", ""}) {
                    if (mode == k1F1B && N > 1) continue;
                    const int n = 7;
                    Pipe p(mlp(K, 16), TMPS_BF16_F32MASTER, 2, N, n, mode == kVsync, mode == k1F1B);
                    const int tasks = mode == k1F1B ? tmps_schedule_plan_1f1b(K, n, nullptr, 0) : tmps_schedule_plan(K, N, n, nullptr, 0);
                    std::vector<int32_t> plan(7 * tasks), log(7 * tasks);
                    if (mode == k1F1B) tmps_schedule_plan_1f1b(K, n, plan.data(), tasks);
                    else tmps_schedule_plan(K, N, n, plan.data(), tasks);
                    setenv("TMPS_ISSUE_THREADS", threads, 1);
                    for (int again = 0; again < 2; ++again) {
                        stub_counters = StubCounters();
                        expect(run(p, mode, n, log.data()) == TMPS_OK, "run");
                        expect(log == plan, "version log");
                        expect(stub_counters.waits_without_record == 0, "a wait for an event that was not recorded");
                        expect(threads[0] != '1' || stub_counters.waits > 0, "K streams were asked for");
                        expect((stub_counters.events > 0) == (stub_counters.waits > 0 && again == 0), "events are kept between runs");
                    }
                    for (tmps_stage* s : p.stages) expect(tmps_stage_version(s) == 2 * n, "updates");
                }
    unsetenv("TMPS_ISSUE_THREADS");
}

// A pass that fails midway: the run ends, reports it, and leaves the stages able to run again.
static void failing_pass() {
    for (const char* threads : {"1", "0"}) {
        Pipe p(mlp(4, 16), TMPS_F32, 2, 2, 6, false, false);
        setenv("TMPS_ISSUE_THREADS", threads, 1);
        for (int good : {0, 1, 3}) {
            kernel_stubs.losses_until_failure = good;
            expect(run(p, kInPlace, 6, nullptr) == TMPS_EHIP, "the failure is reported");
            kernel_stubs.losses_until_failure = -1;
            expect(run(p, kInPlace, 6, nullptr) == TMPS_OK, "the stages run again");
        }
    }
    unsetenv("TMPS_ISSUE_THREADS");
}

// Maps of 5.76 million positions: two micro-batches of one sample fit the convolutions' 24-bit positions, three do not.
static void long_maps() {
    const int h = 2400, n = 2, N = 4;
    Pipe p({{L(TMPS_CONV2D, {h, h, 1, 1, 1, 1, 1, 0})}, {L(TMPS_AVGPOOL, {h, h, 1}), L(TMPS_LINEAR, {1, 10, 0, 1}), L(TMPS_SOFTMAX_CE, {10, 1})}},
           TMPS_BF16_F32MASTER, 1, N, n, false, false);
    for (const char* threads : {"1", "0"}) {
        setenv("TMPS_ISSUE_THREADS", threads, 1);
        stub_counters = StubCounters();
        kernel_stubs.conv_samples.clear();
        const int tasks = tmps_schedule_plan(2, N, n, nullptr, 0);
        std::vector<int32_t> plan(7 * tasks), log(7 * tasks);
        tmps_schedule_plan(2, N, n, plan.data(), tasks);
        expect(run(p, kInPlace, n, log.data()) == TMPS_OK && log == plan, "run over long maps");
        int samples = 0, most = 0;
        for (int b : kernel_stubs.conv_samples) {
            samples += b;
            most = b > most ? b : most;
        }
        expect(samples == n * N && most == 2, "every micro-batch is forwarded once, two at a time at most");
        // (every pass of the second worker waits for every pass of the first whose rows it reads)
        if (threads[0] == '1')
            expect(stub_counters.waits_without_record == 0 && stub_counters.waits == (int)kernel_stubs.conv_samples.size() + n, "waits");
    }
    unsetenv("TMPS_ISSUE_THREADS");
}

int main() {
    short_run();
    k_streams();
    failing_pass();
    long_maps();
    return bad ? 1 : 0;
}
