// Host-only driver of the pipeline runner: which streams and events a run uses.
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

int main() {
    short_run();
    return bad ? 1 : 0;
}
