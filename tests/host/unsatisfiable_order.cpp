// Host-only driver: the pipeline runner on task lists in which a pass waits for one that never comes (a stand-in for the
// planner gives them).  A run must say so instead of reporting a training step that it did not make, and leave the stages
// able to run again.
#include "../../paper_2410_14312_amd/csrc/schedule.h"
#include "run_stages.h"

namespace tmps {
static bool complete = false;
// Two workers, one micro-batch, one mini-batch; incomplete: worker 1 has no backward pass, worker 0's waits for it.
std::vector<Task> plan_nf1b(int, int, int) {
    std::vector<Task> t = {{1, 0, kFwd, 1, 0, 0, 0}, {2, 1, kFwd, 1, 0, 0, 0}};
    if (complete) t.push_back({3, 1, kBwd, 1, -1, 0, 0});
    t.push_back({4, 0, kBwd, 1, -1, 0, 0});
    return t;
}
std::vector<Task> plan_1f1b(int W, int n) { return plan_nf1b(W, 1, n); }
int stash_groups(int, int, int) { return 1; }
int shadow_versions(int, int, int) { return 0; }
}  // namespace tmps
extern "C" int tmps_schedule_stash_groups(int, int, int) { return 1; }
extern "C" int tmps_schedule_shadow_versions(int, int, int) { return 0; }

int main() {
    Pipe p({{L(TMPS_LINEAR, {16, 16, 0, 1})}, {L(TMPS_LINEAR, {16, 10, 0, 1}), L(TMPS_SOFTMAX_CE, {10, 1})}}, TMPS_F32, 4, 1, 1, false, false);
    auto run = [&]() {
        return tmps_schedule_run(p.stages.data(), 2, 1, 1, p.input.data(), p.labels.data(), p.streams.data(), p.losses.data(), nullptr);
    };
    expect(run() == TMPS_EINVAL && strstr(tmps_last_error(), "order"), "an order that cannot be satisfied is reported");
    expect(tmps_stage_version(p.stages[0]) == 0 && tmps_stage_version(p.stages[1]) == 0, "no update was made");
    tmps::complete = true;
    expect(run() == TMPS_OK, "the stages run again");
    expect(tmps_stage_version(p.stages[0]) == 1 && tmps_stage_version(p.stages[1]) == 1, "both updates were made");
    return bad ? 1 : 0;
}
