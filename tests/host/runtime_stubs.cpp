// Stand-ins for the HIP runtime calls that the pipeline runner (paper_2410_14312_amd/csrc/run.cpp) makes, for host-only
// builds beside kernel_stubs.cpp: streams are plain addresses and always idle, events only know whether they have been
// recorded.  A wait for an event that nobody has recorded is counted: on a device it would be no wait at all.
#include "runtime_stubs.h"

#include <deque>
#include <mutex>

StubCounters stub_counters;

namespace {
std::mutex m;
std::deque<bool> recorded;   // (addresses of its elements stand for the events; never freed)
}  // namespace

extern "C" hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    std::lock_guard<std::mutex> lock(m);
    recorded.push_back(false);
    *e = reinterpret_cast<hipEvent_t>(&recorded.back());
    ++stub_counters.events;
    return hipSuccess;
}
extern "C" hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    std::lock_guard<std::mutex> lock(m);
    *reinterpret_cast<bool*>(e) = true;
    ++stub_counters.records;
    return hipSuccess;
}
extern "C" hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned) {
    std::lock_guard<std::mutex> lock(m);
    ++stub_counters.waits;
    if (!*reinterpret_cast<bool*>(e)) ++stub_counters.waits_without_record;
    return hipSuccess;
}
extern "C" hipError_t hipStreamQuery(hipStream_t) { return stub_counters.busy_streams ? hipErrorNotReady : hipSuccess; }
extern "C" hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
extern "C" hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }
extern "C" hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
extern "C" hipError_t hipSetDevice(int) { return hipSuccess; }
