// What the runtime stand-ins of runtime_stubs.cpp have seen, and what they are to pretend.
#pragma once
#include <hip/hip_runtime.h>

struct StubCounters {
    int events = 0, records = 0, waits = 0, waits_without_record = 0;
    bool busy_streams = false;   // hipStreamQuery: work is pending
};
extern StubCounters stub_counters;
