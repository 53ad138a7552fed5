// What the kernel stand-ins of kernel_stubs.cpp keep and can be told.
#pragma once
#include <stddef.h>

#include <atomic>
#include <map>
#include <mutex>
#include <string>
#include <vector>

struct KernelStubs {
    std::mutex m;
    std::vector<int> conv_samples;                // samples of every convolution's forward pass
    std::atomic<int> losses_until_failure{-1};    // the loss layer's forward passes that succeed before one fails (negative: all)

    // Launches that hold several layers' work.  With `joint` they are taken wherever a kernel could have such widths; the launchers that take part then read all of their
    // inputs and write all of their results, so that a sanitizer sees a layout that is too small, and what they touched is kept.
    struct Touched {
        const char* launch;
        const void* at;
        size_t bytes;
        bool write;
    };
    std::atomic<bool> joint{false};
    std::map<std::string, int> launches;
    std::vector<Touched> touched;
    void clear() {
        launches.clear();
        touched.clear();
    }
};
extern KernelStubs kernel_stubs;
