// What the kernel stand-ins of kernel_stubs.cpp keep and can be told.
#pragma once
#include <atomic>
#include <mutex>
#include <vector>

struct KernelStubs {
    std::mutex m;
    std::vector<int> conv_samples;                // samples of every convolution's forward pass
    std::atomic<int> losses_until_failure{-1};    // the loss layer's forward passes that succeed before one fails (negative: all)
};
extern KernelStubs kernel_stubs;
