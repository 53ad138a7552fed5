// Pipelines on plain host memory for the host-only drivers of the pipeline runner.
#pragma once
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <initializer_list>
#include <vector>

#include "../../include/tmps.h"

static int bad = 0;
static void expect(bool ok, const char* what) {
    if (!ok) {
        fprintf(stderr, "FAILED: %s (%s)\n", what, tmps_last_error());
        ++bad;
    }
}

static tmps_layer_desc L(int kind, std::initializer_list<int> dims, int flags = 0) {
    tmps_layer_desc d;
    memset(&d, 0, sizeof(d));
    d.kind = kind;
    int i = 0;
    for (int v : dims) d.dims[i++] = v;
    d.flags = flags;
    return d;
}

struct Pipe {
    std::vector<tmps_stage*> stages;
    std::vector<void*> memory;
    std::vector<char> input;
    std::vector<int32_t> labels;
    std::vector<void*> streams;
    int N;
    std::vector<float> losses;

    // layers[s]: the layers of stage s; groups and kept versions as the mode's schedule needs them (1F1B: N = 1)
    Pipe(const std::vector<std::vector<tmps_layer_desc>>& layers, int dtype, int micro, int N_, int n_minibatches, bool vsync, bool one_f1b) : N(N_) {
        const int K = (int)layers.size();
        for (int s = 0; s < K; ++s) {
            tmps_stage_cfg c;
            memset(&c, 0, sizeof(c));
            c.dtype = dtype; c.micro_batch = micro; c.n_micro = N; c.is_last = s == K - 1; c.borrow_input = 1;
            c.max_stash = N * (one_f1b ? K - s : tmps_schedule_stash_groups(K, N, s));
            c.lr = 0.01f;
            size_t sz[4];
            expect(tmps_stage_bytes(layers[s].data(), (int)layers[s].size(), &c, &sz[0], &sz[1], &sz[2], &sz[3]) == TMPS_OK, "sizes");
            void* r[4];
            for (int i = 0; i < 4; ++i) r[i] = region(sz[i]);
            tmps_stage* st = nullptr;
            expect(tmps_stage_create(&st, layers[s].data(), (int)layers[s].size(), &c, r[0], r[1], r[2], r[3]) == TMPS_OK, "create");
            const int kept = one_f1b ? K - s - 1 : vsync ? tmps_schedule_shadow_versions(K, N, s) : 0;
            if (kept > 0) expect(tmps_stage_set_shadow(st, region(sz[0] * kept), sz[0] * kept, kept) == TMPS_OK, "kept versions");
            stages.push_back(st);
            streams.push_back(reinterpret_cast<void*>((uintptr_t)(64 * (s + 1))));   // (never looked into)
        }
        const size_t rows = (size_t)n_minibatches * N * micro;
        input.resize(rows * tmps_stage_input_elems(stages[0]) * 4);
        labels.resize(rows);
        losses.resize(n_minibatches);
    }
    void* region(size_t bytes) {
        void* p = aligned_alloc(256, (bytes + 255) / 256 * 256 + 256);
        memory.push_back(p);
        return p;
    }
    ~Pipe() {
        for (tmps_stage* s : stages) tmps_stage_destroy(s);
        for (void* p : memory) free(p);
    }
};
