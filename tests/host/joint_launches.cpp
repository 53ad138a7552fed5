// Host-only driver for a sanitizer build of the stage executor's paths that launch several layers' work together (csrc/stage.cpp; the launchers of
// kernel_stubs.cpp read and write all that such a kernel would).  Memory regions are exactly as large as the layout says, and whatever a launch touches among the
// parameters or their gradients has to lie in one layer's.  Every list of layers comes twice: as networks have it, where the launch is taken, and with a layer
// that reads the same values as a map of other channels, where it must not be.
#include <stdint.h>

#include "kernel_stubs.h"
#include "run_stages.h"

struct OneStage {
    std::vector<tmps_layer_desc> layers;
    tmps_stage_cfg c;
    size_t sz[4];
    void* r[4];
    tmps_stage* st = nullptr;

    OneStage(std::vector<tmps_layer_desc> ls, int dtype, int micro, int N) : layers(ls) {
        memset(&c, 0, sizeof(c));
        c.dtype = dtype; c.micro_batch = micro; c.n_micro = N; c.max_stash = N; c.borrow_input = 1;
        c.is_last = ls.back().kind == TMPS_SOFTMAX_CE;
        c.lr = 0.01f;
        expect(tmps_stage_bytes(ls.data(), (int)ls.size(), &c, &sz[0], &sz[1], &sz[2], &sz[3]) == TMPS_OK, "sizes");
        for (int i = 0; i < 4; ++i) {
            r[i] = aligned_alloc(256, sz[i]);
            memset(r[i], 0, sz[i]);
        }
        expect(tmps_stage_create(&st, ls.data(), (int)ls.size(), &c, r[0], r[1], r[2], r[3]) == TMPS_OK, "create");
    }
    ~OneStage() {
        tmps_stage_destroy(st);
        for (void* p : r) free(p);
    }
    // A mini-batch and the update, without and with the gradient of the input, in memory of its own or over the upstream one, with a second place for the result.
    void step() {
        const size_t M = (size_t)c.micro_batch * c.n_micro, in = tmps_stage_input_elems(st) * 4, out = tmps_stage_output_elems(st) * 4;
        std::vector<float> x(M * in), y(c.micro_batch * out), dy(M * out), dx(M * in);   // (on 16 bytes)
        std::vector<int32_t> labels(M);
        std::vector<int> slots;
        const size_t esz = c.dtype == TMPS_F32 ? 4 : 2;
        std::vector<float> same(M * (in > out ? in : out));
        for (int want = 0; want < 3; ++want) {
            slots.clear();
            for (int j = 0; j < c.n_micro; ++j) {
                const char* xj = reinterpret_cast<const char*>(x.data()) + (size_t)j * c.micro_batch * (in / 4) * esz;
                expect(tmps_forward_micro(st, j, xj, y.data(), c.is_last ? labels.data() : nullptr, nullptr, nullptr) == TMPS_OK, "forward");
                slots.push_back(j);
            }
            expect(tmps_backward(st, slots.data(), c.n_micro, c.is_last ? nullptr : want == 2 ? same.data() : dy.data(),
                                 want == 2 ? same.data() : want ? dx.data() : nullptr, nullptr) == TMPS_OK, "backward");
            expect(tmps_update(st, nullptr) == TMPS_OK, "update");
        }
    }
    // Whether [a, a + n) lies in one layer's array: weights or biases, in fp32 or as the working copy; of the gradients also both together.
    bool one_layers(uintptr_t a, size_t n) const {
        const size_t P = (size_t)tmps_stage_param_count(st);
        const uintptr_t master = (uintptr_t)r[0], copy = master + P * 4, grad = (uintptr_t)r[1] + P * 4;
        for (int l = 0; l < (int)layers.size(); ++l) {
            int64_t o[2], k[2];
            for (int which = 0; which < 2; ++which) expect(tmps_stage_param_offset(st, l, which, &o[which], &k[which]) == TMPS_OK, "offset");
            for (int which = 0; which < 2; ++which) {
                if (a >= master + o[which] * 4 && a + n <= master + (o[which] + k[which]) * 4) return true;
                if (a >= copy + o[which] * 2 && a + n <= copy + (o[which] + k[which]) * 2) return true;
            }
            if (a >= grad + o[0] * 4 && a + n <= grad + (o[1] + k[1]) * 4) return true;
        }
        return false;
    }
    void check_parameters() const {
        for (const auto& t : kernel_stubs.touched) {
            const uintptr_t a = (uintptr_t)t.at;
            for (int i = 0; i < 2; ++i)
                if (a >= (uintptr_t)r[i] && a < (uintptr_t)r[i] + sz[i]) {
                    if (!one_layers(a, t.bytes)) fprintf(stderr, "%s: %zu bytes at %zu of region %d\n", t.launch, t.bytes, (size_t)(a - (uintptr_t)r[i]), i);
                    expect(one_layers(a, t.bytes), "a launch stays in one layer's parameters");
                }
        }
    }
};

// `launch` is made this many times in three mini-batches (-1: at all)
static void run(const char* what, std::vector<tmps_layer_desc> layers, int dtype, const char* launch, int times, int micro = 2, int N = 2) {
    kernel_stubs.clear();
    OneStage s(layers, dtype, micro, N);
    if (!s.st) return;
    s.step();
    s.check_parameters();
    const int n = kernel_stubs.launches[launch];
    if (times < 0 ? n == 0 : n != times) fprintf(stderr, "%s: %s %d times\n", what, launch, n);
    expect(times < 0 ? n > 0 : n == times, what);
}

int main() {
    const int R = TMPS_FLAG_RELU, bf16 = TMPS_BF16_F32MASTER;
    kernel_stubs.joint = true;

    // a convolution and the affine layer that reads it
    for (int dtype : {(int)TMPS_F32, bf16}) {
        run("conv and affine", {L(TMPS_CONV2D, {4, 4, 8, 16, 3, 3, 1, 1}), L(TMPS_AFFINE, {4, 4, 16}, R)}, dtype, "conv_affine_forward", 6);
        run("conv and affine of the same channels on another map", {L(TMPS_CONV2D, {4, 4, 8, 16, 3, 3, 1, 1}), L(TMPS_AFFINE, {8, 2, 16}, R)}, dtype, "conv_affine_forward", 6);
        run("conv and affine of other channels", {L(TMPS_CONV2D, {4, 4, 8, 16, 3, 3, 1, 1}), L(TMPS_AFFINE, {8, 8, 4}, R)}, dtype, "conv_affine_forward", 0);
        run("conv and affine of more channels", {L(TMPS_CONV2D, {4, 4, 8, 16, 3, 3, 1, 1}), L(TMPS_AFFINE, {2, 2, 64}, R)}, dtype, "conv_affine_forward", 0);
    }
    // a 1 x 1 convolution and the affine layer that reads it, both gradients
    auto pointwise = [&](tmps_layer_desc aff) {
        return std::vector<tmps_layer_desc>{L(TMPS_CONV2D, {4, 4, 8, 16, 3, 3, 1, 1}, R), L(TMPS_CONV2D, {4, 4, 16, 32, 1, 1, 1, 0}), aff, L(TMPS_LINEAR, {512, 8, 0, 1})};
    };
    run("gradients of conv and affine", pointwise(L(TMPS_AFFINE, {4, 4, 32}, R)), bf16, "affine_pointwise_backward", 2);
    run("gradients of conv and affine of fewer channels", pointwise(L(TMPS_AFFINE, {8, 8, 8}, R)), bf16, "affine_pointwise_backward", 0);
    run("gradients of conv and affine of more channels", pointwise(L(TMPS_AFFINE, {2, 2, 128}, R)), bf16, "affine_pointwise_backward", 0);

    // a join and the next block's first convolution
    auto blocks = [&](tmps_layer_desc conv, tmps_layer_desc aff, tmps_layer_desc last) {
        return std::vector<tmps_layer_desc>{L(TMPS_CONV2D, {4, 4, 8, 256, 1, 1, 1, 0}, R), L(TMPS_CONV2D, {4, 4, 256, 64, 1, 1, 1, 0}), L(TMPS_AFFINE, {4, 4, 64}, R),
                                            L(TMPS_CONV2D, {4, 4, 64, 256, 1, 1, 1, 0}), L(TMPS_AFFINE, {4, 4, 256}), L(TMPS_RESADD, {4, 4, 256, 5}, R), conv, aff, last};
    };
    const auto pair = "pointwise_forward of two";
    run("join and convolution", blocks(L(TMPS_CONV2D, {4, 4, 256, 64, 1, 1, 1, 0}), L(TMPS_AFFINE, {4, 4, 64}, R), L(TMPS_CONV2D, {4, 4, 64, 8, 1, 1, 1, 0})), bf16, pair, 6);
    run("join and convolution that reads other channels", blocks(L(TMPS_CONV2D, {8, 8, 64, 64, 1, 1, 1, 0}), L(TMPS_AFFINE, {8, 8, 64}, R), L(TMPS_CONV2D, {8, 8, 64, 8, 1, 1, 1, 0})),
        bf16, pair, 0);
    run("join, convolution and affine of other channels", blocks(L(TMPS_CONV2D, {4, 4, 256, 64, 1, 1, 1, 0}), L(TMPS_AFFINE, {8, 8, 16}, R), L(TMPS_CONV2D, {8, 8, 16, 8, 1, 1, 1, 0})),
        bf16, pair, 0);

    // max pooling behind an affine layer
    auto pooled = [&](tmps_layer_desc pool, int n) {
        return std::vector<tmps_layer_desc>{L(TMPS_CONV2D, {8, 8, 8, 16, 3, 3, 1, 1}), L(TMPS_AFFINE, {8, 8, 16}, R), pool, L(TMPS_LINEAR, {n, 8, 0, 1})};
    };
    for (int dtype : {(int)TMPS_F32, bf16}) {
        run("pooling and affine", pooled(L(TMPS_MAXPOOL, {8, 8, 16, 3, 2, 1}), 4 * 4 * 16), dtype, "maxpool_affine_backward", 2);
        run("pooling and affine on another map", pooled(L(TMPS_MAXPOOL, {16, 4, 16, 3, 2, 1}), 8 * 2 * 16), dtype, "maxpool_affine_backward", 2);
        run("pooling in larger windows", pooled(L(TMPS_MAXPOOL, {4, 4, 64, 12, 4, 5}), 64), dtype, "maxpool_backward", 3);
        run("pooling and affine of fewer channels", pooled(L(TMPS_MAXPOOL, {4, 4, 64, 3, 2, 1}), 2 * 2 * 64), dtype, "maxpool_affine_backward", 0);
        run("pooling and affine of more channels", pooled(L(TMPS_MAXPOOL, {16, 16, 4, 3, 2, 1}), 8 * 8 * 4), dtype, "maxpool_affine_backward", 0);
    }
    // a layer normalisation and the dense layer behind it
    for (int dtype : {(int)TMPS_F32, bf16})
        run("norm and dense", {L(TMPS_LAYERNORM, {16, 3}), L(TMPS_LINEAR, {16, 24, 0, 3}, TMPS_FLAG_GELU), L(TMPS_LINEAR, {24, 16, 2, 3}), L(TMPS_LAYERNORM, {16, 3}),
                               L(TMPS_LINEAR, {16, 16, 1, 3}, R)}, dtype, "norm_dense_forward", 12);
    // bottleneck blocks: one with a strided projection, whose input gradient waits for the other readers of the block's input, and one without, at the stage input, behind
    // a layer with an activation and one without, and in front of another of either kind
    auto bottleneck = [&](int h, int cin, int width, int stride, bool project) {
        const int ho = (h - 1) / stride + 1, cout = 4 * width;
        std::vector<tmps_layer_desc> b = {L(TMPS_CONV2D, {h, h, cin, width, 1, 1, 1, 0}), L(TMPS_AFFINE, {h, h, width}, R), L(TMPS_CONV2D, {h, h, width, width, 3, 3, stride, 1}),
                                          L(TMPS_AFFINE, {ho, ho, width}, R), L(TMPS_CONV2D, {ho, ho, width, cout, 1, 1, 1, 0}), L(TMPS_AFFINE, {ho, ho, cout})};
        if (project) {
            b.push_back(L(TMPS_CONV2D, {h, h, cin, cout, 1, 1, stride, 0}, TMPS_FLAG_SRC(7)));
            b.push_back(L(TMPS_AFFINE, {ho, ho, cout}));
            b.push_back(L(TMPS_RESADD, {ho, ho, cout, 3}, R));
        } else
            b.push_back(L(TMPS_RESADD, {ho, ho, cout, 7}, R));
        return b;
    };
    for (int below = 0; below < 3; ++below)
        for (int stride = 1; stride < 4; ++stride)
            for (int second = 0; second < 3; ++second)
                for (int last = 0; last < 2; ++last) {
                    std::vector<tmps_layer_desc> ls;
                    if (below) ls.push_back(L(TMPS_CONV2D, {7, 7, 8, 16, 3, 3, 1, 1}, below == 1 ? R : 0));
                    int h = 7, c = 16;
                    auto add = [&](int width, int st, bool project) {
                        const auto b = bottleneck(h, c, width, st, project);
                        ls.insert(ls.end(), b.begin(), b.end());
                        h = (h - 1) / st + 1;
                        c = 4 * width;
                    };
                    add(8, stride, true);
                    if (second) add(8, 1, second == 2);
                    add(8, 2, true);
                    if (last) {
                        ls.push_back(L(TMPS_AVGPOOL, {h, h, c}));
                        ls.push_back(L(TMPS_LINEAR, {c, 10, 0, 1}));
                        ls.push_back(L(TMPS_SOFTMAX_CE, {10, 1}));
                    }
                    run("bottleneck blocks", ls, bf16, "conv_dgrad", -1);
                    run("bottleneck blocks", ls, TMPS_F32, "conv_affine_forward", -1);
                }
    return bad ? 1 : 0;
}
