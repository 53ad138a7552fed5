// Stand-ins for the kernel launchers of libtmps (paper_2410_14312_amd/csrc/kernels.h) in host-only sanitizer builds of
// the stage executor: nothing is launched, every launcher reports success, and the workspace sizes are small fixed
// functions of the shape.  Only the host logic of csrc/stage.cpp (layout, argument checks, slot and buffer
// bookkeeping) is exercised by such a build.
#include "kernel_stubs.h"

#include <string.h>

#include "../../paper_2410_14312_amd/csrc/kernels.h"

KernelStubs kernel_stubs;

// A launch under `joint`: its arrays, read or written whole (null: not given).
static volatile unsigned char sink;
struct Launch {
    const char* name;
    const bool on;
    explicit Launch(const char* n) : name(n), on(kernel_stubs.joint) {
        if (!on) return;
        std::lock_guard<std::mutex> lock(kernel_stubs.m);
        ++kernel_stubs.launches[n];
    }
    void keep(const void* p, size_t bytes, bool write) const {
        std::lock_guard<std::mutex> lock(kernel_stubs.m);
        kernel_stubs.touched.push_back({name, p, bytes, write});
    }
    const Launch& reads(const void* p, size_t bytes) const {
        if (!on || !p) return *this;
        unsigned char sum = 0;
        for (size_t i = 0; i < bytes; ++i) sum += static_cast<const unsigned char*>(p)[i];
        sink = sum;
        keep(p, bytes, false);
        return *this;
    }
    const Launch& writes(void* p, size_t bytes) const {
        if (!on || !p) return *this;
        memset(p, 1, bytes);
        keep(p, bytes, true);
        return *this;
    }
};

namespace tmps {
static size_t esize(int dtype) { return dtype == kBF16 ? 2 : 4; }
size_t affine_workspace_elems(int64_t, int C) { return (size_t)(2 * C * 8); }

hipError_t dense_forward(int dtype, const void* x, const void* w, const float* bias, void* y, int B, int Din, int Dout, int act, int out_f32, const void* res, void* zout, float* ws, hipStream_t s) { return hipSuccess; }
hipError_t dense_dgrad(int dtype, const void* dy, const void* w, void* dx, const void* mask, int mask_mode, const void* add, int B, int Din, int Dout, float* ws, hipStream_t s) { return hipSuccess; }
hipError_t dense_wgrad(int dtype, const void* dy, const void* x, float* gw, int B, int Din, int Dout, const Partials& ws, hipStream_t s) { return hipSuccess; }
hipError_t reduce_all(const Reductions& list, hipStream_t) {
    for (const Reduction& r : list) Launch("reduce").reads(r.part, (size_t)r.slices * r.count * 4).writes(r.out, (size_t)r.count * 4);
    return hipSuccess;
}
hipError_t dense_backward(int, const void*, const void*, const void*, float*, void*, const void*, int, const void*, int, int, int, float*, const Partials&, hipStream_t) { return hipSuccess; }
bool dense_wgrad_groups(int, int64_t, int, int) { return true; }
int64_t dense_wgrad_group_elems(int64_t, const int (*)[2], int n) { return n > 1 ? 1000 : -1; }
hipError_t dense_wgrad_group(int, const DenseWgradJob*, int, int64_t, float*, int64_t, hipStream_t) { return hipSuccess; }
bool norm_dense_takes(int, int64_t, int, int) { return kernel_stubs.joint; }
hipError_t norm_dense_forward(int dtype, const void* x, const float* gamma, const float* beta, void* y, float* stats, float, const void* w, const float* bias, void* out, int rows, int D, int Dout, int, int out_f32, const void* res, void* zout, hipStream_t) {
    const size_t e = esize(dtype), in = (size_t)rows * D * e, eo = out_f32 ? 4 : e, to = (size_t)rows * Dout * eo;
    Launch("norm_dense_forward").reads(x, in).reads(gamma, D * 4).reads(beta, D * 4).writes(y, in).writes(stats, (size_t)rows * 8).reads(w, (size_t)D * Dout * e)
        .reads(bias, (size_t)Dout * 4).reads(res, to).writes(out, to).writes(zout, to);
    return hipSuccess;
}
hipError_t conv_forward(int dtype, const void* x, const void* w, const float* bias, void* y, const ConvShape& c, int relu, float* ws, hipStream_t s) {
    std::lock_guard<std::mutex> lock(kernel_stubs.m);
    kernel_stubs.conv_samples.push_back(c.B);
    return hipSuccess;
}
hipError_t conv_affine_forward(int dtype, const void* x, const void* w, const float* bias, void* z, const float* gain, const float* shift, void* again, const void* res, void* yout, int relu, const ConvShape& c, float* ws, hipStream_t s) {
    const size_t e = esize(dtype), in = (size_t)c.B * c.H * c.W * c.Cin * e, out = (size_t)c.B * c.Ho * c.Wo * c.Cout * e, ch = (size_t)c.Cout * 4;
    Launch("conv_affine_forward").reads(x, in).reads(w, (size_t)c.Cout * c.R * c.S * c.Cin * e).reads(bias, ch).reads(gain, ch).reads(shift, ch).reads(res, out)
        .writes(z, out).writes(yout, out).writes(again, out);
    return hipSuccess;
}
hipError_t conv_dgrad(int dtype, const void* dy, const void* w, void* dx, const void* mask, const void* add, const ConvShape& c, float* ws, hipStream_t s) {
    const size_t e = esize(dtype), in = (size_t)c.B * c.H * c.W * c.Cin * e;
    Launch("conv_dgrad").reads(dy, (size_t)c.B * c.Ho * c.Wo * c.Cout * e).reads(w, (size_t)c.Cout * c.R * c.S * c.Cin * e).reads(mask, in).reads(add, in).writes(dx, in);
    return hipSuccess;
}
hipError_t conv_wgrad(int dtype, const void* dy, const void* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    const size_t e = esize(dtype), count = (size_t)c.Cout * (c.R * c.S * c.Cin + 1);
    Launch("conv_wgrad").reads(dy, (size_t)c.B * c.Ho * c.Wo * c.Cout * e).reads(x, (size_t)c.B * c.H * c.W * c.Cin * e).writes(ws.ws, 2 * count * 4);
    return ws.finish(Reduction{ws.ws, gw, (int64_t)count, 2, false}, s);
}
bool pointwise_forward_takes(int64_t, int Cin, int Cout, bool) { return kernel_stubs.joint && Cout >= Cin; }
hipError_t pointwise_forward(const PointwiseForward& f, const PointwiseForward* next, int64_t P, int Cin, int Cout, hipStream_t) {
    const size_t c = Cin, w = Cout, narrow = (size_t)P * c * 2, wide = (size_t)P * w * 2;
    const Launch l(next ? "pointwise_forward of two" : "pointwise_forward");
    l.reads(f.x, narrow).reads(f.w, w * c * 2).reads(f.bias, w * 4).reads(f.gain, w * 4).reads(f.shift, w * 4).reads(f.res, wide).writes(f.z, wide).writes(f.y, wide)
        .writes(f.again, wide);
    if (next) l.reads(next->w, w * c * 2).reads(next->bias, c * 4).reads(next->gain, c * 4).reads(next->shift, c * 4).writes(next->z, narrow).writes(next->y, narrow);
    return hipSuccess;
}
bool affine_pointwise_takes(int dtype, int64_t, int, int) { return kernel_stubs.joint && dtype == kBF16; }
int affine_pointwise_slabs(int64_t, int, int) { return 3; }
hipError_t affine_pointwise_backward(const void* dy, const void* z, const void* x, const void* w, const float* gain, const void* add, int, void* dx, float* gw_affine, float* gw_conv, const Partials& pa, const Partials& pw, int64_t P, int O, int I, hipStream_t s) {
    const size_t out = (size_t)P * O * 2, in = (size_t)P * I * 2, slabs = affine_pointwise_slabs(P, O, I);
    Launch("affine_pointwise_backward").reads(dy, out).reads(z, out).reads(x, in).reads(w, (size_t)O * I * 2).reads(gain, (size_t)O * 4).reads(add, in).writes(dx, in)
        .writes(pa.ws, slabs * 2 * O * 4).writes(pw.ws, slabs * ((size_t)O * I + O) * 4);
    const hipError_t e = pa.finish(Reduction{pa.ws, gw_affine, 2 * O, (int)slabs, true}, s);
    return e != hipSuccess ? e : pw.finish(Reduction{pw.ws, gw_conv, (int64_t)O * I + O, (int)slabs, false}, s);
}
int maxpool_winner_bytes(int k) { return k <= 11 ? 1 : 4; }
bool maxpool_affine_takes(int, int64_t, int, int, int) { return kernel_stubs.joint; }
static size_t pooled(int B, int H, int W, int C, int k, int stride, int pad) { return (size_t)B * ((H + 2 * pad - k) / stride + 1) * ((W + 2 * pad - k) / stride + 1) * C; }
hipError_t maxpool_affine_backward(int dtype, const void* dy, const void* won, const void* z, const float* gain, void* dz, float* dgain_dshift, const Partials& ws, int B, int H, int W, int C, int k, int stride, int pad, int, hipStream_t s) {
    const size_t e = esize(dtype), in = (size_t)B * H * W * C * e, out = pooled(B, H, W, C, k, stride, pad);
    const int slabs = (int)(affine_workspace_elems((int64_t)B * H * W, C) / (2 * C));
    Launch("maxpool_affine_backward").reads(dy, out * e).reads(won, out).reads(z, in).reads(gain, (size_t)C * 4).writes(dz, in).writes(ws.ws, (size_t)slabs * 2 * C * 4);
    return ws.finish(Reduction{ws.ws, dgain_dshift, 2 * C, slabs, true}, s);
}
hipError_t maxpool_forward(int dtype, const void* x, void* y, void* won, int B, int H, int W, int C, int k, int stride, int pad, hipStream_t s) {
    const size_t e = esize(dtype), out = pooled(B, H, W, C, k, stride, pad);
    Launch("maxpool_forward").reads(x, (size_t)B * H * W * C * e).writes(y, out * e).writes(won, out * maxpool_winner_bytes(k));
    return hipSuccess;
}
hipError_t maxpool_backward(int dtype, const void* dy, const void* won, void* dx, int B, int H, int W, int C, int k, int stride, int pad, int relu_mask, hipStream_t s) {
    const size_t e = esize(dtype), out = pooled(B, H, W, C, k, stride, pad);
    Launch("maxpool_backward").reads(dy, out * e).reads(won, out * maxpool_winner_bytes(k)).writes(dx, (size_t)B * H * W * C * e);
    return hipSuccess;
}
hipError_t affine_forward(int dtype, const void* x, const float* gain, const float* shift, void* y, int64_t rows, int C, int relu, hipStream_t s) {
    const size_t n = (size_t)rows * C * esize(dtype), ch = (size_t)C * 4;
    Launch("affine_forward").reads(x, n).reads(gain, ch).reads(shift, ch).writes(y, n);
    return hipSuccess;
}
hipError_t affine_backward(int dtype, const void* dy, const void* x, const float* gain, void* dx, float* dgain_dshift, const Partials& ws, int64_t rows, int C, hipStream_t s) {
    const size_t n = (size_t)rows * C * esize(dtype), slabs = affine_workspace_elems(rows, C) / (2 * C);
    Launch("affine_backward").reads(dy, n).reads(x, n).reads(gain, (size_t)C * 4).writes(dx, n).writes(ws.ws, slabs * 2 * C * 4);
    return ws.finish(Reduction{ws.ws, dgain_dshift, 2 * C, (int)slabs, true}, s);
}
hipError_t resadd_forward(int dtype, const void* a, const void* b, void* y, int64_t n, int relu, hipStream_t s) { return hipSuccess; }
hipError_t avgpool_forward(int dtype, const void* x, void* y, int B, int HW, int C, hipStream_t s) { return hipSuccess; }
hipError_t avgpool_backward(int dtype, const void* dy, const void* x, void* dx, int B, int HW, int C, int relu_mask, hipStream_t s) { return hipSuccess; }
hipError_t layernorm_forward(int dtype, const void* x, const float* gamma, const float* beta, void* y, float* stats, int64_t rows, int D, float eps, hipStream_t s) { return hipSuccess; }
hipError_t layernorm_backward(int dtype, const void* dy, const void* x, const float* stats, const float* gamma, const void* add, void* dx, float* dgamma_dbeta, const Partials& ws, int64_t rows, int D, hipStream_t s) { return hipSuccess; }
hipError_t attention_forward(int dtype, const void* qkv, void* o, float* lse, int B, int S, int D, int H, hipStream_t s) { return hipSuccess; }
hipError_t attention_backward(int dtype, const void* qkv, const void* o, const void* dout, const float* lse, float* delta, void* dqkv, int B, int S, int D, int H, hipStream_t s) { return hipSuccess; }
hipError_t embedding_forward(int dtype, const int32_t* tok, const void* wte, const void* wpe, void* y, int64_t rows, int S, int D, int vocab, hipStream_t s) { return hipSuccess; }
hipError_t embedding_backward(int dtype, const int32_t* tok, const void* dy, float* dwte, float* dwpe, int64_t B, int S, int D, int vocab, hipStream_t s) { return hipSuccess; }
hipError_t softmax_ce(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* row_loss, int rows, int C, float inv_M, hipStream_t s) {
    return kernel_stubs.losses_until_failure-- == 0 ? hipErrorLaunchFailure : hipSuccess;
}
bool softmax_ce_small_takes(int64_t, int) { return false; }
hipError_t softmax_ce_small(int, const float*, const int32_t*, void*, float*, float*, int, int, int, float, float, float*, hipStream_t) { return hipSuccess; }
hipError_t reduce_scaled_sum(const float* in, int n, float scale, float* out, hipStream_t s) { return hipSuccess; }
hipError_t relu_mask(int dtype, const void* dy, const void* y, void* dz, int64_t n, hipStream_t s) { return hipSuccess; }
hipError_t sgd_momentum(float* w, float* buf, const float* g, void* wcopy_bf16, int64_t n, float lr, float mu, hipStream_t s) { return hipSuccess; }
hipError_t sgd_momentum_all(const Update*, int, hipStream_t) { return hipSuccess; }
hipError_t sgd_momentum_keeping(float* w, float* buf, const float* g, void* wcopy_bf16, int64_t n, float lr, float mu, float* kept_w, void* kept_wcopy, hipStream_t s) {
    memcpy(kept_w, w, (size_t)n * 4);
    if (wcopy_bf16) memcpy(kept_wcopy, wcopy_bf16, (size_t)n * 2);
    return hipSuccess;
}
hipError_t cast_f32_to_bf16(const float* in, void* out, int64_t n, hipStream_t s) { return hipSuccess; }
hipError_t copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t) { memcpy(dst, src, bytes); return hipSuccess; }
GemmPlan plan_gemm(int64_t, int64_t, int64_t) { return GemmPlan{64, 1}; }
size_t conv_wgrad_workspace_elems(int, const ConvShape& c) { return (size_t)(2 * ((int64_t)c.Cout * c.R * c.S * c.Cin + c.Cout)); }
size_t gemm_workspace_elems(int64_t M, int64_t N, int64_t, int with_rowsum) { return (size_t)(2 * (M * N + (with_rowsum ? M : 0))); }
size_t layernorm_workspace_elems(int64_t, int D) { return (size_t)(2 * D * 8); }
size_t attention_workspace_elems(int B, int S, int H) { return (size_t)B * S * H; }
}  // namespace tmps

// Profiling is off in these builds, and the three HIP runtime calls the stage executor makes itself are replaced: a
// "device-to-device" copy is a host memcpy here (the regions are host memory), so that the sanitizer also checks the
// bounds of the stash copies.  Nothing in such a build can reach a GPU.
#include <string.h>

#include "../../paper_2410_14312_amd/csrc/profile.h"

namespace tmps {
bool profile_on() { return false; }
void profile_begin(int, hipStream_t) {}
void profile_end(int, hipStream_t) {}
bool profile_kernel_begin(KernelEvents&) { return false; }
void profile_kernel_end(int, const KernelEvents&) {}
}  // namespace tmps

extern "C" hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t) {
    memcpy(dst, src, bytes);
    return hipSuccess;
}
extern "C" hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
// (graph replay is off in these builds: the calls exist for the linker only)
extern "C" hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
extern "C" hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
extern "C" hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
extern "C" hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
extern "C" hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
extern "C" hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
extern "C" const char* hipGetErrorString(hipError_t) { return "stub"; }
