// Host-side launch interface of the HIP kernels (internal to libtmps).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace tmps {

// dtype codes match TMPS_F32 / TMPS_BF16_F32MASTER
constexpr int kF32 = 0;
constexpr int kBF16 = 1;

inline size_t act_bytes(int dtype) { return dtype == kBF16 ? 2 : 4; }

// Sum of partial results: out[i] = sum over z < slices of part[z * count + i], i < count: eight at a time, in pairs, and the totals in
// order (k-slices of a contraction) or, where many short rows are added up (slabs of a normalisation or affine layer), in sixteen such sums side by side.  What a backward pass adds up of its
// parameter gradients can wait for its end and be one launch: a launcher that is given a list to put its sum on leaves it to
// reduce_all, and its partial results stay in memory of their own until then.
struct Reduction {
    const float* part;
    float* out;
    int64_t count;
    int slices;
    bool rows;
};
typedef std::vector<Reduction> Reductions;
hipError_t reduce_all(const Reductions& list, hipStream_t s);

// Memory for partial results (may be null: then nothing is split) and, if their sum can wait, the list to put it on.
struct Partials {
    float* ws;
    Reductions* later;
    Partials(float* p, Reductions* l = nullptr) : ws(p), later(l) {}
    hipError_t finish(const Reduction& r, hipStream_t s) const {
        if (!later) return reduce_all(Reductions(1, r), s);
        later->push_back(r);
        return hipSuccess;
    }
};

struct ConvShape {
    int B, H, W, Cin, Ho, Wo, Cout, R, S, stride, pad;
    // conv_dgrad, of a pass that adds to dx in place: positions that no filter tap reaches have their final value (the mask applied) already
    int rest_done = 0;
};

// Tile edge (64 or 128) and number of k-slices chosen for a bf16 [M x N x K] contraction.
struct GemmPlan {
    int tile, slices;
};
GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K);
// fp32 workspace elements that the partial sums of a contraction need (0 without a split).  flags: kWsRowSums: a
// weight-gradient GEMM, which also keeps M row sums per slice; kWsF32: fp32 operands.  Every launcher below takes that
// workspace as `ws` (may be null: then nothing is split).
enum { kWsRowSums = 1, kWsF32 = 2 };
size_t gemm_workspace_elems(int64_t M, int64_t N, int64_t K, int flags);

// y[B, Dout] = act(x[B, Din] w^T + b).  w is the working copy (bf16 or fp32 per dtype), bias fp32.
// out_f32: write fp32 regardless of dtype (logits).
// act: 0 none, 1 ReLU, 2 exact GELU (then zout, if not null, receives the derivative gelu'(pre-activation) for the backward
// pass; without GELU it receives y once more).  res (may be
// null): tensor of y's shape and dtype added after the activation (residual connection).
hipError_t dense_forward(int dtype, const void* x, const void* w, const float* bias, void* y, int B,
                         int Din, int Dout, int act, int out_f32, const void* res, void* zout, float* ws,
                         hipStream_t s);
// A layer normalisation (y and stats as layernorm_forward leaves them) and the dense layer that reads it (as dense_forward) in one launch;
// norm_dense_takes: where that is quicker.
bool norm_dense_takes(int dtype, int64_t rows, int D, int Dout);
hipError_t norm_dense_forward(int dtype, const void* x, const float* gamma, const float* beta, void* y, float* stats, float eps, const void* w, const float* bias,
                              void* out, int rows, int D, int Dout, int act, int out_f32, const void* res, void* zout, hipStream_t s);
// dx[B, Din] = dy[B, Dout] w, passed through the activation of the layer below: mask_mode 1: zeroed
// where mask[B, Din] <= 0 (mask = that layer's output); mask_mode 2: times gelu'(mask) (mask = that
// layer's pre-activation).  mask may be null; activation dtype.
hipError_t dense_dgrad(int dtype, const void* dy, const void* w, void* dx, const void* mask, int mask_mode,
                       const void* add, int B, int Din, int Dout, float* ws, hipStream_t s);
// `add` (may be null; may be dx itself): tensor of dx's shape added BEFORE the mask is applied: the
// gradient that other readers of the same input have already contributed.
// gw[Dout, Din] = dy^T x and gb[Dout] = column sums of dy, with gb stored right after gw.
hipError_t dense_wgrad(int dtype, const void* dy, const void* x, float* gw, int B, int Din, int Dout,
                       const Partials& ws, hipStream_t s);

// dense_wgrad and dense_dgrad (neither's result may overlap an operand of the other), in one launch where that is quicker.
hipError_t dense_backward(int dtype, const void* dy, const void* x, const void* w, float* gw, void* dx, const void* mask, int mask_mode,
                          const void* add, int B, int Din, int Dout, float* ws, const Partials& ws_w, hipStream_t s);
// The weight gradients of several dense layers over the same `rows` rows in one launch at the end of a backward pass.
// dense_wgrad_groups: whether a layer's can be part of one.  dense_wgrad_group_elems: fp32 workspace elements of the launch that
// takes these n layers (dims: Din, Dout), -1 where launches of their own are quicker.  In dense_wgrad_group, ws holds ws_elems.
constexpr int kWgradGroupMax = 32;
struct DenseWgradJob {
    const void* dy;
    const void* x;
    float* gw;
    int Din, Dout;
};
bool dense_wgrad_groups(int dtype, int64_t rows, int Din, int Dout);
int64_t dense_wgrad_group_elems(int64_t rows, const int (*dims)[2], int n);
hipError_t dense_wgrad_group(int dtype, const DenseWgradJob* jobs, int n, int64_t rows, float* ws, int64_t ws_elems, hipStream_t s);

hipError_t conv_forward(int dtype, const void* x, const void* w, const float* bias, void* y,
                        const ConvShape& c, int relu, float* ws, hipStream_t s);
// Convolution (no activation of its own) fused with the per-channel affine layer that follows it and, when res is given,
// with the residual join after that: y -> z (the convolution's result), yout and again (may be null) = act(affine + res).
hipError_t conv_affine_forward(int dtype, const void* x, const void* w, const float* bias, void* z, const float* gain,
                               const float* shift, void* again, const void* res, void* yout, int relu, const ConvShape& c,
                               float* ws, hipStream_t s);
hipError_t conv_dgrad(int dtype, const void* dy, const void* w, void* dx, const void* mask, const void* add,
                      const ConvShape& c, float* ws, hipStream_t s);
hipError_t conv_wgrad(int dtype, const void* dy, const void* x, float* gw, const ConvShape& c,
                      const Partials& ws, hipStream_t s);
size_t conv_wgrad_workspace_elems(int dtype, const ConvShape& c);   // fp32, for its partial results

// Forward pass of a 1 x 1 convolution of unit stride over P positions with its affine layer and, if res is given, the join (as conv_affine_forward, bf16);
// next: also the following convolution from those channels back to Cin with its affine layer (its x, res and again are not used).  All of it on 16 bytes.
// pointwise_forward_takes: where that is quicker, without and with a next one.
struct PointwiseForward {
    const void *x, *w, *res;
    const float *bias, *gain, *shift;
    void *z, *y, *again;
    int relu;
};
bool pointwise_forward_takes(int64_t P, int Cin, int Cout, bool next);
hipError_t pointwise_forward(const PointwiseForward& f, const PointwiseForward* next, int64_t P, int Cin, int Cout, hipStream_t s);

// Backward pass of a 1 x 1 convolution of unit stride (x [P][I] -> z [P][O]) and the affine layer that alone reads its result, in one pass: dy is the affine layer's
// incoming gradient, dx the convolution's input gradient (add: joined first, may be dx; masked: then zero where x <= 0), gw_affine and gw_conv as affine_backward and
// conv_wgrad leave them.  affine_pointwise_takes: where that is quicker; affine_pointwise_slabs: partial results of 2 O and O I + O values that pa and pw hold.
bool affine_pointwise_takes(int dtype, int64_t P, int O, int I);
int affine_pointwise_slabs(int64_t P, int O, int I);
hipError_t affine_pointwise_backward(const void* dy, const void* z, const void* x, const void* w, const float* gain, const void* add, int masked, void* dx,
                                     float* gw_affine, float* gw_conv, const Partials& pa, const Partials& pw, int64_t P, int O, int I, hipStream_t s);

// 2-D max pooling, channels-last.  won: every window's winner as the forward pass leaves it, maxpool_winner_bytes each (on as many bytes): the first maximum in
// row-major order, of which NaN is none (nor of the result); in a window of negative infinities and NaN alone the first place inside the map.  relu_mask: also zero
// where the input is <= 0.
int maxpool_winner_bytes(int k);
hipError_t maxpool_forward(int dtype, const void* x, void* y, void* won, int B, int H, int W, int C, int k, int stride, int pad, hipStream_t s);
hipError_t maxpool_backward(int dtype, const void* dy, const void* won, void* dx, int B, int H, int W, int C, int k, int stride, int pad, int relu_mask, hipStream_t s);
// The same behind an affine layer (affine_backward) that only the pooling reads, in one pass: z is that layer's input, dz its gradient (rows positions);
// dy, z, gain and dz on 16 bytes.
bool maxpool_affine_takes(int dtype, int64_t rows, int C, int k, int stride);
hipError_t maxpool_affine_backward(int dtype, const void* dy, const void* won, const void* z, const float* gain, void* dz, float* dgain_dshift, const Partials& ws,
                                   int B, int H, int W, int C, int k, int stride, int pad, int relu_mask, hipStream_t s);

// Per-channel affine layer on channels-last rows: y[r, c] = gain[c] x[r, c] + shift[c], then ReLU if asked.
hipError_t affine_forward(int dtype, const void* x, const float* gain, const float* shift, void* y, int64_t rows, int C,
                          int relu, hipStream_t s);
// dx (may be null) = gain * dy; dgain_dshift: C gain gradients (sum of dy * x) followed by C shift gradients (sum
// of dy); dy has already passed through the layer's own ReLU; ws: affine_workspace_elems.
hipError_t affine_backward(int dtype, const void* dy, const void* x, const float* gain, void* dx, float* dgain_dshift,
                           const Partials& ws, int64_t rows, int C, hipStream_t s);
size_t affine_workspace_elems(int64_t rows, int C);

// y = act(a + b), n elements.
hipError_t resadd_forward(int dtype, const void* a, const void* b, void* y, int64_t n, int relu, hipStream_t s);

// Global average pooling [B, HW, C] -> [B, C] and its gradient (relu_mask: zero where the stored input is <= 0).
hipError_t avgpool_forward(int dtype, const void* x, void* y, int B, int HW, int C, hipStream_t s);
hipError_t avgpool_backward(int dtype, const void* dy, const void* x, void* dx, int B, int HW, int C, int relu_mask,
                            hipStream_t s);

// Layer normalisation over rows of D features.  stats[rows][2] = (mean, 1/std) of the forward pass.
hipError_t layernorm_forward(int dtype, const void* x, const float* gamma, const float* beta, void* y,
                             float* stats, int64_t rows, int D, float eps, hipStream_t s);
// dx (may be null) = gradient w.r.t. x, plus `add` (may be null: gradient of a residual connection that
// joins x); dgamma_dbeta: D gain gradients followed by D shift gradients; ws: layernorm_workspace_elems.
hipError_t layernorm_backward(int dtype, const void* dy, const void* x, const float* stats, const float* gamma,
                              const void* add, void* dx, float* dgamma_dbeta, const Partials& ws, int64_t rows, int D,
                              hipStream_t s);
size_t layernorm_workspace_elems(int64_t rows, int D);

// Causal multi-head self-attention on packed rows [q | k | v] (3*D features, head h owns features
// h*D/H.. of each part).  o[B*S, D]; lse[B, H, S] = log-sum-exp of the scaled scores of each query.
hipError_t attention_forward(int dtype, const void* qkv, void* o, float* lse, int B, int S, int D, int H,
                             hipStream_t s);
// dqkv[B*S, 3*D] from the gradient dout[B*S, D] of the output; delta: workspace of B*H*S floats, for heads and
// addresses that the matrix kernels do not take (those form it as they go).
hipError_t attention_backward(int dtype, const void* qkv, const void* o, const void* dout, const float* lse,
                              float* delta, void* dqkv, int B, int S, int D, int H, hipStream_t s);
size_t attention_workspace_elems(int B, int S, int H);

// y[row] = wte[tok[row]] + wpe[row % S] (tables in the contraction dtype), and the table gradients
// (fp32; dwte cleared, then every occurring token's rows of dy added in row order, no atomic adds; dwpe summed over the batch).
hipError_t embedding_forward(int dtype, const int32_t* tok, const void* wte, const void* wpe, void* y,
                             int64_t rows, int S, int D, int vocab, hipStream_t s);
hipError_t embedding_backward(int dtype, const int32_t* tok, const void* dy, float* dwte, float* dwpe,
                              int64_t B, int S, int D, int vocab, hipStream_t s);

// Softmax cross-entropy of `rows` rows of fp32 logits: row_loss[rows] fp32 and
// dlogits[rows, C] = (softmax - onehot) * inv_M in the gradient dtype.
hipError_t softmax_ce(int dtype, const float* logits, const int32_t* labels, void* dlogits,
                      float* row_loss, int rows, int C, float inv_M, hipStream_t s);
// The same for few rows (softmax_ce_small_takes(rows of the loss, C)) in one workgroup, together with what else the loss layer hands out:
// y (may be null) a copy of the logits; loss_out (may be null) = scale times the sum of row_loss, whose first `before` values other
// passes have left there (this pass's rows follow them).
bool softmax_ce_small_takes(int64_t rows, int C);
hipError_t softmax_ce_small(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* y, float* row_loss, int rows,
                            int C, int before, float inv_M, float scale, float* loss_out, hipStream_t s);
// out[0] = scale * sum(in[0..n))   (deterministic single-block tree)
hipError_t reduce_scaled_sum(const float* in, int n, float scale, float* out, hipStream_t s);

// dz = y > 0 ? dy : 0
hipError_t relu_mask(int dtype, const void* dy, const void* y, void* dz, int64_t n, hipStream_t s);

// buf <- mu*buf + g;  w <- w - lr*buf;  wcopy <- bf16(w) when wcopy != null
hipError_t sgd_momentum(float* w, float* buf, const float* g, void* wcopy_bf16, int64_t n, float lr,
                        float mu, hipStream_t s);
// Up to kUpdateMax of them in one launch.
constexpr int kUpdateMax = 16;
struct Update {
    float* w;
    float* buf;
    const float* g;
    void* wcopy;
    int64_t n;
    float lr, mu;
};
hipError_t sgd_momentum_all(const Update* list, int n, hipStream_t s);
// The same; w and wcopy as they were before go to kept_w and kept_wcopy (arrays that overlap none of the others).
hipError_t sgd_momentum_keeping(float* w, float* buf, const float* g, void* wcopy_bf16, int64_t n, float lr, float mu,
                                float* kept_w, void* kept_wcopy, hipStream_t s);
hipError_t cast_f32_to_bf16(const float* in, void* out, int64_t n, hipStream_t s);
// dst[0..bytes) = src[0..bytes), both on the device, by a kernel
hipError_t copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t s);

}  // namespace tmps
