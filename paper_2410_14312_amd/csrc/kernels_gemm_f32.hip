// fp32 instances of the contractions (dense and convolution, forward and both gradients).
#include "gemm_dispatch.hip.h"

namespace tmps {

hipError_t dense_forward_f32(int kc, const float* x, const float* w, const EpiBiasAct<float>& epi, int B, int Din, int Dout, float* ws, hipStream_t s) {
    return dense_forward_t<float>(kc, x, w, epi, B, Din, Dout, ws, s);
}
bool norm_dense_takes_f32(int64_t rows, int D, int N) { return norm_dense_takes<float>(rows, D, N); }
hipError_t norm_dense_f32(const float* x, const float* gamma, const float* beta, float* y, float* stats, const float* w, const EpiBiasAct<float>& epi, int M, int N,
                          int D, float eps, hipStream_t s) {
    return norm_dense_small<float>(kcDenseFwd, x, gamma, beta, y, stats, w, epi, M, N, D, eps, s);
}
hipError_t dense_dgrad_f32(int kc, const float* dy, const float* w, const EpiMask<float, float>& epi, int B, int Din, int Dout, float* ws, hipStream_t s) {
    return dense_dgrad_t<float>(kc, dy, w, epi, B, Din, Dout, ws, s);
}
hipError_t dense_wgrad_f32(int kc, const float* dy, const float* x, float* gw, int B, int Din, int Dout, const Partials& ws, hipStream_t s) {
    return dense_wgrad_t<float>(kc, dy, x, gw, B, Din, Dout, ws, s);
}
hipError_t small_backward_f32(int kc, const float* dy, const float* x, const float* w, float* gw, const EpiMask<float, float>& epi, int B, int Din, int Dout, hipStream_t s) {
    return small_backward_t<float>(kc, dy, x, w, gw, epi, B, Din, Dout, s);
}
// Both gradients of a dense layer in one launch where dx is few outputs over a long contraction and gw many over a short one: dx on the small kernel's 32 x 32
// tiles (the first `split` workgroups), gw on 64 x 64 tiles of the tiled kernel, which share the compute units with them.
// Each is bound by the latency of its own loads and barriers, a third to a half of the multiplies' rate; together they fill each other's gaps: 235 x 1000 -> 1000
// 11.9 + 10.9 us as two launches, 7 less as one (6.4 at the rate of the multiplies).
__global__ __launch_bounds__(256, 3) void gemm_mixed_backward_kernel(const float* dy, const float* x, const float* w, EpiMask<float, float> ex, EpiWgrad ew, int rows,
                                                                     int Din, int Dout, int split, FastDiv d_x, FastDiv d_n, FastDiv d_w, int wide) {
    const int b = blockIdx.x;
    uint32_t by, bx;
    if (b < split) {
        d_x.divmod((uint32_t)b, by, bx);
        gemm_small_tile<4, 2, 2, false>(SmallOperand<float, true>{dy, rows, Dout}, SmallOperand<float, false>{w, Din, Din}, ex, rows, Din, Dout, (int)bx, (int)by);
    } else {
        d_n.divmod((uint32_t)(b - split), by, bx);
        gemm2_tile<64, 64, 2, true>(DenseRC<float>{dy, Dout, rows, Dout}, DenseRC<float>{x, Din, rows, Din}, ew, Dout, Din, rows, rows, 0, wide, d_w, d_n, (int)bx,
                                    (int)by, 0, (int)d_n.d, (Dout + 63) >> 6, 1);
    }
}
hipError_t mixed_backward_f32(int kc, const float* dy, const float* x, const float* w, float* gw, const EpiMask<float, float>& epi, int B, int Din, int Dout, hipStream_t s) {
    const EpiWgrad ew{gw, Din, (int64_t)Dout * Din, 0};
    constexpr int lx = small_lds_floats(4, 2, 2) * 4, lw = gemm2_lds_bytes<64, 64, DenseRC<float>, DenseRC<float>>();
    const int nx = cdiv(Din, 32), split = nx * cdiv(B, 32), nw = cdiv(Din, 64), tw = nw * cdiv(Dout, 64);
    return launch_timed(kc, gemm_mixed_backward_kernel, dim3(split + tw), dim3(256), lx > lw ? lx : lw, s, dy, x, w, epi, ew, B, Din, Dout, split, FastDiv(nx),
                        FastDiv(nw), FastDiv(tw), Din % 8 == 0 && ew.wide_ok() ? 1 : 0);
}
hipError_t conv_forward_f32(const float* x, const float* w, const EpiBiasAct<float>& epi, const ConvShape& c, float* ws, hipStream_t s) {
    if (pointwise(c)) return dense_forward_t<float>(kcConvFwd, x, w, epi, c.B * c.H * c.W, c.Cin, c.Cout, ws, s);
    return conv_forward_t<float>(x, w, epi, c, ws, s);
}
hipError_t conv_affine_f32(const float* x, const float* w, const EpiConvAffine<float>& epi, const ConvShape& c, float* ws, hipStream_t s) {
    const int M = c.B * c.Ho * c.Wo;
    if (pointwise(c) && c.Cin % 4 == 0 && aligned16(x) && aligned16(w))
        return run2(kcConvFwd, DenseKC<float>{x, M, c.Cin, c.Cin}, DenseKC<float>{w, c.Cout, c.Cin, c.Cin}, epi, M, c.Cout, c.Cin, ws, s);
    return conv_forward_t<float>(x, w, epi, c, ws, s);
}
hipError_t conv_dgrad_f32(const float* dy, const float* w, const EpiMask<float, float>& epi, const ConvShape& c, float* ws, hipStream_t s) {
    if (pointwise(c)) return dense_dgrad_t<float>(kcConvDgrad, dy, w, epi, c.B * c.H * c.W, c.Cin, c.Cout, ws, s);
    return conv_dgrad_t<float>(dy, w, epi, c, ws, s);
}
hipError_t conv_wgrad_f32(const float* dy, const float* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    if (pointwise(c)) return dense_wgrad_t<float>(kcConvWgrad, dy, x, gw, c.B * c.H * c.W, c.Cin, c.Cout, ws, s);
    return conv_wgrad_t<float>(dy, x, gw, c, ws, s);
}

}  // namespace tmps
