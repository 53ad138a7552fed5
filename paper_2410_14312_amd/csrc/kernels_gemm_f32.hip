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
