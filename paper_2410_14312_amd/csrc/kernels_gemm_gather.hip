// Contractions whose operands cannot be fetched in 16-byte chunks: convolutions over channel counts that are not whole
// chunks (an RGB image in fp32, where channels are not padded), matrices with rows of less than a chunk.  One source
// file for both types; the 64 x 64 instance of the tiled kernel with gathering loaders.
#include "gemm_dispatch.hip.h"

namespace tmps {

template <class T> static Gather<T, true, MatrixView<true>> mat_kc(const T* p, int rows, int K) { return {p, {rows, K, K}}; }
template <class T> static Gather<T, false, MatrixView<false>> mat_rc(const T* p, int rows, int K) { return {p, {rows, K, rows}}; }

template <class T, class Epi> hipError_t gather_dense_kc_kc(int kc, const T* a, const T* b, const Epi& epi, int M, int N, int K, float* ws, hipStream_t s) {
    return run2(kc, mat_kc(a, M, K), mat_kc(b, N, K), epi, M, N, K, ws, s);
}
template <class T> hipError_t gather_dense_dgrad(int kc, const T* dy, const T* w, const EpiMask<T, T>& epi, int M, int N, int K, float* ws, hipStream_t s) {
    return run2(kc, mat_kc(dy, M, K), mat_rc(w, N, K), epi, M, N, K, ws, s);
}
template <class T> hipError_t gather_dense_wgrad(int kc, const T* dy, const T* x, float* gw, int rows, int cols, int K, const Partials& ws, hipStream_t s) {
    return run2_wgrad(kc, mat_rc(dy, rows, K), mat_rc(x, cols, K), gw, rows, cols, K, ws, s);
}

template <class T, class Epi> hipError_t gather_conv_forward(const T* x, const T* w, const Epi& epi, const ConvShape& c, float* ws, hipStream_t s) {
    const int M = c.B * c.Ho * c.Wo, K = c.R * c.S * c.Cin;
    Gather<T, true, PatchView> A{x, {geom2(c), M, K}};
    if (K >= ElemTile<T>::V) return run2(kcConvFwd, A, RaggedKC<T>{w, c.Cout, K, K}, epi, M, c.Cout, K, ws, s);
    return run2(kcConvFwd, A, mat_kc(w, c.Cout, K), epi, M, c.Cout, K, ws, s);
}
template <class T> hipError_t gather_conv_dgrad(const T* dy, const T* w, const EpiMask<T, T>& epi, const ConvShape& c, float* ws, hipStream_t s) {
    const int M = c.B * c.H * c.W, K = c.R * c.S * c.Cout;
    Gather<T, true, BackPatchView> A{dy, {geom2(c), M, K}};
    Gather<T, false, BackTapView> B{w, {geom2(c), c.Cin, K}};
    return run2(kcConvDgrad, A, B, epi, M, c.Cin, K, ws, s);
}
template <class T> hipError_t gather_conv_wgrad(const T* dy, const T* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    const int rows = c.Cout, cols = c.R * c.S * c.Cin, K = c.B * c.Ho * c.Wo;
    Gather<T, false, TapView> B{x, {{geom2(c), K, cols}}};
    if (rows >= ElemTile<T>::V) return run2_wgrad(kcConvWgrad, RaggedRC<T>{dy, rows, K, rows}, B, gw, rows, cols, K, ws, s);
    return run2_wgrad(kcConvWgrad, mat_rc(dy, rows, K), B, gw, rows, cols, K, ws, s);
}

#define TMPS_GATHER(T)                                                                                                                     \
    template hipError_t gather_dense_dgrad<T>(int, const T*, const T*, const EpiMask<T, T>&, int, int, int, float*, hipStream_t);           \
    template hipError_t gather_dense_wgrad<T>(int, const T*, const T*, float*, int, int, int, const Partials&, hipStream_t);                        \
    template hipError_t gather_dense_kc_kc<T, EpiBiasAct<T>>(int, const T*, const T*, const EpiBiasAct<T>&, int, int, int, float*, hipStream_t); \
    template hipError_t gather_conv_forward<T, EpiBiasAct<T>>(const T*, const T*, const EpiBiasAct<T>&, const ConvShape&, float*, hipStream_t); \
    template hipError_t gather_conv_forward<T, EpiConvAffine<T>>(const T*, const T*, const EpiConvAffine<T>&, const ConvShape&, float*, hipStream_t); \
    template hipError_t gather_conv_dgrad<T>(const T*, const T*, const EpiMask<T, T>&, const ConvShape&, float*, hipStream_t);              \
    template hipError_t gather_conv_wgrad<T>(const T*, const T*, float*, const ConvShape&, const Partials&, hipStream_t);
TMPS_GATHER(float)
TMPS_GATHER(bf16_t)
template hipError_t gather_dense_kc_kc<bf16_t, EpiBiasAct<float>>(int, const bf16_t*, const bf16_t*, const EpiBiasAct<float>&, int, int, int, float*, hipStream_t);

}  // namespace tmps
