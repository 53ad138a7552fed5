// Instances of conv_first.hip.h and what they take.
#include "conv_first.hip.h"
#include "gemm_dispatch.hip.h"

namespace tmps {

// Forward pass and weight gradient with its slices' sum, on the tiled kernels and here (us): 3 x 3, 64 columns: 128 images of 32 x 32 14.3 / 20.7 and 7.8 / 12.7,
// 32 of them 6.5 / 12.9 and 4.5 / 11.2, 2 of them 6.2 / 9.6 and 4.0 / 8.8, 64 of 64 x 64 24.6 / 33 and 11.9 / 15.1, 64 of 8 x 8 5.9 / 10.6 and 3.9 / 8.9; 7 x 7,
// stride 2: 64 images of 224 x 224 118 / 158 and 54 / 76 (131 and 73 with an affine layer), 8 of them 22.7 / 32 and 14.8 / 24, 30 of 99 x 99 x 32 18.9 / 26 and
// 10.9 / 22.  The fixed part of a workgroup is larger with 49 taps: forward 16 images of 32 x 32 (32 tiles of 8 x 16 positions) 8.0 and 6.6, one (2 tiles)
// 5.4 and 6.4; weight gradient one image of 224 x 224 (98 tiles) 14.0 and 16.1, 16 of 32 x 32 (32) 11.3 and 12.4.
enum { kFirst3x3 = 1, kFirst7x7 = 2 };
int conv_first_kind(const ConvShape& c, bool wgrad) {
    if (c.Cin != 8 || c.Cout % 8 != 0 || c.R != c.S || !small_enough(c)) return 0;
    if (c.R == 3 && c.stride == 1) return kFirst3x3;
    const int64_t tiles = (int64_t)c.B * cdiv(c.Ho, 8) * cdiv(c.Wo, 16);
    return c.R == 7 && c.stride == 2 && tiles >= (wgrad ? kCUs : 16) ? kFirst7x7 : 0;
}

static ConvFirst first_of(const bf16_t* x, const bf16_t* o, const ConvShape& c) {
    ConvFirst cv;
    cv.x = x;
    cv.o = o;
    cv.H = c.H; cv.W = c.W; cv.Ho = c.Ho; cv.Wo = c.Wo; cv.N = c.Cout; cv.pad = c.pad;
    const int rows = cdiv(c.Ho, 8), cols = cdiv(c.Wo, 16);
    cv.tiles = c.B * rows * cols;
    cv.per = 0;
    cv.d_img = FastDiv(rows * cols);
    cv.d_row = FastDiv(cols);
    return cv;
}

// Two workgroups to a unit walk the tiles.
template <int R, int STRIDE, class Epi>
static hipError_t launch_first(const ConvFirst& cv, const Epi& epi, hipStream_t s) {
    constexpr int lds = conv_first_lds<R, R, STRIDE>();
    auto kern = conv_first_kernel<R, R, STRIDE, Epi>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    const int slots = 2 * kCUs;
    return launch_timed(kcConvFwd, kern, dim3(cv.tiles < slots ? cv.tiles : slots, cdiv(cv.N, 64)), dim3(256), lds, s, cv, epi);
}
template <class Epi> hipError_t conv_first(int kind, const bf16_t* x, const bf16_t* w, const Epi& epi, const ConvShape& c, hipStream_t s) {
    const ConvFirst cv = first_of(x, w, c);
    return kind == kFirst3x3 ? launch_first<3, 1>(cv, epi, s) : launch_first<7, 2>(cv, epi, s);
}
template hipError_t conv_first<EpiBiasAct<bf16_t>>(int, const bf16_t*, const bf16_t*, const EpiBiasAct<bf16_t>&, const ConvShape&, hipStream_t);
template hipError_t conv_first<EpiConvAffine<bf16_t>>(int, const bf16_t*, const bf16_t*, const EpiConvAffine<bf16_t>&, const ConvShape&, hipStream_t);

// Tiles of a workgroup of the weight gradient: as few as leave no more workgroups than the device has units.
static int first_wgrad_per(const ConvShape& c, int tiles) { return cdiv((int64_t)tiles * cdiv(c.Cout, 64), kCUs); }
int conv_first_wgrad_slices(const ConvShape& c) {
    const int tiles = first_of(nullptr, nullptr, c).tiles;
    return cdiv(tiles, first_wgrad_per(c, tiles));
}
template <int R, int STRIDE, int SETS>
static hipError_t launch_first_wgrad(const ConvFirst& cv, const EpiWgrad& epi, int slices, hipStream_t s) {
    constexpr int lds = conv_first_wgrad_lds<R, R, STRIDE>();
    auto kern = conv_first_wgrad_kernel<R, R, STRIDE, SETS>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    return launch_timed(kcConvWgrad, kern, dim3(slices, cdiv(cv.N, 64)), dim3(512), lds, s, cv, epi);
}
hipError_t conv_first_wgrad(int kind, const bf16_t* dy, const bf16_t* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    ConvFirst cv = first_of(x, dy, c);
    cv.per = first_wgrad_per(c, cv.tiles);
    const int slices = cdiv(cv.tiles, cv.per);
    const int64_t cols = (int64_t)c.R * c.S * 8, count = cols * c.Cout + c.Cout;
    const EpiWgrad epi{slices > 1 ? ws.ws : gw, cols, cols * c.Cout, count};
    const hipError_t e = kind == kFirst3x3 ? launch_first_wgrad<3, 1, 1>(cv, epi, slices, s) : launch_first_wgrad<7, 2, 4>(cv, epi, slices, s);
    if (e != hipSuccess || slices <= 1) return e;
    return ws.finish(Reduction{ws.ws, gw, count, slices, true}, s);
}

}  // namespace tmps
