// Instances of conv_rows.hip.h and the rule that chooses them.
#include <math.h>

#include "conv_rows.hip.h"
#include "gemm_dispatch.hip.h"

namespace tmps {

// LDS of a variant
static int rows_patch_bytes(int wm, const ConvShape& c) { return ((64 * wm + (c.R - 1) * c.W + c.S - 1) / 8 + 1) * 1024; }   // (a zero row behind the run)
static int rows_lds(int nw, int wm, int ns, const ConvShape& c, int C) {
    const int main = ns * (nw / wm) * 8192 + (C > 64 ? 2 : 1) * rows_patch_bytes(wm, c);
    return main > nw * 16384 ? main : nw * 16384;
}

template <int NW, int WM, int NS, bool DGRAD, class Epi>
static hipError_t launch_rows(int kc, ConvRows cv, const Epi& epi, const ConvShape& c, hipStream_t s) {
    constexpr int BM = 64 * WM;
    cv.patch_rows = BM + (c.R - 1) * c.W + c.S - 1;
    cv.patch_bytes = rows_patch_bytes(WM, c);
    auto kern = conv_rows_kernel<NW, WM, NS, DGRAD, Epi>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (attr != hipSuccess) return attr;
    const int tn = cdiv(cv.N, 64);
    return launch_timed(kc, kern, dim3(cdiv(cv.M, BM) * tn), dim3(64 * NW), rows_lds(NW, WM, NS, c, cv.C), s, cv, epi, FastDiv(tn));
}

// Variants (waves, of them along the positions, stages of weights), by what bounds their tiles:
//   443  256 positions, every wave all taps: the fewest copies of weights; two workgroups to a unit with one run of rows
//   422  128 positions, two groups of waves: two workgroups to a unit
//   823  128 positions, four groups: one workgroup with eight waves, for about as many tiles as units
//   413  64 positions, four groups: for fewer tiles than that
// Estimated time (us) of a variant: rounds of the device (a last round that is not full counts half way) times a fixed part
// (launch, the first copies, the sum of the groups' partial tiles, the epilogue) and the steps.  Fitted to 3 x 3 filters over 64 to 512
// channels and 1 to 300 images of 2 x 2 to 224 x 224; the variant chosen is within 5 % of the best almost everywhere.
static double rows_us(int nw, int wm, int ns, const ConvShape& c, int64_t M, int N, int C) {
    const int lds = rows_lds(nw, wm, ns, c, C), kg = nw / wm;
    if (lds > kMaxLds) return 1e9;
    const int per_cu = nw == 4 && wm > 1 && 2 * lds <= kMaxLds ? 2 : 1;
    const double tiles = (double)cdiv(M, 64 * wm) * cdiv(N, 64), x = tiles / (kCUs * per_cu);
    const double rounds = x <= 1.0 ? 1.0 : 0.5 * (x + ceil(x)), steps = (double)cdiv((int64_t)C / 64 * c.R * c.S, kg);
    const bool shared = per_cu == 2 && tiles > kCUs;
    const double fixed = wm == 1 ? 5.0 : nw == 8 ? 6.0 : wm == 4 ? (shared ? 8.0 : 5.0) : (shared ? 7.0 : 3.0);
    const double step = wm == 1 ? 0.68 : nw == 8 ? 0.88 : wm == 4 ? (shared ? 1.1 : 0.75) : 0.9;
    return rounds * (fixed + step * steps);
}

int conv_rows_variant(const ConvShape& c, int64_t M, int N, int C, double other_us) {
    if (c.stride != 1 || c.R != 2 * c.pad + 1 || c.S != 2 * c.pad + 1 || c.R * c.S < 9 || c.R * c.S > 32 || C % 64 != 0 || N % 8 != 0 || !small_enough(c)) return 0;
    int best = 0;
    // What the other kernels' plan estimates is too low for convolutions: over 84 passes of 3 x 3 filters (42 shapes, 3 to 128 images of
    // 2 x 2 to 100 x 100, 64 to 512 channels) they took 0.8 to 2.1 times as long, quartiles 1.07, 1.34 and 1.45.  The factor stands here
    // because the choice among those kernels was fitted to the estimates as they are.  With it the kernel taken was within 1 % of the
    // best one in nine passes of ten, at worst 16 % off (64 images of 2 x 2 x 512: 18.6 us against 16.1).
    double best_us = 1.3 * other_us;
    for (int v : {413, 422, 443, 823}) {
        const double us = rows_us(v / 100, v / 10 % 10, v % 10, c, M, N, C);
        if (us < best_us) {
            best_us = us;
            best = v;
        }
    }
    return best;
}

template <bool DGRAD, class Epi>
hipError_t conv_rows(int variant, int kc, const bf16_t* x, const bf16_t* w, const Epi& epi, const ConvShape& c, hipStream_t s) {
    ConvRows cv;
    cv.x = x;
    cv.w = w;
    cv.M = c.B * c.H * c.W;
    cv.N = DGRAD ? c.Cin : c.Cout;
    cv.C = DGRAD ? c.Cout : c.Cin;
    cv.H = c.H; cv.W = c.W; cv.S = c.S; cv.RS = c.R * c.S; cv.pad = c.pad;
    cv.two = cv.C > 64 ? 1 : 0;
    cv.d_hw = FastDiv(c.H * c.W);
    cv.d_w = FastDiv(c.W);
    cv.d_s = FastDiv(c.S);
    switch (variant) {
        case 413: return launch_rows<4, 1, 3, DGRAD>(kc, cv, epi, c, s);
        case 443: return launch_rows<4, 4, 3, DGRAD>(kc, cv, epi, c, s);
        case 823: return launch_rows<8, 2, 3, DGRAD>(kc, cv, epi, c, s);
        default: return launch_rows<4, 2, 2, DGRAD>(kc, cv, epi, c, s);
    }
}
template hipError_t conv_rows<false, EpiBiasAct<bf16_t>>(int, int, const bf16_t*, const bf16_t*, const EpiBiasAct<bf16_t>&, const ConvShape&, hipStream_t);
template hipError_t conv_rows<false, EpiConvAffine<bf16_t>>(int, int, const bf16_t*, const bf16_t*, const EpiConvAffine<bf16_t>&, const ConvShape&, hipStream_t);
template hipError_t conv_rows<true, EpiMask<bf16_t, bf16_t>>(int, int, const bf16_t*, const bf16_t*, const EpiMask<bf16_t, bf16_t>&, const ConvShape&, hipStream_t);

}  // namespace tmps
