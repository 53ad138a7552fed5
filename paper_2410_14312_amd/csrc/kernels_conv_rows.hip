// Instances of conv_rows.hip.h and the rule that chooses them.
#include <math.h>

#include "conv_rows.hip.h"
#include "conv_wgrad_rows.hip.h"
#include "gemm_dispatch.hip.h"

namespace tmps {

// LDS of a variant
static int rows_patch_bytes(int wm, const ConvShape& c) { return ((64 * wm + (c.R - 1) * c.W + c.S - 1) / 8 + 1) * 1024; }   // (a zero row behind the run)
static int rows_lds(int nw, int wm, int tn, int ns, const ConvShape& c, int C) {
    const int main = ns * (nw / wm) * tn * 4096 + (C > 64 ? 2 : 1) * rows_patch_bytes(wm, c), sums = nw * tn * 8192;
    return main > sums ? main : sums;
}

template <int NW, int WM, int TN, int NS, bool DGRAD, class Epi>
static hipError_t launch_rows(int kc, ConvRows cv, const Epi& epi, const ConvShape& c, hipStream_t s) {
    constexpr int BM = 64 * WM;
    cv.patch_rows = BM + (c.R - 1) * c.W + c.S - 1;
    cv.patch_bytes = rows_patch_bytes(WM, c);
    auto kern = conv_rows_kernel<NW, WM, TN, NS, DGRAD, Epi>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (attr != hipSuccess) return attr;
    const int tn = cdiv(cv.N, 32 * TN);
    return launch_timed(kc, kern, dim3(cdiv(cv.M, BM) * tn), dim3(64 * NW), rows_lds(NW, WM, TN, NS, c, cv.C), s, cv, epi, FastDiv(tn));
}

// Variants (waves, of them along the positions, stages of weights; in front, a 1 for tiles of 32 columns instead of 64), by what bounds their tiles:
//   443  256 positions, every wave all taps: the fewest copies of weights; two workgroups to a unit with one run of rows
//   422  128 positions, two groups of waves: two workgroups to a unit
//   823  128 positions, four groups: one workgroup with eight waves, for about as many tiles as units
//   413  64 positions, four groups: for fewer tiles than that
//  1413  the same in tiles of 32 columns, for at most half as many: twice the workgroups, with half as many copies, reads and multiplies in
//        a step each (3 x 3 over 512 channels, forward / input gradient, 413 and 1413, us: 128 images of 2 x 2 15.0 / 16.4 and 12.1 / 14.5, 64 of
//        4 x 4 15.5 / 16.3 and 12.5 / 14.8; over 256, 32 of 4 x 4 10.1 / 10.2 and 8.0 / 8.3; the gradient's copies are of 64 bytes in a row)
// Estimated time (us) of a variant: rounds of the device (a last round that is not full counts half way) times a fixed part
// (launch, the first copies, the sum of the groups' partial tiles, the epilogue) and the steps.  Fitted to 110 passes of 3 x 3 filters
// (55 shapes, 64 to 512 channels, 1 to 512 images of 2 x 2 to 56 x 56); the variant chosen is within 0.2 % of the best of the five on average, at worst 5 %.
static double rows_us(int variant, const ConvShape& c, int64_t M, int N, int C) {
    const int tn = variant > 1000 ? 1 : 2, nw = variant / 100 % 10, wm = variant / 10 % 10, ns = variant % 10;
    const int lds = rows_lds(nw, wm, tn, ns, c, C), kg = nw / wm;
    if (lds > kMaxLds) return 1e9;
    const int per_cu = nw == 4 && (wm > 1 || tn == 1) && 2 * lds <= kMaxLds ? 2 : 1;
    const double tiles = (double)cdiv(M, 64 * wm) * cdiv(N, 32 * tn), x = tiles / (kCUs * per_cu);
    const double rounds = x <= 1.0 ? 1.0 : 0.5 * (x + ceil(x)), steps = (double)cdiv((int64_t)C / 64 * c.R * c.S, kg);
    const bool shared = per_cu == 2 && tiles > kCUs;
    if (tn == 1 && tiles > 2 * kCUs) return 1e9;   // (a second round of half as much work each: never the best)
    double fixed, step;
    switch (variant) {
        case 1413: fixed = shared ? 3.4 : 3.9; step = shared ? 0.82 : 0.50; break;
        case 413: fixed = 4.8; step = 0.62; break;
        case 422: fixed = shared ? 6.3 : 4.5; step = shared ? 0.88 : 0.69; break;
        case 443: fixed = shared ? 8.0 : 6.8; step = shared ? 0.95 : 0.44; break;
        default: fixed = tiles > 0.95 * kCUs ? 8.5 : 6.0; step = 0.75; break;   // (a full round of them pays for copies that wait for each other)
    }
    return rounds * (fixed + step * steps);
}

int conv_rows_variant(const ConvShape& c, int64_t M, int N, int C, double other_us) {
    if (c.stride != 1 || c.R != 2 * c.pad + 1 || c.S != 2 * c.pad + 1 || c.R * c.S < 9 || c.R * c.S > 32 || C % 64 != 0 || N % 8 != 0 || !small_enough(c)) return 0;
    int best = 0;
    // What the other kernels' plan estimates is too low for convolutions: over 84 passes of 3 x 3 filters (42 shapes, 3 to 128 images of
    // 2 x 2 to 100 x 100, 64 to 512 channels) they took 0.8 to 2.1 times as long, quartiles 1.07, 1.34 and 1.45.  The factor stands here
    // because the choice among those kernels was fitted to the estimates as they are.  In the 110 passes above the best variant
    // took 0.41 to 0.95 of what they did.
    double best_us = 2.0 * other_us;
    for (int v : {1413, 413, 422, 443, 823}) {
        const double us = rows_us(v, c, M, N, C);
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
        case 413: return launch_rows<4, 1, 2, 3, DGRAD>(kc, cv, epi, c, s);
        case 1413: return launch_rows<4, 1, 1, 3, DGRAD>(kc, cv, epi, c, s);
        case 443: return launch_rows<4, 4, 2, 3, DGRAD>(kc, cv, epi, c, s);
        case 823: return launch_rows<8, 2, 2, 3, DGRAD>(kc, cv, epi, c, s);
        default: return launch_rows<4, 2, 2, 2, DGRAD>(kc, cv, epi, c, s);
    }
}
template hipError_t conv_rows<false, EpiBiasAct<bf16_t>>(int, int, const bf16_t*, const bf16_t*, const EpiBiasAct<bf16_t>&, const ConvShape&, hipStream_t);
template hipError_t conv_rows<false, EpiConvAffine<bf16_t>>(int, int, const bf16_t*, const bf16_t*, const EpiConvAffine<bf16_t>&, const ConvShape&, hipStream_t);
template hipError_t conv_rows<true, EpiMask<bf16_t, bf16_t>>(int, int, const bf16_t*, const bf16_t*, const EpiMask<bf16_t, bf16_t>&, const ConvShape&, hipStream_t);


// Weight gradients: the number of k-slices with the least estimated time, which is rounds of the device times a fixed part and 128 positions at a time, and
// what slices write and are added up for (5 TB/s).  Estimated, on this kernel and on the others (us): 128 images of 2 x 2 x 512 10.0, 10.6, 13.8, of
// 4 x 4 x 512 21, 22, 29, of 8 x 8 x 256 27, 26, 30, of 16 x 16 x 128 27, 28, 31, of 32 x 32 x 64 27, 28, 40; 64 images of 56 x 56 x 64 32, 34,
// 53, of 28 x 28 x 512 311, 300, 337; 8 of 7 x 7 x 512 10.0, 9.9, 12.6.  The other kernels' plan estimates up to 1.4 times
// too little (see conv_rows_variant); with 1.5 the one taken is within 3 % of the better one in 29 of 30 shapes, in the other one 9 % off (7.5 us against 6.9).
// A wave rounds a sum twice a chunk.  A slice has no more chunks than 64, which leaves its sums 2.75e-7 (2-norm) from those in 64 bits, or than make as many
// roundings as the other kernels' plan would.  Unlimited, the slice of 98 chunks that 64 images of 14 x 14 x 512 made and the one of 128 of 256
// images of 8 x 8 x 512 were 3.3 and 3.8e-7 off, the other kernels 2.7 and 3.0e-7; in four slices they are
// 1.6 and 1.8e-7 off and take no longer (103 and 118 us; in one 105 and 122).
static int64_t roundings(const Plan2& p, int64_t K) {
    const int chains = p.kind == kByK ? 4 : p.kind == kAsync || p.bm * p.bn == 4096 ? 2 : 1;   // waves or wave groups by k, alternating accumulators
    return cdiv(K, (int64_t)16 * p.slices * chains);
}
static int wgrad_run_groups(const ConvShape& c) { return (128 + 2 * c.W + 2 + 7) / 8; }

WgradRowsPlan conv_wgrad_rows_plan(const ConvShape& c, const Plan2& other) {
    WgradRowsPlan best{0, 0};
    if (c.R != 3 || c.S != 3 || c.stride != 1 || c.pad != 1 || c.Cin % 64 != 0 || c.Cout % 64 != 0 || !small_enough(c)) return best;
    if (conv_wgrad_rows_lds(wgrad_run_groups(c)) > kMaxLds) return best;
    const int64_t M = (int64_t)c.B * c.H * c.W, count = (int64_t)c.Cout * (9 * c.Cin + 1);
    const int64_t other_chunks = roundings(other, M) / 2, most = other_chunks > 64 ? other_chunks : 64;
    const int chunks = cdiv(M, 128), tiles = c.Cout / 64 * (c.Cin / 64) * 3;
    double best_us = 1e9;
    for (int s = 1; s <= 128 && s <= chunks; ++s) {
        const int per = cdiv(chunks, s);
        if (cdiv(chunks, per) != s || per > most) continue;
        const double us = cdiv((int64_t)tiles * s, kCUs) * (6.3 + 0.93 * per) + (s > 1 ? 3.5 + s * count * 8.0 / 5e6 : 0.0);
        if (us < best_us) {
            best_us = us;
            best = WgradRowsPlan{s, per * 128};
        }
    }
    return best_us < 1.5 * other.cost / 2400.0 ? best : WgradRowsPlan{0, 0};
}

hipError_t conv_wgrad_rows(const WgradRowsPlan& p, const bf16_t* dy, const bf16_t* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    ConvWgradRows cv;
    cv.dy = dy;
    cv.x = x;
    cv.M = c.B * c.H * c.W;
    cv.N = c.Cout; cv.C = c.Cin; cv.H = c.H; cv.W = c.W;
    cv.run_groups = wgrad_run_groups(c);
    cv.per_slice = p.per_slice;
    const int per_row = c.Cin / 64 * 3, tiles = c.Cout / 64 * per_row;
    cv.d_tiles = FastDiv(tiles);
    cv.d_row = FastDiv(per_row);
    cv.d_w = FastDiv(c.W);
    cv.d_h = FastDiv(c.H);
    const int64_t cols = (int64_t)9 * c.Cin, count = cols * c.Cout + c.Cout;
    const EpiWgrad epi{p.slices > 1 ? ws.ws : gw, cols, cols * c.Cout, count};
    const int lds = conv_wgrad_rows_lds(cv.run_groups);
    auto kern = conv_wgrad_rows_kernel<kWgradStages>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (attr != hipSuccess) return attr;
    hipError_t e = launch_timed(kcConvWgrad, kern, dim3(tiles * p.slices), dim3(512), lds, s, cv, epi);
    if (e != hipSuccess || p.slices <= 1) return e;
    return ws.finish(Reduction{ws.ws, gw, count, p.slices, false}, s);
}

}  // namespace tmps
