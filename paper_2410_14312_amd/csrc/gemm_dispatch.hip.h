// Dispatch of the contractions, written once for bf16 and fp32 operands and instantiated in one source file per type
// (kernels_gemm.hip, kernels_gemm_f32.hip; the gathering bf16 instances in kernels_gemm_gather.hip): tile sizes and
// k-splits, the choice between the kernels, and the dense and convolution passes in terms of them.
#pragma once
#include <hip/hip_ext.h>

#include "gemm5.hip.h"
#include "gemm_small.hip.h"
#include "kernels.h"
#include "launch.h"
#include "profile.h"

namespace tmps {

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// What a contraction runs on: the tiled kernel with a tile shape, the k-sharing kernel (64 x 64) or the 128 x 128 kernel with
// asynchronous copies, and k-slices.
enum { kTiled = 0, kByK, kAsync };
struct Plan2 {
    int bm, bn, slices, kind;
    double cost;   // estimated cycles (2.4 GHz)
};

constexpr int kCUs = 256;   // compute units of the device the rules below are written for

// ---- plans ----------------------------------------------------------------------------------------
// The plan of least estimated time for the tiled kernel alone (kByKNo) or for it and the kernels with asynchronous copies, on matrices
// or with an operand that a convolution's loader addresses.  esize: bytes of an operand element.
enum { kByKNo = 0, kByKDense, kByKConv };
Plan2 plan_for(int64_t M, int64_t N, int64_t K, bool rowsum, int esize, int by_k);
// Tiles (16 tm x 16 tn) of the small kernel (gemm_small.hip.h) for a contraction and its estimated cycles; whether a dense contraction
// runs on it rather than by the given plan.
struct SmallPlan {
    int tm, tn;
    double cost;
};
SmallPlan small_plan(int64_t M, int64_t N, int64_t K, int esize);
bool small_is_better(int64_t M, int64_t N, int64_t K, int esize, const Plan2& other);

// slice length (whole k-tiles) and the number of slices really launched
static void slice_geometry(int64_t K, int want, int ktile, int& per, int& nz) {
    if (want < 1) want = 1;
    per = cdiv(cdiv(K, want), ktile) * ktile;
    if (per < ktile) per = ktile;
    nz = K > 0 ? cdiv(K, per) : 1;
}


// (gathering loaders put a chunk together from eight or four loads: one small tile, a short ring)
template <class Op> struct IsGather { static constexpr bool value = false; };
template <class T, bool KC, class View> struct IsGather<Gather<T, KC, View>> { static constexpr bool value = true; };

// how the k-sharing kernel can take a pair of loaders (it needs a chunk's address)
template <class Op> struct IsMatrix { static constexpr bool value = false; };
template <class T> struct IsMatrix<DenseKC<T>> { static constexpr bool value = true; };
template <class T> struct IsMatrix<DenseRC<T>> { static constexpr bool value = true; };
template <class T> struct IsMatrix<StridedKC<T>> { static constexpr bool value = true; };
template <class Op> constexpr bool has_addr() { return !IsGather<Op>::value && !Op::kSettle; }
template <class AOp, class BOp> constexpr int by_k_mode() {
    return !has_addr<AOp>() || !has_addr<BOp>() ? kByKNo : IsMatrix<AOp>::value && IsMatrix<BOp>::value ? kByKDense : kByKConv;
}

// ---- launches -------------------------------------------------------------------------------------
// How the XCDs share the tiles of a launch (xcd_tile) and what its d_minor divides by.  Strips: the XCDs split the operand with more rows between
// them and each reads the other one whole.  Rectangles where tiles divide evenly and an XCD's share of both operands has fewer rows than that (matrices only:
// rows of a convolution's operand overlap in memory).
struct XcdOrder {
    int order, minor;
};
static XcdOrder xcd_order(int gx, int gy, int nz, int64_t M, int64_t N, bool matrices) {
    XcdOrder o = N > M ? XcdOrder{1, gy} : XcdOrder{0, gx};
    if (!matrices || nz != 1) return o;
    int64_t best = N > M ? M + N / 8 : N + M / 8;
    for (int lb = 1; lb <= 2; ++lb) {
        const int64_t rows = M / (8 >> lb) + N / (1 << lb);
        if (gx % (1 << lb) == 0 && gy % (8 >> lb) == 0 && rows < best) {
            best = rows;
            o = XcdOrder{2 + lb, gx >> lb};
        }
    }
    return o;
}

template <int BM, int BN, int D, bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t launch2_inst(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int per,
                               int nz, hipStream_t s) {
    constexpr int lds = gemm2_lds_bytes<BM, BN, AOp, BOp>();
    auto kern = gemm2_kernel<BM, BN, D, ROWSUM, AOp, BOp, Epi>;
    if (lds > 64 * 1024) {
        // more LDS than the default per-workgroup limit: raise it once per kernel instance
        static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (attr != hipSuccess) return attr;
    }
    dim3 grid(cdiv(N, BN), cdiv(M, BM), nz);
    const XcdOrder o = xcd_order(grid.x, grid.y, nz, M, N, by_k_mode<AOp, BOp>() == kByKDense);
    return launch_timed(kc, kern, grid, dim3(256), lds, s, A, B, epi, M, N, K, per, o.order,
                        (N % 8 == 0 && epi.wide_ok()) ? 1 : 0, FastDiv(grid.x * grid.y), FastDiv(o.minor));
}


// f(epi) with the epilogue as its form's type where it has one
template <int F = 0, class Epi, class Fn> static hipError_t with_form(int form, const Epi& epi, Fn&& f) {
    if constexpr (F < Epi::kForms) return form == F ? f(EpiForm<Epi, F>{epi}) : with_form<F + 1>(form, epi, f);
    else return f(epi);
}

template <bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t launch4_form(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int per, int nz, hipStream_t s) {
    auto kern = gemm4_kernel<ROWSUM, AOp, BOp, Epi>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kGemm4Lds);
    if (attr != hipSuccess) return attr;
    dim3 grid(cdiv(N, 64), cdiv(M, 64), nz);
    const XcdOrder o = xcd_order(grid.x, grid.y, nz, M, N, by_k_mode<AOp, BOp>() == kByKDense);
    return launch_timed(kc, kern, grid, dim3(256), kGemm4Lds, s, A, B, epi, M, N, K, per, o.order, (N % 8 == 0 && epi.wide_ok()) ? 1 : 0,
                        FastDiv(grid.x * grid.y), FastDiv(o.minor));
}


template <bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t launch4(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int per, int nz, hipStream_t s) {
    if constexpr (sizeof(typename AOp::T) == 2 && by_k_mode<AOp, BOp>() == kByKDense && Epi::kForms > 1) {
        if (N % 8 == 0 && epi.wide_ok())
            return with_form(epi.form(), epi, [&](const auto& e) { return launch4_form<ROWSUM>(kc, A, B, e, M, N, K, per, nz, s); });
    }
    return launch4_form<ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
}

template <bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t launch5_form(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int per, int nz, hipStream_t s) {
    constexpr int lds = kGemm5Lds;
    auto kern = gemm5_kernel<ROWSUM, AOp, BOp, Epi>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    dim3 grid(cdiv(N, 128), cdiv(M, 128), nz);
    const XcdOrder o = xcd_order(grid.x, grid.y, nz, M, N, by_k_mode<AOp, BOp>() == kByKDense);
    return launch_timed(kc, kern, grid, dim3(64 * kGemm5Waves), lds, s, A, B, epi, M, N, K, per, o.order, FastDiv(grid.x * grid.y), FastDiv(o.minor));
}

// (dense layers' epilogues in their forms, as the persistent kernel has them)
template <bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t launch5(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int per, int nz, hipStream_t s) {
    if constexpr (by_k_mode<AOp, BOp>() == kByKDense && Epi::kForms > 1)
        return with_form(epi.form(), epi, [&](const auto& e) { return launch5_form<ROWSUM>(kc, A, B, e, M, N, K, per, nz, s); });
    else return launch5_form<ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
}

template <bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t launch2_tile(int kc, const Plan2& p, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int per,
                               int nz, hipStream_t s) {
    if constexpr (IsGather<AOp>::value || IsGather<BOp>::value) return launch2_inst<64, 64, 1, ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
    else {
        if constexpr (by_k_mode<AOp, BOp>() != kByKNo) {
            if (p.kind == kByK) return launch4<ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
            if constexpr (sizeof(typename AOp::T) == 2) {
                // (its epilogue has only the 16-byte form)
                if (p.kind == kAsync && N % 8 == 0 && epi.wide_ok()) return launch5<ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
            }
        }
        if (p.bm == 128 && p.bn == 128) return launch2_inst<128, 128, 2, ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
        if constexpr (!ROWSUM && !AOp::kSettle) {
            if (p.bm == 128) return launch2_inst<128, 64, 2, false>(kc, A, B, epi, M, N, K, per, nz, s);
        }
        // (fp32: a k-tile is multiplied for 1000 cycles, and two in flight are enough; ragged operands: no registers for four)
        constexpr int D = sizeof(typename AOp::T) == 4 || AOp::kSettle ? 2 : 4;
        return launch2_inst<64, 64, D, ROWSUM>(kc, A, B, epi, M, N, K, per, nz, s);
    }
}

// Forward / input-gradient style GEMM: epilogue `epi` applied once per output element.
// tile: 0 = the plan's choice, else the edge of the square tiles to use (the slices stay the plan's)
template <class AOp, class BOp, class Epi>
static hipError_t run2(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, float* ws, hipStream_t s, int tile = 0) {
    typedef typename AOp::T T;
    if (M <= 0 || N <= 0) return hipSuccess;
    Plan2 p = plan_for(M, N, K, false, sizeof(T), by_k_mode<AOp, BOp>());
    if (tile && p.kind != kByK) {
        if (tile != p.bm) p.kind = kTiled;
        p.bm = p.bn = tile;
    }
    int per, nz;
    slice_geometry(K, ws ? p.slices : 1, ElemTile<T>::BK, per, nz);
    if (nz <= 1) return launch2_tile<false>(kc, p, A, B, epi, M, N, K, per, nz, s);
    EpiPartial part{ws, N, (int64_t)M * N};
    hipError_t e = launch2_tile<false>(kc, p, A, B, part, M, N, K, per, nz, s);
    if (e != hipSuccess) return e;
    int64_t total = (int64_t)M * N;
    if (N % 8 == 0 && epi.wide_ok() && aligned16(ws))
        return launch_timed(kcSplitFinish, splitk_finish8_kernel<Epi, SameRows>, dim3(cdiv(total / 8, 256)), dim3(256), 0, s,
                            (const float*)ws, epi, M, N, nz, SameRows{});
    return launch_timed(kcSplitFinish, splitk_finish_kernel<Epi>, dim3(cdiv(total, 256)), dim3(256), 0, s,
                        (const float*)ws, epi, M, N, nz);
}

// The same of rows that lie apart in the result (every tensor of the epilogue 16-byte aligned, N a multiple of 8).
template <class T, class BOp, class Epi>
static hipError_t run2_strided(int kc, const StridedKC<T>& A, const BOp& B, const Epi& epi, int M, int N, int K, float* ws, hipStream_t s) {
    const Plan2 p = plan_for(M, N, K, false, sizeof(T), by_k_mode<StridedKC<T>, BOp>());
    int per, nz;
    slice_geometry(K, aligned16(ws) && ws ? p.slices : 1, ElemTile<T>::BK, per, nz);
    if (nz <= 1) return launch2_tile<false>(kc, p, A, B, epi, M, N, K, per, nz, s);
    const hipError_t e = launch2_tile<false>(kc, p, static_cast<const DenseKC<T>&>(A), B, EpiPartial{ws, N, (int64_t)M * N}, M, N, K, per, nz, s);
    if (e != hipSuccess) return e;
    return launch_timed(kcSplitFinish, splitk_finish8_kernel<Epi, StridedKC<T>>, dim3(cdiv((int64_t)M * N / 8, 256)), dim3(256), 0, s, (const float*)ws, epi, M, N, nz, A);
}

// Weight-gradient style GEMM: fp32 result [rows x cols] followed by the row sums of A (bias gradient).
template <class AOp, class BOp>
static hipError_t run2_wgrad(int kc, const AOp& A, const BOp& B, float* gw, int rows, int cols, int64_t K, const Partials& ws, hipStream_t s) {
    typedef typename AOp::T T;
    const Plan2 p = plan_for(rows, cols, K, true, sizeof(T), by_k_mode<AOp, BOp>());
    int per, nz;
    slice_geometry(K, ws.ws ? p.slices : 1, ElemTile<T>::BK, per, nz);
    int64_t count = (int64_t)rows * cols + rows;
    EpiWgrad epi{nz > 1 ? ws.ws : gw, cols, (int64_t)rows * cols, count};
    hipError_t e = launch2_tile<true>(kc, p, A, B, epi, rows, cols, (int)K, per, nz, s);
    if (e != hipSuccess || nz <= 1) return e;
    return ws.finish(Reduction{ws.ws, gw, count, nz, false}, s);
}

// Small kernel: eight waves; four for a contraction of at most four steps and for 32 x 32 outputs in fp32 (256 x 1024 x 1024 10.3 us against 10.9).
template <int NW, int TM, int TN, bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t small_inst(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, hipStream_t s) {
    return launch_timed(kc, gemm_small_kernel<NW, TM, TN, ROWSUM, AOp, BOp, Epi>, dim3(cdiv(N, 16 * TN), cdiv(M, 16 * TM)), dim3(64 * NW),
                        small_lds_floats(NW, TM, TN) * 4, s, A, B, epi, M, N, K);
}
template <bool ROWSUM, class AOp, class BOp, class Epi>
static hipError_t run_small(int kc, const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, hipStream_t s) {
    const SmallPlan p = small_plan(M, N, K, sizeof(typename AOp::T));
    constexpr int esize = sizeof(typename AOp::T);
    if (p.tm == 2 && (esize == 4 || K <= 4 * (64 / esize))) return small_inst<4, 2, 2, ROWSUM>(kc, A, B, epi, M, N, K, s);
    if (K <= 4 * (64 / esize)) {
        if (p.tn == 2) return small_inst<4, 1, 2, ROWSUM>(kc, A, B, epi, M, N, K, s);
        return small_inst<4, 1, 1, ROWSUM>(kc, A, B, epi, M, N, K, s);
    }
    if (p.tm == 2) return small_inst<8, 2, 2, ROWSUM>(kc, A, B, epi, M, N, K, s);
    if (p.tn == 2) return small_inst<8, 1, 2, ROWSUM>(kc, A, B, epi, M, N, K, s);
    return small_inst<8, 1, 1, ROWSUM>(kc, A, B, epi, M, N, K, s);
}

// A layer normalisation and the dense layer behind it on the small kernel: rows of one piece to a lane, a contraction that four waves share in one step
// each, and a dense layer that this kernel takes in 16 x 16 tiles by itself.
// Forward and backward pass of both layers, bound by their launches, in two launches and in one (us): bf16, 64 -> 192 over 16, 64 and 256 rows 20.9 / 22.0 / 20.3 and
// 18.7 / 19.6 / 18.3, 32 -> 32 over 2048 rows 21.0 and 18.8, 128 -> 512 over 64 rows 20.3 and 18.0; fp32 64 -> 192 20.3 / 20.5 / 20.0 and 18.9 / 18.2 / 17.5, 64 -> 4096 over 16
// rows 26.2 and 23.7.  The line, where the dense layer alone moves to larger tiles, is on the safe side: in 16 x 16 tiles all the same one launch would take 19.5 for 21.3 (fp32
// 64 -> 192 over 512 rows), 19.3 for 21.1 (bf16 64 -> 256 over 1024), 20.9 for 21.4 (bf16 64 -> 64 over 2048).
template <class T> static bool norm_dense_takes(int64_t rows, int D, int N) {
    constexpr int esize = sizeof(T);
    if (D % 8 != 0 || D > 4 * (64 / esize) || !small_is_better(rows, N, D, esize, plan_for(rows, N, D, false, esize, kByKDense))) return false;
    const SmallPlan p = small_plan(rows, N, D, esize);
    return p.tm == 1 && p.tn == 1;
}
template <class T, class Epi>
static hipError_t norm_dense_small(int kc, const T* x, const float* gamma, const float* beta, T* y, float* stats, const T* w, const Epi& epi, int M, int N, int D,
                                   float eps, hipStream_t s) {
    const int lds = small_lds_floats(kNormWaves, 1, 1) * 4 + 16 * small_norm_ld<T>(D) * (int)sizeof(T);
    return launch_timed(kc, norm_dense_small_kernel<T, Epi>, dim3(cdiv(N, 16), cdiv(M, 16)), dim3(64 * kNormWaves), lds, s, x, gamma, beta, y, stats, w, epi, M, N, D, eps);
}

// ---- element-wise gathering instances (kernels_gemm_gather.hip, both types) ------------------------------
template <class T, class Epi> hipError_t gather_dense_kc_kc(int kc, const T* a, const T* b, const Epi& epi, int M, int N, int K, float* ws, hipStream_t s);
template <class T> hipError_t gather_dense_dgrad(int kc, const T* dy, const T* w, const EpiMask<T, T>& epi, int M, int N, int K, float* ws, hipStream_t s);
template <class T> hipError_t gather_dense_wgrad(int kc, const T* dy, const T* x, float* gw, int rows, int cols, int K, const Partials& ws, hipStream_t s);
template <class T, class Epi> hipError_t gather_conv_forward(const T* x, const T* w, const Epi& epi, const ConvShape& c, float* ws, hipStream_t s);
template <class T> hipError_t gather_conv_dgrad(const T* dy, const T* w, const EpiMask<T, T>& epi, const ConvShape& c, float* ws, hipStream_t s);
template <class T> hipError_t gather_conv_wgrad(const T* dy, const T* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s);

static inline ConvGeom2 geom2(const ConvShape& c) {
    ConvGeom2 g;
    g.B = c.B; g.H = c.H; g.W = c.W; g.Cin = c.Cin; g.Ho = c.Ho; g.Wo = c.Wo; g.Cout = c.Cout;
    g.R = c.R; g.S = c.S; g.stride = c.stride; g.pad = c.pad;
    g.d_howo = FastDiv(c.Ho * c.Wo); g.d_wo = FastDiv(c.Wo);
    g.d_hw = FastDiv(c.H * c.W); g.d_w = FastDiv(c.W);
    g.d_scin = FastDiv(c.S * c.Cin); g.d_cin = FastDiv(c.Cin);
    g.d_scout = FastDiv(c.S * c.Cout); g.d_cout = FastDiv(c.Cout);
    g.d_stride = FastDiv(c.stride);
    return g;
}

// ---- dense passes (without the persistent kernel) -----------------------------------------------------
// Rows in whole 16-byte chunks take the plain loaders, ragged ones of a chunk or more the ragged loaders, the rest is gathered.
template <class T, class Epi>
static hipError_t dense_forward_t(int kc, const T* x, const T* w, const Epi& epi, int B, int Din, int Dout, float* ws, hipStream_t s) {
    constexpr int V = ElemTile<T>::V;
    if (small_is_better(B, Dout, Din, sizeof(T), plan_for(B, Dout, Din, false, sizeof(T), kByKDense)))
        return run_small<false>(kc, SmallOperand<T, true>{x, B, Din}, SmallOperand<T, true>{w, Dout, Din}, epi, B, Dout, Din, s);
    if (Din % V == 0 && aligned16(x) && aligned16(w))
        return run2(kc, DenseKC<T>{x, B, Din, Din}, DenseKC<T>{w, Dout, Din, Din}, epi, B, Dout, Din, ws, s);
    if (Din >= V) return run2(kc, RaggedKC<T>{x, B, Din, Din}, RaggedKC<T>{w, Dout, Din, Din}, epi, B, Dout, Din, ws, s);
    return gather_dense_kc_kc<T>(kc, x, w, epi, B, Dout, Din, ws, s);
}

// dx[m, n] = sum_k dy[m, k] * w[k, n]:  A = dy (k-contiguous), B(n, k) = w[k*Din + n] (row-contiguous)
template <class T>
static hipError_t dense_dgrad_t(int kc, const T* dy, const T* w, const EpiMask<T, T>& epi, int B, int Din, int Dout, float* ws, hipStream_t s) {
    constexpr int V = ElemTile<T>::V;
    if (small_is_better(B, Din, Dout, sizeof(T), plan_for(B, Din, Dout, false, sizeof(T), kByKDense)))
        return run_small<false>(kc, SmallOperand<T, true>{dy, B, Dout}, SmallOperand<T, false>{w, Din, Din}, epi, B, Din, Dout, s);
    if (Dout % V == 0 && Din % V == 0 && aligned16(dy) && aligned16(w))
        return run2(kc, DenseKC<T>{dy, B, Dout, Dout}, DenseRC<T>{w, Din, Dout, Din}, epi, B, Din, Dout, ws, s);
    if (Dout >= V && Din >= V)
        return run2(kc, RaggedKC<T>{dy, B, Dout, Dout}, RaggedRC<T>{w, Din, Dout, Din}, epi, B, Din, Dout, ws, s);
    return gather_dense_dgrad<T>(kc, dy, w, epi, B, Din, Dout, ws, s);
}

// gw[m, n] = sum_k dy[k, m] * x[k, n]: both operands row-contiguous, contraction over the batch
template <class T>
static hipError_t dense_wgrad_t(int kc, const T* dy, const T* x, float* gw, int B, int Din, int Dout, const Partials& ws, hipStream_t s) {
    constexpr int V = ElemTile<T>::V;
    if (small_is_better(Dout, Din, B, sizeof(T), plan_for(Dout, Din, B, true, sizeof(T), kByKDense)))
        return run_small<true>(kc, SmallOperand<T, false>{dy, Dout, Dout}, SmallOperand<T, false>{x, Din, Din},
                               EpiWgrad{gw, Din, (int64_t)Dout * Din, 0}, Dout, Din, B, s);
    if (Dout % V == 0 && Din % V == 0 && aligned16(dy) && aligned16(x))
        return run2_wgrad(kc, DenseRC<T>{dy, Dout, B, Dout}, DenseRC<T>{x, Din, B, Din}, gw, Dout, Din, B, ws, s);
    if (Dout >= V && Din >= V)
        return run2_wgrad(kc, RaggedRC<T>{dy, Dout, B, Dout}, RaggedRC<T>{x, Din, B, Din}, gw, Dout, Din, B, ws, s);
    return gather_dense_wgrad<T>(kc, dy, x, gw, Dout, Din, B, ws, s);
}

// Both gradients of a dense layer in one launch of the small kernel.
enum { kTwo = 0, kOneSmall, kOneTiled };
int backward_kind(int64_t B, int64_t Din, int64_t Dout, int esize);
int small_backward_tile(int64_t M, int64_t N, int esize);   // 1 or 2: tiles of 16 x 16 or 32 x 32 outputs
template <int TX, int TW, class T>
static hipError_t small_backward_inst(int kc, const T* dy, const T* x, const T* w, float* gw, const EpiMask<T, T>& epi, int B, int Din, int Dout, hipStream_t s) {
    const int of_x = cdiv(Din, 16 * TX) * cdiv(B, 16 * TX), of_w = cdiv(Din, 16 * TW) * cdiv(Dout, 16 * TW), grid = of_x + of_w;
    constexpr int lx = small_lds_floats(4, TX, TX), lw = small_lds_floats(4, TW, TW);
    return launch_timed(kc, gemm_small_backward_kernel<4, TX, TW, T>, dim3(grid), dim3(256), (lx > lw ? lx : lw) * 4, s, dy, x, w, epi,
                        EpiWgrad{gw, Din, (int64_t)Dout * Din, 0}, B, Din, Dout, Dout >= B ? of_x : of_w);
}
template <class T>
static hipError_t small_backward_t(int kc, const T* dy, const T* x, const T* w, float* gw, const EpiMask<T, T>& epi, int B, int Din, int Dout, hipStream_t s) {
    const int tx = small_backward_tile(B, Din, sizeof(T)), tw = small_backward_tile(Dout, Din, sizeof(T));
    if (tx == 2 && tw == 2) return small_backward_inst<2, 2>(kc, dy, x, w, gw, epi, B, Din, Dout, s);
    if (tx == 2) return small_backward_inst<2, 1>(kc, dy, x, w, gw, epi, B, Din, Dout, s);
    if (tw == 2) return small_backward_inst<1, 2>(kc, dy, x, w, gw, epi, B, Din, Dout, s);
    return small_backward_inst<1, 1>(kc, dy, x, w, gw, epi, B, Din, Dout, s);
}

// ---- convolution passes -------------------------------------------------------------------------------
// The chunked loaders index positions with 24-bit multiplies and tensors with 32-bit element offsets.
static inline bool small_enough(const ConvShape& c) {
    const int64_t pin = (int64_t)c.B * c.H * c.W, pout = (int64_t)c.B * c.Ho * c.Wo;
    const int64_t wel = (int64_t)c.Cout * c.R * c.S * c.Cin;
    return pin < (1 << 24) && pout < (1 << 24) && pin * c.Cin < (int64_t(1) << 31) &&
           pout * c.Cout < (int64_t(1) << 31) && wel < (int64_t(1) << 31) && c.Cin < (1 << 20) && c.Cout < (1 << 20);
}

// Convolutions on runs of rows (kernels_conv_rows.hip, bf16): the variant to launch, 0 for a convolution that the kernel cannot
// take or where the other kernels, estimated at other_us, are quicker.
constexpr int kMaxLds = 160 * 1024;
int conv_rows_variant(const ConvShape& c, int64_t M, int N, int C, double other_us);
template <bool DGRAD, class Epi>
hipError_t conv_rows(int variant, int kc, const bf16_t* x, const bf16_t* w, const Epi& epi, const ConvShape& c, hipStream_t s);

// Weight gradients on runs of rows (there too): k-slices (0: not to be taken) and the positions of each.
struct WgradRowsPlan {
    int slices, per_slice;
};
WgradRowsPlan conv_wgrad_rows_plan(const ConvShape& c, const Plan2& other);
hipError_t conv_wgrad_rows(const WgradRowsPlan& p, const bf16_t* dy, const bf16_t* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s);

// Convolutions over eight channels (kernels_conv_first.hip, bf16): which of them it is, 0 for any other and where the other kernels are quicker; slices
// of its weight gradient.
int conv_first_kind(const ConvShape& c, bool wgrad);
template <class Epi> hipError_t conv_first(int kind, const bf16_t* x, const bf16_t* w, const Epi& epi, const ConvShape& c, hipStream_t s);
int conv_first_wgrad_slices(const ConvShape& c);
hipError_t conv_first_wgrad(int kind, const bf16_t* dy, const bf16_t* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s);

template <class T, class Epi>
static hipError_t conv_forward_t(const T* x, const T* w, const Epi& epi, const ConvShape& c, float* ws, hipStream_t s) {
    const int M = c.B * c.Ho * c.Wo, K = c.R * c.S * c.Cin;
    if constexpr (sizeof(T) == 2) {
        const int first = conv_first_kind(c, false);
        if (first && epi.wide_ok() && aligned16(x) && aligned16(w)) return conv_first(first, x, w, epi, c, s);
        const int v = conv_rows_variant(c, M, c.Cout, c.Cin, plan_for(M, c.Cout, K, false, 2, kByKConv).cost / 2400.0);
        if (v && epi.wide_ok() && aligned16(x) && aligned16(w)) return conv_rows<false>(v, kcConvFwd, x, w, epi, c, s);
    }
    if (c.Cin % ElemTile<T>::V == 0 && aligned16(x) && aligned16(w) && small_enough(c))
        return run2(kcConvFwd, ConvFwdA2<T>{x, geom2(c), M, K}, DenseKC<T>{w, c.Cout, K, K}, epi, M, c.Cout, K, ws, s);
    return gather_conv_forward<T>(x, w, epi, c, ws, s);
}

template <class T>
static hipError_t conv_dgrad_t(const T* dy, const T* w, const EpiMask<T, T>& epi, const ConvShape& c, float* ws, hipStream_t s) {
    const int M = c.B * c.H * c.W, K = c.R * c.S * c.Cout;
    constexpr int V = ElemTile<T>::V, BK = ElemTile<T>::BK;
    if (c.Cin % V != 0 || c.Cout % V != 0 || !aligned16(dy) || !aligned16(w) || !small_enough(c)) return gather_conv_dgrad<T>(dy, w, epi, c, ws, s);
    if constexpr (sizeof(T) == 2) {
        const int v = conv_rows_variant(c, M, c.Cin, c.Cout, plan_for(M, c.Cin, K, false, 2, kByKConv).cost / 2400.0);
        if (v && epi.wide_ok()) return conv_rows<true>(v, kcConvDgrad, dy, w, epi, c, s);
    }
    if (c.rest_done && c.R == 1 && c.S == 1 && c.pad == 0 && epi.add == epi.out && epi.wide_ok()) {
        // A 1 x 1 filter with a stride reaches one position of stride^2: a dense product over those, added where they lie.  (In k-slices, which small
        // maps need, the partial sums are of those positions too: a block's forward and backward pass in fp32, in one slice and in as many as the plan has, 4 images of
        // 8 x 8 x 64 into 4096 channels 283 and 202 us, one of 14 x 14 x 1024 into 2048 211 and 173.)  Over the whole map three positions in four were read and written for nothing, for a
        // dx that the layer beside it then read once more: 64 images of 56 x 56 x 256 from 512 channels 138 us, of 14 x 14 x 1024 from 2048 119.
        const int Mo = c.B * c.Ho * c.Wo;
        const StridedKC<T> A(DenseKC<T>{dy, Mo, c.Cout, c.Cout}, c.H, c.W, c.stride, c.Ho, c.Wo);
        return run2_strided(kcConvDgrad, A, DenseRC<T>{w, c.Cin, c.Cout, c.Cin}, epi, Mo, c.Cin, c.Cout, ws, s);
    }
    if (c.stride == 2 && c.H % 2 == 0 && c.W % 2 == 0 && c.Cin % 8 == 0) {
        // Rows ordered by the parity of their position, each class walking only the filter taps that reach it:
        // k extent of the largest class; every class a whole number of tiles; the 16-byte epilogue (the one
        // that asks the loader where a row lies in memory), also for the partial sums of a split.
        const int Kp = ((c.R + 1) / 2) * ((c.S + 1) / 2) * c.Cout;
        const Plan2 plan = plan_for(M, c.Cin, Kp, false, sizeof(T), kByKConv);
        const int edge = plan.bn;   // (64 for the tall tiles: this order needs square ones)
        const int Mc = M / 4;
        int per, nz;
        slice_geometry(Kp, ws ? plan.slices : 1, BK, per, nz);
        const bool split_ok = nz <= 1 || (aligned16(ws) && ((int64_t)M * c.Cin) % 4 == 0);
        // (where a class is no whole number of the plan's tiles, smaller tiles still pay for a filter with
        // several taps; a 1x1 filter's launch is mostly epilogue either way and keeps the plain order then)
        const int tile = (Mc % edge == 0 || c.R * c.S == 1) ? edge : 64;
        if (Mc % tile == 0 && epi.wide_ok() && split_ok) {
            ParityGeom pg;
            pg.Mc = Mc;
            pg.W2 = c.W / 2;
            pg.d_mc = FastDiv(Mc);
            pg.d_h2w2 = FastDiv((c.H / 2) * (c.W / 2));
            pg.d_w2 = FastDiv(c.W / 2);
            return run2(kcConvDgrad, ConvDgradA2P<T>{dy, geom2(c), M, Kp, pg, {}}, ConvDgradB2P<T>{w, geom2(c), c.Cin, Kp, pg, {}}, epi, M,
                        c.Cin, Kp, ws, s, tile);
        }
    }
    return run2(kcConvDgrad, ConvDgradA2<T>{dy, geom2(c), M, K}, ConvDgradB2<T>{w, geom2(c), c.Cin, K}, epi, M, c.Cin, K, ws, s);
}

template <class T> static hipError_t conv_wgrad_t(const T* dy, const T* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    const int rows = c.Cout, cols = c.R * c.S * c.Cin;
    const int64_t K = (int64_t)c.B * c.Ho * c.Wo;
    constexpr int V = ElemTile<T>::V, BK = ElemTile<T>::BK;
    if (c.Cin % V != 0 || c.Cout % V != 0 || !aligned16(dy) || !aligned16(x) || !small_enough(c)) return gather_conv_wgrad<T>(dy, x, gw, c, ws, s);
    if constexpr (sizeof(T) == 2) {
        const int first = conv_first_kind(c, true);
        if (first && (conv_first_wgrad_slices(c) == 1 ? aligned16(gw) : ws.ws && aligned16(ws.ws))) return conv_first_wgrad(first, dy, x, gw, c, ws, s);
        const WgradRowsPlan p = conv_wgrad_rows_plan(c, plan_for(rows, cols, K, true, 2, kByKConv));
        if (p.slices && (p.slices == 1 ? aligned16(gw) : ws.ws && aligned16(ws.ws))) return conv_wgrad_rows(p, dy, x, gw, c, ws, s);
    }
    const int rows_bk = BK / c.Wo;
    ConvWgradB2<T> Bv{x, geom2(c), cols, (int)K, BK % c.Wo, rows_bk % c.Ho, rows_bk / c.Ho};
    return run2_wgrad(kcConvWgrad, DenseRC<T>{dy, rows, (int)K, c.Cout}, Bv, gw, rows, cols, K, ws, s);
}

// A 1x1 convolution with unit stride and no padding on NHWC tensors IS a dense layer over the B*H*W positions
// (weights [Cout][Cin]) and takes the dense paths.
static inline bool pointwise(const ConvShape& c) {
    return c.R == 1 && c.S == 1 && c.stride == 1 && c.pad == 0 && (int64_t)c.B * c.H * c.W < (int64_t(1) << 31);
}

// fp32 passes (kernels_gemm_f32.hip)
hipError_t dense_forward_f32(int kc, const float* x, const float* w, const EpiBiasAct<float>& epi, int B, int Din, int Dout, float* ws, hipStream_t s);
bool norm_dense_takes_f32(int64_t rows, int D, int N);
hipError_t norm_dense_f32(const float* x, const float* gamma, const float* beta, float* y, float* stats, const float* w, const EpiBiasAct<float>& epi, int M, int N,
                          int D, float eps, hipStream_t s);
hipError_t dense_dgrad_f32(int kc, const float* dy, const float* w, const EpiMask<float, float>& epi, int B, int Din, int Dout, float* ws, hipStream_t s);
hipError_t dense_wgrad_f32(int kc, const float* dy, const float* x, float* gw, int B, int Din, int Dout, const Partials& ws, hipStream_t s);
hipError_t small_backward_f32(int kc, const float* dy, const float* x, const float* w, float* gw, const EpiMask<float, float>& epi, int B, int Din, int Dout, hipStream_t s);
hipError_t mixed_backward_f32(int kc, const float* dy, const float* x, const float* w, float* gw, const EpiMask<float, float>& epi, int B, int Din, int Dout, hipStream_t s);
hipError_t conv_forward_f32(const float* x, const float* w, const EpiBiasAct<float>& epi, const ConvShape& c, float* ws, hipStream_t s);
hipError_t conv_affine_f32(const float* x, const float* w, const EpiConvAffine<float>& epi, const ConvShape& c, float* ws, hipStream_t s);
hipError_t conv_dgrad_f32(const float* dy, const float* w, const EpiMask<float, float>& epi, const ConvShape& c, float* ws, hipStream_t s);
hipError_t conv_wgrad_f32(const float* dy, const float* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s);

}  // namespace tmps
