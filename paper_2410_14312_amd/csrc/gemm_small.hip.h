// Dense contractions of few output tiles, bound by latency: C[m, n] = sum_k A(m, k) * B(n, k).
//
// A workgroup owns a 32 x 32 tile of C and its NW waves share the k range, each with fragments fetched straight from
// global memory into registers (no LDS tile, no barrier in the k-loop; the loads of the next D fragment pairs are in
// flight), so that a short contraction costs about one memory latency and a long one is walked
// NW times as fast; the partial tiles are added through LDS in the order of the waves and the epilogue follows in the
// same launch.  The tiled kernel needs k-slices and a second launch for such shapes, or walks the whole k range in one
// workgroup: 47 x 1000 x 1000 in fp32 took 132 us there with a k-loop on the vector units.
// A 32 x 32 tile reads 64 elements per k for 2048 operations, so this pays while the tiles are few (the rule is in
// gemm_dispatch.hip.h).
#pragma once
#include "gemm2.hip.h"

namespace tmps {

// Operand of the small kernel.  KC: element (row, k) at p[row * ld + k], otherwise at p[k * ld + row].
template <class T_, bool KC> struct SmallOperand {
    typedef T_ T;
    static constexpr bool kContig = KC;
    const T* p;
    int rows;
    int64_t ld;
};

// Fragment of lane (row lane % 32, half lane / 32): V elements from k on, at p (k-contiguous) or p, p + ld, ...
template <class T, bool KC> __device__ __forceinline__ typename Frag<T>::type small_frag(const T* p, int64_t ld) {
    constexpr int V = ElemTile<T>::V;
    union { typename Frag<T>::type f; T e[V]; } r;
    if constexpr (KC) __builtin_memcpy(&r, p, 16);   // (element-aligned)
    else {
#pragma unroll
        for (int e = 0; e < V; ++e) r.e[e] = p[e * ld];
    }
    return r.f;
}
// the same where only the first n of the V elements exist
template <class T, bool KC> __device__ __forceinline__ typename Frag<T>::type small_frag_tail(const T* p, int64_t ld, int n) {
    constexpr int V = ElemTile<T>::V;
    union { typename Frag<T>::type f; T e[V]; } r;
#pragma unroll
    for (int e = 0; e < V; ++e) r.e[e] = e < n ? p[KC ? e : e * ld] : T(0.0f);
    return r.f;
}

// Tile (bx, by) of the contraction by a workgroup of NW waves.
template <int NW, bool ROWSUM, class AOp, class BOp, class Epi>
__device__ __forceinline__ void gemm_small_tile(const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int bx, int by) {
    typedef typename AOp::T T;
    typedef typename Frag<T>::type frag_t;
    constexpr bool AKC = AOp::kContig, BKC = BOp::kContig;
    constexpr int V = ElemTile<T>::V, GK = 2 * V;     // k of a fragment pair
    // pairs in flight (16 waves leave 128 registers per lane, and row-contiguous fragments need more addresses)
    constexpr int D = NW == 16 && !(AKC && BKC) ? 4 : 6;
    extern __shared__ __attribute__((aligned(16))) float part[];   // [NW][32][32], then [NW][32] row sums
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = by * 32, n0 = bx * 32;
    const int ra = min(m0 + (lane & 31), M - 1), rb = min(n0 + (lane & 31), N - 1);
    const T* const pa = AKC ? A.p + (int64_t)ra * A.ld + half * V : A.p + (int64_t)(half * V) * A.ld + ra;
    const T* const pb = BKC ? B.p + (int64_t)rb * B.ld + half * V : B.p + (int64_t)(half * V) * B.ld + rb;
    const int groups = K / GK;   // whole fragment pairs; wave w takes w, w + NW, ...
    f32x16_t acc[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.0f;
    float rsum = 0.0f;
    auto multiply = [&](const frag_t& a, const frag_t& b, int d) {
        if constexpr (sizeof(T) == 2) acc[d & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[d & 1], 0, 0, 0);
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc[e & 1], 0, 0, 0);
        }
        if (ROWSUM) rsum = add_frag(rsum, a);
    };
    frag_t fa[D], fb[D];   // ring: pair i of this wave in place i % D
    auto fetch = [&](int d, int i) {
        const int64_t k = (int64_t)(wave + i * NW) * GK;
        fa[d] = small_frag<T, AKC>(pa + (AKC ? k : k * A.ld), A.ld);
        fb[d] = small_frag<T, BKC>(pb + (BKC ? k : k * B.ld), B.ld);
    };
    const int mine_n = wave < groups ? (groups - wave + NW - 1) / NW : 0;
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < mine_n) fetch(d, d);
    int i = 0;
    // (no branch around a load here: the compiler then waits for a pair with the younger ones still in flight)
    for (; i + 2 * D <= mine_n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(fa[d], fb[d], d);
            fetch(d, i + D + d);
        }
    }
    for (; i < mine_n; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (i + d < mine_n) multiply(fa[d], fb[d], d);
            if (i + D + d < mine_n) fetch(d, i + D + d);
        }
    }
    if (groups * GK < K && groups % NW == wave) {
        const int k = groups * GK, n = K - k - half * V;
        const frag_t a = small_frag_tail<T, AKC>(pa + (AKC ? (int64_t)k : k * A.ld), A.ld, n);
        const frag_t b = small_frag_tail<T, BKC>(pb + (BKC ? (int64_t)k : k * B.ld), B.ld, n);
        multiply(a, b, 0);
    }
    float* const mine = part + wave * 1024;
#pragma unroll
    for (int r = 0; r < 16; ++r) mine[(8 * (r >> 2) + 4 * half + (r & 3)) * 32 + (lane & 31)] = acc[0][r] + acc[1][r];
    float* const sums = part + NW * 1024;
    if (ROWSUM) {
        const float both = rsum + __shfl_xor(rsum, 32, 64);
        if (lane < 32) sums[wave * 32 + lane] = both;
    }
    __syncthreads();
#pragma unroll
    for (int i = tid; i < 1024; i += 64 * NW) {
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += part[w * 1024 + i];
        const int m = m0 + (i >> 5), n = n0 + (i & 31);
        if (m < M && n < N) epi.at(epi.column(n), (int64_t)m * epi.ld + n, v, 0);
    }
    if (ROWSUM && bx == 0 && tid < 32 && m0 + tid < M) {
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += sums[w * 32 + tid];
        epi.rowsum(m0 + tid, v, 0);
    }
}

template <int NW, bool ROWSUM, class AOp, class BOp, class Epi>
__global__ __launch_bounds__(64 * NW) void gemm_small_kernel(AOp A, BOp B, Epi epi, int M, int N, int K) {
    gemm_small_tile<NW, ROWSUM>(A, B, epi, M, N, K, blockIdx.x, blockIdx.y);
}

// Input and weight gradient of a dense layer in one launch: dx[B, Din] = dy w (the first `split` workgroups, the longer contractions
// where a batch is small) and gw[Dout, Din] = dy^T x.  Neither depends on the other, and a launch of its own costs each more than its work:
// 32 x 128 -> 128 in fp32 4.2 us against 7.5 in two launches (the rule, backward_kind, has the others).
template <int NW, class T>
__global__ __launch_bounds__(64 * NW) void gemm_small_backward_kernel(const T* dy, const T* x, const T* w, EpiMask<T, T> ex, EpiWgrad ew,
                                                                      int rows, int Din, int Dout, int split) {
    const int tiles_n = (Din + 31) >> 5;   // (both outputs have Din columns)
    const int b = blockIdx.x, i = b < split ? b : b - split;
    const int by = i / tiles_n, bx = i - by * tiles_n;
    if (b < split)
        gemm_small_tile<NW, false>(SmallOperand<T, true>{dy, rows, Dout}, SmallOperand<T, false>{w, Din, Din}, ex, rows, Din, Dout, bx, by);
    else
        gemm_small_tile<NW, true>(SmallOperand<T, false>{dy, Dout, Dout}, SmallOperand<T, false>{x, Din, Din}, ew, Dout, Din, rows, bx, by);
}

}  // namespace tmps
