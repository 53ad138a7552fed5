// Dense contractions of few outputs, bound by latency: C[m, n] = sum_k A(m, k) * B(n, k).
//
// A workgroup owns 16 TM x 16 TN outputs and its NW waves share the k range, each with fragments fetched straight from
// global memory into registers (no LDS tile, no barrier in the k-loop; the loads of the next D steps are in
// flight), so that a short contraction costs about one memory latency and a long one is walked
// NW times as fast; the partial tiles are added through LDS in a fixed order and the epilogue follows in the
// same launch.  The tiled kernel needs k-slices and a second launch for such shapes, or walks the whole k range in one
// workgroup.  What bounds it is the number of cache lines that the fragment loads of a compute unit touch: multiplies of 16 x 16 read 64
// consecutive bytes of a row with four lanes (those of 32 x 32 only 32 bytes), and an output of few rows is cut into the smallest tiles
// that the device has units for, which each load the least.  Launch to launch, with 32 x 32 multiplies and with these (us): fp32
// 32 x 64 -> 128 3.1 and 2.2, 47 x 1000 -> 1000 8.9 and 4.8, 128 x 1024 -> 1024 9.8 and 7.7, 256 x 1024 -> 1024 10.1 and 10.3; bf16 64 x 1024 -> 1024 5.7 and
// 3.8, 64 x 3072 -> 1024 11.7 (in k-slices) and 7.4, 256 x 1024 -> 1024 5.9 and 5.8 (what its sums' second set takes of that stands below).
#pragma once
#include "gemm2.hip.h"
#include "wave.hip.h"

namespace tmps {

// Operand of the small kernel.  KC: element (row, k) at p[row * ld + k], otherwise at p[k * ld + row].
template <class T_, bool KC> struct SmallOperand {
    typedef T_ T;
    static constexpr bool kContig = KC, kLocal = false;
    const T* p;
    int rows;
    int64_t ld;
    __device__ __forceinline__ void prepare() const {}
};

// Fragment of a lane (row lane % 16, quarter lane / 16): V elements from k on, at p (k-contiguous) or p, p + ld, ...
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

constexpr int small_lds_floats(int nw, int tm, int tn) { return nw * (tm * tn * 256 + tm * 16); }

// Tile (bx, by) of the contraction by a workgroup of NW waves.
template <int NW, int TM, int TN, bool ROWSUM, class AOp, class BOp, class Epi>
__device__ __forceinline__ void gemm_small_tile(const AOp& A, const BOp& B, const Epi& epi, int M, int N, int K, int bx, int by) {
    typedef typename AOp::T T;
    typedef typename Frag<T>::type frag_t;
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    constexpr bool AKC = AOp::kContig, BKC = BOp::kContig;
    constexpr int V = ElemTile<T>::V, GK = 4 * V;     // k of a step
    constexpr int BM = 16 * TM, BN = 16 * TN;
    constexpr int D = TM + TN <= 2 ? 6 : 4;   // steps in flight
    extern __shared__ __attribute__((aligned(16))) float part[];   // [NW][BM][BN], then [NW][BM] row sums
    const int tid = threadIdx.x, lane = tid & 63, quarter = lane >> 4, row = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = by * BM, n0 = bx * BN;
    const T *pa[TM], *pb[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = AOp::kLocal ? 16 * i + row : min(m0 + 16 * i + row, M - 1);
        pa[i] = AKC ? A.p + (int64_t)r * A.ld + quarter * V : A.p + (int64_t)(quarter * V) * A.ld + r;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int r = min(n0 + 16 * j + row, N - 1);
        pb[j] = BKC ? B.p + (int64_t)r * B.ld + quarter * V : B.p + (int64_t)(quarter * V) * B.ld + r;
    }
    const int groups = K / GK;   // whole steps; wave w takes w, w + NW, ...
    // A step is one multiply in bf16 and four in fp32, of two roundings each.  They go to accumulators in turn (as many as there are registers for), which
    // also keeps the multiplies of a single output from waiting for each other, and every D steps these are added to a second sum and start
    // again at zero: the roundings of a chain do not grow with the contraction.  Errors (2-norm, against 64 bits) in one chain a wave and so, fp32:
    // 235 x 1000 -> 1000 forward 2.9e-7 and 1.0e-7, weight gradients of 112 x 108 over 3432 rows 3.7e-7 and 1.2e-7, of 4936 x 24 over 8059 rows 8.0e-7 and
    // 1.6e-7; bf16, of 4096 x 64 over 2048 rows 1.3e-7 and 0.8e-7.  Where the multiplies set the time, as in fp32 in 32 x 32 tiles, that takes 2 to 15 % more:
    // forward 47 x 1000 -> 1000 4.9 and 4.9 us, 235 x 784 -> 1000 7.1 and 8.2, 235 x 1000 -> 1000 8.7 and 9.9; both gradients of 235 x 784 -> 1000 17.2 and 19.2.
    constexpr int NACC = sizeof(T) == 4 ? (TM * TN == 1 || !ROWSUM ? 4 : 2) : TM * TN == 1 ? 2 : 1;
    f32x4_t acc[NACC][TM][TN];
    float rsum[TM];
    auto clear = [&]() {   // (costs nothing where multiplies follow: they take a constant for the sum)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            rsum[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int a = 0; a < NACC; ++a) acc[a][i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    f32x4_t tot[TM][TN];
    float rsum_tot[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        rsum_tot[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < TN; ++j) tot[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
    auto add_to_totals = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            rsum_tot[i] += rsum[i];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v = acc[0][i][j][r];
                    if constexpr (NACC == 2) v += acc[NACC - 1][i][j][r];
                    if constexpr (NACC == 4) v = (v + acc[NACC - 3][i][j][r]) + (acc[NACC - 2][i][j][r] + acc[NACC - 1][i][j][r]);
                    tot[i][j][r] += v;
                }
        }
    };
    auto multiply = [&](const frag_t (&a)[TM], const frag_t (&b)[TN], int d) {
#pragma unroll
        for (int e = 0; e < (sizeof(T) == 2 ? 1 : 4); ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    f32x4_t& c = acc[(sizeof(T) == 2 ? d : e) % NACC][i][j];
                    if constexpr (sizeof(T) == 2) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], c, 0, 0, 0);
                    else c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], c, 0, 0, 0);
                }
        if (ROWSUM) {
#pragma unroll
            for (int i = 0; i < TM; ++i) rsum[i] = add_frag(rsum[i], a[i]);
        }
    };
    frag_t fa[D][TM], fb[D][TN];   // ring: step i of this wave in place i % D
    auto fetch_a = [&](int d, int i) {
        const int64_t k = (int64_t)(wave + i * NW) * GK;
#pragma unroll
        for (int t = 0; t < TM; ++t) fa[d][t] = small_frag<T, AKC>(pa[t] + (AKC ? k : k * A.ld), A.ld);
    };
    auto fetch_b = [&](int d, int i) {
        const int64_t k = (int64_t)(wave + i * NW) * GK;
#pragma unroll
        for (int t = 0; t < TN; ++t) fb[d][t] = small_frag<T, BKC>(pb[t] + (BKC ? k : k * B.ld), B.ld);
    };
    auto fetch = [&](int d, int i) {
        fetch_a(d, i);
        fetch_b(d, i);
    };
    const int mine_n = wave < groups ? (groups - wave + NW - 1) / NW : 0;
    if constexpr (AOp::kLocal) {   // (formed by the workgroup itself, while its first fragments of B are on their way)
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < mine_n) fetch_b(d, d);
        A.prepare();
        __syncthreads();
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < mine_n) fetch_a(d, d);
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < mine_n) fetch(d, d);
    }
    int i = 0;
    // (no branch around a load here: the compiler then waits for a step with the younger ones still in flight)
    for (; i + 2 * D <= mine_n; i += D) {
        clear();
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(fa[d], fb[d], d);
            fetch(d, i + D + d);
        }
        add_to_totals();
    }
    for (; i < mine_n; i += D) {
        clear();
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (i + d < mine_n) multiply(fa[d], fb[d], d);
            if (i + D + d < mine_n) fetch(d, i + D + d);
        }
        add_to_totals();
    }
    if (groups * GK < K && groups % NW == wave) {
        const int k = groups * GK, n = K - k - quarter * V;
        frag_t a[TM], b[TN];
        clear();
#pragma unroll
        for (int t = 0; t < TM; ++t) a[t] = small_frag_tail<T, AKC>(pa[t] + (AKC ? (int64_t)k : k * A.ld), A.ld, n);
#pragma unroll
        for (int t = 0; t < TN; ++t) b[t] = small_frag_tail<T, BKC>(pb[t] + (BKC ? (int64_t)k : k * B.ld), B.ld, n);
        multiply(a, b, 0);
        add_to_totals();
    }
    // register r of a lane: row 4 (lane / 16) + r, column lane % 16
    float* const mine = part + wave * (BM * BN);
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(16 * t + 4 * quarter + r) * BN + 16 * j + row] = tot[t][j][r];
    float* const sums = part + NW * (BM * BN);
    if (ROWSUM) {
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            float all = rsum_tot[t] + __shfl_xor(rsum_tot[t], 16, 64);
            all += __shfl_xor(all, 32, 64);
            if (lane < 16) sums[wave * BM + 16 * t + lane] = all;
        }
    }
    __syncthreads();
#pragma unroll
    for (int o = tid; o < BM * BN; o += 64 * NW) {
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; w += 2) v += part[w * (BM * BN) + o] + part[(w + 1) * (BM * BN) + o];   // (half the chain of additions)
        const int m = m0 + o / BN, n = n0 + o % BN;
        if (m < M && n < N) epi.at(epi.column(n), (int64_t)m * epi.ld + n, v, 0);
    }
    if (ROWSUM && bx == 0 && tid < BM && m0 + tid < M) {
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += sums[w * BM + tid];
        epi.rowsum(m0 + tid, v, 0);
    }
}

template <int NW, int TM, int TN, bool ROWSUM, class AOp, class BOp, class Epi>
__global__ __launch_bounds__(64 * NW, sizeof(typename AOp::T) == 4 ? 3 : 1) void gemm_small_kernel(AOp A, BOp B, Epi epi, int M, int N, int K) {
    gemm_small_tile<NW, TM, TN, ROWSUM>(A, B, epi, M, N, K, blockIdx.x, blockIdx.y);
}

// A layer normalisation and the dense layer that reads it: y = normalise(x) gamma + beta (with the rows' statistics, as the normalisation's own kernel
// leaves them), C = y w^T.  Every workgroup normalises its 16 rows itself, four to a wave, rounds them to LDS and multiplies from there; those of the
// first column of tiles store them.  For rows that one piece of V features to a lane holds, where the layer's launch costs as much as all of
// its work: 256 x 64 -> 192 in fp32 4.9 us for 2.6 and 3.2 in two launches, and 3 us less of a host thread that issues nothing but short launches
// (two mini-batches of two transformer blocks of width 64, two stages: 332 and 314 us).
template <class T> struct SmallNormalised : SmallOperand<T, true> {
    static constexpr bool kLocal = true;
    static constexpr int V = sizeof(T) == 2 ? 8 : 1;
    const T* x;        // [M][D] in global memory
    const float* gamma;
    const float* beta;
    T* y;              // null: not to be stored by this workgroup
    float* stats;
    int m0, M, D;
    float eps;
    __device__ __forceinline__ void prepare() const {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane * V;
        T* const tile = const_cast<T*>(this->p);
        float v[4][V], g[V], b[V];
        const bool mine = c < D;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = min(m0 + wave * 4 + r, M - 1);
            if (mine) {
                if constexpr (V == 8) load8(x + (int64_t)row * D + c, v[r]);
                else v[r][0] = to_f32(x[(int64_t)row * D + c]);
            }
        }
        if (mine) {
            if constexpr (V == 8) {
                load8(gamma + c, g);
                load8(beta + c, b);
            } else {
                g[0] = gamma[c];
                b[0] = beta[c];
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float s = 0.0f, q = 0.0f;
            if (mine) {
#pragma unroll
                for (int e = 0; e < V; ++e) s += v[r][e];
            }
            const float mean = wsum(s) / (float)D;
            if (mine) {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float d = v[r][e] - mean;
                    q += d * d;
                }
            }
            const float rstd = 1.0f / sqrtf(wsum(q) / (float)D + eps);
            const int local = wave * 4 + r, row = m0 + local;
            if (mine) {
                float o[V];
#pragma unroll
                for (int e = 0; e < V; ++e) o[e] = (v[r][e] - mean) * rstd * g[e] + b[e];
                if constexpr (V == 8) {
                    store8(tile + local * this->ld + c, o);
                    if (y && row < M) store8(y + (int64_t)row * D + c, o);
                } else {
                    tile[local * this->ld + c] = from_f32<T>(o[0]);
                    if (y && row < M) y[(int64_t)row * D + c] = from_f32<T>(o[0]);
                }
            }
            if (y && lane == 0 && row < M) {
                stats[2 * row] = mean;
                stats[2 * row + 1] = rstd;
            }
        }
    }
};
constexpr int kNormWaves = 4;
template <class T> constexpr int small_norm_ld(int D) { return D + 16 / (int)sizeof(T); }   // elements of a row in LDS
template <class T, class Epi>
__global__ __launch_bounds__(64 * kNormWaves) void norm_dense_small_kernel(const T* x, const float* gamma, const float* beta, T* y, float* stats, const T* w, Epi epi,
                                                                          int M, int N, int D, float eps) {
    extern __shared__ __attribute__((aligned(16))) float part[];
    SmallNormalised<T> A;
    A.p = reinterpret_cast<const T*>(part + small_lds_floats(kNormWaves, 1, 1));
    A.rows = 16;
    A.ld = small_norm_ld<T>(D);
    A.x = x; A.gamma = gamma; A.beta = beta; A.stats = stats;
    A.y = blockIdx.x == 0 ? y : nullptr;
    A.m0 = blockIdx.y * 16; A.M = M; A.D = D; A.eps = eps;
    gemm_small_tile<kNormWaves, 1, 1, false>(A, SmallOperand<T, true>{w, N, D}, epi, M, N, D, blockIdx.x, blockIdx.y);
}

// Input and weight gradient of a dense layer in one launch: dx[B, Din] = dy w and gw[Dout, Din] = dy^T x, the longer contraction by the first
// `split` workgroups, since the launch lasts as long as the last of them (weight gradients last and first, us: fp32 916 x 1336 -> 136 28.8 and 15.9,
// 2299 x 456 -> 32 13.0 and 11.1; bf16 2192 x 752 -> 24 13.5 and 8.2, 2752 x 288 -> 560 23.0 and 15.8).  Neither depends on the other, and
// a launch of its own costs each more than its work: 32 x 64 -> 128 in fp32 2.5 us against 4.4 in two launches (the rule, backward_kind, has the others).
// (TX, TW: tiles of 16 TX square outputs of dx and 16 TW square ones of gw)
template <int NW, int TX, int TW, class T>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 4 ? 3 : 1) void gemm_small_backward_kernel(const T* dy, const T* x, const T* w, EpiMask<T, T> ex, EpiWgrad ew,
                                                                      int rows, int Din, int Dout, int split) {
    const bool early = (int)blockIdx.x < split;
    const int b = early ? blockIdx.x : blockIdx.x - split;
    if (early == (Dout >= rows)) {
        const int tiles_n = (Din + 16 * TX - 1) / (16 * TX), by = b / tiles_n, bx = b - by * tiles_n;
        gemm_small_tile<NW, TX, TX, false>(SmallOperand<T, true>{dy, rows, Dout}, SmallOperand<T, false>{w, Din, Din}, ex, rows, Din, Dout, bx, by);
    } else {
        const int tiles_n = (Din + 16 * TW - 1) / (16 * TW), by = b / tiles_n, bx = b - by * tiles_n;
        gemm_small_tile<NW, TW, TW, true>(SmallOperand<T, false>{dy, Dout, Dout}, SmallOperand<T, false>{x, Din, Din}, ew, Dout, Din, rows, bx, by);
    }
}

}  // namespace tmps
