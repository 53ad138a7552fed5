// Max pooling over channels-last maps.  The forward pass keeps every window's winner (the first maximum in row-major order) beside the
// result, as a byte (for windows of 12 x 12 and more as four), so that the backward pass reads these instead of finding them again in the input: a quarter (2 x 2) or
// less of its bytes, and none of the comparisons that bound it before.  Backward pass with the input searched and by winners (us, bf16): 64 maps of 56 x 56 x 64, 3 x 3
// windows of stride 1 91 and 30, 5 x 5 of stride 2 99 and 23, 12 x 12 of stride 12 672 and 13; 64 of 13 x 13 x 512, 9 x 9 of stride 1 12197 and 68; 16 of 19 x 19 x 512, 13 x 13
// of stride 1 29656 and 147.
#include "gemm.hip.h"
#include "gemm2.hip.h"
#include "kernels.h"
#include "launch.h"

namespace tmps {

static inline int cdiv_pool(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
static inline bool al16p(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// A winner of a window whose places a byte tells apart: r * k + q of its place, with kNotPositive where it is not above zero (what the ReLU of the layer below then
// stops).  Of a larger one: its position in the map, h W + w, in 31 bits (which tell apart the positions of any window that spans fewer), and the highest bit for that.  In a window of negative infinities and NaN alone: the first
// place inside the map.  kNoWinner: no such window.
constexpr unsigned kNotPositive = 128, kNoWinner = 255;
template <class W> constexpr uint32_t not_positive() { return sizeof(W) == 1 ? kNotPositive : 0x80000000u; }
__device__ __forceinline__ uint32_t map_position(int h, int w, int width) { return ((uint32_t)h * (uint32_t)width + (uint32_t)w) & 0x7FFFFFFFu; }

struct PoolDims {
    int B, H, W, C, Ho, Wo, k, stride, pad;
};
static PoolDims pool_dims(int B, int H, int W, int C, int k, int stride, int pad) {
    return PoolDims{B, H, W, C, (H + 2 * pad - k) / stride + 1, (W + 2 * pad - k) / stride + 1, k, stride, pad};
}

// V consecutive elements (16 bytes, or one) and V winners
template <class T, int V> struct PoolVec {
    union {
        uint4 raw;
        T e[16 / sizeof(T)];
    } u;
    __device__ __forceinline__ void load(const T* p) {
        if constexpr (V == 1) u.e[0] = *p;
        else u.raw = *reinterpret_cast<const uint4*>(p);
    }
    __device__ __forceinline__ void store(T* p) const {
        if constexpr (V == 1) *p = u.e[0];
        else *reinterpret_cast<uint4*>(p) = u.raw;
    }
};
template <class W, int V> struct Winners;
template <int V> struct Winners<uint8_t, V> {
    uint32_t w[V > 4 ? V / 4 : 1];
    __device__ __forceinline__ void load(const uint8_t* p) {
        if constexpr (V == 1) w[0] = *p;
        else if constexpr (V == 4) w[0] = *reinterpret_cast<const uint32_t*>(p);
        else {
            const uint2 t = *reinterpret_cast<const uint2*>(p);
            w[0] = t.x;
            w[1] = t.y;
        }
    }
    __device__ __forceinline__ void store(uint8_t* p) const {
        if constexpr (V == 1) *p = (uint8_t)w[0];
        else if constexpr (V == 4) *reinterpret_cast<uint32_t*>(p) = w[0];
        else *reinterpret_cast<uint2*>(p) = make_uint2(w[0], w[1]);
    }
    __device__ __forceinline__ uint32_t at(int e) const { return (w[e >> 2] >> (8 * (e & 3))) & 255u; }
    __device__ __forceinline__ void set(int e, uint32_t v) {   // (in order, from the first one on)
        if ((e & 3) == 0) w[e >> 2] = v;
        else w[e >> 2] |= v << (8 * (e & 3));
    }
    __device__ __forceinline__ void fill(uint32_t byte) {
#pragma unroll
        for (int i = 0; i < (V > 4 ? V / 4 : 1); ++i) w[i] = byte * 0x01010101u;
    }
    __device__ __forceinline__ void mask(uint32_t byte) {
#pragma unroll
        for (int i = 0; i < (V > 4 ? V / 4 : 1); ++i) w[i] &= byte * 0x01010101u;
    }
};
template <int V> struct Winners<uint32_t, V> {
    uint32_t w[V];
    __device__ __forceinline__ void load(const uint32_t* p) {
        if constexpr (V == 1) w[0] = *p;
        else {
#pragma unroll
            for (int i = 0; i < V; i += 4) {
                const uint4 t = *reinterpret_cast<const uint4*>(p + i);
                w[i] = t.x; w[i + 1] = t.y; w[i + 2] = t.z; w[i + 3] = t.w;
            }
        }
    }
    __device__ __forceinline__ void store(uint32_t* p) const {
        if constexpr (V == 1) *p = w[0];
        else {
#pragma unroll
            for (int i = 0; i < V; i += 4) *reinterpret_cast<uint4*>(p + i) = make_uint4(w[i], w[i + 1], w[i + 2], w[i + 3]);
        }
    }
    __device__ __forceinline__ uint32_t at(int e) const { return w[e]; }
    __device__ __forceinline__ void set(int e, uint32_t v) { w[e] = v; }
    __device__ __forceinline__ void mask(uint32_t bits) {
#pragma unroll
        for (int e = 0; e < V; ++e) w[e] &= bits;
    }
};

// One thread per window and V channels.  K: the window where it is known at compile time (0: the argument); all of its elements are then requested at
// once (8 images of 112 x 112 x 64, 3 x 3 windows of stride 2: 6.7 us; a loop that waits for one at a time 8.5).
template <class T, int V, int K, class W>
__global__ __launch_bounds__(256) void maxpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ y, W* __restrict__ won, PoolDims p) {
    constexpr bool kByte = sizeof(W) == 1;
    const int CV = p.C / V;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)p.B * p.Ho * p.Wo * CV) return;
    const int c = (int)(i % CV) * V;
    int64_t t = i / CV;
    const int wo = (int)(t % p.Wo); t /= p.Wo;
    const int ho = (int)(t % p.Ho);
    const int n = (int)(t / p.Ho);
    const int h0 = ho * p.stride - p.pad, w0 = wo * p.stride - p.pad, hl = max(h0, 0), wl = max(w0, 0);   // (the first place inside the map)
    const T* const xn = x + (int64_t)n * p.H * p.W * p.C + c;
    auto place = [&](int h, int w) { return kByte ? (uint32_t)((h - h0) * (K ? K : p.k) + w - w0) : map_position(h, w, p.W); };
    float best[V];
    uint32_t where[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        best[e] = -INFINITY;
        where[e] = place(hl, wl);
    }
    auto look = [&](const PoolVec<T, V>& o, uint32_t me) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float v = to_f32(o.u.e[e]);
            if (v > best[e]) {   // strict: the first maximum stays
                best[e] = v;
                where[e] = me;
            }
        }
    };
    if constexpr (K > 0) {
        PoolVec<T, V> o[K * K];
#pragma unroll
        for (int a = 0; a < K * K; ++a) {
            const int hh = min(max(h0 + a / K, 0), p.H - 1), ww = min(max(w0 + a % K, 0), p.W - 1);
            o[a].load(xn + ((int64_t)hh * p.W + ww) * p.C);
        }
#pragma unroll
        for (int a = 0; a < K * K; ++a)   // (padding never wins)
            if ((unsigned)(h0 + a / K) < (unsigned)p.H && (unsigned)(w0 + a % K) < (unsigned)p.W) look(o[a], a);
    } else if constexpr (kByte) {
        for (int r = 0; r < p.k; ++r)
            for (int q = 0; q < p.k; ++q) {
                const int h = h0 + r, w = w0 + q;
                if ((unsigned)h >= (unsigned)p.H || (unsigned)w >= (unsigned)p.W) continue;
                PoolVec<T, V> o;
                o.load(xn + ((int64_t)h * p.W + w) * p.C);
                look(o, place(h, w));
            }
    } else {
        // (long rows, four of whose elements are requested at a time: 14 x 14 windows of 64 maps of 56 x 56 x 64 in bf16 85 and 36 us; rows of four and five lose by it,
        // 4 x 4 of stride 2 over 30 x 30 8.7 and 12.0)
        const int h1 = min(h0 + p.k, p.H), w1 = min(w0 + p.k, p.W);
        for (int h = hl; h < h1; ++h) {
            const T* const row = xn + (int64_t)h * p.W * p.C;
#pragma unroll 4
            for (int w = wl; w < w1; ++w) {
                PoolVec<T, V> o;
                o.load(row + (int64_t)w * p.C);
                look(o, place(h, w));
            }
        }
    }
    PoolVec<T, V> out;
    Winners<W, V> win;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        out.u.e[e] = from_f32<T>(best[e]);
        win.set(e, best[e] > 0.0f ? where[e] : where[e] | not_positive<W>());
    }
    out.store(y + i * V);
    win.store(won + i * V);
}

// The input gradients of an S x S block of positions, (i S + a - pad, j S + b - pad) for a, b < S, each the sum of the upstream gradients of the windows
// that it won, in row-major order.  A block shares its windows: (i - dh, j - dw), in which it has the places (a + dh S, b + dw S).
template <class T, int V, int K, int S>
__device__ __forceinline__ void pool_block(const PoolDims& p, const T* dy, const uint8_t* won, int n, int i, int j, int c, bool relu, float (&acc)[S * S][V]) {
    constexpr int NA = (K - 1) / S + 1;
    PoolVec<T, V> g[NA * NA];
    Winners<uint8_t, V> win[NA * NA];
#pragma unroll
    for (int a = 0; a < NA * NA; ++a) {
        const int ho = i - a / NA, wo = j - a % NA;
        const bool ok = (unsigned)ho < (unsigned)p.Ho && (unsigned)wo < (unsigned)p.Wo;
        const int64_t at = (((int64_t)n * p.Ho + (ok ? ho : 0)) * p.Wo + (ok ? wo : 0)) * p.C + c;
        g[a].load(dy + at);
        win[a].load(won + at);
        if (!relu) win[a].mask(kNotPositive - 1);
        if (!ok) win[a].fill(kNoWinner);
    }
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < S; ++b) {
#pragma unroll
            for (int e = 0; e < V; ++e) acc[a * S + b][e] = 0.0f;
#pragma unroll
            for (int dh = (K - 1 - a) / S; dh >= 0; --dh)
#pragma unroll
                for (int dw = (K - 1 - b) / S; dw >= 0; --dw)
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        acc[a * S + b][e] += win[dh * NA + dw].at(e) == (unsigned)((a + dh * S) * K + b + dw * S) ? to_f32(g[dh * NA + dw].u.e[e]) : 0.0f;
        }
}

struct PoolBlocks {
    int nh, nw;          // blocks of a map
    FastDiv d_c, d_w, d_h;   // by pieces of channels, nw and nh
};

// One thread per block and V channels: upstream gradients and winners once (but for what neighbouring blocks share), the result once.
// 128 images of 32 x 32 x 64 in bf16, 2 x 2 windows: 8.1 us (11.1 with the input read and searched).
template <class T, int V, int K, int S>
__global__ __launch_bounds__(256) void maxpool_bwd_kernel(const T* __restrict__ dy, const uint8_t* __restrict__ won, T* __restrict__ dx, PoolDims p, PoolBlocks blocks,
                                                          int total, int relu) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= total) return;
    uint32_t q, c, j, i, n;
    blocks.d_c.divmod((uint32_t)t, q, c);
    blocks.d_w.divmod(q, q, j);
    blocks.d_h.divmod(q, n, i);
    float acc[S * S][V];
    pool_block<T, V, K, S>(p, dy, won, (int)n, (int)i, (int)j, (int)c * V, relu != 0, acc);
#pragma unroll
    for (int a = 0; a < S * S; ++a) {
        const int h = (int)i * S + a / S - p.pad, w = (int)j * S + a % S - p.pad;
        if ((unsigned)h >= (unsigned)p.H || (unsigned)w >= (unsigned)p.W) continue;
        PoolVec<T, V> out;
#pragma unroll
        for (int e = 0; e < V; ++e) out.u.e[e] = from_f32<T>(acc[a][e]);
        out.store(dx + (((int64_t)n * p.H + h) * p.W + w) * p.C + (int)c * V);
    }
}

// Any window, stride and channel count: one thread per position and V channels.
template <class T, int V, class W>
__global__ __launch_bounds__(256) void maxpool_bwd_any_kernel(const T* __restrict__ dy, const W* __restrict__ won, T* __restrict__ dx, PoolDims p, int relu) {
    const int CV = p.C / V;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)p.B * p.H * p.W * CV) return;
    const int c = (int)(i % CV) * V;
    int64_t t = i / CV;
    const int w = (int)(t % p.W); t /= p.W;
    const int h = (int)(t % p.H);
    const int n = (int)(t / p.H);
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.0f;
    const int hp = h + p.pad, wp = w + p.pad;
    const int ho_lo = hp - p.k + 1 > 0 ? (hp - p.k + p.stride) / p.stride : 0;
    const int wo_lo = wp - p.k + 1 > 0 ? (wp - p.k + p.stride) / p.stride : 0;
    for (int ho = ho_lo; ho < p.Ho && ho * p.stride <= hp; ++ho)
        for (int wo = wo_lo; wo < p.Wo && wo * p.stride <= wp; ++wo) {
            const int64_t at = (((int64_t)n * p.Ho + ho) * p.Wo + wo) * p.C + c;
            PoolVec<T, V> g;
            Winners<W, V> win;
            g.load(dy + at);
            win.load(won + at);
            if (!relu) win.mask(not_positive<W>() - 1);
            const uint32_t me = sizeof(W) == 1 ? (uint32_t)((hp - ho * p.stride) * p.k + wp - wo * p.stride) : map_position(h, w, p.W);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] += win.at(e) == me ? to_f32(g.u.e[e]) : 0.0f;
        }
    PoolVec<T, V> out;
#pragma unroll
    for (int e = 0; e < V; ++e) out.u.e[e] = from_f32<T>(acc[e]);
    out.store(dx + i * V);
}

// Max pooling behind a per-channel affine layer that nothing else reads: the affine layer's backward pass (dz = gain * da and the sums of da * z and of
// da, a slab of blocks to a workgroup: part[slab][0][C], part[slab][1][C]) with da = the pooling's input gradient, rounded as it would have been stored, in
// registers.  Bound by its bytes: winners, upstream gradient and z once, dz once.  64 images of 112 x 112 x 64 in bf16 56 us; the
// two passes one after the other, with the winners found again, 87 and 51.
template <class T, int V, int K, int S>
__global__ __launch_bounds__(256) void maxpool_affine_bwd_kernel(const T* __restrict__ dy, const uint8_t* __restrict__ won, const T* __restrict__ z,
                                                                 const float* __restrict__ gain, T* __restrict__ dz, float* __restrict__ part, PoolDims p,
                                                                 PoolBlocks blocks, int total, int per_slab, int relu) {
    constexpr int L = 64 / V, R = 256 / L;   // lanes that hold 64 channels, blocks at a time
    __shared__ float sg[R][65], sb[R][65];
    const int cg = threadIdx.x % L, rl = threadIdx.x / L, col = blockIdx.x * 64 + cg * V;
    const int q1 = min(total, (int)(blockIdx.y + 1) * per_slab);
    float dg[V], db[V], g[V];
#pragma unroll
    for (int e = 0; e < V; ++e) dg[e] = db[e] = 0.0f;
    if (col < p.C) {
#pragma unroll
        for (int e = 0; e < V; ++e) g[e] = gain[col + e];
        for (int q = (int)blockIdx.y * per_slab + rl; q < q1; q += R) {
            uint32_t t, j, i, n;
            blocks.d_w.divmod((uint32_t)q, t, j);
            blocks.d_h.divmod(t, n, i);
            int64_t at[S * S];
            bool ok[S * S];
            PoolVec<T, V> zv[S * S];
#pragma unroll
            for (int a = 0; a < S * S; ++a) {
                const int h = (int)i * S + a / S - p.pad, w = (int)j * S + a % S - p.pad;
                ok[a] = (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
                at[a] = (((int64_t)n * p.H + (ok[a] ? h : 0)) * p.W + (ok[a] ? w : 0)) * p.C + col;
                zv[a].load(z + at[a]);
            }
            float acc[S * S][V];
            pool_block<T, V, K, S>(p, dy, won, (int)n, (int)i, (int)j, col, relu != 0, acc);
#pragma unroll
            for (int a = 0; a < S * S; ++a) {
                if (!ok[a]) continue;
                PoolVec<T, V> out;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float d = to_f32(from_f32<T>(acc[a][e]));
                    dg[e] += d * to_f32(zv[a].u.e[e]);
                    db[e] += d;
                    out.u.e[e] = from_f32<T>(d * g[e]);
                }
                out.store(dz + at[a]);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
        sg[rl][cg * V + e] = dg[e];
        sb[rl][cg * V + e] = db[e];
    }
    __syncthreads();
    const int mine = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x < 64 && mine < p.C) {
        float a = 0.0f, b = 0.0f;
#pragma unroll 8
        for (int r = 0; r < R; ++r) {
            a += sg[r][threadIdx.x];
            b += sb[r][threadIdx.x];
        }
        part[((int64_t)blockIdx.y * 2 + 0) * p.C + mine] = a;
        part[((int64_t)blockIdx.y * 2 + 1) * p.C + mine] = b;
    }
}

int maxpool_winner_bytes(int k) { return (int64_t)k * k < (int64_t)kNotPositive ? 1 : 4; }

template <class T, class W>
static hipError_t forward_t(const T* x, T* y, W* won, const PoolDims& p, hipStream_t s) {
    constexpr int V = 16 / sizeof(T);
    const int64_t n = (int64_t)p.B * p.Ho * p.Wo * p.C;
    if (p.C % V == 0 && al16p(x) && al16p(y)) {
        const dim3 grid(cdiv_pool(n / V, 256));
        if constexpr (sizeof(W) == 1) {
            if (p.k == 2) return launch_timed(kcPoolFwd, maxpool_fwd_kernel<T, V, 2, W>, grid, dim3(256), 0, s, x, y, won, p);
            if (p.k == 3) return launch_timed(kcPoolFwd, maxpool_fwd_kernel<T, V, 3, W>, grid, dim3(256), 0, s, x, y, won, p);
        }
        return launch_timed(kcPoolFwd, maxpool_fwd_kernel<T, V, 0, W>, grid, dim3(256), 0, s, x, y, won, p);
    }
    return launch_timed(kcPoolFwd, maxpool_fwd_kernel<T, 1, 0, W>, dim3(cdiv_pool(n, 256)), dim3(256), 0, s, x, y, won, p);
}

hipError_t maxpool_forward(int dtype, const void* x, void* y, void* won, int B, int H, int W, int C, int k, int stride, int pad, hipStream_t s) {
    const PoolDims p = pool_dims(B, H, W, C, k, stride, pad);
    if ((int64_t)B * p.Ho * p.Wo * C <= 0) return hipSuccess;
    if (maxpool_winner_bytes(k) == 1)
        return dtype == kBF16 ? forward_t((const bf16_t*)x, (bf16_t*)y, (uint8_t*)won, p, s) : forward_t((const float*)x, (float*)y, (uint8_t*)won, p, s);
    if ((int64_t)(k < H ? k : H) * W >= (int64_t(1) << 31)) return hipErrorInvalidValue;   // (a window's positions would not all differ in 31 bits)
    return dtype == kBF16 ? forward_t((const bf16_t*)x, (bf16_t*)y, (uint32_t*)won, p, s) : forward_t((const float*)x, (float*)y, (uint32_t*)won, p, s);
}

static PoolBlocks pool_blocks(const PoolDims& p, int V) {
    PoolBlocks b;
    b.nh = (p.H - 1 + p.pad) / p.stride + 1;
    b.nw = (p.W - 1 + p.pad) / p.stride + 1;
    b.d_c = FastDiv((uint32_t)(p.C / V));
    b.d_w = FastDiv((uint32_t)b.nw);
    b.d_h = FastDiv((uint32_t)b.nh);
    return b;
}

template <class T, class W>
static hipError_t backward_t(const T* dy, const W* won, T* dx, const PoolDims& p, int relu, hipStream_t s) {
    constexpr int V = 16 / sizeof(T);
    const int64_t n = (int64_t)p.B * p.H * p.W * p.C;
    if (p.C % V != 0 || !al16p(dy) || !al16p(dx))
        return launch_timed(kcPoolBwd, maxpool_bwd_any_kernel<T, 1, W>, dim3(cdiv_pool(n, 256)), dim3(256), 0, s, dy, won, dx, p, relu);
    if constexpr (sizeof(W) == 1) {
        const PoolBlocks b = pool_blocks(p, V);
        const int64_t total = (int64_t)p.B * b.nh * b.nw * (p.C / V);
        if (p.stride == 2 && (p.k == 2 || p.k == 3) && total < (int64_t(1) << 30)) {
            const dim3 grid(cdiv_pool(total, 256));
            if (p.k == 2) return launch_timed(kcPoolBwd, maxpool_bwd_kernel<T, V, 2, 2>, grid, dim3(256), 0, s, dy, won, dx, p, b, (int)total, relu);
            return launch_timed(kcPoolBwd, maxpool_bwd_kernel<T, V, 3, 2>, grid, dim3(256), 0, s, dy, won, dx, p, b, (int)total, relu);
        }
    }
    return launch_timed(kcPoolBwd, maxpool_bwd_any_kernel<T, V, W>, dim3(cdiv_pool(n / V, 256)), dim3(256), 0, s, dy, won, dx, p, relu);
}

hipError_t maxpool_backward(int dtype, const void* dy, const void* won, void* dx, int B, int H, int W, int C, int k, int stride, int pad, int relu_mask, hipStream_t s) {
    const PoolDims p = pool_dims(B, H, W, C, k, stride, pad);
    if ((int64_t)B * H * W * C <= 0) return hipSuccess;
    if (maxpool_winner_bytes(k) == 1)
        return dtype == kBF16 ? backward_t((const bf16_t*)dy, (const uint8_t*)won, (bf16_t*)dx, p, relu_mask, s)
                              : backward_t((const float*)dy, (const uint8_t*)won, (float*)dx, p, relu_mask, s);
    return dtype == kBF16 ? backward_t((const bf16_t*)dy, (const uint32_t*)won, (bf16_t*)dx, p, relu_mask, s)
                          : backward_t((const float*)dy, (const uint32_t*)won, (float*)dx, p, relu_mask, s);
}

bool maxpool_affine_takes(int dtype, int64_t rows, int C, int k, int stride) {
    return k == 3 && stride == 2 && C % (dtype == kBF16 ? 8 : 4) == 0 && rows < (int64_t(1) << 30);
}

template <class T>
static hipError_t affine_t(const T* dy, const uint8_t* won, const T* z, const float* gain, T* dz, float* ws, int slabs_at_most, const PoolDims& p, int relu, int& slabs,
                           hipStream_t s) {
    constexpr int V = 16 / sizeof(T), R = 256 / (64 / V);
    const PoolBlocks b = pool_blocks(p, V);
    const int total = p.B * b.nh * b.nw, per_slab = cdiv_pool(cdiv_pool(total, slabs_at_most), R) * R;
    slabs = cdiv_pool(total, per_slab);
    return launch_timed(kcPoolBwd, maxpool_affine_bwd_kernel<T, V, 3, 2>, dim3(cdiv_pool(p.C, 64), slabs), dim3(256), 0, s, dy, won, z, gain, dz, ws, p, b, total, per_slab,
                        relu);
}

hipError_t maxpool_affine_backward(int dtype, const void* dy, const void* winners, const void* z, const float* gain, void* dz, float* dgain_dshift, const Partials& partials,
                                   int B, int H, int W, int C, int k, int stride, int pad, int relu_mask, hipStream_t s) {
    const PoolDims p = pool_dims(B, H, W, C, k, stride, pad);
    if ((int64_t)B * H * W * C <= 0) return hipSuccess;
    const int room = (int)(affine_workspace_elems((int64_t)B * H * W, C) / (2 * (size_t)C));   // as many slabs as the affine layer alone has
    const uint8_t* const won = (const uint8_t*)winners;
    int slabs = 0;
    const hipError_t e = dtype == kBF16 ? affine_t((const bf16_t*)dy, won, (const bf16_t*)z, gain, (bf16_t*)dz, partials.ws, room, p, relu_mask, slabs, s)
                                        : affine_t((const float*)dy, won, (const float*)z, gain, (float*)dz, partials.ws, room, p, relu_mask, slabs, s);
    if (e != hipSuccess) return e;
    return partials.finish(Reduction{partials.ws, dgain_dshift, 2 * C, slabs, true}, s);
}

}  // namespace tmps

extern "C" int tmps_pool_affine_gradients_joint(int dtype, int64_t positions, int channels, int window, int stride) {
    return tmps::maxpool_affine_takes(dtype, positions, channels, window, stride) ? 1 : 0;
}
