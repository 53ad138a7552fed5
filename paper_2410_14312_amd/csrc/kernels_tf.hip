// Transformer-stage kernels for gfx950 beside attention (kernels_attn.hip): layer normalisation, token + position
// embedding.
#include <type_traits>
#include <cstdlib>
#include "gemm2.hip.h"
#include "kernels.h"
#include "launch.h"
#include "wave.hip.h"

namespace tmps {

static inline int cdiv_tf(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

__global__ void zero_f32_kernel(float* __restrict__ p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0.0f;
}

// ------------------------------------------------------------------------------ layer normalisation
// One wave per row.  The row is read three times (mean, variance, output); it stays in cache.
template <typename T>
__global__ __launch_bounds__(256) void layernorm_fwd_kernel(const T* __restrict__ x, const float* __restrict__ gamma,
                                                            const float* __restrict__ beta, T* __restrict__ y,
                                                            float* __restrict__ stats, int64_t rows, int D, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const T* xr = x + row * D;
    float s = 0.0f;
    for (int i = lane; i < D; i += 64) s += to_f32(xr[i]);
    const float mean = wsum(s) / (float)D;
    float v = 0.0f;
    for (int i = lane; i < D; i += 64) {
        const float d = to_f32(xr[i]) - mean;
        v += d * d;
    }
    const float rstd = 1.0f / sqrtf(wsum(v) / (float)D + eps);
    T* yr = y + row * D;
    for (int i = lane; i < D; i += 64) yr[i] = from_f32<T>((to_f32(xr[i]) - mean) * rstd * gamma[i] + beta[i]);
    if (lane == 0) {
        stats[2 * row] = mean;
        stats[2 * row + 1] = rstd;
    }
}

// The same with 8 bf16 per lane and access (D % 8 == 0, 16-byte aligned rows), for rows that registers do not hold.
__global__ __launch_bounds__(256) void layernorm_fwd_bf16x8_kernel(const bf16_t* __restrict__ x,
                                                                   const float* __restrict__ gamma,
                                                                   const float* __restrict__ beta, bf16_t* __restrict__ y,
                                                                   float* __restrict__ stats, int64_t rows, int D,
                                                                   float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const bf16_t* xr = x + row * D;
    const int nch = D >> 3;
    float s = 0.0f;
    for (int c = lane; c < nch; c += 64) {
        Pack8 p;
        p.u = *reinterpret_cast<const uint4*>(xr + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (float)p.h[e];
    }
    const float mean = wsum(s) / (float)D;
    float v = 0.0f;
    for (int c = lane; c < nch; c += 64) {
        Pack8 p;
        p.u = *reinterpret_cast<const uint4*>(xr + c * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float d = (float)p.h[e] - mean;
            v += d * d;
        }
    }
    const float rstd = 1.0f / sqrtf(wsum(v) / (float)D + eps);
    bf16_t* yr = y + row * D;
    for (int c = lane; c < nch; c += 64) {
        Pack8 p, o;
        p.u = *reinterpret_cast<const uint4*>(xr + c * 8);
        const float4 g0 = *reinterpret_cast<const float4*>(gamma + c * 8), g1 = *reinterpret_cast<const float4*>(gamma + c * 8 + 4);
        const float4 b0 = *reinterpret_cast<const float4*>(beta + c * 8), b1 = *reinterpret_cast<const float4*>(beta + c * 8 + 4);
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) o.h[e] = (bf16_t)(((float)p.h[e] - mean) * rstd * g[e] + b[e]);
        *reinterpret_cast<uint4*>(yr + c * 8) = o.u;
    }
    if (lane == 0) {
        stats[2 * row] = mean;
        stats[2 * row + 1] = rstd;
    }
}

// The same for rows of at most 64 V N features: a lane requests its N pieces of V features, gains and shifts among them, before it needs the first, and
// keeps the row in registers.  (Read three times over, the row comes from the caches, but each time after the sum before it.)  Before and here (us): bf16,
// 1024 rows of 768 3.8 and 3.1, 8192 rows 8.0 and 6.9 (3.6 TB/s), 999 rows of 512 3.1 and 2.5; fp32, 256 rows of 64 2.8 and 2.3, 1024 of 768 6.4 and 4.0.
// What is left of the short ones is the launch, one latency and two sums over the wave.  Sums are in the order of the kernels above.
template <typename T, int V, int N>
__global__ __launch_bounds__(256) void layernorm_fwd_row_kernel(const T* __restrict__ x, const float* __restrict__ gamma,
                                                                const float* __restrict__ beta, T* __restrict__ y,
                                                                float* __restrict__ stats, int64_t rows, int D, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    float v[N][V], g[N][V], b[N][V];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = (lane + 64 * i) * V;
        if (c < D) {
            if constexpr (V == 8) load8(x + row * D + c, v[i]);
            else v[i][0] = to_f32(x[row * D + c]);
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = (lane + 64 * i) * V;
        if (c < D) {
            if constexpr (V == 8) {
                load8(gamma + c, g[i]);
                load8(beta + c, b[i]);
            } else {
                g[i][0] = gamma[c];
                b[i][0] = beta[c];
            }
        }
    }
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if ((lane + 64 * i) * V < D) {
#pragma unroll
            for (int e = 0; e < V; ++e) s += v[i][e];
        }
    const float mean = wsum(s) / (float)D;
    float q = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i)
        if ((lane + 64 * i) * V < D) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float d = v[i][e] - mean;
                q += d * d;
            }
        }
    const float rstd = 1.0f / sqrtf(wsum(q) / (float)D + eps);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = (lane + 64 * i) * V;
        if (c < D) {
            float o[V];
#pragma unroll
            for (int e = 0; e < V; ++e) o[e] = (v[i][e] - mean) * rstd * g[i][e] + b[i][e];
            if constexpr (V == 8) store8(y + row * D + c, o);
            else y[row * D + c] = from_f32<T>(o[0]);
        }
    }
    if (lane == 0) {
        stats[2 * row] = mean;
        stats[2 * row + 1] = rstd;
    }
}

// dx = rstd * (g - mean(g) - xhat * mean(g * xhat)) [+ add],  g = dy * gamma, xhat = (x - mean) * rstd with the
// statistics of the forward pass.  `add` is the gradient of a residual connection that joins this layer's input.
template <typename T>
__global__ __launch_bounds__(256) void layernorm_bwd_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                            const float* __restrict__ stats,
                                                            const float* __restrict__ gamma, const T* __restrict__ add,
                                                            T* __restrict__ dx, int64_t rows, int D) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const T* xr = x + row * D;
    const T* gr = dy + row * D;
    const float mean = stats[2 * row], rstd = stats[2 * row + 1];
    float s1 = 0.0f, s2 = 0.0f;
    for (int i = lane; i < D; i += 64) {
        const float g = to_f32(gr[i]) * gamma[i];
        s1 += g;
        s2 += g * (to_f32(xr[i]) - mean) * rstd;
    }
    const float m1 = wsum(s1) / (float)D, m2 = wsum(s2) / (float)D;
    T* dr = dx + row * D;
    for (int i = lane; i < D; i += 64) {
        const float g = to_f32(gr[i]) * gamma[i];
        const float xh = (to_f32(xr[i]) - mean) * rstd;
        float v = rstd * (g - m1 - xh * m2);
        if (add) v += to_f32(add[row * D + i]);
        dr[i] = from_f32<T>(v);
    }
}

// Gain / shift gradients: block = 64 columns x 4 row lanes over one slab of rows; partial sums
// part[slab][0][D] (gain) and part[slab][1][D] (shift).
template <typename T>
__global__ __launch_bounds__(256) void layernorm_pgrad_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                              const float* __restrict__ stats, float* __restrict__ part,
                                                              int64_t rows, int D, int rows_per_slab) {
    __shared__ float sg[4][64], sb[4][64];
    const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
    const int col = blockIdx.x * 64 + cl;
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_slab;
    const int64_t r1 = r0 + rows_per_slab < rows ? r0 + rows_per_slab : rows;
    float dg = 0.0f, db = 0.0f;
    if (col < D)
        for (int64_t r = r0 + rl; r < r1; r += 4) {
            const float d = to_f32(dy[r * D + col]);
            dg += d * (to_f32(x[r * D + col]) - stats[2 * r]) * stats[2 * r + 1];
            db += d;
        }
    sg[rl][cl] = dg;
    sb[rl][cl] = db;
    __syncthreads();
    if (rl == 0 && col < D) {
        part[((int64_t)blockIdx.y * 2 + 0) * D + col] = (sg[0][cl] + sg[1][cl]) + (sg[2][cl] + sg[3][cl]);
        part[((int64_t)blockIdx.y * 2 + 1) * D + col] = (sb[0][cl] + sb[1][cl]) + (sb[2][cl] + sb[3][cl]);
    }
}

// Input gradient AND the per-slab partial sums of the gain / shift gradients in one pass over dy and x: 8 features
// per lane and access, D % 8 == 0 and D <= 1024 (at most two 8-feature chunks per lane).  A wave takes R rows of its
// workgroup's slab of 4 R rows; the four waves' partial sums are combined through LDS.  (256 rows of 64 in fp32: 3.7 us, the two
// kernels above 2.9 and 4.5.)
template <typename T, int R>
__global__ __launch_bounds__(256) void layernorm_bwd_fused_kernel(const T* __restrict__ dy, const T* __restrict__ x,
                                                                  const float* __restrict__ stats,
                                                                  const float* __restrict__ gamma, const T* __restrict__ add,
                                                                  T* __restrict__ dx, float* __restrict__ part,
                                                                  int64_t rows, int D) {
    __shared__ float sred[4][2][1024];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nch = D >> 3;
    float g[2][8], ag[2][8], ab[2][8];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) load8(gamma + c * 8, g[i]);
#pragma unroll
        for (int e = 0; e < 8; ++e) ag[i][e] = ab[i][e] = 0.0f;
    }
    const int64_t r0 = (int64_t)blockIdx.x * (4 * R) + wave * R;
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
        const int64_t row = r0 + rr;
        if (row >= rows) break;   // uniform per wave
        const float mean = stats[2 * row], rstd = stats[2 * row + 1];
        float dyv[2][8], xh[2][8];
        float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = lane + 64 * i;
            if (c < nch) {
                float xv[8];
                load8(dy + row * D + c * 8, dyv[i]);
                load8(x + row * D + c * 8, xv);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    xh[i][e] = (xv[e] - mean) * rstd;
                    const float t = dyv[i][e] * g[i][e];
                    s1 += t;
                    s2 += t * xh[i][e];
                    ag[i][e] += dyv[i][e] * xh[i][e];
                    ab[i][e] += dyv[i][e];
                }
            }
        }
        const float m1 = wsum(s1) / (float)D, m2 = wsum(s2) / (float)D;
        if (dx) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int c = lane + 64 * i;
                if (c < nch) {
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = rstd * (dyv[i][e] * g[i][e] - m1 - xh[i][e] * m2);
                    if (add) {
                        float a[8];
                        load8(add + row * D + c * 8, a);
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] += a[e];
                    }
                    store8(dx + row * D + c * 8, v);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                sred[wave][0][c * 8 + e] = ag[i][e];
                sred[wave][1][c * 8 + e] = ab[i][e];
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * D; i += 256) {
        const int w = i >= D ? 1 : 0, col = i - w * D;
        part[((int64_t)blockIdx.x * 2 + w) * D + col] = (sred[0][w][col] + sred[1][w][col]) + (sred[2][w][col] + sred[3][w][col]);
    }
}

// Rows per wave of the fused backward kernel: its workgroups are to cover the device (1024 rows in slabs of 16 are 64 of them:
// both passes of 1024 x 768 18.2 us, in slabs of 4 12.6 us), and every slab costs a row of partial sums.
static int ln_rows_per_wave(int64_t rows) { return rows >= 4096 ? 4 : rows >= 2048 ? 2 : 1; }
static int ln_slab_rows(int64_t rows) { return rows > 4096 ? 128 : 32; }

size_t layernorm_workspace_elems(int64_t rows, int D) {
    // (the slabs of the fused backward kernel; those of the others are longer)
    return (size_t)cdiv_tf(rows, 4 * ln_rows_per_wave(rows)) * 2 * (size_t)D;
}

hipError_t layernorm_forward(int dtype, const void* x, const float* gamma, const float* beta, void* y, float* stats,
                             int64_t rows, int D, float eps, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    dim3 grid(cdiv_tf(rows, 4));
    if (dtype == kBF16) {
        const bool vec = D % 8 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) |
                                         reinterpret_cast<uintptr_t>(gamma) | reinterpret_cast<uintptr_t>(beta)) & 15) == 0;
        if (vec && D <= 1024) {
            auto kern = D <= 512 ? layernorm_fwd_row_kernel<bf16_t, 8, 1> : layernorm_fwd_row_kernel<bf16_t, 8, 2>;
            return launch_timed(kcLayerNorm, kern, grid, dim3(256), 0, s, (const bf16_t*)x, gamma, beta, (bf16_t*)y, stats, rows, D, eps);
        }
        if (vec)
            return launch_timed(kcLayerNorm, layernorm_fwd_bf16x8_kernel, grid, dim3(256), 0, s, (const bf16_t*)x, gamma,
                                beta, (bf16_t*)y, stats, rows, D, eps);
        return launch_timed(kcLayerNorm, layernorm_fwd_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)x, gamma, beta,
                            (bf16_t*)y, stats, rows, D, eps);
    }
    auto kern = D <= 64 ? layernorm_fwd_row_kernel<float, 1, 1> : D <= 256 ? layernorm_fwd_row_kernel<float, 1, 4>
              : D <= 1024 ? layernorm_fwd_row_kernel<float, 1, 16> : layernorm_fwd_kernel<float>;
    return launch_timed(kcLayerNorm, kern, grid, dim3(256), 0, s, (const float*)x, gamma, beta, (float*)y, stats, rows, D, eps);
}

template <typename T>
static hipError_t ln_backward(const T* dy, const T* x, const float* stats, const float* gamma, const T* add, T* dx, float* dgamma_dbeta,
                              const Partials& partials, int64_t rows, int D, hipStream_t s) {
    float* const ws = partials.ws;
    hipError_t e;
    if (D % 8 == 0 && D <= 1024 && ((reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(gamma) |
                                     reinterpret_cast<uintptr_t>(add) | reinterpret_cast<uintptr_t>(dx)) & 15) == 0) {
        const int per_wave = ln_rows_per_wave(rows), slabs = cdiv_tf(rows, 4 * per_wave);
        auto kern = per_wave == 4 ? layernorm_bwd_fused_kernel<T, 4> : per_wave == 2 ? layernorm_bwd_fused_kernel<T, 2> : layernorm_bwd_fused_kernel<T, 1>;
        e = launch_timed(kcLayerNorm, kern, dim3(slabs), dim3(256), 0, s, dy, x, stats, gamma, add, dx, ws, rows, D);
        if (e != hipSuccess) return e;
        return partials.finish(Reduction{ws, dgamma_dbeta, 2 * D, slabs, true}, s);
    }
    const int slab = ln_slab_rows(rows), slabs = cdiv_tf(rows, slab);
    if (dx) {
        e = launch_timed(kcLayerNorm, layernorm_bwd_kernel<T>, dim3(cdiv_tf(rows, 4)), dim3(256), 0, s, dy, x, stats, gamma, add, dx, rows, D);
        if (e != hipSuccess) return e;
    }
    e = launch_timed(kcLayerNorm, layernorm_pgrad_kernel<T>, dim3(cdiv_tf(D, 64), slabs), dim3(256), 0, s, dy, x, stats, ws, rows, D, slab);
    if (e != hipSuccess) return e;
    return partials.finish(Reduction{ws, dgamma_dbeta, 2 * D, slabs, true}, s);
}

hipError_t layernorm_backward(int dtype, const void* dy, const void* x, const float* stats, const float* gamma,
                              const void* add, void* dx, float* dgamma_dbeta, const Partials& partials, int64_t rows, int D,
                              hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    if (dtype == kBF16)
        return ln_backward<bf16_t>((const bf16_t*)dy, (const bf16_t*)x, stats, gamma, (const bf16_t*)add, (bf16_t*)dx, dgamma_dbeta, partials, rows, D, s);
    return ln_backward<float>((const float*)dy, (const float*)x, stats, gamma, (const float*)add, (float*)dx, dgamma_dbeta, partials, rows, D, s);
}

// ----------------------------------------------------------------------------------------- embedding
// y[row] = wte[tok[row]] + wpe[row % S]; a token outside the vocabulary gives a NaN row, never a wild read.
template <typename T>
__global__ __launch_bounds__(256) void embedding_fwd_kernel(const int32_t* __restrict__ tok, const T* __restrict__ wte,
                                                            const T* __restrict__ wpe, T* __restrict__ y, int64_t rows,
                                                            int S, int D, int vocab) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int t = tok[row];
    const bool ok = t >= 0 && t < vocab;
    const T* a = wte + (int64_t)(ok ? t : 0) * D;
    const T* b = wpe + (int64_t)(row % S) * D;
    T* yr = y + row * D;
    for (int i = lane; i < D; i += 64) yr[i] = ok ? from_f32<T>(to_f32(a[i]) + to_f32(b[i])) : from_f32<T>(NAN);
}

template <typename T>
__global__ void embedding_bwd_pos_kernel(const T* __restrict__ dy, float* __restrict__ dwpe, int64_t B, int64_t SD) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= SD) return;
    float a = 0.0f;
    for (int64_t b = 0; b < B; ++b) a += to_f32(dy[b * SD + i]);
    dwpe[i] = a;
}

// Token-table gradient, deterministic: dwte[t] = sum of the rows of dy whose token is t, added in row order.  One wave
// per row.  The wave of a token's FIRST row (no earlier row has the token: a scan of the rows before it) collects the
// later rows with the same token (a scan of the rows after it, 256 tokens per step) and adds them up in increasing row
// order; every other wave leaves.  No atomic adds, so the sum does not depend on which wave arrives first; rows of
// tokens that do not occur are zero (the table gradient is cleared before).
template <typename T>
__global__ __launch_bounds__(256) void embedding_bwd_tok_kernel(const int32_t* __restrict__ tok, const T* __restrict__ dy,
                                                                float* __restrict__ dwte, int64_t rows, int D, int vocab) {
    constexpr int CAP = 128;   // later occurrences kept in LDS per wave; a token with more is summed by rescanning
    __shared__ int later[4][CAP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row = (int64_t)blockIdx.x * 4 + wave;
    if (row >= rows) return;
    const int t = tok[row];
    if (t < 0 || t >= vocab) return;
    for (int64_t base = 0; base < row; base += 256) {
        bool hit = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + u * 64 + lane;
            hit |= j < row && tok[j] == t;
        }
        if (__ballot(hit)) return;   // not the first row of this token (uniform over the wave)
    }
    int n = 0;
    for (int64_t base = row + 1; base < rows; base += 256) {
        int v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t j = base + u * 64 + lane;
            v[u] = j < rows ? tok[j] : -1;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            unsigned long long m = __ballot(v[u] == t);
            while (m) {
                const int b = __ffsll((long long)m) - 1;
                m &= m - 1;
                if (n < CAP && lane == 0) later[wave][n] = (int)(base + u * 64 + b);
                ++n;
            }
        }
    }
    // lane 0 wrote the list, every lane reads it: LDS operations of one wave complete in order; keep the compiler
    // from moving the reads up
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    float* dst = dwte + (int64_t)t * D;
    if (n <= CAP) {
        for (int i = lane; i < D; i += 64) {
            float a = to_f32(dy[row * D + i]);
            for (int k = 0; k < n; ++k) a += to_f32(dy[(int64_t)later[wave][k] * D + i]);
            dst[i] = a;
        }
    } else {
        for (int i = lane; i < D; i += 64) {
            float a = to_f32(dy[row * D + i]);
            for (int64_t j = row + 1; j < rows; ++j)
                if (tok[j] == t) a += to_f32(dy[j * D + i]);
            dst[i] = a;
        }
    }
}

// Both table gradients of small tables in one launch: a wave to a token, which collects the rows that have it in row order (none: its row is zero), and
// behind those workgroups a thread to an element of the position table.  The sums are those of the two kernels above, bit for bit.  256 rows of
// 64 features, 96 tokens: one launch of 3.4 us for three of 1.9, 4.3 and 2.6.
template <typename T>
__global__ __launch_bounds__(256) void embedding_bwd_small_kernel(const int32_t* __restrict__ tok, const T* __restrict__ dy, float* __restrict__ dwte,
                                                                  float* __restrict__ dwpe, int rows, int D, int vocab, int tok_blocks, int B, int64_t SD) {
    if ((int)blockIdx.x >= tok_blocks) {
        const int64_t i = (int64_t)(blockIdx.x - tok_blocks) * 256 + threadIdx.x;
        if (i >= SD) return;
        float a = 0.0f;
#pragma unroll 4
        for (int b = 0; b < B; ++b) a += to_f32(dy[b * SD + i]);
        dwpe[i] = a;
        return;
    }
    constexpr int CAP = 64;   // rows collected before they are added up
    __shared__ int list[4][CAP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = blockIdx.x * 4 + wave;
    if (t >= vocab) return;
    float* const dst = dwte + (int64_t)t * D;
    int n = 0;
    bool begun = false;
    auto add_up = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the list is one wave's: its LDS operations complete in order)
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < D; i += 64) {
            float a = begun ? dst[i] : n > 0 ? to_f32(dy[(int64_t)list[wave][0] * D + i]) : 0.0f;
#pragma unroll 4
            for (int k = begun ? 0 : 1; k < n; ++k) a += to_f32(dy[(int64_t)list[wave][k] * D + i]);
            dst[i] = a;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        begun = true;
        n = 0;
    };
    for (int base = 0; base < rows; base += 256) {
        int v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = base + u * 64 + lane;
            v[u] = j < rows ? tok[j] : -1;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned long long m = __ballot(v[u] == t);
            if (!m) continue;
            if (n + __popcll(m) > CAP) add_up();
            if (v[u] == t) list[wave][n + __popcll(m & ((1ull << lane) - 1))] = base + u * 64 + lane;
            n += __popcll(m);
        }
    }
    if (n > 0 || !begun) add_up();
}

hipError_t embedding_forward(int dtype, const int32_t* tok, const void* wte, const void* wpe, void* y, int64_t rows, int S,
                             int D, int vocab, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    dim3 grid(cdiv_tf(rows, 4));
    if (dtype == kBF16)
        return launch_timed(kcEmbedding, embedding_fwd_kernel<bf16_t>, grid, dim3(256), 0, s, tok, (const bf16_t*)wte,
                            (const bf16_t*)wpe, (bf16_t*)y, rows, S, D, vocab);
    return launch_timed(kcEmbedding, embedding_fwd_kernel<float>, grid, dim3(256), 0, s, tok, (const float*)wte,
                        (const float*)wpe, (float*)y, rows, S, D, vocab);
}

hipError_t embedding_backward(int dtype, const int32_t* tok, const void* dy, float* dwte, float* dwpe, int64_t B, int S,
                              int D, int vocab, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    const int64_t nw = (int64_t)vocab * D, SD = (int64_t)S * D, rows = B * S;
    // (a wave to a token reads all rows' tokens, 16 thousand steps of 64 at most, some 16 to a SIMD; with larger tables the launches below, a wave to a
    // row, are the ones with less to read, and their three launches are no longer what counts.  Forward and backward pass in three launches and in one, 64 features (us): 8192
    // rows of 96 tokens to 1024 of 1000 17 to 18 and 11.5; 10000 rows, 100 tokens 52 and 24; 16 rows, 65536 tokens 18.4 and 13.5.  The waves that find no row cost
    // 0.1 us for a thousand tokens: 10 rows, 100000 tokens 19.0 and 16.1; 8 rows, 131072 18.2 and 19.6; 2 rows, 500000 23 and 57)
    if (rows * vocab <= (int64_t(1) << 20) && vocab <= 100000 && SD <= (int64_t(1) << 20)) {
        const int tok_blocks = cdiv_tf(vocab, 4);
        const dim3 grid(tok_blocks + cdiv_tf(SD, 256));
        if (dtype == kBF16)
            return launch_timed(kcEmbedding, embedding_bwd_small_kernel<bf16_t>, grid, dim3(256), 0, s, tok, (const bf16_t*)dy, dwte, dwpe, (int)rows, D, vocab,
                                tok_blocks, (int)B, SD);
        return launch_timed(kcEmbedding, embedding_bwd_small_kernel<float>, grid, dim3(256), 0, s, tok, (const float*)dy, dwte, dwpe, (int)rows, D, vocab,
                            tok_blocks, (int)B, SD);
    }
    int zb = cdiv_tf(nw, 256);
    if (zb > 4096) zb = 4096;
    hipError_t e = launch_timed(kcEmbedding, zero_f32_kernel, dim3(zb), dim3(256), 0, s, dwte, nw);
    if (e != hipSuccess) return e;
    if (dtype == kBF16) {
        e = launch_timed(kcEmbedding, embedding_bwd_pos_kernel<bf16_t>, dim3(cdiv_tf(SD, 256)), dim3(256), 0, s,
                         (const bf16_t*)dy, dwpe, B, SD);
        if (e != hipSuccess) return e;
        return launch_timed(kcEmbedding, embedding_bwd_tok_kernel<bf16_t>, dim3(cdiv_tf(rows, 4)), dim3(256), 0, s, tok,
                            (const bf16_t*)dy, dwte, rows, D, vocab);
    }
    e = launch_timed(kcEmbedding, embedding_bwd_pos_kernel<float>, dim3(cdiv_tf(SD, 256)), dim3(256), 0, s, (const float*)dy,
                     dwpe, B, SD);
    if (e != hipSuccess) return e;
    return launch_timed(kcEmbedding, embedding_bwd_tok_kernel<float>, dim3(cdiv_tf(rows, 4)), dim3(256), 0, s, tok,
                        (const float*)dy, dwte, rows, D, vocab);
}

}  // namespace tmps
