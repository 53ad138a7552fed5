// Causal multi-head self-attention for gfx950: forward and the query and key/value gradients.
//
// The MFMA path (32 or 64 features per head, bf16 or fp32) is a flash-style kernel: a wave owns 32 query rows (or 32 key
// rows where the gradients of keys and values are formed), streams blocks of keys (queries) through LDS and keeps running softmax
// statistics, so the S x S score matrix never exists in memory.  Products are arranged so that the softmax reduction runs
// over a lane's own registers: scores are computed TRANSPOSED (keys along the accumulator registers, queries along the
// lanes), and the probabilities leave the accumulators straight into the B operand of the next MFMA with no shuffle.
// Operands that the next product needs transposed (V^T, K^T, Q^T, dO^T) are read from their row-major LDS tile: in bf16
// with the transpose read of gfx950, in fp32 value by value (an fp32 MFMA takes one value per lane).
// The generic path (any head size) is a plain one-row-per-wave kernel.  The fp32 configurations ran on it before they had
// an MFMA path: 98 positions, 90 (batch, head) pairs of 64 features, 70 us forward and 260 us backward.
#include <math.h>

#include <cstdlib>
#include <type_traits>

#include "gemm2.hip.h"
#include "kernels.h"
#include "launch.h"
#include "wave.hip.h"

namespace tmps {

static inline int cdiv_at(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------------- generic path
// qkv rows are [q | k | v] of D features each; head h owns features h*dh .. h*dh+dh-1 of each part.
// One wave per (batch, head, query row).  Dynamic LDS: S floats (probabilities).
template <typename T>
__global__ __launch_bounds__(64) void attn_fwd_row_kernel(const T* __restrict__ qkv, T* __restrict__ o,
                                                          float* __restrict__ lse, int S, int D, int H, float scale) {
    extern __shared__ float sp[];
    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
    const int dh = D / H;
    const int64_t ld = 3 * (int64_t)D;
    const T* base = qkv + (int64_t)b * S * ld + h * dh;
    const T* qi = base + i * ld;
    float mx = -INFINITY;
    for (int j = lane; j <= i; j += 64) {
        const T* kj = base + j * ld + D;
        float a = 0.0f;
        for (int d = 0; d < dh; ++d) a += to_f32(qi[d]) * to_f32(kj[d]);
        a *= scale;
        sp[j] = a;
        mx = fmaxf(mx, a);
    }
    mx = wmax(mx);
    float sum = 0.0f;
    for (int j = lane; j <= i; j += 64) {
        const float e = expf(sp[j] - mx);
        sp[j] = e;
        sum += e;
    }
    sum = wsum(sum);
    __syncthreads();
    const float inv = 1.0f / sum;
    for (int d = lane; d < dh; d += 64) {
        float a = 0.0f;
        for (int j = 0; j <= i; ++j) a += sp[j] * to_f32(base[j * ld + 2 * D + d]);
        o[((int64_t)b * S + i) * D + h * dh + d] = from_f32<T>(a * inv);
    }
    if (lane == 0) lse[((int64_t)b * H + h) * S + i] = mx + logf(sum);
}

// delta[b, h, i] = sum_d dO[i, d] * O[i, d]
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_kernel(const T* __restrict__ o, const T* __restrict__ dout,
                                                         float* __restrict__ delta, int64_t BS, int S, int D, int H) {
    const int lane = threadIdx.x & 63;
    const int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // (b*S + i)*H + h
    if (idx >= BS * H) return;
    const int h = (int)(idx % H);
    const int64_t bi = idx / H;
    const int dh = D / H;
    float a = 0.0f;
    for (int d = lane; d < dh; d += 64) a += to_f32(o[bi * D + h * dh + d]) * to_f32(dout[bi * D + h * dh + d]);
    a = wsum(a);
    if (lane == 0) delta[((bi / S) * H + h) * S + (bi % S)] = a;
}

// Query gradient, one wave per (b, h, i).  Dynamic LDS: S floats (dS row).
template <typename T>
__global__ __launch_bounds__(64) void attn_bwd_q_row_kernel(const T* __restrict__ qkv, const T* __restrict__ dout,
                                                            const float* __restrict__ lse, const float* __restrict__ delta,
                                                            T* __restrict__ dqkv, int S, int D, int H, float scale) {
    extern __shared__ float sp[];
    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
    const int dh = D / H;
    const int64_t ld = 3 * (int64_t)D;
    const T* base = qkv + (int64_t)b * S * ld + h * dh;
    const T* qi = base + i * ld;
    const T* doi = dout + ((int64_t)b * S + i) * D + h * dh;
    const float L = lse[((int64_t)b * H + h) * S + i], dl = delta[((int64_t)b * H + h) * S + i];
    for (int j = lane; j <= i; j += 64) {
        const T* kj = base + j * ld + D;
        const T* vj = base + j * ld + 2 * D;
        float a = 0.0f, dp = 0.0f;
        for (int d = 0; d < dh; ++d) {
            a += to_f32(qi[d]) * to_f32(kj[d]);
            dp += to_f32(doi[d]) * to_f32(vj[d]);
        }
        sp[j] = expf(a * scale - L) * (dp - dl);
    }
    __syncthreads();
    for (int d = lane; d < dh; d += 64) {
        float a = 0.0f;
        for (int j = 0; j <= i; ++j) a += sp[j] * to_f32(base[j * ld + D + d]);
        dqkv[((int64_t)b * S + i) * ld + h * dh + d] = from_f32<T>(a * scale);
    }
}

// Key / value gradients, one wave per (b, h, j).  Dynamic LDS: 2*S floats (P and dS columns).
template <typename T>
__global__ __launch_bounds__(64) void attn_bwd_kv_row_kernel(const T* __restrict__ qkv, const T* __restrict__ dout,
                                                             const float* __restrict__ lse, const float* __restrict__ delta,
                                                             T* __restrict__ dqkv, int S, int D, int H, float scale) {
    extern __shared__ float sp[];
    float* sds = sp + S;
    const int j = blockIdx.x, h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x;
    const int dh = D / H;
    const int64_t ld = 3 * (int64_t)D;
    const T* base = qkv + (int64_t)b * S * ld + h * dh;
    const T* kj = base + j * ld + D;
    const T* vj = base + j * ld + 2 * D;
    for (int i = j + lane; i < S; i += 64) {
        const T* qi = base + i * ld;
        const T* doi = dout + ((int64_t)b * S + i) * D + h * dh;
        float a = 0.0f, dp = 0.0f;
        for (int d = 0; d < dh; ++d) {
            a += to_f32(qi[d]) * to_f32(kj[d]);
            dp += to_f32(doi[d]) * to_f32(vj[d]);
        }
        const float p = expf(a * scale - lse[((int64_t)b * H + h) * S + i]);
        sp[i] = p;
        sds[i] = p * (dp - delta[((int64_t)b * H + h) * S + i]);
    }
    __syncthreads();
    for (int d = lane; d < dh; d += 64) {
        float dk = 0.0f, dv = 0.0f;
        for (int i = j; i < S; ++i) {
            dk += sds[i] * to_f32(base[i * ld + d]);
            dv += sp[i] * to_f32(dout[((int64_t)b * S + i) * D + h * dh + d]);
        }
        dqkv[((int64_t)b * S + j) * ld + D + h * dh + d] = from_f32<T>(dk * scale);
        dqkv[((int64_t)b * S + j) * ld + 2 * D + h * dh + d] = from_f32<T>(dv);
    }
}

// ---------------------------------------------------------------------------- MFMA path
// Exponentials use the hardware exp2 (one ulp; the library expf costs some 25 instructions and made the softmax, not the
// MFMAs, the bulk of the bf16 kernels).  Scores are kept in units of log 2 (scale * log2(e) folded into one factor), so
// that a probability costs one fused multiply-add and one exp2.
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
// 16 bytes in flight between global memory and LDS (a native vector: arrays of it stay in registers)
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// v plus another lane's (CTRL: the data-parallel-primitive control that names it)
template <int CTRL> __device__ __forceinline__ float add_lanes(float v) {
    return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// What depends on the element type and the features per head.
template <class T, int DH> struct Attn {
    static constexpr bool BF = sizeof(T) == 2;
    static constexpr int V = 16 / (int)sizeof(T);     // elements of a 16-byte chunk
    static constexpr int FT = DH / 32;                // 32-feature tiles
    static constexpr int NF = DH / (2 * V);           // fragments of a row: 16 features each in bf16, 8 in fp32
    static constexpr int P = DH + V;                  // LDS row pitch (16 bytes over: rows of a fragment on other banks)
    static constexpr int R = BF ? 64 : 32;            // rows of an LDS tile
    // bf16: the probabilities (and their gradients) enter the second product rounded to bf16 for 64 features per head; for 32, where
    // the kernels by rows used to take them in fp32, as the sum of three bf16 terms, which is as exact.
    static constexpr int TERMS = DH == 32 ? 3 : 1;
    typedef typename Frag<T>::type frag_t;

    // Fragment t of 32 rows (lane: row lane % 32, V features from 2 V t + V (lane / 32)): from global memory (rows
    // clamped to the last valid one) or from an LDS tile.
    static __device__ __forceinline__ frag_t gfrag(const T* base, int64_t ld, int row, int max_row, int t, int lane) {
        int r = row + (lane & 31);
        r = r < max_row ? r : max_row - 1;
        return *reinterpret_cast<const frag_t*>(base + r * ld + t * 2 * V + (lane >> 5) * V);
    }
    static __device__ __forceinline__ frag_t lfrag(const T* tile, int row0, int t, int lane) {
        return *reinterpret_cast<const frag_t*>(tile + (row0 + (lane & 31)) * P + t * 2 * V + (lane >> 5) * V);
    }
    // acc += rows of a times rows of b over one fragment's features
    static __device__ __forceinline__ f32x16_t mul(frag_t a, frag_t b, f32x16_t acc) {
        if constexpr (BF) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
            return acc;
        }
    }
    // out[i] += transposed tile rows r0 .. r0+31 (features 32 i ..) times p, whose accumulator registers run over those
    // rows: register r of a lane in half h belongs to row r0 + 8 (r / 4) + 4 h + r % 4.
    static __device__ __forceinline__ void mul_t(const T* tile, int r0, const f32x16_t& p, f32x16_t (&out)[FT], int lane) {
        if constexpr (BF) {
            typedef __attribute__((address_space(3))) s16x4_t* lds_ptr_t;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bf16x8_t pf[TERMS];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float rest = p[8 * t + e];
#pragma unroll
                    for (int k = 0; k < TERMS; ++k) {
                        pf[k][e] = (bf16_t)rest;
                        rest -= (float)pf[k][e];
                    }
                }
#pragma unroll
                for (int i = 0; i < FT; ++i) {
                    // two transpose reads of 4 rows each: slot (half, e) is row r0 + 16 t + 8 (e / 4) + 4 half + e % 4
                    const int row = r0 + 16 * t + 4 * (lane >> 5) + ((lane & 15) >> 2);
                    const int col = 32 * i + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
                    const T* p0 = tile + row * P + col;
                    union { s16x4_t h[2]; bf16x8_t v; } u;
                    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p0));
                    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p0 + 8 * P));
#pragma unroll
                    for (int k = TERMS - 1; k >= 0; --k) out[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u.v, pf[k], out[i], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int i = 0; i < FT; ++i) {
                    const T a = tile[(r0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * P + 32 * i + (lane & 31)];
                    out[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, p[r], out[i], 0, 0, 0);
                }
        }
    }
    // four consecutive features of a row
    static __device__ __forceinline__ void store4(T* p, float a, float b, float c, float d) {
        if constexpr (BF) {
            union { bf16_t hv[4]; uint2 u; } pk;
            pk.hv[0] = (bf16_t)a; pk.hv[1] = (bf16_t)b; pk.hv[2] = (bf16_t)c; pk.hv[3] = (bf16_t)d;
            *reinterpret_cast<uint2*>(p) = pk.u;
        } else *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
    }
    // a result with features along the registers, times f, to one row
    static __device__ __forceinline__ void store_row(T* row, const f32x16_t (&v)[FT], float f, int half) {
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                store4(row + 32 * i + 8 * g + 4 * half, v[i][4 * g] * f, v[i][4 * g + 1] * f, v[i][4 * g + 2] * f, v[i][4 * g + 3] * f);
    }
    // Cooperative copy of R rows into an LDS tile in two halves, so that the global loads of the next tile are in flight
    // while the current one is multiplied: fetch() issues the loads, put() writes them to LDS.  Rows >= max_row are clamped.
    template <int NT> struct Fetch {
        static constexpr int C = DH / V, N = (R * C + NT - 1) / NT;   // chunks of a row, chunks of a thread
        u32x4_t r[N];
        __device__ __forceinline__ void fetch(const T* base, int64_t ld, int row0, int max_row, int tid) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int c = tid + i * NT;
                int row = row0 + c / C;
                row = row < max_row ? row : max_row - 1;
                r[i] = *reinterpret_cast<const u32x4_t*>(base + row * ld + (c % C) * V);
            }
        }
        __device__ __forceinline__ void put(T* tile, int tid) const {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int c = tid + i * NT;
                if (R * C % NT == 0 || c < R * C) *reinterpret_cast<u32x4_t*>(tile + (c / C) * P + (c % C) * V) = r[i];
            }
        }
        // dots[row] = the row times the other one's, summed over the C neighbouring lanes that hold it
        __device__ __forceinline__ void put_dots(const Fetch& other, float* dots, int tid) const {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const frag_t x = __builtin_bit_cast(frag_t, r[i]), y = __builtin_bit_cast(frag_t, other.r[i]);
                float d = 0.0f;
#pragma unroll
                for (int e = 0; e < V; ++e) d = fmaf((float)x[e], (float)y[e], d);
                d = add_lanes<0xB1>(d);                       // lanes 1 apart
                d = add_lanes<0x4E>(d);                       // 2 apart
                if constexpr (C >= 8) d = add_lanes<0x141>(d);    // the other four of eight
                if constexpr (C >= 16) d = add_lanes<0x140>(d);   // the other eight of sixteen
                const int c = tid + i * NT;
                if (c % C == 0 && (R * C % NT == 0 || c < R * C)) dots[c / C] = d;
            }
        }
    };
};

template <int FT> __device__ __forceinline__ void clear(f32x16_t (&v)[FT]) {
#pragma unroll
    for (int i = 0; i < FT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) v[i][r] = 0.0f;
}

// N 32-key blocks of the running softmax of 32 queries (one per lane pair; keys along the registers).  st holds the
// raw scores q.k and leaves as unnormalised probabilities; m_run (in units of log 2) and l_run are the running
// maximum and sum, ot the running output, rescaled here.  MASK: keys after the query are excluded (the first block's
// first key is kb).  Blocks below the diagonal skip the three mask instructions per element.
template <bool MASK, int N, int FT>
__device__ __forceinline__ void softmax_blocks(f32x16_t (&st)[N], int kb, int q, int half, float scale2, float& m_run, float& l_run,
                                               f32x16_t (&ot)[FT]) {
    float mx[N], ls[N];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        mx[n] = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if constexpr (MASK) {
                const int key = kb + 32 * n + 8 * (r >> 2) + 4 * half + (r & 3);
                st[n][r] = key <= q ? st[n][r] : -INFINITY;
            }
            mx[n] = fmaxf(mx[n], st[n][r]);
        }
    }
    float mt = N == 2 ? fmaxf(mx[0], mx[N - 1]) : mx[0];
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    const float m_new = fmaxf(m_run, mt * scale2);       // scale2 > 0: the maximum commutes with the scaling
    const float m_use = m_new == -INFINITY ? 0.0f : m_new;   // a query with no key yet keeps zeros
    const float alpha = exp2_hw(m_run - m_use);
#pragma unroll
    for (int n = 0; n < N; ++n) {
        ls[n] = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            st[n][r] = exp2_hw(fmaf(st[n][r], scale2, -m_use));
            ls[n] += st[n][r];
        }
    }
    l_run = l_run * alpha + (N == 2 ? ls[0] + ls[N - 1] : ls[0]);
    m_run = m_new;
#pragma unroll
    for (int i = 0; i < FT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) ot[i][r] *= alpha;
}

// ---- results that are not finite ----
// The kernels below multiply whole 32 x 32 blocks: on the diagonal, and past the end of the sequence, a probability of zero
// meets rows that the query (or key) does not see, and an infinity or a NaN there (0 * inf) would reach results that do not
// depend on it; where probabilities are a sum of bf16 terms, a term of zero does the same to a row that is seen.  Rows of the
// result that are not finite although their statistics are (not_finite_rows) are therefore formed again, by rows
// and over the visible pairs alone, with the probabilities in fp32.  Finite data pay one three-operand maximum (the kind that
// keeps a NaN) for two result registers.
template <int FT> __device__ __forceinline__ uint32_t not_finite_rows(const f32x16_t (&v)[FT], bool statistics_ok) {
    float z[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < FT; ++i)
#pragma unroll
        for (int r = 0; r < 16; r += 2)
            z[(r >> 1) & 1] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(z[(r >> 1) & 1], __builtin_fabsf(v[i][r])), __builtin_fabsf(v[i][r + 1]));
    const uint64_t lanes = __ballot(!(__builtin_elementwise_maximum(z[0], z[1]) < INFINITY) && statistics_ok);
    return (uint32_t)(lanes | (lanes >> 32));   // (a lane pair holds a row)
}

template <class T, int DH> __device__ __forceinline__ float row_dot(const T* a, const T* b) {
    typedef Attn<T, DH> X;
    float s = 0.0f;
#pragma unroll 1
    for (int c = 0; c < DH; c += X::V) {
        const typename X::frag_t x = *reinterpret_cast<const typename X::frag_t*>(a + c), y = *reinterpret_cast<const typename X::frag_t*>(b + c);
#pragma unroll
        for (int e = 0; e < X::V; ++e) s = fmaf((float)x[e], (float)y[e], s);
    }
    return s;
}

// One query's output by a whole wave: a lane to each key of 64, then a lane to each feature.  m (in units of log 2) and l: the
// query's maximum and sum.
template <class T, int DH>
__device__ __forceinline__ void output_row(const T* base, int64_t ld, int D, int q, float scale2, float m, float l, T* out, int lane) {
    const int f = lane % DH;
    float a = 0.0f;
#pragma unroll 1
    for (int j0 = 0; j0 <= q; j0 += 64) {
        const int n = min(64, q + 1 - j0);
        const float p = exp2_hw(fmaf(row_dot<T, DH>(base + q * ld, base + D + (j0 + min(lane, n - 1)) * ld), scale2, -m));
#pragma unroll 1
        for (int t = 0; t < n; ++t) a = fmaf(__shfl(p, t, 64), (float)base[2 * D + (j0 + t) * ld + f], a);
    }
    if (lane < DH) out[f] = (T)(a / l);
}

// One query's gradient.  dout: the output gradient's rows of this (batch, head), D elements apart; L2: log-sum-exp in units of log 2.
template <class T, int DH>
__device__ __forceinline__ void query_gradient_row(const T* base, const T* dout, int64_t ld, int D, int q, float scale, float L2, float dl, T* dq, int lane) {
    const int f = lane % DH;
    const float scale2 = scale * kLog2e;
    float a = 0.0f;
#pragma unroll 1
    for (int j0 = 0; j0 <= q; j0 += 64) {
        const int n = min(64, q + 1 - j0);
        const T* kj = base + D + (j0 + min(lane, n - 1)) * ld;
        const float p = exp2_hw(fmaf(row_dot<T, DH>(base + q * ld, kj), scale2, -L2));
        const float ds = p * (row_dot<T, DH>(dout + (int64_t)q * D, kj + D) - dl);
#pragma unroll 1
        for (int t = 0; t < n; ++t) a = fmaf(__shfl(ds, t, 64), (float)base[D + (j0 + t) * ld + f], a);
    }
    if (lane < DH) dq[f] = (T)(a * scale);
}

// One key's and value's gradients, over the queries from that position on.  o: the outputs' rows, as dout's; lse: the statistics of this (batch, head).
template <class T, int DH>
__device__ __forceinline__ void key_value_gradient_row(const T* base, const T* o, const T* dout, int64_t ld, int D, int S, int key, float scale,
                                                       const float* lse, T* dk_row, T* dv_row, int lane) {
    const int f = lane % DH;
    const float scale2 = scale * kLog2e;
    float dk = 0.0f, dv = 0.0f;
#pragma unroll 1
    for (int i0 = key; i0 < S; i0 += 64) {
        const int n = min(64, S - i0), i = i0 + min(lane, n - 1);
        const float p = exp2_hw(fmaf(row_dot<T, DH>(base + D + key * ld, base + i * ld), scale2, -lse[i] * kLog2e));
        const float ds = p * (row_dot<T, DH>(base + 2 * D + key * ld, dout + (int64_t)i * D) - row_dot<T, DH>(o + (int64_t)i * D, dout + (int64_t)i * D));
#pragma unroll 1
        for (int t = 0; t < n; ++t) {
            dk = fmaf(__shfl(ds, t, 64), (float)base[(i0 + t) * ld + f], dk);
            dv = fmaf(__shfl(p, t, 64), (float)dout[(int64_t)(i0 + t) * D + f], dv);
        }
    }
    if (lane < DH) {
        dk_row[f] = (T)(dk * scale);
        dv_row[f] = (T)dv;
    }
}

// Workgroups go to the 8 XCDs (each with its own L2) round-robin in launch order (x fastest, then y, then z).  Hand
// every XCD a contiguous run of that order instead: the query (or key) blocks of one (batch, head) then sit on one XCD,
// and the keys and values (queries and output gradients) they all read come in from memory once, not once per XCD.
__device__ __forceinline__ void xcd_local_block(int& x, int& y, int& z) {
    const int gx = gridDim.x, gy = gridDim.y, plane = gx * gy, total = plane * gridDim.z;
    x = blockIdx.x; y = blockIdx.y; z = blockIdx.z;
    if (total < 16) return;
    const int lin = (z * gy + y) * gx + x;
    const int xcd = lin & 7, idx = lin >> 3, q = total >> 3, r = total & 7;
    int moved = xcd * q + min(xcd, r) + idx;
    z = moved / plane;
    moved -= z * plane;
    y = moved / gx;
    x = moved - y * gx;
}

// The same for grids of (slots per (batch, head) pair x heads, batches), whose workgroups differ in their way along the diagonal: an XCD gets
// an eighth of the pairs, and slot 0, which has the longest way, of all of them first.
__device__ __forceinline__ void longest_first(int slots, int H, int& slot, int& h, int& b) {
    const int total = gridDim.x * gridDim.y, lin = blockIdx.y * gridDim.x + blockIdx.x, xcd = lin & 7;
    const int u = total < 16 ? lin : xcd * (total >> 3) + min(xcd, total & 7) + (lin >> 3);
    const int pairs = gridDim.y * H, group = max(1, pairs >> 3), per = slots * group;
    const int g = u / per, r = u - g * per, n = min(group, pairs - g * group);
    slot = r / n;
    const int pair = g * group + (r - slot * n);
    b = pair / H;
    h = pair - b * H;
}

// Forward.  A workgroup's NW waves own 32 * NW query rows of one (batch, head).  Bound by latency, as the gradients below, and for the same
// reasons: a bf16 tile's two blocks of 32 keys go side by side, with one rescaling of the output for both, and the longest way comes first.  Blocks one
// after the other in eight waves, and this (us), positions x heads x sequences: 512 x 12 x 16 27 and 19, x 8 17.0 and 13.3; 2048 x 8 x 8 86 and 58;
// 333 x 8 x 12 12.7 and 10.3; 512 x 8 x 16 of 32 features 19.5 and 15.0.  (Side by side in the kernel below: 9.9 and 12.1 for 512 x 12 x 2, whose waves
// have four blocks each at most and would have two pairs.)
template <class T, int DH, int NW>
__global__ __launch_bounds__(64 * NW, 2) void attn_fwd_mfma_kernel(const T* __restrict__ qkv, T* __restrict__ o, float* __restrict__ lse, int S,
                                                                int D, int H, int blocks, float scale) {
    typedef Attn<T, DH> X;
    __shared__ __attribute__((aligned(16))) T sKb[2][X::R * X::P];
    __shared__ __attribute__((aligned(16))) T sVb[2][X::R * X::P];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    int slot, h, b;
    longest_first(blocks, H, slot, h, b);
    const int qb = blocks - 1 - slot;
    const int64_t ld = 3 * (int64_t)D;
    const T* base = qkv + (int64_t)b * S * ld + h * DH;
    const int q0 = (qb * NW + wave) * 32;
    const int q = q0 + (lane & 31);
    typename X::template Fetch<64 * NW> fk, fv;
    fk.fetch(base + D, ld, 0, S, tid);
    fv.fetch(base + 2 * D, ld, 0, S, tid);
    typename X::frag_t qf[X::NF];
#pragma unroll
    for (int t = 0; t < X::NF; ++t) qf[t] = X::gfrag(base, ld, q0, S, t, lane);
    f32x16_t ot[X::FT];
    clear(ot);
    float m_run = -INFINITY, l_run = 0.0f;
    const float scale2 = scale * kLog2e;
    const int kv_end = min(S, (qb + 1) * NW * 32);
    fk.put(sKb[0], tid);
    fv.put(sVb[0], tid);
    __syncthreads();
    for (int kv0 = 0, it = 0; kv0 < kv_end; kv0 += X::R, ++it) {
        const T* sK = sKb[it & 1];
        const T* sV = sVb[it & 1];
        // the next tile's loads fly while this one is multiplied (past the last tile they re-read clamped, valid rows
        // and the copy lands in the buffer that nobody reads again)
        fk.fetch(base + D, ld, kv0 + X::R, S, tid);
        fv.fetch(base + 2 * D, ld, kv0 + X::R, S, tid);
        // the first N blocks of 32 keys of the tile; MASK: the last of them straddles the diagonal
        auto key_blocks = [&](auto nc, auto maskc) {
            constexpr int N = decltype(nc)::value;
            f32x16_t st[N];
            clear(st);
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int t = 0; t < X::NF; ++t) st[n] = X::mul(X::lfrag(sK, 32 * n, t, lane), qf[t], st[n]);
            softmax_blocks<decltype(maskc)::value>(st, kv0, q, half, scale2, m_run, l_run, ot);
#pragma unroll
            for (int n = 0; n < N; ++n) X::mul_t(sV, 32 * n, st[n], ot, lane);
        };
        constexpr int NB = X::R / 32;
        const std::integral_constant<int, NB> all;
        if (kv0 + X::R <= q0) key_blocks(all, std::false_type());
        else if (kv0 + X::R - 32 == q0) key_blocks(all, std::true_type());
        else if (NB == 2 && kv0 == q0) key_blocks(std::integral_constant<int, 1>(), std::true_type());
        fk.put(sKb[(it + 1) & 1], tid);   // the other buffer was last read before the previous barrier
        fv.put(sVb[(it + 1) & 1], tid);
        __syncthreads();
    }
    const float l = l_run + __shfl_xor(l_run, 32, 64);
    const uint32_t redo = not_finite_rows(ot, l > 0.0f);
    if (q < S) {
        if (!((redo >> (lane & 31)) & 1)) X::store_row(o + ((int64_t)b * S + q) * D + h * DH, ot, 1.0f / l, half);
        if (half == 0) lse[((int64_t)b * H + h) * S + q] = fmaf(m_run, kLn2, logf(l));
    }
    for (uint32_t todo = redo; todo; todo &= todo - 1) {
        const int r = __builtin_ctz(todo);
        if (q0 + r < S) output_row<T, DH>(base, ld, D, q0 + r, scale2, __shfl(m_run, r, 64), __shfl(l, r, 64), o + ((int64_t)b * S + q0 + r) * D + h * DH, lane);
    }
}

// Forward for launches with few (batch, head) pairs, where the kernel above leaves most of the chip idle and its
// longest workgroup walks the whole key range alone.  A workgroup owns 32 query rows; its NW waves take the 32-key
// blocks up to the diagonal in turn (wave w: blocks w, w + NW, ...) with their own running statistics, and the
// partial results are merged at the end: O = sum_w e^{m_w - m} O_w, l = sum_w e^{m_w - m} l_w, m = max_w m_w.
// Nothing is shared between the waves inside the loop, so there is no workgroup barrier in it: K fragments come
// straight from global memory, V passes through a wave-private LDS tile.
template <class T, int DH, int NW>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 2 ? 3 : 1) void attn_fwd_split_kernel(const T* __restrict__ qkv, T* __restrict__ o, float* __restrict__ lse, int S,
                                                                 int D, int H, float scale) {
    typedef Attn<T, DH> X;
    constexpr int FT = X::FT, C = DH / X::V, NV = 32 * C / 64;   // 16-byte chunks of a row, chunks per lane of 32 rows
    __shared__ __attribute__((aligned(16))) T sVw[NW][32 * X::P];
    __shared__ float sOw[NW - 1][16 * FT][64];
    __shared__ float sMw[NW - 1][32], sLw[NW - 1][32];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    int bx, h, b;
    xcd_local_block(bx, h, b);
    const int qb = gridDim.x - 1 - bx;
    const int64_t ld = 3 * (int64_t)D;
    const T* base = qkv + (int64_t)b * S * ld + h * DH;
    const int q0 = qb * 32;
    const int q = q0 + (lane & 31);
    T* const sV = sVw[wave];
    typename X::frag_t qf[X::NF], kn[X::NF];
    u32x4_t vn[NV];
    auto fetch = [&](int j) {   // rows are clamped: a fetch past the diagonal re-reads valid rows and is never used
#pragma unroll
        for (int t = 0; t < X::NF; ++t) kn[t] = X::gfrag(base + D, ld, 32 * j, S, t, lane);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i;
            int row = 32 * j + c / C;
            row = row < S ? row : S - 1;
            vn[i] = *reinterpret_cast<const u32x4_t*>(base + 2 * D + row * ld + (c % C) * X::V);
        }
    };
    fetch(wave);
#pragma unroll
    for (int t = 0; t < X::NF; ++t) qf[t] = X::gfrag(base, ld, q0, S, t, lane);
    f32x16_t ot[FT];
    clear(ot);
    float m_run = -INFINITY, l_run = 0.0f;
    const float scale2 = scale * kLog2e;
    for (int j = wave; j <= qb; j += NW) {
        typename X::frag_t kf[X::NF];
#pragma unroll
        for (int t = 0; t < X::NF; ++t) kf[t] = kn[t];
        // LDS serves a wave's accesses in order: the reads of the previous block are done before these writes
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int c = lane + 64 * i;
            *reinterpret_cast<u32x4_t*>(sV + (c / C) * X::P + (c % C) * X::V) = vn[i];
        }
        __builtin_amdgcn_wave_barrier();
        fetch(j + NW);
        const int kb = 32 * j;
        f32x16_t st[1];
        clear(st);
#pragma unroll
        for (int t = 0; t < X::NF; ++t) st[0] = X::mul(kf[t], qf[t], st[0]);
        if (kb + 31 <= q0) softmax_blocks<false>(st, kb, q, half, scale2, m_run, l_run, ot);
        else softmax_blocks<true>(st, kb, q, half, scale2, m_run, l_run, ot);
        X::mul_t(sV, 0, st[0], ot, lane);
    }
    float l = l_run + __shfl_xor(l_run, 32, 64);
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) sOw[wave - 1][16 * i + r][lane] = ot[i][r];
        if (half == 0) {
            sMw[wave - 1][lane] = m_run;
            sLw[wave - 1][lane] = l;
        }
    }
    __syncthreads();
    if (wave != 0) return;
    // wave 0 always owns key block 0, which every query sees: its maximum is finite
    float m = m_run;
#pragma unroll
    for (int w = 0; w < NW - 1; ++w) m = fmaxf(m, sMw[w][lane & 31]);
    const float f0 = exp2_hw(m_run - m);
    l *= f0;
#pragma unroll
    for (int i = 0; i < FT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) ot[i][r] *= f0;
#pragma unroll
    for (int w = 0; w < NW - 1; ++w) {
        const float fw = exp2_hw(sMw[w][lane & 31] - m);   // a wave that had no block holds -inf: factor 0
        l += fw * sLw[w][lane & 31];
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) ot[i][r] += fw * sOw[w][16 * i + r][lane];
    }
    const uint32_t redo = not_finite_rows(ot, l > 0.0f);
    if (q < S) {
        if (!((redo >> (lane & 31)) & 1)) X::store_row(o + ((int64_t)b * S + q) * D + h * DH, ot, 1.0f / l, half);
        if (half == 0) lse[((int64_t)b * H + h) * S + q] = fmaf(m, kLn2, logf(l));
    }
    for (uint32_t todo = redo; todo; todo &= todo - 1) {
        const int r = __builtin_ctz(todo);
        if (q0 + r < S) output_row<T, DH>(base, ld, D, q0 + r, scale2, __shfl(m, r, 64), __shfl(l, r, 64), o + ((int64_t)b * S + q0 + r) * D + h * DH, lane);
    }
}

// Gradients: one launch, in which a workgroup of NW waves forms the gradient of 32 NW queries or those of 32 NW keys and values.  Both read
// tiles of R rows through LDS, the next one's loads in flight; both form delta[q] = dO[q] . O[q] for themselves, which costs the keys' workgroups
// a sixth more vector work and spares the pass a second launch behind the first, with its own way to the end of the longest diagonal.
// What bounds them is latency: products, exponentials and products again that depend on each other, in two waves per SIMD, all that the
// registers allow (28 multiplies and about 260 vector instructions for 32 x 32 pairs take 10 and 13 us of the 55 for 16 x 12 heads over 512 positions).
// So the two 32-row blocks of a bf16 tile go side by side, whose chains fill each other's gaps, a workgroup has four waves
// (eight wait for the one with the longest way), and the workgroups with the longest way start first.  Two kernels with the blocks one after the
// other and eight / four / two waves, and this (us), bf16, positions x heads x sequences: 512 x 12 x 16 87 and 55, x 2 33 and 20; 1024 x 12 x 2 59 and
// 35; 2048 x 8 x 8 255 and 169; 333 x 8 x 12 35 and 23; 96 x 8 x 64 32 and 24; 32 features per head, 512 x 8 x 16 53 and 36, 128 x 4 x 16 13.2 and 7.9;
// fp32, 512 x 4 x 4, 32 features 83 and 48; 256 x 8 x 8, 64 features 75 and 49; 32 x 2 x 16 10.4 and 6.2.
template <class T, int DH, int NW> struct AttnBwdTiles {
    typedef Attn<T, DH> X;
    T a[2][X::R * X::P], b[2][X::R * X::P];   // keys and values, or queries and output gradients
    float L2[2][X::R], delta[2][X::R];        // log-sum-exp (in units of log 2) and delta of the queries
};

// Query gradient.  Same arrangement as the forward pass: P^T and dS^T have keys along the registers.
template <class T, int DH, int NW>
__device__ __forceinline__ void attn_bwd_q(AttnBwdTiles<T, DH, NW>& sm, const T* __restrict__ base, const T* __restrict__ ob, const T* __restrict__ dob,
                                           const float* __restrict__ lse, T* __restrict__ dbase, int qb, int S, int D, float scale) {
    typedef Attn<T, DH> X;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int64_t ld = 3 * (int64_t)D;
    typename X::template Fetch<64 * NW> fk, fv;
    fk.fetch(base + D, ld, 0, S, tid);
    fv.fetch(base + 2 * D, ld, 0, S, tid);
    const int q0 = (qb * NW + wave) * 32;
    const int q = q0 + (lane & 31);
    const int qc = q < S ? q : S - 1;
    typename X::frag_t qf[X::NF], dof[X::NF], of[X::NF];
#pragma unroll
    for (int t = 0; t < X::NF; ++t) {
        qf[t] = X::gfrag(base, ld, q0, S, t, lane);
        dof[t] = X::gfrag(dob, D, q0, S, t, lane);
        of[t] = X::gfrag(ob, D, q0, S, t, lane);
    }
    const float L2 = lse[qc] * kLog2e;
    float dl = 0.0f;
#pragma unroll
    for (int t = 0; t < X::NF; ++t)
#pragma unroll
        for (int e = 0; e < X::V; ++e) dl += (float)of[t][e] * (float)dof[t][e];
    dl += __shfl_xor(dl, 32, 64);
    const float scale2 = scale * kLog2e;
    f32x16_t dq[X::FT];
    clear(dq);
    const int kv_end = min(S, (qb + 1) * NW * 32);
    fk.put(sm.a[0], tid);
    fv.put(sm.b[0], tid);
    __syncthreads();
    for (int kv0 = 0, it = 0; kv0 < kv_end; kv0 += X::R, ++it) {
        const T* sK = sm.a[it & 1];
        const T* sV = sm.b[it & 1];
        fk.fetch(base + D, ld, kv0 + X::R, S, tid);
        fv.fetch(base + 2 * D, ld, kv0 + X::R, S, tid);
        // the first N blocks of 32 keys of the tile; MASK: the last of them straddles the diagonal
        auto blocks = [&](auto nc, auto maskc) {
            constexpr int N = decltype(nc)::value;
            constexpr bool MASK = decltype(maskc)::value;
            f32x16_t st[N], dp[N];
            clear(st);
            clear(dp);
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int t = 0; t < X::NF; ++t) {
                    st[n] = X::mul(X::lfrag(sK, 32 * n, t, lane), qf[t], st[n]);
                    dp[n] = X::mul(X::lfrag(sV, 32 * n, t, lane), dof[t], dp[n]);
                }
#pragma unroll
            for (int n = 0; n < N; ++n) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float p = exp2_hw(fmaf(st[n][r], scale2, -L2));
                    if (MASK && n == N - 1) p = kv0 + 32 * n + 8 * (r >> 2) + 4 * half + (r & 3) <= q ? p : 0.0f;
                    st[n][r] = p * (dp[n][r] - dl);
                }
                X::mul_t(sK, 32 * n, st[n], dq, lane);
            }
        };
        constexpr int NB = X::R / 32;
        const std::integral_constant<int, NB> all;
        if (kv0 + X::R <= q0) blocks(all, std::false_type());
        else if (kv0 + X::R - 32 == q0) blocks(all, std::true_type());
        else if (NB == 2 && kv0 == q0) blocks(std::integral_constant<int, 1>(), std::true_type());
        fk.put(sm.a[(it + 1) & 1], tid);
        fv.put(sm.b[(it + 1) & 1], tid);
        __syncthreads();
    }
    // (a log-sum-exp that is not finite, or a delta that is NaN, stands in every term of the row)
    const uint32_t redo = not_finite_rows(dq, fabsf(L2) < INFINITY && dl == dl);
    if (q < S && !((redo >> (lane & 31)) & 1)) X::store_row(dbase + q * ld, dq, scale, half);
    for (uint32_t todo = redo; todo; todo &= todo - 1) {
        const int r = __builtin_ctz(todo);
        if (q0 + r < S)
            query_gradient_row<T, DH>(base, dob, ld, D, q0 + r, scale, __shfl(L2, r, 64), __shfl(dl, r, 64), dbase + (q0 + r) * ld, lane);
    }
}

// Key and value gradients.  A wave owns 32 keys (lanes); queries run along the accumulator registers, so the
// per-query statistics (log-sum-exp, delta) are read per register from LDS.
template <class T, int DH, int NW>
__device__ __forceinline__ void attn_bwd_kv(AttnBwdTiles<T, DH, NW>& sm, const T* __restrict__ base, const T* __restrict__ ob, const T* __restrict__ dob,
                                            const float* __restrict__ lse, T* __restrict__ dbase, int kblk, int S, int D, float scale) {
    typedef Attn<T, DH> X;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int64_t ld = 3 * (int64_t)D;
    const int k0 = (kblk * NW + wave) * 32;
    const int key = k0 + (lane & 31);
    const float scale2 = scale * kLog2e;
    typename X::frag_t kf[X::NF], vf[X::NF];
#pragma unroll
    for (int t = 0; t < X::NF; ++t) {
        kf[t] = X::gfrag(base + D, ld, k0, S, t, lane);
        vf[t] = X::gfrag(base + 2 * D, ld, k0, S, t, lane);
    }
    f32x16_t dk[X::FT], dv[X::FT];
    clear(dk);
    clear(dv);
    const int qstart = (kblk * NW * 32) / X::R * X::R;   // first query block that can see a key of this workgroup
    typename X::template Fetch<64 * NW> fq, fg, fo;
    float pl = 0.0f;   // log-sum-exp of query qb0 + tid (threads 0 .. R-1)
    auto fetch = [&](int qb0) {
        fq.fetch(base, ld, qb0, S, tid);
        fg.fetch(dob, D, qb0, S, tid);
        fo.fetch(ob, D, qb0, S, tid);
        if (tid < X::R) pl = lse[qb0 + tid < S ? qb0 + tid : S - 1];
    };
    auto put = [&](int buf) {
        fq.put(sm.a[buf], tid);
        fg.put(sm.b[buf], tid);
        fo.put_dots(fg, sm.delta[buf], tid);
        if (tid < X::R) sm.L2[buf][tid] = pl * kLog2e;
    };
    fetch(qstart);
    put(0);
    __syncthreads();
    for (int qb0 = qstart, it = 0; qb0 < S; qb0 += X::R, ++it) {
        const T* sQ = sm.a[it & 1];
        const T* sO = sm.b[it & 1];
        const float* sL = sm.L2[it & 1];
        const float* sDl = sm.delta[it & 1];
        fetch(qb0 + X::R);
        // the last N blocks of 32 queries of the tile; MASK: some of their queries do not see all keys of this wave, or do not exist
        auto blocks = [&](auto nc, auto maskc) {
            constexpr int N = decltype(nc)::value, B0 = X::R / 32 - N;
            constexpr bool MASK = decltype(maskc)::value;
            f32x16_t st[N], dp[N];
            clear(st);
            clear(dp);
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int t = 0; t < X::NF; ++t) {
                    st[n] = X::mul(X::lfrag(sQ, 32 * (B0 + n), t, lane), kf[t], st[n]);
                    dp[n] = X::mul(X::lfrag(sO, 32 * (B0 + n), t, lane), vf[t], dp[n]);
                }
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int row = 32 * (B0 + n);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    // statistics of the 4 consecutive queries of a register group in one LDS read each
                    const float4 l4 = *reinterpret_cast<const float4*>(sL + row + 8 * g + 4 * half);
                    const float4 d4 = *reinterpret_cast<const float4*>(sDl + row + 8 * g + 4 * half);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r = 4 * g + e;
                        const float Lq = e == 0 ? l4.x : e == 1 ? l4.y : e == 2 ? l4.z : l4.w;
                        const float Dq = e == 0 ? d4.x : e == 1 ? d4.y : e == 2 ? d4.z : d4.w;
                        float p = exp2_hw(fmaf(st[n][r], scale2, -Lq));
                        if (MASK) {
                            const int qq = qb0 + row + 8 * g + 4 * half + e;
                            p = (key <= qq && qq < S) ? p : 0.0f;
                        }
                        st[n][r] = p;
                        dp[n][r] = p * (dp[n][r] - Dq);
                    }
                }
                X::mul_t(sO, row, st[n], dv, lane);
                X::mul_t(sQ, row, dp[n], dk, lane);
            }
        };
        constexpr int NB = X::R / 32;
        const std::integral_constant<int, NB> all;
        if (qb0 > k0 && qb0 + X::R <= S) blocks(all, std::false_type());
        else if (qb0 >= k0) blocks(all, std::true_type());
        else if (NB == 2 && qb0 + 32 == k0) blocks(std::integral_constant<int, 1>(), std::true_type());
        put((it + 1) & 1);
        __syncthreads();
    }
    const uint32_t dk_rows = not_finite_rows(dk, true), dv_rows = not_finite_rows(dv, true);
    uint32_t redo = dk_rows | dv_rows;
    if (redo) {
        // every key sees the last query: a NaN in that one's log-sum-exp stands in every row of both gradients, one in its delta
        // in every row of the key gradient
        const float dl = row_dot<T, DH>(ob + (int64_t)(S - 1) * D, dob + (int64_t)(S - 1) * D);
        const bool lse_ok = lse[S - 1] == lse[S - 1], delta_ok = dl == dl;
        redo = (lse_ok && delta_ok ? dk_rows : 0) | (lse_ok ? dv_rows : 0);
    }
    if (key < S && !((redo >> (lane & 31)) & 1)) {
        T* drow = dbase + key * ld;
        X::store_row(drow + D, dk, scale, half);
        X::store_row(drow + 2 * D, dv, 1.0f, half);
    }
    for (uint32_t todo = redo; todo; todo &= todo - 1) {
        const int r = __builtin_ctz(todo);
        T* drow = dbase + (k0 + r) * ld;
        if (k0 + r < S) key_value_gradient_row<T, DH>(base, ob, dob, ld, D, S, k0 + r, scale, lse, drow + D, drow + 2 * D, lane);
    }
}

template <class T, int DH, int NW>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 4 ? 1 : 2) void attn_bwd_mfma_kernel(const T* __restrict__ qkv, const T* __restrict__ o,
                                                                   const T* __restrict__ dout, const float* __restrict__ lse, T* __restrict__ dqkv, int S, int D, int H,
                                                                   int blocks, float scale) {
    __shared__ __attribute__((aligned(16))) AttnBwdTiles<T, DH, NW> sm;
    int slot, h, b;
    longest_first(2 * blocks, H, slot, h, b);
    const T* base = qkv + (int64_t)b * S * 3 * D + h * DH;
    const T* ob = o + (int64_t)b * S * D + h * DH;
    const T* dob = dout + (int64_t)b * S * D + h * DH;
    T* dbase = dqkv + (int64_t)b * S * 3 * D + h * DH;
    lse += ((int64_t)b * H + h) * S;
    if (slot & 1) attn_bwd_q<T, DH, NW>(sm, base, ob, dob, lse, dbase, blocks - 1 - (slot >> 1), S, D, scale);
    else attn_bwd_kv<T, DH, NW>(sm, base, ob, dob, lse, dbase, slot >> 1, S, D, scale);
}

// (of the kernels that take a row at a time: heads of other sizes than 32 and 64 features, and these where an operand is not aligned, which a caller decides
// only with the pointers of a pass)
size_t attention_workspace_elems(int B, int S, int H) { return (size_t)B * S * H; }

// The kernel with the key range split over a workgroup's waves, where the tiled one has too few workgroups: its time is that of the longest way (3.5 us
// and 1 us per 64 keys in bf16) until there are more than a round of them.  Split and tiled (us), bf16, positions x heads x sequences: 512 x 12 x 1
// 6.6 and -, x 2 9.9 and 11.5, x 4 13.8 and 11.8, x 5 16.5 and 12.1; 1024 x 12 x 2 20.7 and 19.6; 2048 x 12 x 1 30.7 and 35; 128 x 4 x 16 with 32 features
// 4.0 and 5.5; fp32, 256 x 8 x 8 17.2 and 23.6, 512 x 4 x 4 9.9 and 25.5.  A single block of 32 keys leaves nothing to split: 32 x 2 x 16, fp32, 4.4 and 3.9.
// Four waves per workgroup of the tiled kernel in bf16 (two cover 64 rows; 8 and 4: 512 x 12 x 16 20.8 and 19.3, x 8 16.7 and 13.3, 2048 x 8 x 8 63
// and 58, 96 x 8 x 64 10.4 and 8.1).  fp32: the MFMAs take sixteen times as long, and workgroups stay small for balance along the diagonal.
template <class T, int DH>
static hipError_t forward_mfma(const T* qkv, T* o, float* lse, int B, int S, int D, int H, float scale, hipStream_t s) {
    const int64_t tiles = (int64_t)cdiv_at(S, 64) * B * H;
    const bool split = S > 32 && (sizeof(T) == 2 && S <= 1024 ? tiles < 256 : tiles < 512);
    if (split)
        return launch_timed(kcAttnFwd, attn_fwd_split_kernel<T, DH, 4>, dim3(cdiv_at(S, 32), H, B), dim3(256), 0, s, qkv, o, lse, S, D, H, scale);
    auto go = [&](auto nwc) {
        constexpr int NW = decltype(nwc)::value;
        const int blocks = cdiv_at(S, 32 * NW);
        return launch_timed(kcAttnFwd, attn_fwd_mfma_kernel<T, DH, NW>, dim3(blocks * H, B), dim3(64 * NW), 0, s, qkv, o, lse, S, D, H, blocks, scale);
    };
    if (S <= 64 || (sizeof(T) == 4 && (int64_t)cdiv_at(S, 128) * B * H < 1024)) return go(std::integral_constant<int, 2>{});
    return go(std::integral_constant<int, 4>{});
}

// Four waves per workgroup, or two where four would leave compute units without one (128 positions x 4 heads x 16 sequences in bf16 7.9 us
// against 8.8) and registers allow it: bf16 rows of 64 features are staged in twice the registers by half the waves, and spill (512 x 12 x 2 33 us against 20).
template <class T, int DH>
static hipError_t backward_mfma(const T* qkv, const T* o, const T* dout, const float* lse, T* dqkv, int B, int S, int D, int H, float scale, hipStream_t s) {
    auto go = [&](auto nwc) {
        constexpr int NW = decltype(nwc)::value;
        const int blocks = cdiv_at(S, 32 * NW);
        return launch_timed(kcAttnBwd, attn_bwd_mfma_kernel<T, DH, NW>, dim3(2 * blocks * H, B), dim3(64 * NW), 0, s, qkv, o, dout, lse, dqkv, S, D, H,
                            blocks, scale);
    };
    if constexpr (sizeof(T) == 4 || DH == 32)
        if ((int64_t)2 * cdiv_at(S, 128) * B * H < 256) return go(std::integral_constant<int, 2>{});
    return go(std::integral_constant<int, 4>{});
}

template <class T> static hipError_t forward_t(const T* qkv, T* o, float* lse, int B, int S, int D, int H, hipStream_t s) {
    const float scale = 1.0f / sqrtf((float)(D / H));
    const bool aligned = ((reinterpret_cast<uintptr_t>(qkv) | reinterpret_cast<uintptr_t>(o)) & 15) == 0;
    if (aligned && D == 64 * H) return forward_mfma<T, 64>(qkv, o, lse, B, S, D, H, scale, s);
    if (aligned && D == 32 * H) return forward_mfma<T, 32>(qkv, o, lse, B, S, D, H, scale, s);
    return launch_timed(kcAttnFwd, attn_fwd_row_kernel<T>, dim3(S, H, B), dim3(64), (unsigned)S * 4, s, qkv, o, lse, S, D, H, scale);
}

template <class T>
static hipError_t backward_t(const T* qkv, const T* o, const T* dout, const float* lse, float* delta, T* dqkv, int B, int S, int D, int H, hipStream_t s) {
    const float scale = 1.0f / sqrtf((float)(D / H));
    const bool aligned = ((reinterpret_cast<uintptr_t>(qkv) | reinterpret_cast<uintptr_t>(o) | reinterpret_cast<uintptr_t>(dout) |
                           reinterpret_cast<uintptr_t>(dqkv)) & 15) == 0;
    if (aligned && D == 64 * H) return backward_mfma<T, 64>(qkv, o, dout, lse, dqkv, B, S, D, H, scale, s);
    if (aligned && D == 32 * H) return backward_mfma<T, 32>(qkv, o, dout, lse, dqkv, B, S, D, H, scale, s);
    const int64_t BS = (int64_t)B * S;
    hipError_t e = launch_timed(kcAttnBwd, attn_delta_kernel<T>, dim3(cdiv_at(BS * H, 4)), dim3(256), 0, s, o, dout, delta, BS, S, D, H);
    if (e != hipSuccess) return e;
    const dim3 grid(S, H, B);
    e = launch_timed(kcAttnBwd, attn_bwd_q_row_kernel<T>, grid, dim3(64), (unsigned)S * 4, s, qkv, dout, lse, (const float*)delta, dqkv, S, D, H, scale);
    if (e != hipSuccess) return e;
    return launch_timed(kcAttnBwd, attn_bwd_kv_row_kernel<T>, grid, dim3(64), (unsigned)S * 8, s, qkv, dout, lse, (const float*)delta, dqkv, S, D, H, scale);
}

hipError_t attention_forward(int dtype, const void* qkv, void* o, float* lse, int B, int S, int D, int H, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    if (dtype == kBF16) return forward_t<bf16_t>((const bf16_t*)qkv, (bf16_t*)o, lse, B, S, D, H, s);
    return forward_t<float>((const float*)qkv, (float*)o, lse, B, S, D, H, s);
}

hipError_t attention_backward(int dtype, const void* qkv, const void* o, const void* dout, const float* lse, float* delta,
                              void* dqkv, int B, int S, int D, int H, hipStream_t s) {
    if (B <= 0) return hipSuccess;
    if (dtype == kBF16)
        return backward_t<bf16_t>((const bf16_t*)qkv, (const bf16_t*)o, (const bf16_t*)dout, lse, delta, (bf16_t*)dqkv, B, S, D, H, s);
    return backward_t<float>((const float*)qkv, (const float*)o, (const float*)dout, lse, delta, (float*)dqkv, B, S, D, H, s);
}

}  // namespace tmps
