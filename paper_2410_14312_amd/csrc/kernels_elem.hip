// Bandwidth-bound kernels of the stage step: softmax cross-entropy, momentum update,
// ReLU gradient mask, casts and small reductions.
#include "gemm.hip.h"
#include "kernels.h"
#include "wave.hip.h"

namespace tmps {

static inline int cdiv64(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------------- softmax cross-entropy
// One wave per row; 4 rows per block.  dlogits = (softmax - onehot) * inv_M, loss = lse - z[label].
template <typename TG>
__global__ __launch_bounds__(256) void softmax_ce_kernel(const float* __restrict__ logits,
                                                         const int32_t* __restrict__ labels,
                                                         TG* __restrict__ dlogits,
                                                         float* __restrict__ row_loss, int rows, int C,
                                                         float inv_M) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float* z = logits + (int64_t)row * C;
    float mx = -INFINITY;
    for (int c = lane; c < C; c += 64) mx = fmaxf(mx, z[c]);
    mx = wmax(mx);
    float sum = 0.0f;
    for (int c = lane; c < C; c += 64) sum += expf(z[c] - mx);
    sum = wsum(sum);
    const float inv = 1.0f / sum;
    const int label = labels[row];
    const bool label_ok = label >= 0 && label < C;  // an out-of-range label gives a NaN loss, never a wild read
    TG* g = dlogits + (int64_t)row * C;
    for (int c = lane; c < C; c += 64) {
        float p = expf(z[c] - mx) * inv;
        g[c] = from_f32<TG>((p - (c == label ? 1.0f : 0.0f)) * inv_M);
    }
    if (lane == 0) row_loss[row] = label_ok ? logf(sum) - (z[label] - mx) : NAN;
}

// Wide rows (a vocabulary): one 256-thread block per row.  First pass keeps a running (max, sum) per thread
// (online softmax), combined across the block; second pass writes the gradient.
template <typename TG>
__global__ __launch_bounds__(256) void softmax_ce_wide_kernel(const float* __restrict__ logits,
                                                              const int32_t* __restrict__ labels,
                                                              TG* __restrict__ dlogits, float* __restrict__ row_loss,
                                                              int C, float inv_M) {
    __shared__ float sm[4], ss[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const float* z = logits + row * C;
    float mx = -INFINITY, sum = 0.0f;
    for (int c = tid; c < C; c += 256) {
        const float v = z[c];
        if (v > mx) {
            sum = sum * expf(mx - v) + 1.0f;
            mx = v;
        } else {
            sum += expf(v - mx);
        }
    }
    const float wm = wmax(mx);
    sum = wsum(sum * expf(mx - wm));   // a thread that saw nothing has sum 0 and mx -inf: 0 * exp(-inf) = 0
    if (lane == 0) {
        sm[wave] = wm;
        ss[wave] = sum;
    }
    __syncthreads();
    const float bm = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
    float bs = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) bs += ss[w] * expf(sm[w] - bm);
    const float inv = 1.0f / bs;
    const int label = labels[row];
    const bool label_ok = label >= 0 && label < C;
    TG* g = dlogits + row * C;
    for (int c = tid; c < C; c += 256) {
        const float p = expf(z[c] - bm) * inv;
        g[c] = from_f32<TG>((p - (c == label ? 1.0f : 0.0f)) * inv_M);
    }
    if (tid == 0) row_loss[row] = label_ok ? logf(bs) - (z[label] - bm) : NAN;
}

// Wide rows that fit in LDS (C fp32 values, C % 4 == 0): one 1024-thread block per row reads the row from HBM ONCE,
// keeps it in LDS for the maximum, the sum and the gradient, and writes the gradient: algorithmic traffic exactly.
// A row of a large vocabulary takes most of a compute unit's LDS, so one workgroup is all a unit holds: 16 waves
// (not 4) keep enough loads in flight.  Exponentials on the hardware exp2 (a few ulp of fp32).
constexpr int kCeThreads = 1024;
template <typename TG>
__global__ __launch_bounds__(kCeThreads) void softmax_ce_lds_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                                    TG* __restrict__ dlogits, float* __restrict__ row_loss, int C,
                                                                    float inv_M) {
    extern __shared__ __attribute__((aligned(16))) float srow[];
    constexpr int NWV = kCeThreads / 64;
    __shared__ float sm[NWV], ss[NWV];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const float4* z4 = reinterpret_cast<const float4*>(logits + row * C);
    float4* s4 = reinterpret_cast<float4*>(srow);
    const int C4 = C >> 2;
    float mx = -INFINITY;
    for (int c = tid; c < C4; c += kCeThreads) {
        const float4 v = z4[c];
        s4[c] = v;
        mx = fmaxf(fmaxf(mx, fmaxf(v.x, v.y)), fmaxf(v.z, v.w));
    }
    mx = wmax(mx);
    if (lane == 0) sm[wave] = mx;
    __syncthreads();
    float bm = sm[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) bm = fmaxf(bm, sm[w]);
    float sum = 0.0f;
    for (int c = tid; c < C4; c += kCeThreads) {
        float4 v = s4[c];
        v.x = __expf(v.x - bm); v.y = __expf(v.y - bm); v.z = __expf(v.z - bm); v.w = __expf(v.w - bm);
        s4[c] = v;   // keep the exponentials: the gradient needs them again
        sum += (v.x + v.y) + (v.z + v.w);
    }
    sum = wsum(sum);
    if (lane == 0) ss[wave] = sum;
    __syncthreads();
    float bs = 0.0f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) bs += ss[w];
    const float inv = 1.0f / bs;
    const int label = labels[row];
    const bool label_ok = label >= 0 && label < C;
    TG* g = dlogits + row * C;
    for (int c = tid; c < C4; c += kCeThreads) {
        const float4 e = s4[c];
        float p[4] = {e.x * inv, e.y * inv, e.z * inv, e.w * inv};
        const int c0 = c * 4;
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = (p[k] - (c0 + k == label ? 1.0f : 0.0f)) * inv_M;
        if constexpr (sizeof(TG) == 2) {
            union { bf16_t h[4]; uint2 u; } pk;
#pragma unroll
            for (int k = 0; k < 4; ++k) pk.h[k] = (bf16_t)p[k];
            *reinterpret_cast<uint2*>(g + c0) = pk.u;
        } else {
            *reinterpret_cast<float4*>(g + c0) = make_float4(p[0], p[1], p[2], p[3]);
        }
    }
    if (tid == 0) row_loss[row] = label_ok ? logf(bs) - (logits[row * C + label] - bm) : NAN;
}

// The same with the row in registers (C <= 4096 * NV): NV 16-byte pieces per thread, no LDS beyond the block reductions,
// so that a compute unit holds two rows at a time and one row's memory phase overlaps the other's arithmetic (with the row
// in LDS a unit holds one).  The same values are combined in the same order as above: the results are the same bit for bit.
template <typename TG, int NV>
__global__ __launch_bounds__(kCeThreads, 8) void softmax_ce_reg_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                                       TG* __restrict__ dlogits, float* __restrict__ row_loss, int C,
                                                                       float inv_M) {
    constexpr int NWV = kCeThreads / 64;
    __shared__ float sm[NWV], ss[NWV];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const float4* z4 = reinterpret_cast<const float4*>(logits + row * C);
    const int C4 = C >> 2;
    float4 v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c = tid + k * kCeThreads;
        if (c < C4) v[k] = z4[c];
    }
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < NV; ++k)
        if (tid + k * kCeThreads < C4) mx = fmaxf(fmaxf(mx, fmaxf(v[k].x, v[k].y)), fmaxf(v[k].z, v[k].w));
    mx = wmax(mx);
    if (lane == 0) sm[wave] = mx;
    __syncthreads();
    float bm = sm[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) bm = fmaxf(bm, sm[w]);
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < NV; ++k)
        if (tid + k * kCeThreads < C4) {
            v[k].x = __expf(v[k].x - bm); v[k].y = __expf(v[k].y - bm); v[k].z = __expf(v[k].z - bm); v[k].w = __expf(v[k].w - bm);
            sum += (v[k].x + v[k].y) + (v[k].z + v[k].w);
        }
    sum = wsum(sum);
    if (lane == 0) ss[wave] = sum;
    __syncthreads();
    float bs = 0.0f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) bs += ss[w];
    const float inv = 1.0f / bs;
    const int label = labels[row];
    const bool label_ok = label >= 0 && label < C;
    TG* g = dlogits + row * C;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int c = tid + k * kCeThreads;
        if (c < C4) {
            float p[4] = {v[k].x * inv, v[k].y * inv, v[k].z * inv, v[k].w * inv};
            const int c0 = c * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = (p[e] - (c0 + e == label ? 1.0f : 0.0f)) * inv_M;
            if constexpr (sizeof(TG) == 2) {
                union { bf16_t h[4]; uint2 u; } pk;
#pragma unroll
                for (int e = 0; e < 4; ++e) pk.h[e] = (bf16_t)p[e];
                *reinterpret_cast<uint2*>(g + c0) = pk.u;
            } else {
                *reinterpret_cast<float4*>(g + c0) = make_float4(p[0], p[1], p[2], p[3]);
            }
        }
    }
    if (tid == 0) row_loss[row] = label_ok ? logf(bs) - (logits[row * C + label] - bm) : NAN;
}

// Rows of any length and alignment, up to T NE values: a block of T threads reads a row once, a value at a time, and keeps it in registers.  Values of neighbouring
// threads are neighbours in memory, so this costs wider rows' bandwidth little: 999 x 5003 values in bf16 19.8 us as two passes of softmax_ce_wide_kernel
// and 10.8 so.  (Exponentials as there: expf.)
template <typename TG, int T, int NE>
__global__ __launch_bounds__(T) void softmax_ce_any_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels, TG* __restrict__ dlogits,
                                                          float* __restrict__ row_loss, int C, float inv_M) {
    constexpr int NWV = T / 64;
    __shared__ float sm[NWV], ss[NWV];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const float* const z = logits + row * C;
    float v[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) v[k] = tid + k * T < C ? z[tid + k * T] : -INFINITY;
    float mx = v[0];
#pragma unroll
    for (int k = 1; k < NE; ++k) mx = fmaxf(mx, v[k]);
    mx = wmax(mx);
    if (lane == 0) sm[wave] = mx;
    __syncthreads();
    float bm = sm[0];
#pragma unroll
    for (int w = 1; w < NWV; ++w) bm = fmaxf(bm, sm[w]);
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < NE; ++k)
        if (tid + k * T < C) {
            v[k] = expf(v[k] - bm);
            sum += v[k];
        }
    sum = wsum(sum);
    if (lane == 0) ss[wave] = sum;
    __syncthreads();
    float bs = 0.0f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) bs += ss[w];
    const float inv = 1.0f / bs;
    const int label = labels[row];
    const bool label_ok = label >= 0 && label < C;
    TG* const g = dlogits + row * C;
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int c = tid + k * T;
        if (c < C) g[c] = from_f32<TG>((v[k] * inv - (c == label ? 1.0f : 0.0f)) * inv_M);
    }
    if (tid == 0) row_loss[row] = label_ok ? logf(bs) - (z[label] - bm) : NAN;
}
template <int T, int NE>
static hipError_t softmax_ce_any(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* row_loss, int rows, int C, float inv_M, hipStream_t s) {
    if (dtype == kBF16) hipLaunchKernelGGL((softmax_ce_any_kernel<bf16_t, T, NE>), dim3(rows), dim3(T), 0, s, logits, labels, (bf16_t*)dlogits, row_loss, C, inv_M);
    else hipLaunchKernelGGL((softmax_ce_any_kernel<float, T, NE>), dim3(rows), dim3(T), 0, s, logits, labels, (float*)dlogits, row_loss, C, inv_M);
    return hipGetLastError();
}

hipError_t softmax_ce(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* row_loss,
                      int rows, int C, float inv_M, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    if (C > 2048 && C % 4 == 0 && C <= 4096 * 8 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0 &&
        (reinterpret_cast<uintptr_t>(dlogits) & 15) == 0) {
        const bool small = C <= 4096 * 4;
        if (dtype == kBF16) {
            if (small) hipLaunchKernelGGL((softmax_ce_reg_kernel<bf16_t, 4>), dim3(rows), dim3(kCeThreads), 0, s, logits, labels, (bf16_t*)dlogits, row_loss, C, inv_M);
            else hipLaunchKernelGGL((softmax_ce_reg_kernel<bf16_t, 8>), dim3(rows), dim3(kCeThreads), 0, s, logits, labels, (bf16_t*)dlogits, row_loss, C, inv_M);
        } else {
            if (small) hipLaunchKernelGGL((softmax_ce_reg_kernel<float, 4>), dim3(rows), dim3(kCeThreads), 0, s, logits, labels, (float*)dlogits, row_loss, C, inv_M);
            else hipLaunchKernelGGL((softmax_ce_reg_kernel<float, 8>), dim3(rows), dim3(kCeThreads), 0, s, logits, labels, (float*)dlogits, row_loss, C, inv_M);
        }
        return hipGetLastError();
    }
    if (C > 2048 && C % 4 == 0 && (size_t)C * 4 <= 150 * 1024 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0 &&
        (reinterpret_cast<uintptr_t>(dlogits) & 15) == 0) {
        const unsigned lds = (unsigned)C * 4;
        if (dtype == kBF16) {
            static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(softmax_ce_lds_kernel<bf16_t>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
            if (attr != hipSuccess) return attr;
            hipLaunchKernelGGL(softmax_ce_lds_kernel<bf16_t>, dim3(rows), dim3(kCeThreads), lds, s, logits, labels, (bf16_t*)dlogits,
                               row_loss, C, inv_M);
        } else {
            static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(softmax_ce_lds_kernel<float>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
            if (attr != hipSuccess) return attr;
            hipLaunchKernelGGL(softmax_ce_lds_kernel<float>, dim3(rows), dim3(kCeThreads), lds, s, logits, labels, (float*)dlogits,
                               row_loss, C, inv_M);
        }
        return hipGetLastError();
    }
    if (C > 2048 && C <= 1024 * 32) {
        if (C <= 256 * 16) return softmax_ce_any<256, 16>(dtype, logits, labels, dlogits, row_loss, rows, C, inv_M, s);
        if (C <= 512 * 16) return softmax_ce_any<512, 16>(dtype, logits, labels, dlogits, row_loss, rows, C, inv_M, s);
        if (C <= 1024 * 16) return softmax_ce_any<1024, 16>(dtype, logits, labels, dlogits, row_loss, rows, C, inv_M, s);
        return softmax_ce_any<1024, 32>(dtype, logits, labels, dlogits, row_loss, rows, C, inv_M, s);
    }
    if (C > 2048) {
        if (dtype == kBF16)
            hipLaunchKernelGGL(softmax_ce_wide_kernel<bf16_t>, dim3(rows), dim3(256), 0, s, logits, labels,
                               (bf16_t*)dlogits, row_loss, C, inv_M);
        else
            hipLaunchKernelGGL(softmax_ce_wide_kernel<float>, dim3(rows), dim3(256), 0, s, logits, labels,
                               (float*)dlogits, row_loss, C, inv_M);
        return hipGetLastError();
    }
    dim3 grid(cdiv64(rows, 4));
    if (dtype == kBF16)
        hipLaunchKernelGGL(softmax_ce_kernel<bf16_t>, grid, dim3(256), 0, s, logits, labels, (bf16_t*)dlogits,
                           row_loss, rows, C, inv_M);
    else
        hipLaunchKernelGGL(softmax_ce_kernel<float>, grid, dim3(256), 0, s, logits, labels, (float*)dlogits,
                           row_loss, rows, C, inv_M);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void reduce_scaled_sum_kernel(const float* __restrict__ in, int n,
                                                                float scale, float* __restrict__ out) {
    __shared__ float part[4];
    float a = 0.0f;
    for (int i = threadIdx.x; i < n; i += 256) a += in[i];
    a = wsum(a);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (part[0] + part[1] + part[2] + part[3]) * scale;
}

hipError_t reduce_scaled_sum(const float* in, int n, float scale, float* out, hipStream_t s) {
    hipLaunchKernelGGL(reduce_scaled_sum_kernel, dim3(1), dim3(256), 0, s, in, n, scale, out);
    return hipGetLastError();
}

// Few rows: one 1024-thread workgroup, LPR lanes to a row with up to 8 of its values each in registers, so that 1024 / LPR rows are
// in flight at once; then the mean over all rows of the loss, summed in the order of reduce_scaled_sum_kernel.  What such a launch
// takes is latency: 47 rows of 10 classes run as long as one row does, and the launch replaces two or three of 4 to 5 us each
// (five micro-batches of a four-layer fp32 MLP, backward pass and update: 269 -> 257 us).
template <typename TG, int LPR>
__global__ __launch_bounds__(1024) void softmax_ce_small_kernel(const float* __restrict__ logits, const int32_t* __restrict__ labels,
                                                                TG* __restrict__ dlogits, float* __restrict__ y, float* row_loss,
                                                                int rows, int C, int before, float inv_M, float scale,
                                                                float* __restrict__ loss_out) {
    const int tid = threadIdx.x, sub = tid & (LPR - 1);
    for (int row = tid / LPR; row < rows; row += 1024 / LPR) {
        const float* z = logits + (int64_t)row * C;
        float v[8];
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = sub + e * LPR;
            v[e] = c < C ? z[c] : -INFINITY;
            mx = fmaxf(mx, v[e]);
        }
        if (y) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = sub + e * LPR;
                if (c < C) y[(int64_t)row * C + c] = v[e];
            }
        }
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        const int label = labels[row];
        const bool label_ok = label >= 0 && label < C;  // an out-of-range label gives a NaN loss, never a wild read
        float sum = 0.0f, hit = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = sub + e * LPR;
            if (c < C) {
                v[e] -= mx;
                if (c == label) hit = v[e];
                v[e] = expf(v[e]);
                sum += v[e];
            }
        }
#pragma unroll
        for (int o = LPR / 2; o > 0; o >>= 1) {
            sum += __shfl_xor(sum, o, 64);
            hit += __shfl_xor(hit, o, 64);   // (one lane's value and zeros)
        }
        const float inv = 1.0f / sum;
        TG* g = dlogits + (int64_t)row * C;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int c = sub + e * LPR;
            if (c < C) g[c] = from_f32<TG>((v[e] * inv - (c == label ? 1.0f : 0.0f)) * inv_M);
        }
        if (sub == 0) row_loss[before + row] = label_ok ? logf(sum) - hit : NAN;
    }
    if (!loss_out) return;
    __shared__ float part[4];
    __syncthreads();   // (the row losses are this workgroup's own stores, or an earlier launch's)
    if (tid < 256) {
        float a = 0.0f;
        for (int i = tid; i < before + rows; i += 256) a += row_loss[i];
        a = wsum(a);
        if ((tid & 63) == 0) part[tid >> 6] = a;
    }
    __syncthreads();
    if (tid == 0) loss_out[0] = (part[0] + part[1] + part[2] + part[3]) * scale;
}

// Lanes to a row, and what is taken: all rows of the loss at once.  (256 rows of 96 in four rounds take 12 us, a wave to a row in 64 workgroups and the mean in
// a launch of its own 7.)
static constexpr int ce_small_lanes(int C) { return C <= 16 ? 2 : C <= 64 ? 8 : C <= 128 ? 16 : 64; }
bool softmax_ce_small_takes(int64_t rows, int C) { return C <= 512 && rows * ce_small_lanes(C) <= 1024; }

template <typename TG, int LPR>
static hipError_t launch_ce_small(const float* logits, const int32_t* labels, void* dlogits, float* y, float* row_loss, int rows, int C,
                                  int before, float inv_M, float scale, float* loss_out, hipStream_t s) {
    hipLaunchKernelGGL((softmax_ce_small_kernel<TG, LPR>), dim3(1), dim3(1024), 0, s, logits, labels, (TG*)dlogits, y, row_loss, rows, C, before,
                       inv_M, scale, loss_out);
    return hipGetLastError();
}

template <typename TG>
static hipError_t ce_small_of(const float* logits, const int32_t* labels, void* dlogits, float* y, float* row_loss, int rows, int C, int before,
                              float inv_M, float scale, float* loss_out, hipStream_t s) {
    if (C <= 16) return launch_ce_small<TG, 2>(logits, labels, dlogits, y, row_loss, rows, C, before, inv_M, scale, loss_out, s);
    if (C <= 64) return launch_ce_small<TG, 8>(logits, labels, dlogits, y, row_loss, rows, C, before, inv_M, scale, loss_out, s);
    if (C <= 128) return launch_ce_small<TG, 16>(logits, labels, dlogits, y, row_loss, rows, C, before, inv_M, scale, loss_out, s);
    return launch_ce_small<TG, 64>(logits, labels, dlogits, y, row_loss, rows, C, before, inv_M, scale, loss_out, s);
}

hipError_t softmax_ce_small(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* y, float* row_loss, int rows,
                            int C, int before, float inv_M, float scale, float* loss_out, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    if (dtype == kBF16) return ce_small_of<bf16_t>(logits, labels, dlogits, y, row_loss, rows, C, before, inv_M, scale, loss_out, s);
    return ce_small_of<float>(logits, labels, dlogits, y, row_loss, rows, C, before, inv_M, scale, loss_out, s);
}

// ------------------------------------------------------------------------------- ReLU gradient
template <typename T>
__global__ void relu_mask_kernel(const T* __restrict__ dy, const T* __restrict__ y, T* __restrict__ dz,
                                 int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) dz[i] = to_f32(y[i]) > 0.0f ? dy[i] : T(0.0f);
}

// bf16, 8 elements (16 bytes) per thread and access
__global__ __launch_bounds__(256) void relu_mask_bf16x8_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ y,
                                                               bf16_t* __restrict__ dz, int64_t n8) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8) return;
    Pack8 g, v;
    g.u = reinterpret_cast<const uint4*>(dy)[i];
    v.u = reinterpret_cast<const uint4*>(y)[i];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (!((float)v.h[e] > 0.0f)) g.h[e] = (bf16_t)0.0f;
    reinterpret_cast<uint4*>(dz)[i] = g.u;
}

hipError_t relu_mask(int dtype, const void* dy, const void* y, void* dz, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (dtype == kBF16 && n % 8 == 0 && ((reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(dz)) & 15) == 0) {
        hipLaunchKernelGGL(relu_mask_bf16x8_kernel, dim3(cdiv64(n / 8, 256)), dim3(256), 0, s, (const bf16_t*)dy, (const bf16_t*)y,
                           (bf16_t*)dz, n / 8);
        return hipGetLastError();
    }
    int blocks = cdiv64(n, 256);
    if (blocks > 4096) blocks = 4096;
    if (dtype == kBF16)
        hipLaunchKernelGGL(relu_mask_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t*)dy,
                           (const bf16_t*)y, (bf16_t*)dz, n);
    else
        hipLaunchKernelGGL(relu_mask_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float*)dy,
                           (const float*)y, (float*)dz, n);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------- momentum update
// 4 parameters per thread: 16-byte loads of w, buf, g; 16-byte stores of w, buf; 8-byte store of the
// bf16 working copy.  The tail (n % 4) is handled by the last threads one element at a time.
// KEEP: the parameters as they were (masters and working copy) go to kept_w and kept_wc as well: the copy of a version that
// forward or backward passes may still ask for costs its stores (and the old working copy's load) instead of a pass of its own
// over the parameters.  (Two mini-batches of VGG-16 with vertical weight stashing 2325 -> 2258 us, one of GPT-2 in 1F1B order
// 23.29 -> 22.83 ms, whose copies of 0.13 to 0.26 GB took 52 us each.)
template <bool KEEP>
__device__ __forceinline__ void sgd_momentum_block(int block, int blocks, float* __restrict__ w, float* __restrict__ buf,
                                                   const float* __restrict__ g, bf16_t* __restrict__ wc, int64_t n, float lr,
                                                   float mu, float* __restrict__ kept_w, bf16_t* __restrict__ kept_wc) {
    const int64_t n4 = n >> 2;
    int64_t i = (int64_t)block * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)blocks * blockDim.x;
    for (; i < n4; i += stride) {
        float4 wv = reinterpret_cast<const float4*>(w)[i];
        float4 bv = reinterpret_cast<const float4*>(buf)[i];
        float4 gv = reinterpret_cast<const float4*>(g)[i];
        if (KEEP) {
            reinterpret_cast<float4*>(kept_w)[i] = wv;
            if (wc) reinterpret_cast<uint2*>(kept_wc)[i] = reinterpret_cast<const uint2*>(wc)[i];
        }
        bv.x = mu * bv.x + gv.x; bv.y = mu * bv.y + gv.y; bv.z = mu * bv.z + gv.z; bv.w = mu * bv.w + gv.w;
        wv.x -= lr * bv.x; wv.y -= lr * bv.y; wv.z -= lr * bv.z; wv.w -= lr * bv.w;
        reinterpret_cast<float4*>(buf)[i] = bv;
        reinterpret_cast<float4*>(w)[i] = wv;
        if (wc) {
            union { bf16_t h[4]; uint2 u; } pk;
            pk.h[0] = (bf16_t)wv.x; pk.h[1] = (bf16_t)wv.y; pk.h[2] = (bf16_t)wv.z; pk.h[3] = (bf16_t)wv.w;
            reinterpret_cast<uint2*>(wc)[i] = pk.u;
        }
    }
    int64_t t = (n4 << 2) + (int64_t)block * blockDim.x + threadIdx.x;
    if (t < n) {
        float b = mu * buf[t] + g[t];
        if (KEEP) {
            kept_w[t] = w[t];
            if (wc) kept_wc[t] = wc[t];
        }
        float x = w[t] - lr * b;
        buf[t] = b;
        w[t] = x;
        if (wc) wc[t] = (bf16_t)x;
    }
}

template <bool KEEP>
__global__ __launch_bounds__(256) void sgd_momentum_kernel(float* __restrict__ w, float* __restrict__ buf,
                                                           const float* __restrict__ g,
                                                           bf16_t* __restrict__ wc, int64_t n, float lr,
                                                           float mu, float* __restrict__ kept_w, bf16_t* __restrict__ kept_wc) {
    sgd_momentum_block<KEEP>(blockIdx.x, gridDim.x, w, buf, g, wc, n, lr, mu, kept_w, kept_wc);
}

// The updates of several stages in one launch.  A run on one stream is bound by its launches where the stages are small, 2.5 to 3 us each on the device and 3.1 on the host.
struct SgdJobs {
    int first[kUpdateMax + 1];   // first workgroup of a stage; behind the last one the number of workgroups
    Update job[kUpdateMax];
};
__global__ __launch_bounds__(256) void sgd_momentum_all_kernel(SgdJobs all) {
    int j = 0;
#pragma unroll
    for (int k = 1; k < kUpdateMax; ++k) j += (int)blockIdx.x >= all.first[k] ? 1 : 0;
    const Update u = all.job[j];
    sgd_momentum_block<false>(blockIdx.x - all.first[j], all.first[j + 1] - all.first[j], u.w, u.buf, u.g, (bf16_t*)u.wcopy, u.n, u.lr, u.mu, nullptr, nullptr);
}

static int sgd_blocks(int64_t n) {
    const int blocks = cdiv64((n >> 2) + 4, 256);
    return blocks > 2048 ? 2048 : blocks;
}

hipError_t sgd_momentum_all(const Update* list, int n, hipStream_t s) {
    if (n < 1 || n > kUpdateMax) return n < 1 ? hipSuccess : hipErrorInvalidValue;
    SgdJobs all;
    int blocks = 0;
    for (int k = 0; k <= kUpdateMax; ++k) {
        all.first[k] = blocks;
        if (k == kUpdateMax) break;
        all.job[k] = k < n ? list[k] : Update{};
        if (k < n && list[k].n > 0) blocks += sgd_blocks(list[k].n);
    }
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(sgd_momentum_all_kernel, dim3(blocks), dim3(256), 0, s, all);
    return hipGetLastError();
}

hipError_t sgd_momentum(float* w, float* buf, const float* g, void* wcopy_bf16, int64_t n, float lr, float mu,
                        hipStream_t s) {
    return sgd_momentum_keeping(w, buf, g, wcopy_bf16, n, lr, mu, nullptr, nullptr, s);
}

hipError_t sgd_momentum_keeping(float* w, float* buf, const float* g, void* wcopy_bf16, int64_t n, float lr, float mu,
                                float* kept_w, void* kept_wcopy, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int blocks = sgd_blocks(n);
    if (kept_w)
        hipLaunchKernelGGL(sgd_momentum_kernel<true>, dim3(blocks), dim3(256), 0, s, w, buf, g, (bf16_t*)wcopy_bf16, n,
                           lr, mu, kept_w, (bf16_t*)kept_wcopy);
    else
        hipLaunchKernelGGL(sgd_momentum_kernel<false>, dim3(blocks), dim3(256), 0, s, w, buf, g, (bf16_t*)wcopy_bf16, n,
                           lr, mu, (float*)nullptr, (bf16_t*)nullptr);
    return hipGetLastError();
}

__global__ void cast_f32_to_bf16_kernel(const float* __restrict__ in, bf16_t* __restrict__ out, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) out[i] = (bf16_t)in[i];
}

hipError_t cast_f32_to_bf16(const float* in, void* out, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int blocks = cdiv64(n, 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(cast_f32_to_bf16_kernel, dim3(blocks), dim3(256), 0, s, in, (bf16_t*)out, n);
    return hipGetLastError();
}

// dst[0..bytes) = src[0..bytes) as a kernel (a captured graph of the backward pass then holds kernel nodes only):
// 16 bytes per thread and step where both addresses allow it, single bytes for the rest.
__global__ void copy_bytes_kernel(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst, int64_t n16, int64_t bytes) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t; i < n16; i += stride) reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(src)[i];
    for (int64_t i = n16 * 16 + t; i < bytes; i += stride) dst[i] = src[i];
}

hipError_t copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    const bool wide = ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15) == 0;
    const int64_t n16 = wide ? (int64_t)(bytes / 16) : 0;
    int blocks = cdiv64(wide ? (n16 > 0 ? n16 : 1) : (int64_t)bytes, 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(copy_bytes_kernel, dim3(blocks), dim3(256), 0, s, (const unsigned char*)src, (unsigned char*)dst, n16,
                       (int64_t)bytes);
    return hipGetLastError();
}

}  // namespace tmps
