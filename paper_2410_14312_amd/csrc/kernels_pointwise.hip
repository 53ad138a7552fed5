// Backward pass of a 1 x 1 convolution with a per-channel affine layer behind it, in one pass over memory (bf16, unit stride).
//
// On the way back the affine layer forms g = gain dY and its own sums, the convolution dW = g^T x and dx = mask(g W + add).  As launches of their own these
// read dY, z and x, write g, read it twice more and read x again for the mask; the bottleneck blocks' maps of 64 and 256 channels are bound by exactly that.
// Here a workgroup takes a run of positions, 64 at a time, and reads dY, z, x and add once: g and x go to LDS, dx comes from there and from W, which lies in LDS too,
// transposed, for the workgroup's whole run and is read there in every step, and dW stays in the accumulators until the workgroup's last position.  One workgroup of eight waves to a compute unit; the next positions' loads are on
// their way during all of a step's multiplies.  What remains beside the maps is each workgroup's partial sums, 66 KB for 256 x 64.
//
// g is rounded to bf16 as where it was stored, dx once after add and mask: the same values but for the order of sums.
//
// Maps of 56 x 56 x 256 from 64, 64 images (200704 positions, 258 MB): 52 us, 5 TB/s, for 118 in three launches (55 among a run's other kernels); 64 from 256 with a gradient
// to join 70 for 143 (69); the first group of ResNet-50's blocks as a stage 2248 -> 1871 us.  Forward and backward pass and update of both layers, before and now (us): 256 from 64 at 65536
// positions 76 and 58, 16384 39 and 31, 64 from 64 at 65536 43 and 27, at 4096 and below 27 and 22 (the launches).  Errors of dW against 64 bits (2-norm) over 200704,
// 16384 and 1024 positions 1.8, 1.0 and 0.7e-7 before, 1.2, 1.0 and 0.7e-7 now.
#include <algorithm>

#include "gemm3.hip.h"
#include "kernels.h"
#include "launch.h"

namespace tmps {

typedef float f32x4v_t __attribute__((ext_vector_type(4)));

static constexpr int kPwThreads = 512, kPwRows = 64;   // positions of a step
// Row strides in LDS, bytes: whole 16-byte pieces, an odd number of them modulo 16, so that 16 rows read at one column and 4 rows of 64 bytes read transposed
// fall on different banks (64 values: the latter two by two).
__host__ __device__ constexpr int pw_stride(int n) { return n == 32 ? 80 : n == 64 ? 144 : n == 128 ? 336 : 592; }
template <int O, int I> constexpr int pw_lds_bytes() { return kPwRows * (pw_stride(O) + pw_stride(I) + (I + 4) * 4) + I * pw_stride(O); }

__device__ __forceinline__ void pw_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// dy, z: [P][O]; x, add (may be null), dx: [P][I]; w: [O][I].  Workgroup b takes positions b per .. b per + per - 1 (per: a multiple of 16).
// part_a: [workgroups][2][O] sums of dy z and of dy; part_w: [workgroups][O I + O] dW, then the sums of g.
template <int O, int I>
__global__ __launch_bounds__(kPwThreads) void affine_pointwise_bwd_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ z, const bf16_t* __restrict__ x,
                                                                          const bf16_t* __restrict__ w, const float* __restrict__ gain, const bf16_t* add, int masked,
                                                                          bf16_t* dx, float* __restrict__ part_a, float* __restrict__ part_w, int P, int per) {
    constexpr int CO = O / 8, CI = I / 8;                               // 16-byte pieces of a row
    constexpr int RO = kPwThreads / CO, RI = kPwThreads / CI;           // rows that the workgroup's threads cover at a time
    constexpr int NO = kPwRows / RO, NI = kPwRows / RI;                 // pieces of a thread
    constexpr int SG = pw_stride(O), SX = pw_stride(I), SD = I + 4;     // row strides in LDS: bytes, bytes, floats
    constexpr int CB = I / 64, KS = O / 32;                             // dx: 16-column blocks and 32-k steps of a wave
    constexpr int TO = O / 32, TI = I / 32, PW = TO * TI >= 8 ? TO * TI / 8 : 1;   // dW: 32 x 32 blocks of a wave
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const lds_t G = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const lds_t X = G + kPwRows * SG, D = X + kPwRows * SX, W = D + kPwRows * SD * 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quarter = lane >> 4;
    const int co = tid % CO, ro = tid / CO, ci = tid % CI, ri = tid / CI;
    const int p0 = blockIdx.x * per, p1 = min(P, p0 + per);

    float gn[8], s_g[8], s_dy[8], s_dyz[8];   // (a step's values are summed by themselves first, here and in dW: no chain of roundings over all positions)
    load8(gain + co * 8, gn);
#pragma unroll
    for (int e = 0; e < 8; ++e) s_g[e] = s_dy[e] = s_dyz[e] = 0.0f;

    // W transposed, [I][O]
#pragma unroll
    for (int n = 0; n < O * I / kPwThreads; ++n) {
        const int at = n * kPwThreads + tid;
        *lds_ptr<bf16_t>(W + at % I * SG + at / I * 2) = w[at];
    }
    // dx: wave (column group, half of the positions)
    const int cg = wave & 3, ph = wave >> 2;

    // dW: a wave's blocks share the block of the wider side
    const int wide = O >= I ? TO : TI;
    const int b_wide = wave % wide, b_other = wave / wide * PW;
    const bool multiplies = TO * TI >= 8 || wave < TO * TI;
    f32x16_t dw[PW];
#pragma unroll
    for (int b = 0; b < PW; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) dw[b][r] = 0.0f;
    // transposed fragment: rows (channels) 32 block + .., k (positions) 16 kk + 8 (lane / 32) + 0 .. 7
    const int tk = (lane >> 5) * 8 + ((lane & 15) >> 2), tc = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    auto fragment = [&](lds_t tile, int stride, int block, int kk) {
        const lds_t a = tile + (kk * 16 + tk) * stride + (block * 32 + tc) * 2;
        union { s16x4_t h[2]; bf16x8_t v; } u;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(a));
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(a + 4 * stride));
        return u.v;
    };

    bf16x8_t vdy[NO], vz[NO], vx[NI], va[NI];
    const bf16x8_t none = {};
    // (positions from here on are the workgroup's own: 32-bit offsets)
    const int mine = p1 - p0;
    dy += (int64_t)p0 * O;
    z += (int64_t)p0 * O;
    x += (int64_t)p0 * I;
    dx += (int64_t)p0 * I;
    if (add) add += (int64_t)p0 * I;
    auto request = [&](int base) {
#pragma unroll
        for (int n = 0; n < NO; ++n) {
            const int p = base + ro + n * RO;
            const uint32_t at = (uint32_t)(p * O + co * 8);
            vdy[n] = p < mine ? *reinterpret_cast<const bf16x8_t*>(dy + at) : none;
            vz[n] = p < mine ? *reinterpret_cast<const bf16x8_t*>(z + at) : none;
        }
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int p = base + ri + n * RI;
            const uint32_t at = (uint32_t)(p * I + ci * 8);
            vx[n] = p < mine ? *reinterpret_cast<const bf16x8_t*>(x + at) : none;
            va[n] = add && p < mine ? *reinterpret_cast<const bf16x8_t*>(add + at) : none;
        }
    };
    if (mine > 0) request(0);
    for (int base = 0; base < mine; base += kPwRows) {
        float t_g[8] = {}, t_dy[8] = {}, t_dyz[8] = {};
#pragma unroll
        for (int n = 0; n < NO; ++n) {
            bf16x8_t g;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = (float)vdy[n][e];
                t_dy[e] += d;
                t_dyz[e] += d * (float)vz[n][e];
                g[e] = (bf16_t)(d * gn[e]);
                t_g[e] += (float)g[e];
            }
            *lds_ptr<bf16x8_t>(G + (ro + n * RO) * SG + co * 16) = g;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            s_g[e] += t_g[e];
            s_dy[e] += t_dy[e];
            s_dyz[e] += t_dyz[e];
        }
        bf16x8_t keep[NI];
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            *lds_ptr<bf16x8_t>(X + (ri + n * RI) * SX + ci * 16) = vx[n];
            keep[n] = va[n];
        }
        if (base + kPwRows < mine) request(base + kPwRows);
        pw_barrier();

        f32x4v_t d[2][CB];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < CB; ++c) d[h][c] = f32x4v_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            bf16x8_t af[2], wf[CB];
#pragma unroll
            for (int c = 0; c < CB; ++c) wf[c] = *lds_ptr<const bf16x8_t>(W + (cg * (I / 4) + c * 16 + l16) * SG + k * 64 + quarter * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) af[h] = *lds_ptr<const bf16x8_t>(G + (ph * 32 + h * 16 + l16) * SG + k * 64 + quarter * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < CB; ++c) d[h][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[h], wf[c], d[h][c], 0, 0, 0);
        }
        // register r of a lane: position 4 (lane / 16) + r, column lane % 16
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *lds_ptr<float>(D + ((ph * 32 + h * 16 + quarter * 4 + r) * SD + cg * (I / 4) + c * 16 + l16) * 4) = d[h][c][r];
        if (multiplies) {
#pragma unroll
            for (int b = 0; b < PW; ++b) {
                f32x16_t t = {};
#pragma unroll
                for (int kk = 0; kk < kPwRows / 16; ++kk)
                    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fragment(G, SG, O >= I ? b_wide : b_other + b, kk), fragment(X, SX, O >= I ? b_other + b : b_wide, kk), t, 0, 0, 0);
                dw[b] += t;
            }
        }
        pw_barrier();
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const int row = ri + n * RI, p = base + row;
            if (p < mine) {
                const f32x4v_t lo = *lds_ptr<const f32x4v_t>(D + (row * SD + ci * 8) * 4), hi = *lds_ptr<const f32x4v_t>(D + (row * SD + ci * 8 + 4) * 4);
                float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                const bf16x8_t t = *lds_ptr<const bf16x8_t>(X + row * SX + ci * 16);   // (this thread's own piece)
                bf16x8_t out;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (add) v[e] += (float)keep[n][e];
                    if (masked && !((float)t[e] > 0.0f)) v[e] = 0.0f;
                    out[e] = (bf16_t)v[e];
                }
                *reinterpret_cast<bf16x8_t*>(dx + (uint32_t)(p * I + ci * 8)) = out;
            }
        }
    }

    float* const pw = part_w + (int64_t)blockIdx.x * (O * I + O);
    if (multiplies) {
        // register r of a lane: row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
#pragma unroll
        for (int b = 0; b < PW; ++b) {
            const int o = (O >= I ? b_wide : b_other + b) * 32, i = (O >= I ? b_other + b : b_wide) * 32;
#pragma unroll
            for (int r = 0; r < 16; ++r) pw[(o + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * I + i + (lane & 31)] = dw[b][r];
        }
    }
    // sums over the rows of the threads that hold the same channels
    float* const sums = reinterpret_cast<float*>(smem_raw);   // [RO][O]
#pragma unroll
    for (int which = 0; which < 3; ++which) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) sums[ro * O + co * 8 + e] = which == 0 ? s_dyz[e] : which == 1 ? s_dy[e] : s_g[e];
        __syncthreads();
        if (tid < O) {
            float v = 0.0f;
            for (int r = 0; r < RO; r += 8) {
                float t[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) t[u] = sums[(r + u) * O + tid];
                v += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
            }
            if (which < 2) part_a[((int64_t)blockIdx.x * 2 + which) * O + tid] = v;
            else pw[O * I + tid] = v;
        }
    }
}

// ---- forward: C channels to W, and from those to C again -----------------------------------------------------------------------------------------------------
// z = x w^T + bias, y = act(gain z + shift + res) as EpiConvAffine forms and rounds them; PAIR: and the next block's first convolution, which reads y, with its
// affine layer, from LDS instead of memory.  A workgroup takes a run of positions, 64 at a time; it has a wave for every 32 of the wide result's channels (which also has 16 of
// the narrow one's for its share of the positions) and keeps their weights in registers; x and res of the next step are on their way during a step.  A wave's two blocks of 16
// channels are interleaved in fours, so that a lane holds 8 consecutive channels of a position.
struct PwWide {
    const bf16_t *x, *w, *res;   // [P][C], [W][C], [P][W] or null
    const float *bias, *gain, *shift;
    bf16_t *z, *y, *again;   // [P][W] each; again: y once more, or null
    int relu;
};
struct PwNarrow {
    const bf16_t* w;   // [C][W]
    const float *bias, *gain, *shift;
    bf16_t *z, *y;     // [P][C] each
    int relu;
};

template <int C, int W, bool PAIR>
__global__ __launch_bounds__(2 * W) void pointwise_fwd_kernel(PwWide a, PwNarrow b, int P, int per) {
    constexpr int T = 2 * W, SX = pw_stride(C), SY = pw_stride(W), CP = C / 8;
    constexpr int NX = kPwRows * CP / T, KX = C / 32;                    // pieces of x of a thread; steps of 32 k of the wide result
    constexpr int CB = C / 16, NH = PAIR ? 4 * CB * 32 / W : 1, KN = PAIR ? W / 32 : 1;   // narrow result: blocks of channels, of a wave's positions; steps
    static_assert(NX >= 1 && W >= 2 * C, "a piece of x to every thread, a block of the narrow result's channels to every wave");
    __shared__ __attribute__((aligned(16))) unsigned char xs[kPwRows * SX];
    __shared__ __attribute__((aligned(16))) unsigned char ys[PAIR ? kPwRows * SY : 16];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p0 = blockIdx.x * per, mine = min(P - p0, per);
    if (mine <= 0) return;
    const bf16_t* const x = a.x + (int64_t)p0 * C;
    const bf16_t* const res = a.res ? a.res + (int64_t)p0 * W : nullptr;
    bf16_t *const z = a.z + (int64_t)p0 * W, *const y = a.y + (int64_t)p0 * W, *const again = a.again ? a.again + (int64_t)p0 * W : nullptr;

    const bf16x8_t none = {};
    const int xr = tid / CP, xc = tid % CP * 8;
    const int ch = wave * 32 + quarter * 8;   // this lane's channels of the wide result: ch .. ch + 7
    bf16x8_t vx[NX], vr[4];
    auto request_x = [&](int base) {
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            const int p = base + xr + n * (T / CP);
            vx[n] = p < mine ? *reinterpret_cast<const bf16x8_t*>(x + (uint32_t)(p * C + xc)) : none;
        }
    };
    auto keep_x = [&]() {
#pragma unroll
        for (int n = 0; n < NX; ++n) *reinterpret_cast<bf16x8_t*>(xs + (xr + n * (T / CP)) * SX + xc * 2) = vx[n];
    };
    auto request_res = [&](int base) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int p = base + c * 16 + l16;
            vr[c] = res && p < mine ? *reinterpret_cast<const bf16x8_t*>(res + (uint32_t)(p * W + ch)) : none;
        }
    };
    request_x(0);
    request_res(0);

    bf16x8_t wf[2][KX];   // [block][step of 32 k]: row l16 of block j is channel 32 wave + 8 (l16 / 4) + 4 j + l16 % 4
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int k = 0; k < KX; ++k) wf[j][k] = *reinterpret_cast<const bf16x8_t*>(a.w + (wave * 32 + (l16 >> 2) * 8 + j * 4 + (l16 & 3)) * C + k * 32 + quarter * 8);
    float g[8], sh[8], bi[8];
    load8(a.gain + ch, g);
    load8(a.shift + ch, sh);
#pragma unroll
    for (int e = 0; e < 8; ++e) bi[e] = a.bias ? a.bias[ch + e] : 0.0f;
    // the narrow result: channels 16 (wave % CB) + 4 quarter + 0 .. 3, positions 16 NH (wave / CB) + 16 h + l16
    const int cn = wave % CB * 16, pn = wave / CB * (16 * NH);
    bf16x8_t wn[KN];
    float gn[4], sn[4], bn[4];
    if constexpr (PAIR) {
#pragma unroll
        for (int k = 0; k < KN; ++k) wn[k] = *reinterpret_cast<const bf16x8_t*>(b.w + (cn + l16) * W + k * 32 + quarter * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            gn[e] = b.gain[cn + quarter * 4 + e];
            sn[e] = b.shift[cn + quarter * 4 + e];
            bn[e] = b.bias ? b.bias[cn + quarter * 4 + e] : 0.0f;
        }
    }

    keep_x();
    for (int base = 0; base < mine; base += kPwRows) {
        const bool more = base + kPwRows < mine;
        if (more) request_x(base + kPwRows);
        pw_barrier();
        f32x4v_t d[2][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int j = 0; j < 2; ++j) d[j][c] = f32x4v_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < KX; ++k) {
                const bf16x8_t f = *reinterpret_cast<const bf16x8_t*>(xs + (c * 16 + l16) * SX + k * 64 + quarter * 16);
#pragma unroll
                for (int j = 0; j < 2; ++j) d[j][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j][k], f, d[j][c], 0, 0, 0);
            }
        }
        // register r of block j: channel ch + 4 j + r of position 16 c + l16
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int p = base + c * 16 + l16;
            bf16x8_t zo, yo;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                zo[e] = (bf16_t)(d[e >> 2][c][e & 3] + bi[e]);
                float v = (float)(bf16_t)(g[e] * (float)zo[e] + sh[e]);   // rounded as the stored tensor would be
                if (res) v += (float)vr[c][e];
                if (a.relu) v = v > 0.0f ? v : 0.0f;
                yo[e] = (bf16_t)v;
            }
            if (p < mine) {
                const uint32_t at = (uint32_t)(p * W + ch);
                __builtin_nontemporal_store(zo, reinterpret_cast<bf16x8_t*>(z + at));
                *reinterpret_cast<bf16x8_t*>(y + at) = yo;
                if (again) *reinterpret_cast<bf16x8_t*>(again + at) = yo;
            }
            if constexpr (PAIR) *reinterpret_cast<bf16x8_t*>(ys + (c * 16 + l16) * SY + ch * 2) = yo;
        }
        if (more) request_res(base + kPwRows);
        pw_barrier();
        if (more) keep_x();
        if constexpr (PAIR) {
            f32x4v_t n[NH];
#pragma unroll
            for (int h = 0; h < NH; ++h) n[h] = f32x4v_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < KN; ++k)
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    n[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wn[k], *reinterpret_cast<const bf16x8_t*>(ys + (pn + h * 16 + l16) * SY + k * 64 + quarter * 16), n[h], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const int p = base + pn + h * 16 + l16;
                typedef bf16_t bf16x4_t __attribute__((ext_vector_type(4)));
                bf16x4_t zo, yo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    zo[e] = (bf16_t)(n[h][e] + bn[e]);
                    float v = (float)(bf16_t)(gn[e] * (float)zo[e] + sn[e]);
                    if (b.relu) v = v > 0.0f ? v : 0.0f;
                    yo[e] = (bf16_t)v;
                }
                if (p < mine) {
                    const int64_t at = (int64_t)(p0 + p) * C + cn + quarter * 4;
                    *reinterpret_cast<bf16x4_t*>(b.z + at) = zo;
                    *reinterpret_cast<bf16x4_t*>(b.y + at) = yo;
                }
            }
        }
    }
}

// Layers that widen 32 or 64 channels to twice or four times as many (a bottleneck block's last one).  The contractions' kernels and this one over 1024, 4096, 16384, 65536
// and 200704 positions (us): 32 -> 64 5.0 / 5.5 / 6.4 / 10.4 / 20.0 and 4.5 / 4.9 / 5.0 / 8.0 / 13.0, 32 -> 128 5.3 / 5.3 / 8.5 / 11.7 / 31.0 and 5.0 / 5.0 / 6.9 / 10.2 /
// 20.4, 64 -> 128 5.0 / 6.0 / 8.4 / 11.7 / 32.1 and 5.4 / 5.6 / 7.5 / 10.6 / 23.0, 64 -> 256 5.0 / 6.2 / 9.9 / 20.3 / 64 and 6.1 / 6.3 / 8.5 / 15.1 / 40.  As wide as
// their input they gain at some sizes and lose at others (64 -> 64 over 32768 8.5 and 6.8, over 65536 9.4 and 9.7), and from 128 channels, whose weights take the registers of
// what should be on its way, they lose (128 -> 256 over 65536 15.5 and 21, 128 -> 512 over 4096 6.3 and 9.1).  With the next convolution a launch is saved as well: all
// convolutions of a block and the next one's first over 256, 1024, 4096, 16384 and 200704 positions, 32 and 64 channels 18.0 / 18.5 / 18.9 / 19.0 / 75 and 13.2 / 13.0 / 13.9 /
// 16.7 / 57, 32 and 128 17.5 / 18.3 / 19.0 / 20.8 / 98 and 13.7 / 13.4 / 14.9 / 17.0 / 71, 64 and 128 17.8 / 18.4 / 19.0 / 21.5 / 103 and 14.5 / 15.2 / 15.6 / 19.6 / 88, 64
// and 256 18.1 / 19.5 / 19.2 / 23.2 / 173 and 17.0 / 17.8 / 17.6 / 20.2 / 155.
bool pointwise_forward_takes(int64_t P, int Cin, int Cout, bool next) {
    return (Cin == 32 || Cin == 64) && (Cout == 2 * Cin || Cout == 4 * Cin) && P >= (next ? 256 : 4096) && P < (int64_t(1) << 31) - 4096;
}

// Sixteen waves to a compute unit, eight with a second layer.
template <int C, int W, bool PAIR>
static hipError_t launch_pointwise_forward(const PwWide& a, const PwNarrow& b, int64_t P, hipStream_t s) {
    constexpr int most = (PAIR ? 8 : 16) * 256 * 32 / W;
    const int grid = (int)std::min<int64_t>(most, (P + 31) / 32), per = (int)((P + grid - 1) / grid);
    return launch_timed(kcConvFwd, pointwise_fwd_kernel<C, W, PAIR>, dim3(grid), dim3(2 * W), 0, s, a, b, (int)P, per);
}

hipError_t pointwise_forward(const PointwiseForward& f, const PointwiseForward* next, int64_t P, int Cin, int Cout, hipStream_t s) {
    const PwWide a{(const bf16_t*)f.x, (const bf16_t*)f.w, (const bf16_t*)f.res, f.bias, f.gain, f.shift, (bf16_t*)f.z, (bf16_t*)f.y, (bf16_t*)f.again, f.relu};
    PwNarrow b{};
    if (next) b = PwNarrow{(const bf16_t*)next->w, next->bias, next->gain, next->shift, (bf16_t*)next->z, (bf16_t*)next->y, next->relu};
#define TMPS_POINTWISE(c, w) \
    if (Cin == c && Cout == w) return next ? launch_pointwise_forward<c, w, true>(a, b, P, s) : launch_pointwise_forward<c, w, false>(a, b, P, s)
    TMPS_POINTWISE(32, 64);
    TMPS_POINTWISE(32, 128);
    TMPS_POINTWISE(64, 128);
    TMPS_POINTWISE(64, 256);
#undef TMPS_POINTWISE
    return hipErrorInvalidValue;
}

// Partial results stay within the 16 MB that a backward pass keeps until its end, a workgroup to a compute unit.
int affine_pointwise_slabs(int64_t P, int O, int I) {
    const int64_t most = std::min<int64_t>(256, (int64_t(1) << 22) / (O * I + O)), per = ((P + most - 1) / most + 15) / 16 * 16;
    return (int)((P + per - 1) / per);
}

// From 1024 positions on: below, a step of 64 is mostly the workgroup's start and end.  dW has to fit the accumulators of a workgroup beside what is on its way.
bool affine_pointwise_takes(int dtype, int64_t P, int O, int I) {
    auto width = [](int n) { return n == 64 || n == 128 || n == 256; };
    return dtype == kBF16 && width(O) && width(I) && O * I <= 16384 && P >= 1024 && P < (int64_t(1) << 31) - 4096;
}

template <int O, int I>
static hipError_t launch_pointwise(const void* dy, const void* z, const void* x, const void* w, const float* gain, const void* add, int masked, void* dx,
                                   float* gw_affine, float* gw_conv, const Partials& pa, const Partials& pw, int P, hipStream_t s) {
    constexpr int lds = pw_lds_bytes<O, I>();
    auto kern = affine_pointwise_bwd_kernel<O, I>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    const int slabs = affine_pointwise_slabs(P, O, I), per = ((P + slabs - 1) / slabs + 15) / 16 * 16;
    hipError_t e = launch_timed(kcAffine, kern, dim3(slabs), dim3(kPwThreads), lds, s, (const bf16_t*)dy, (const bf16_t*)z, (const bf16_t*)x, (const bf16_t*)w, gain,
                                (const bf16_t*)add, masked, (bf16_t*)dx, pa.ws, pw.ws, P, per);
    if (e != hipSuccess) return e;
    if ((e = pa.finish(Reduction{pa.ws, gw_affine, 2 * O, slabs, true}, s)) != hipSuccess) return e;
    return pw.finish(Reduction{pw.ws, gw_conv, (int64_t)O * I + O, slabs, false}, s);
}

hipError_t affine_pointwise_backward(const void* dy, const void* z, const void* x, const void* w, const float* gain, const void* add, int masked, void* dx,
                                     float* gw_affine, float* gw_conv, const Partials& pa, const Partials& pw, int64_t P, int O, int I, hipStream_t s) {
#define TMPS_POINTWISE(o, i) \
    if (O == o && I == i) return launch_pointwise<o, i>(dy, z, x, w, gain, add, masked, dx, gw_affine, gw_conv, pa, pw, (int)P, s)
    TMPS_POINTWISE(64, 64);
    TMPS_POINTWISE(64, 128);
    TMPS_POINTWISE(128, 64);
    TMPS_POINTWISE(128, 128);
    TMPS_POINTWISE(64, 256);
    TMPS_POINTWISE(256, 64);
#undef TMPS_POINTWISE
    return hipErrorInvalidValue;
}

}  // namespace tmps

extern "C" int tmps_pointwise_gradients_joint(int dtype, int64_t positions, int cin, int cout) {
    return tmps::affine_pointwise_takes(dtype, positions, cout, cin) ? 1 : 0;
}
extern "C" int tmps_pointwise_forward_joint(int dtype, int64_t positions, int cin, int cout) {
    return dtype == tmps::kBF16 && tmps::pointwise_forward_takes(positions, cin, cout, true) ? 1 : 0;
}
