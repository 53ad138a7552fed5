// What the contraction kernels of the stage step share: element types, conversions, 8-wide loads and stores, and the
// epilogues that end a GEMM C[m, n] = sum_k A(m, k) * B(n, k).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace tmps {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }

union Pack8 {
    uint4 u;
    bf16_t h[8];
};

// ------------------------------------------------------------------------------------------
// Epilogues: called once per output element (at) or once per 8 consecutive columns of a row (at8, where every tensor is
// 16-byte aligned and columns come in eights) with the fp32 accumulators.  `z` is the split-K slice.
// ------------------------------------------------------------------------------------------

// Exact GELU z * Phi(z) and its derivative Phi(z) + z * phi(z), Phi(z) = (1 + erf(z / sqrt 2)) / 2.
// erf by the rational-times-Gaussian formula of Abramowitz & Stegun 7.1.26 (|error| < 1.5e-7, at the level of fp32
// rounding), with the hardware reciprocal and exp2: the library erff costs several dozen instructions per element,
// which made the GELU epilogues longer than the k-loops of the GEMMs they end.  E = exp(-z^2 / 2) serves both the
// erf and the density phi(z) = E / sqrt(2 pi).
__device__ __forceinline__ void gelu_parts(float z, float& Phi, float& E) {
    const float x = fabsf(z) * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
    E = __expf(-x * x);
    float p = fmaf(1.061405429f, t, -1.453152027f);
    p = fmaf(p, t, 1.421413741f);
    p = fmaf(p, t, -0.284496736f);
    p = fmaf(p, t, 0.254829592f);
    const float er = 1.0f - p * t * E;             // erf(|z| / sqrt 2)
    Phi = 0.5f * (1.0f + copysignf(er, z));
}
__device__ __forceinline__ float gelu_f(float z) {
    float Phi, E;
    gelu_parts(z, Phi, E);
    return z * Phi;
}
__device__ __forceinline__ float gelu_grad_f(float z) {
    float Phi, E;
    gelu_parts(z, Phi, E);
    return Phi + z * 0.3989422804014327f * E;
}
// both at once: y = gelu(z), d = gelu'(z)
__device__ __forceinline__ void gelu_both(float z, float& y, float& d) {
    float Phi, E;
    gelu_parts(z, Phi, E);
    y = z * Phi;
    d = Phi + z * 0.3989422804014327f * E;
}

enum { kActNone = 0, kActRelu = 1, kActGelu = 2 };

// 8 consecutive elements with 16-byte accesses (the address is 16-byte aligned)
__device__ __forceinline__ void store8(bf16_t* p, const float (&v)[8]) {
    // (in pairs: one conversion makes two values in the halves of a register, one by one they are put together with a permutation more each)
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{v[2 * e], v[2 * e + 1]}), bf16x2_t));
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
    Pack8 pk;
    pk.u = *reinterpret_cast<const uint4*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)pk.h[e];
}
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// 8 consecutive elements fetched now and converted later: the 8-wide epilogues request what they read from memory
// (a residual source, a mask, the gradient already collected) for several rows at once, BEFORE the results of those
// rows are ready, so that the memory latency is paid once per group of rows and not once per row.
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
    uint4 u;
    __device__ __forceinline__ void load(const bf16_t* p) { u = *reinterpret_cast<const uint4*>(p); }
    // (from whole words: as an array of 16-bit values the compiler takes them apart where they arrive and holds twice the registers)
    __device__ __forceinline__ void get(float (&v)[8]) const {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = __builtin_bit_cast(float, w[e] << 16);
            v[2 * e + 1] = __builtin_bit_cast(float, w[e] & 0xffff0000u);
        }
    }
};
template <> struct Raw8<float> {
    float4 a, b;
    __device__ __forceinline__ void load(const float* p) {
        a = *reinterpret_cast<const float4*>(p);
        b = *reinterpret_cast<const float4*>(p + 4);
    }
    __device__ __forceinline__ void get(float (&v)[8]) const {
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
};
struct NoCol8 {};
struct NoRow8 {};

// Forms of an epilogue.  What an epilogue does hangs on arguments that are the same for a whole launch (an activation, a mask, a second result); asked for
// at every 8 elements, those questions are branches and moves that a kernel with a wave or two to a SIMD waits for.  E::form() names the combination (below 0:
// none of those that have an instance of their own); EpiForm is E for one of them, with the elements at `base` (the same for the wave) + `off` (of
// the lane): a load takes a scalar base and a 32-bit offset, a store one addition in the vector unit.  (Bytes are counted on the pointer: behind a cast to an integer and back the compiler
// no longer knows that it points to global memory and takes generic accesses, which count as LDS accesses too, so that it waits for all of both.)
template <class T> __device__ __forceinline__ T* at_lane(T* p, int64_t base, uint32_t off) {
    typedef std::conditional_t<std::is_const<T>::value, const char, char> byte_t;
    return reinterpret_cast<T*>(reinterpret_cast<byte_t*>(p + base) + (uint32_t)(off * (uint32_t)sizeof(T)));
}
constexpr int64_t kFormMaxLd = 1 << 22;   // 128 rows of fp32 are then less than 2^32 bytes
// The forms of the epilogues below by what they are given.
int bias_act_form(int act, bool bias, bool res, bool second, int64_t ld);
int conv_affine_form(bool bias, bool again, bool res, bool relu, int64_t ld);
int mask_form(int mode, bool mask, bool add, int64_t ld);
template <class E, int F> struct EpiForm : E {
    static constexpr bool kFormed = true;
    typedef decltype(E::template raw8f<F>()) Row8;
    __device__ __forceinline__ Row8 row8f(int64_t base, uint32_t off) const { return E::template request8f<F>(base, off); }
    __device__ __forceinline__ void at8f(const typename E::Col8& c, const Row8& p, int64_t base, uint32_t off, float (&v)[8], int z) const {
        E::template finish8f<F>(c, p, base, off, v, z);
    }
    // (for kernels whose rows lie where their loader says)
    __device__ __forceinline__ Row8 row8(int64_t idx, bool ok) const {
        Row8 p;
        if (ok) p = E::template request8f<F>(idx, 0);
        return p;
    }
    __device__ __forceinline__ void at8(const typename E::Col8& c, const Row8& p, int64_t idx, float (&v)[8], int z) const {
        E::template finish8f<F>(c, p, idx, 0, v, z);
    }
};

// Host-side test for the 8-wide (16-byte) form of an epilogue: every tensor it touches is 16-byte aligned and a row
// start keeps that alignment.
static inline bool epi_al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// out[m, n] = act(v + bias[n]) + res[m, n].  With GELU the DERIVATIVE gelu'(v + bias[n]) is stored as well (zout): the
// backward pass then multiplies by a stored factor, as it does for ReLU, instead of evaluating an erf and an
// exponential per element in the epilogue of the input-gradient GEMM (where that cost more than the GEMM's k-loop).
// res: a residual connection's source, same shape as out.  Without GELU zout is a second place for the result (what a stage hands to the next worker).
template <typename TOut> struct EpiBiasAct {
    TOut* out;
    const float* bias;  // may be null
    int64_t ld;
    int relu;           // kActNone / kActRelu / kActGelu
    const TOut* res = nullptr;
    TOut* zout = nullptr;
    __device__ __forceinline__ void finish(int64_t idx, float v) const {
        if (relu == kActRelu) v = v > 0.0f ? v : 0.0f;
        else if (relu == kActGelu) {
            float d;
            gelu_both(v, v, d);
            if (zout) zout[idx] = from_f32<TOut>(d);
        }
        if (res) v += to_f32(res[idx]);
        out[idx] = from_f32<TOut>(v);
        if (relu != kActGelu && zout) zout[idx] = from_f32<TOut>(v);
    }
    bool wide_ok() const { return ld % 8 == 0 && epi_al16(out) && epi_al16(bias) && epi_al16(res) && epi_al16(zout); }
    // the same in two steps: column(n) fetches the bias once, at() finishes element idx = m*ld + n
    __device__ __forceinline__ float column(int n) const { return bias ? bias[n] : 0.0f; }
    __device__ __forceinline__ void at(float b, int64_t idx, float v, int) const { finish(idx, v + b); }
    // the same with the column data (bias) and the row data (residual source) requested ahead of time
    struct Col8 { float b[8]; };
    struct Row8 { Raw8<TOut> r; };
    __device__ __forceinline__ Col8 col8(int n) const {
        Col8 c;
        if (bias) load8(bias + n, c.b);
        return c;
    }
    __device__ __forceinline__ Row8 row8(int64_t idx, bool ok) const {
        Row8 p;
        if (res && ok) p.r.load(res + idx);
        return p;
    }
    __device__ __forceinline__ void at8(const Col8& c, const Row8& p, int64_t idx, float (&v)[8], int) const {
        if (bias) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += c.b[e];
        }
        if (relu == kActRelu) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
        } else if (relu == kActGelu) {
            float d[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) gelu_both(v[e], v[e], d[e]);
            if (zout) store8(zout + idx, d);
        }
        if (res) {
            float r[8];
            p.r.get(r);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += r[e];
        }
        store8(out + idx, v);
        if (relu != kActGelu && zout) store8(zout + idx, v);
    }
    // 0: bias only, 1: ReLU, 2: GELU and its derivative, 3: a residual source.  (The last layer of a stage, whose result leaves twice, keeps the general
    // epilogue, with a residual source or without; an instance of its own for it has not been measured.)
    static constexpr bool kFormed = false;
    static constexpr int kForms = sizeof(TOut) == 2 ? 4 : 1;
    int form() const { return bias_act_form(relu, bias, res, zout, ld); }
    template <int F> static __device__ __host__ auto raw8f() {
        if constexpr (F == 3) return Row8{};
        else return NoRow8{};
    }
    template <int F> __device__ __forceinline__ auto request8f(int64_t base, uint32_t off) const {
        decltype(raw8f<F>()) p;
        if constexpr (F == 3) p.r.load(at_lane(res, base, off));
        return p;
    }
    template <int F, class R> __device__ __forceinline__ void finish8f(const Col8& c, const R& p, int64_t base, uint32_t off, float (&v)[8], int) const {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += c.b[e];
        if constexpr (F == 1) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
        } else if constexpr (F == 2) {
            float d[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) gelu_both(v[e], v[e], d[e]);
            store8(at_lane(zout, base, off), d);
        } else if constexpr (F == 3) {
            float r[8];
            p.r.get(r);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += r[e];
        }
        store8(at_lane(out, base, off), v);
    }
    __device__ __forceinline__ void rowsum(int, float, int) const {}
};

// Convolution followed by a per-channel affine layer and, optionally, a residual join, in one epilogue:
//   z = v + bias[n]                        -> out   (the convolution's result, kept for the affine layer's gradient)
//   a = gain[n] * z + shift[n]             (not stored: the backward pass of the affine layer needs z, that of the join only y)
//   y = act(a + res[m, n])                 -> yout and, if it is given, again (res may be null)
// Every stored tensor is rounded to its storage type before the next step reads it, exactly as if the three layers
// had run one after the other.
template <typename TOut> struct EpiConvAffine {
    TOut* out;
    const float* bias;   // may be null
    int64_t ld;
    const float* gain;
    const float* shift;
    TOut* again;         // a second place for y (what a stage hands to the next worker); may be null
    const TOut* res;     // second source of the residual join; may be null
    TOut* yout;
    int relu;
    struct Col { float b, g, s; };
    bool wide_ok() const {
        return ld % 8 == 0 && epi_al16(out) && epi_al16(bias) && epi_al16(gain) && epi_al16(shift) && epi_al16(again) &&
               epi_al16(res) && epi_al16(yout);
    }
    __device__ __forceinline__ Col column(int n) const { return Col{bias ? bias[n] : 0.0f, gain[n], shift[n]}; }
    __device__ __forceinline__ void at(const Col& c, int64_t idx, float v, int) const {
        const TOut z = from_f32<TOut>(v + c.b);
        out[idx] = z;
        const TOut ar = from_f32<TOut>(c.g * to_f32(z) + c.s);   // rounded as the stored tensor would be, stored or not
        float a = to_f32(ar);
        if (res) a += to_f32(res[idx]);
        if (relu) a = a > 0.0f ? a : 0.0f;
        yout[idx] = from_f32<TOut>(a);
        if (again) again[idx] = from_f32<TOut>(a);
    }
    struct Col8 { float b[8], g[8], s[8]; };
    struct Row8 { Raw8<TOut> r; };
    __device__ __forceinline__ Col8 col8(int n) const {
        Col8 c;
        load8(gain + n, c.g);
        load8(shift + n, c.s);
        if (bias) load8(bias + n, c.b);
        return c;
    }
    __device__ __forceinline__ Row8 row8(int64_t idx, bool ok) const {
        Row8 p;
        if (res && ok) p.r.load(res + idx);
        return p;
    }
    __device__ __forceinline__ void at8(const Col8& c, const Row8& p, int64_t idx, float (&v)[8], int) const {
        if (bias) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += c.b[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = to_f32(from_f32<TOut>(v[e]));
        store8(out + idx, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = to_f32(from_f32<TOut>(c.g[e] * v[e] + c.s[e]));   // rounded as the stored tensor would be
        if (res) {
            float r[8];
            p.r.get(r);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += r[e];
        }
        if (relu) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
        }
        store8(yout + idx, v);
        if (again) store8(again + idx, v);
    }
    // without a bias and a second copy (not measured as instances of their own): 0 the layers alone, 1 with ReLU, 2 with a residual source and ReLU
    static constexpr bool kFormed = false;
    static constexpr int kForms = sizeof(TOut) == 2 ? 3 : 0;
    int form() const { return conv_affine_form(bias, again, res, relu, ld); }
    template <int F> static __device__ __host__ auto raw8f() {
        if constexpr (F == 2) return Row8{};
        else return NoRow8{};
    }
    template <int F> __device__ __forceinline__ auto request8f(int64_t base, uint32_t off) const {
        decltype(raw8f<F>()) p;
        if constexpr (F == 2) p.r.load(at_lane(res, base, off));
        return p;
    }
    template <int F, class R> __device__ __forceinline__ void finish8f(const Col8& c, const R& p, int64_t base, uint32_t off, float (&v)[8], int) const {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = to_f32(from_f32<TOut>(v[e]));
        store8(at_lane(out, base, off), v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = to_f32(from_f32<TOut>(c.g[e] * v[e] + c.s[e]));   // rounded as the stored tensor would be
        if constexpr (F == 2) {
            float r[8];
            p.r.get(r);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += r[e];
        }
        if constexpr (F >= 1) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
        }
        store8(at_lane(yout, base, off), v);
    }
    __device__ __forceinline__ void rowsum(int, float, int) const {}
};

// Gradient through the stored activation of the layer below: mode kActRelu: v where mask[m, n] > 0 else 0
// (mask = that layer's output); mode kActGelu: v * mask[m, n] (mask = the derivative stored by that layer's forward pass).
// add (may be null, may be out itself): what other readers of the same tensor have already contributed to its
// gradient; it joins v before the mask is applied.
template <typename TOut, typename TMask> struct EpiMask {
    TOut* out;
    const TMask* mask;  // may be null
    int64_t ld;
    int mode = kActRelu;
    const TOut* add = nullptr;
    __device__ __forceinline__ void finish(int64_t i, float v) const {
        if (add) v += to_f32(add[i]);
        if (mask) {
            const float t = to_f32(mask[i]);
            if (mode == kActGelu) v *= t;
            else if (!(t > 0.0f)) v = 0.0f;
        }
        out[i] = from_f32<TOut>(v);
    }
    bool wide_ok() const { return ld % 8 == 0 && epi_al16(out) && epi_al16(mask) && epi_al16(add); }
    __device__ __forceinline__ int column(int) const { return 0; }
    __device__ __forceinline__ void at(int, int64_t i, float v, int) const { finish(i, v); }
    typedef NoCol8 Col8;
    struct Row8 { Raw8<TOut> a; Raw8<TMask> t; };
    __device__ __forceinline__ Col8 col8(int) const { return Col8{}; }
    __device__ __forceinline__ Row8 row8(int64_t i, bool ok) const {
        Row8 p;
        if (add && ok) p.a.load(add + i);
        if (mask && ok) p.t.load(mask + i);
        return p;
    }
    __device__ __forceinline__ void at8(const Col8&, const Row8& p, int64_t i, float (&v)[8], int) const {
        if (add) {
            float a[8];
            p.a.get(a);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += a[e];
        }
        if (mask) {
            float t[8];
            p.t.get(t);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (mode == kActGelu) v[e] *= t[e];
                else if (!(t[e] > 0.0f)) v[e] = 0.0f;
            }
        }
        store8(out + i, v);
    }
    // 0: no mask, 1: ReLU's, 2: GELU's, 3: what others have contributed and ReLU's
    static constexpr bool kFormed = false;
    static constexpr int kForms = sizeof(TOut) == 2 && sizeof(TMask) == 2 ? 4 : 0;
    int form() const { return mask_form(mode, mask, add, ld); }
    struct Mask8 { Raw8<TMask> t; };
    template <int F> static __device__ __host__ auto raw8f() {
        if constexpr (F == 3) return Row8{};
        else if constexpr (F > 0) return Mask8{};
        else return NoRow8{};
    }
    template <int F> __device__ __forceinline__ auto request8f(int64_t base, uint32_t off) const {
        decltype(raw8f<F>()) p;
        if constexpr (F == 3) p.a.load(at_lane(add, base, off));
        if constexpr (F > 0) p.t.load(at_lane(mask, base, off));
        return p;
    }
    template <int F, class R> __device__ __forceinline__ void finish8f(const Col8&, const R& p, int64_t base, uint32_t off, float (&v)[8], int) const {
        if constexpr (F == 3) {
            float a[8];
            p.a.get(a);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += a[e];
        }
        if constexpr (F > 0) {
            float t[8];
            p.t.get(t);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if constexpr (F == 2) v[e] *= t[e];
                else if (!(t[e] > 0.0f)) v[e] = 0.0f;
            }
        }
        store8(at_lane(out, base, off), v);
    }
    __device__ __forceinline__ void rowsum(int, float, int) const {}
};

// Weight gradient: fp32 [rows, cols] followed by the bias gradient [rows]; slice z writes its own
// copy at out + z*slice_stride (reduced afterwards), or the final location when there is one slice.
struct EpiWgrad {
    float* out;
    int64_t ld;            // cols
    int64_t bias_off;      // rows*cols
    int64_t slice_stride;  // rows*cols + rows
    bool wide_ok() const { return ld % 8 == 0 && slice_stride % 4 == 0 && epi_al16(out); }
    __device__ __forceinline__ int column(int) const { return 0; }
    __device__ __forceinline__ void at(int, int64_t idx, float v, int z) const {
        out[z * slice_stride + idx] = v;
    }
    typedef NoCol8 Col8;
    typedef NoRow8 Row8;
    __device__ __forceinline__ Col8 col8(int) const { return Col8{}; }
    __device__ __forceinline__ Row8 row8(int64_t, bool) const { return Row8{}; }
    __device__ __forceinline__ void at8(const Col8&, const Row8&, int64_t idx, float (&v)[8], int z) const {
        store8(out + z * slice_stride + idx, v);
    }
    static constexpr bool kFormed = false;
    static constexpr int kForms = 1;
    int form() const { return ld > kFormMaxLd ? -1 : 0; }
    template <int> static __device__ __host__ NoRow8 raw8f() { return NoRow8{}; }
    template <int> __device__ __forceinline__ NoRow8 request8f(int64_t, uint32_t) const { return NoRow8{}; }
    template <int> __device__ __forceinline__ void finish8f(const Col8&, const NoRow8&, int64_t base, uint32_t off, float (&v)[8], int z) const {
        store8(at_lane(out + z * slice_stride, base, off), v);
    }
    __device__ __forceinline__ void rowsum(int m, float v, int z) const {
        out[z * slice_stride + bias_off + m] = v;
    }
};

}  // namespace tmps
