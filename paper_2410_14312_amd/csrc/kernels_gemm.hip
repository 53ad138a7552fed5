// Launchers of the contraction kernels: dense and convolution forward, input gradient and weight gradient, for both
// element types; the bf16 instances of the tiled, the small and the persistent kernel (the fp32 ones are in
// kernels_gemm_f32.hip, those with gathering loaders in kernels_gemm_gather.hip).
#include <math.h>

#include <algorithm>

#include "gemm_dispatch.hip.h"

namespace tmps {

// ------------------------------------------------------------------------------------------
// Tile size and k-split of a [M x N x K] contraction.  Small outputs are split along k until the grid
// has a few hundred workgroups, as long as the fp32 partial sums do not outweigh the operands.
// ------------------------------------------------------------------------------------------
GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K) {
    GemmPlan p;
    const int64_t t128 = (int64_t)cdiv(M, 128) * cdiv(N, 128);
    const int64_t t64 = (int64_t)cdiv(M, 64) * cdiv(N, 64);
    const bool wide = N > 64 && M > 64;
    // An output with fewer 128-tiles than compute units and a contraction that is not long is latency-bound: more,
    // smaller workgroups finish sooner (measured on 1024-row transformer GEMMs: 13 us against 16 us; a row limit of
    // 2048 that used to stand here cost ResNet-50 1.6 % and VGG-16 2.8 % per step).
    const bool short_rows = t128 < 256 && K <= 4096;
    // (a long contraction is cut into slices anyway: then a dozen 128-tiles suffice to fill the device)
    // 128 x 128 tiles for outputs of 512 such tiles or more, for 64 or more with a contraction of 2048 or longer, and
    // for a dozen with a very long one; in between, the smaller tiles (128 x 64 for tall outputs) do better with
    // the stages' kernels sharing the device (swept on the ResNet-50, VGG-16 and GPT-2 workloads: a short contraction
    // is mostly epilogue, which the smaller tiles spread over more workgroups)
    p.tile = (wide && !short_rows && (t128 >= 512 || (t128 >= 64 && K >= 2048) || (K > 4096 && t128 >= 8))) ? 128 : 64;
    const int64_t tiles = p.tile == 128 ? t128 : t64;
    const int64_t target = 384;  // swept 32..2048 on the VGG workload: flat optimum around 384-512
    int64_t s = 1;
    // (short outputs with 64 tiles or more and a short contraction are not split: the finishing kernel costs
    // more than the split saves; swept 1..256)
    if (tiles < target && !(short_rows && tiles >= 64)) {
        s = (target + tiles - 1) / tiles;
        const int64_t by_k = K / 128;
        const int64_t by_bytes = ((M + N) * K) / (2 * M * N);
        if (s > by_k) s = by_k;
        if (s > by_bytes) s = by_bytes;
        if (s > 64) s = 64;
        if (s < 1) s = 1;
    }
    p.slices = (int)s;
    return p;
}

// ---- estimates (cycles at 2.4 GHz) ----
// what a k-split costs beside its kernel: the finishing launch and the partial sums' way through memory (5 TB/s)
static double split_cost(int64_t M, int64_t N, int64_t slices) { return slices > 1 ? 9000.0 + (double)slices * M * N * 8.0 / 2083.0 : 0.0; }

// Tiled kernel in bf16: cycles of a k-tile of a workgroup alone on its unit, and of each of several that share one
// (1024 rows x 768: 0.3 us; 1024 x 2304 and 3072 in 128 x 64 tiles and 8192 x 768 in 128 x 128: two to a unit).  With a
// convolution's loaders a k-tile takes longer (8 x 8 x 256 -> 256 on 32 images: 1000 cycles forward, 1400 in the gradients), and
// with both operands read across k in a weight gradient (1024 and 4096 rows x 768 -> 2304 and 3072).
static double tiled_cost_bf16(int64_t M, int64_t N, int64_t K, int bm, int bn, bool rowsum, int by_k, int64_t slices) {
    const bool conv = by_k == kByKConv;
    const double alone = bm * bn == 4096 ? (conv ? 1100.0 : rowsum ? 880.0 : 720.0) : bm * bn == 8192 ? 1140.0 : (conv ? 1800.0 : 1500.0);
    const double shared = bm * bn == 4096 ? (rowsum ? 670.0 : conv ? 600.0 : 400.0) : alone;
    const double rounds = (double)cdiv((int64_t)cdiv(M, bm) * cdiv(N, bn) * slices, kCUs);
    return 5300.0 + (double)cdiv(cdiv(K, 64), slices) * fmax(alone, shared * rounds) + split_cost(M, N, slices);
}

// fp32: the busiest compute unit's multiplies (1024 cycles for a k-tile of a 64 x 64 tile; small tiles weighed up for the
// LDS traffic they need more of per product) and what a workgroup alone on its unit cannot hide.
static double tiled_cost_f32(int64_t M, int64_t N, int64_t K, int bm, int bn, int64_t slices) {
    const double per_ktile = (bm / 64) * (bn / 64) * 1024.0, weight = bm * bn == 4096 ? 1.10 : bm * bn == 8192 ? 1.04 : 1.0;
    const double nk = (double)cdiv(cdiv(K, 32), slices), rounds = (double)cdiv((int64_t)cdiv(M, bm) * cdiv(N, bn) * slices, kCUs);
    return rounds * nk * per_ktile * weight + (rounds <= 1.0 ? 300.0 * nk : 0.0) + 5000.0 + split_cost(M, N, slices);
}

// k-sharing kernel: a wave's k-tile takes 1800 cycles in bf16 (80 bytes/ns into the unit; 1024 x 768 x 3072), 2250 in a weight
// gradient (8192 x 768 -> 768), 2500 where addresses are a convolution's (8 x 8 x 256 -> 256), and 4300 in fp32 (its multiplies);
// one workgroup to a unit, prologue and epilogue not overlapped.
static double by_k_cost(int64_t M, int64_t N, int64_t K, int esize, bool rowsum, int by_k, int64_t slices) {
    const int64_t nk = cdiv(cdiv(K, 128 / esize), slices);
    const double rounds = (double)cdiv((int64_t)cdiv(M, 64) * cdiv(N, 64) * slices, kCUs);
    const double per_ktile = esize == 4 ? 4300.0 : by_k == kByKConv ? 2500.0 : rowsum ? 2250.0 : 1800.0;
    return 5500.0 + rounds * ((double)cdiv(nk, 4) * per_ktile + 3500.0) + split_cost(M, N, slices);
}

// 128 x 128 kernel with asynchronous copies: two k-tiles a step, one workgroup to a unit (1024 and 4096 rows x 768 to 3072).
static double async_cost(int64_t M, int64_t N, int64_t K, int by_k, int64_t slices) {
    const double steps = (double)cdiv(cdiv(cdiv(K, 64), slices), 2);
    const double rounds = (double)cdiv((int64_t)cdiv(M, 128) * cdiv(N, 128) * slices, kCUs);
    return rounds * (11300.0 + steps * (by_k == kByKConv ? 2900.0 : 2470.0)) + split_cost(M, N, slices);
}

Plan2 plan_for(int64_t M, int64_t N, int64_t K, bool rowsum, int esize, int by_k) {
    Plan2 best{64, 64, 1, kTiled, 0.0};
    auto each_split = [&](auto&& f) {   // (at most 64 MB of partial sums, at least 128 k to a slice)
        for (int64_t sl = 1; sl <= 64; sl += sl < 8 ? 1 : sl < 16 ? 2 : 8) {
            if (sl > 1 && (K < sl * 128 || sl * M * N > (int64_t(1) << 24))) break;
            f(sl);
        }
    };
    if (esize == 4) {
        static const int shape[3][2] = {{64, 64}, {128, 64}, {128, 128}};
        for (const auto& sh : shape) {
            if (rowsum && sh[0] != sh[1]) continue;
            each_split([&](int64_t sl) {
                const double t = tiled_cost_f32(M, N, K, sh[0], sh[1], sl);
                if (best.cost == 0.0 || t < best.cost) best = {sh[0], sh[1], (int)sl, kTiled, t};
            });
        }
    } else {
        const GemmPlan p = plan_gemm(M, N, K);
        // Where the plan's edge is 64, the output has 512 rows or more and 128 x 64 tiles still make 192 workgroups, the
        // tiles are 128 rows tall: a 128 x 64 tile reads a quarter less LDS per MFMA than a 64 x 64 one, and with the
        // stages' kernels sharing the device that outweighs having half as many workgroups (measured: GPT-2 and ResNet-50
        // steps 1 % shorter, VGG-16 1-2 %; 128 x 128 and 64 x 128 for the same launches did worse; below 192 workgroups
        // the launch itself gets slower and the step no faster).
        const bool tall = p.tile == 64 && !rowsum && M >= 512 && (int64_t)cdiv(M, 128) * cdiv(N, 64) * p.slices >= 192;
        best = {tall ? 128 : p.tile, p.tile, p.slices, kTiled, 0.0};
        best.cost = tiled_cost_bf16(M, N, K, best.bm, best.bn, rowsum, by_k, best.slices);
    }
    if (by_k != kByKNo) {
        Plan2 k{64, 64, 1, kByK, 0.0};
        each_split([&](int64_t sl) {
            const double t = by_k_cost(M, N, K, esize, rowsum, by_k, sl);
            if (k.cost == 0.0 || t < k.cost) k = {64, 64, (int)sl, kByK, t};
            const double ta = esize == 2 ? async_cost(M, N, K, by_k, sl) : t;
            if (ta < k.cost) k = {128, 128, (int)sl, kAsync, ta};
        });
        if (k.cost < 0.9 * best.cost) best = k;
    }
    return best;
}

// Small kernel: the smallest tiles that are no more than the compute units.  What a unit's fragment loads touch sets the pace: cycles per k
// of 16 x 16, 16 x 32 and 32 x 32 outputs 9, 14 and 18.5 in fp32, 4.2, 6.2 and 9.2 in bf16 (64 to 256 rows x 768 to 1024, K = 64 to 3072), and a fixed part.
// (20 for the third, as alone it measures, sends fp32 layers of some 300 such outputs to the tiled kernel in slices: forward 235 x 748 -> 1581 and 69 x 1518 -> 1730, both gradients
// with them, 38.5 and 38.9 us instead of 37.4 and 37.1; sums 1.7e-7 (2-norm) from those in 64 bits instead of 1.0e-7.)
SmallPlan small_plan(int64_t M, int64_t N, int64_t K, int esize) {
    static const int shape[3][2] = {{1, 1}, {1, 2}, {2, 2}};
    static const double per_k[2][3] = {{9.0, 14.0, 18.5}, {4.2, 6.2, 9.2}};
    for (int i = 0;; ++i) {
        const int64_t tiles = (int64_t)cdiv(M, 16 * shape[i][0]) * cdiv(N, 16 * shape[i][1]);
        if (i == 2 || tiles <= kCUs) return SmallPlan{shape[i][0], shape[i][1], 2500.0 + (double)cdiv(tiles, kCUs) * K * per_k[esize == 4 ? 0 : 1][i]};
    }
}
bool small_is_better(int64_t M, int64_t N, int64_t K, int esize, const Plan2& other) {
    if ((int64_t)cdiv(M, 32) * cdiv(N, 32) > 2 * kCUs) return false;
    return small_plan(M, N, K, esize).cost < other.cost;
}

int g3_wgrad_slices(int64_t M, int64_t N, int64_t K);
int g3_long_k_slices(int64_t M, int64_t N, int64_t K);

size_t gemm_workspace_elems(int64_t M, int64_t N, int64_t K, int flags) {
    const bool with_rowsum = (flags & kWsRowSums) != 0;
    const int esize = (flags & kWsF32) ? 4 : 2;
    int slices = 1;   // (which plan a launch takes depends on what its operands are and on their alignment)
    for (int by_k : {kByKNo, kByKDense, kByKConv}) slices = std::max(slices, plan_for(M, N, K, with_rowsum, esize, by_k).slices);
    if (esize == 2) {   // a weight gradient, or an input gradient with a very long contraction, may go to the persistent path
        const int s3 = with_rowsum ? g3_wgrad_slices(M, N, K) : g3_long_k_slices(M, N, K);
        if (s3 > slices) slices = s3;
    }
    if (slices <= 1) return 0;
    return (size_t)(slices + 1) * ((size_t)M * N + (with_rowsum ? (size_t)M : 0));
}

// ---- sums of partial results ----------------------------------------------------------------------------
// A job's outputs are shared out over workgroups of 256 threads: 1024 of them, four to a thread, where they lie in 16-byte pieces; 256; or, where many
// short rows are added up, 16, by sixteen lanes of rows each, combined through LDS.  Eight partial results in flight are added in pairs, then to the
// sum: an eighth of the roundings in its chain (bias gradients of 32 x 32 x 64 over 128 images 1.6e-7 (2-norm, against 64 bits) in order and 0.8e-7 so, layer
// normalisation's gains over 16384 rows 1.6e-7 and 1.2e-7).  Alone such a sum takes
// 4.5 us for a few hundred kilobytes, and a mini-batch of ResNet-50 has 97 of them: two mini-batches 14.88 ms with a launch for each, 14.20
// with one launch at the end of every backward pass; its first group of blocks as a stage 2.70 and 2.60 ms.
constexpr int kReduceMax = 64;
struct ReduceJob {
    const float* part;
    float* out;
    int64_t count;
    int slices, form;   // form: 0 four outputs to a thread, 1 one, 2 rows, 3 rows of four outputs
};
struct ReduceJobs {
    int first[kReduceMax];   // first workgroup of a job; where there is none, the number of workgroups
    ReduceJob job[kReduceMax];
};

__global__ __launch_bounds__(256) void reduce_kernel(ReduceJobs all) {
    __shared__ float sp[16][16];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int j = __builtin_amdgcn_readfirstlane(__popcll(__ballot(b >= all.first[tid & 63])) - 1);
    const ReduceJob r = all.job[j];
    const int blk = b - all.first[j];
    if (r.form == 0) {
        const int64_t i = ((int64_t)blk * 256 + tid) * 4;
        if (i >= r.count) return;
        const float* p = r.part + i;
        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        int z = 0;
        for (; z + 8 <= r.slices; z += 8) {   // eight loads in flight
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(p + u * r.count);
#pragma unroll
            for (int h = 4; h > 0; h >>= 1)
#pragma unroll
                for (int u = 0; u < h; ++u) {
                    v[u].x += v[u + h].x; v[u].y += v[u + h].y; v[u].z += v[u + h].z; v[u].w += v[u + h].w;
                }
            a.x += v[0].x; a.y += v[0].y; a.z += v[0].z; a.w += v[0].w;
            p += 8 * r.count;
        }
        for (; z < r.slices; ++z) {
            const float4 v = *reinterpret_cast<const float4*>(p);
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
            p += r.count;
        }
        *reinterpret_cast<float4*>(r.out + i) = a;
        return;
    }
    if (r.form == 3) {
        // sixteen lanes of rows, four outputs to a thread, eight rows in flight
        __shared__ float4 sp4[16][16];
        const int64_t i = (int64_t)blk * 64 + (tid & 15) * 4;
        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        auto plus = [](float4& x, const float4& y) { x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w; };
        if (i < r.count) {
            const float* p = r.part + (int64_t)(tid >> 4) * r.count + i;
            const int64_t step = 16 * r.count;
            int z = tid >> 4;
            for (; z + 7 * 16 < r.slices; z += 8 * 16) {
                float4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(p + u * step);
#pragma unroll
                for (int h = 4; h > 0; h >>= 1)
#pragma unroll
                    for (int u = 0; u < h; ++u) plus(v[u], v[u + h]);
                plus(a, v[0]);
                p += 8 * step;
            }
            for (; z < r.slices; z += 16) {
                plus(a, *reinterpret_cast<const float4*>(p));
                p += step;
            }
        }
        sp4[tid >> 4][tid & 15] = a;
        __syncthreads();
        if (tid < 16 && i < r.count) {
            float4 t[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) t[k] = sp4[k][tid];
#pragma unroll
            for (int h = 8; h > 0; h >>= 1)
#pragma unroll
                for (int k = 0; k < h; ++k) plus(t[k], t[k + h]);
            *reinterpret_cast<float4*>(r.out + i) = t[0];
        }
        return;
    }
    const bool rows = r.form == 2;
    const int lane_z = rows ? tid >> 4 : 0, lanes = rows ? 16 : 1;
    const int64_t i = rows ? (int64_t)blk * 16 + (tid & 15) : (int64_t)blk * 256 + tid;
    float a = 0.0f;
    if (i < r.count) {
        const float* p = r.part + (int64_t)lane_z * r.count + i;
        const int64_t step = (int64_t)lanes * r.count;
        int z = lane_z;
        for (; z + 7 * lanes < r.slices; z += 8 * lanes) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[u * step];
#pragma unroll
            for (int h = 4; h > 0; h >>= 1)
#pragma unroll
                for (int u = 0; u < h; ++u) v[u] += v[u + h];
            a += v[0];
            p += 8 * step;
        }
        for (; z < r.slices; z += lanes) {
            a += *p;
            p += step;
        }
    }
    if (!rows) {
        if (i < r.count) r.out[i] = a;
        return;
    }
    sp[lane_z][tid & 15] = a;
    __syncthreads();
    if (lane_z == 0 && i < r.count) {
        float t[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) t[k] = sp[k][tid & 15];
#pragma unroll
        for (int h = 8; h > 0; h >>= 1)
#pragma unroll
            for (int k = 0; k < h; ++k) t[k] += t[k + h];
        r.out[i] = t[0];
    }
}

hipError_t reduce_all(const Reductions& list, hipStream_t s) {
    for (size_t at = 0; at < list.size(); at += kReduceMax) {
        const int n = (int)(list.size() - at < (size_t)kReduceMax ? list.size() - at : kReduceMax);
        ReduceJobs all;
        int64_t blocks = 0;
        for (int k = 0; k < kReduceMax; ++k) {
            all.first[k] = (int)blocks;
            all.job[k] = ReduceJob{nullptr, nullptr, 0, 0, 1};
            if (k >= n) continue;
            const Reduction& r = list[at + k];
            const bool wide = r.count % 4 == 0 && aligned16(r.part) && aligned16(r.out);
            const int form = r.rows ? 2 : !wide ? 1 : r.slices >= 32 && r.count <= (1 << 18) ? 3 : 0;
            all.job[k] = ReduceJob{r.part, r.out, r.count, r.slices, form};
            blocks += cdiv(r.count, form == 0 ? 1024 : form == 1 ? 256 : form == 2 ? 16 : 64);
            if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
        }
        if (blocks == 0) continue;
        const hipError_t e = launch_timed(kcSliceSum, reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, s, all);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---- forms of the dense epilogues ------------------------------------------------------------------------
int bias_act_form(int act, bool bias, bool res, bool second, int64_t ld) {
    if (!bias || ld > kFormMaxLd) return -1;
    if (act == kActGelu) return second && !res ? 2 : -1;
    return second ? -1 : act == kActRelu ? (res ? -1 : 1) : (res ? 3 : 0);
}
int conv_affine_form(bool bias, bool again, bool res, bool relu, int64_t ld) {
    return bias || again || ld > kFormMaxLd ? -1 : res ? (relu ? 2 : -1) : relu ? 1 : 0;
}
int mask_form(int mode, bool mask, bool add, int64_t ld) {
    if (ld > kFormMaxLd) return -1;
    if (add) return mask && mode == kActRelu ? 3 : -1;
    return !mask ? 0 : mode == kActGelu ? 2 : 1;
}

// ---- persistent MFMA path (gemm3.hip.h): large dense contractions --------------------------------------
static int compute_units() {
    static int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
            v = 256;
        return v;
    }();
    return n;
}

constexpr int kG3Tile = 256;
static int64_t g3_tiles(int64_t M, int64_t N) { return (int64_t)cdiv(M, kG3Tile) * cdiv(N, kG3Tile); }
// k-slices of a weight-gradient contraction on the persistent path (0: leave it to the other path).  Measured in whole runs:
// the path pays once a launch has about as many (tile, slice) units as the device has compute units.  Alone on the device (us, persistent and other kernels, with the
// sums of their slices): 4096 x 4096 over 1024 / 4096 rows 42 and 57 / 122 and 174, 4096 x 2048 over 4096 85 and 90, 3072 x 768 over 8192 58 and 67; but also 3072 x 3072, 144 units, which
// the line leaves to the others, over 1024 / 4096 32 and 38 / 89 and 123, and 2048 x 2048 over 4096, 4096 x 2048 over 2048 and 2048 x 1024 over 8192, 256 units each, which
// it does not, 56 and 43, 58 and 49, 56 and 49.
int g3_wgrad_slices(int64_t M, int64_t N, int64_t K) {
    if (K % 64 != 0 || M % 8 != 0 || N % 8 != 0) return 0;
    const int64_t tiles = g3_tiles(M, N);
    int64_t s = tiles >= 192 ? 1 : 256 / tiles;
    if (s > K / 1024) s = K / 1024;
    if (s < 1) s = 1;
    return tiles * s >= 200 ? (int)s : 0;   // (swept: 144..200 units are quicker on the other path, ResNet-50 step -1.7 %)
}
// Not for a contraction of a single k-tile, which is all epilogue (many small workgroups keep more memory requests in
// flight than one persistent workgroup per compute unit), nor when more than a quarter of the 256-wide tiles would be
// padding (measured on the 1x1 convolutions of the residual networks).  192 tiles: swept in whole runs from 128 to 450, which changed nothing, when a k-tile took a fifth longer.  Alone on
// the device now (us, persistent and other kernels), 1024 columns over 256 / 768 / 3072: 256 tiles 16 and 22 / 28 and 40 / 87 and 124, 192 tiles 14 and 18 / 24 and 30 / 71 and 94; also
// 176, 160 and 144 tiles, which the line leaves to the others, 14 and 18 / 23 and 29 / 62 to 67 and 89, and only 128 no longer, 14 and 13 / 22 and 22 / 64 and 64.
bool g3_forward_ok(int64_t M, int64_t N, int64_t K) {
    return K % 64 == 0 && K >= 128 && N % 8 == 0 && g3_tiles(M, N) >= 192 && (int64_t)cdiv(N, 256) * 256 * 3 <= N * 4;
}

// A tall, narrow output (the 8192 x 768 input gradients of a transformer block: 96 tiles of 256 x 256, which leave most
// of the device idle) goes to the persistent kernel in 256 x 128 tiles with four waves of 128 x 64 each, where every unit has a
// compute unit to itself, the same output in 128 x 128 tiles would not (then the kernel with asynchronous copies walks it in
// one round: 256 tiles of 4096 x 1024, contraction 1024, 14.5 us against 17.7, 215 tiles of 640 x 5504 13.5 against 17.6), and a k-loop of at least 8
// k-tiles carries the unit's prologue and epilogue.  Input gradients alone on the device, persistent and other kernels (us), contractions over 512 /
// 1024 / 2048 / 4096: 8448 x 512 (264 tiles of 128 x 128) 11.5 / 16.6 / 25 / 44 and 15.5 / 23 / 42 / 72, 16384 x 512 (512 tiles)
// 14.3 / 21 / 35 / 62 and 18.1 / 28 / 47 / 87; the 8192 x 768 of a transformer block, over 2304 / 768 / 3072, 32 / 16 / 40 and 46 / 20 / 59.  (The 8 k-tiles are where both took
// 15 to 18 us when the line was drawn; over 256, 8192 x 1024 takes 10.8 and 12.7 now.)
bool g3_narrow_ok(int64_t M, int64_t N, int64_t K) {
    if (K % 64 != 0 || K < 512 || N % 128 != 0) return false;
    return (int64_t)cdiv(M, 256) * (N / 128) <= compute_units() && (int64_t)cdiv(M, 128) * (N / 128) > compute_units();
}

// An output of few 256-wide tiles with a very long contraction (the input gradient of a vocabulary-wide output layer:
// 96 tiles, k = 32000) goes to the persistent kernel in k-slices: the slice count is the one whose (tile, slice) units
// fill whole rounds of the device best, weighed against the fp32 partial sums it writes and the finishing pass reads
// (rates: 1 PFLOP/s in the k-loop, 5 TB/s for the partial sums; the k-loop is at 1.2 to 1.3 now, which leaves the choice as it is).  Of 2 to 16 slices the choice is the quickest of those measured, alone on the device
// (us, in brackets the slices; then the tiled kernel): 8192 x 768 over 32000 380 (5) and 459, 4096 x 768 187 (5) and 243, 8192 x 512 240 (4) and 305, 8192 x 1024 over 16384 238 (2) and 284,
// 4096 x 2048 over 8192 130 (2) and 142, 4096 x 1024 76 (4) and 72.  0: leave it to the tiled kernel.
int g3_long_k_slices(int64_t M, int64_t N, int64_t K) {
    if (K % 64 != 0 || N % 8 != 0 || K < 8192) return 0;
    const int64_t tiles = g3_tiles(M, N);
    if (tiles >= 192 || tiles < 32 || (int64_t)cdiv(N, 256) * 256 * 3 > N * 4) return 0;
    const int cus = compute_units();
    int best = 0;
    double best_us = 0.0;
    for (int sl = 2; sl <= 16; ++sl) {
        if (K / sl < 2048) break;
        const int64_t units = tiles * sl;
        const double fill = (double)units / (double)((units + cus - 1) / cus * cus);
        const double us = 2.0 * M * N * K / (fill * 1e9) + (double)sl * M * N * 8.0 / 5e6;
        if (best == 0 || us < best_us) {
            best = sl;
            best_us = us;
        }
    }
    return best;
}

static G3Plan g3_plan(int M, int N, int K, int slices, int bm = kG3Tile, int bn = kG3Tile) {
    G3Plan p;
    p.tiles_m = cdiv(M, bm);
    p.tiles_n = cdiv(N, bn);
    int per = cdiv(cdiv(K, slices), 64) * 64;
    p.k_per_slice = per;
    p.slices = cdiv(K, per);
    p.units = p.tiles_m * p.tiles_n * p.slices;
    p.col_major = N > M ? 1 : 0;   // the XCDs split the operand with more rows between them and each reads the other one whole
    p.d_tn = FastDiv(p.col_major ? p.tiles_m : p.tiles_n);
    p.d_tiles = FastDiv(p.tiles_m * p.tiles_n);
    // Blocks of 32 tiles for outputs wide enough that a run of 32 tiles would span few rows and all columns (or the
    // other way round): the squarest block whose sides divide the tile counts.
    p.gm = p.gn = 0;
    if (p.tiles_m >= 8 && p.tiles_n >= 8) {
        for (int gn : {4, 8, 2, 16}) {
            const int gm = 32 / gn;
            if (p.tiles_n % gn == 0 && p.tiles_m % gm == 0) {
                p.gm = gm;
                p.gn = gn;
                break;
            }
        }
    }
    if (p.gm) {
        p.d_blk = FastDiv(32);
        p.d_gn = FastDiv(p.gn);
        p.d_nbn = FastDiv(p.tiles_n / p.gn);
    }
    return p;
}

// Whether a tile of `rows` rows of an operand is copied at 32-bit offsets from a base that a wave shares.  Launches with longer rows are instances with
// addresses in each lane, which every length fits: the tiled kernels, whose grids hold fewer than 65536 rows of tiles, would refuse a weight gradient of so many.  Forward
// passes in 256 x 256 tiles have none (eight waves have no registers for such addresses beside that epilogue, 42 spills) and leave those rows to the tiled
// kernels: 192 tiles of 8.4 million k are 315 GB of operands, masters and momentum at the least.
bool g3_lane_offsets(bool k_contiguous, int rows, int64_t ld) {
    return k_contiguous ? g3_offsets_fit(rows, 64, ld) : g3_offsets_fit(64, rows, ld);
}
static bool g3_forward_takes(int64_t M, int64_t N, int64_t K) { return g3_forward_ok(M, N, K) && g3_lane_offsets(true, kG3Tile, K); }

// 256 x 256 x 64 tiles, 8 waves (2 x 4), two LDS stages: the configuration that did best on every large shape tried.
template <int BM, int BN, int WM, int WN, int NS, int PER_CU, bool AKC, bool BKC, bool ROWSUM, bool WIDE, class Epi>
static hipError_t launch3_form(int kc, const G3Operand<AKC>& A, const G3Operand<BKC>& B, const Epi& epi, int M, int N, int K,
                               const G3Plan& plan, hipStream_t s) {
    constexpr int lds = gemm3_lds_bytes<BM, BN, 64, NS>(WM * WN);
    auto kern = gemm3_kernel<BM, BN, 64, WM, WN, NS, AKC, BKC, ROWSUM, WIDE, Epi>;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    const int slots = compute_units() * PER_CU;
    const int grid = plan.units < slots ? plan.units : slots;
    return launch_timed(kc, kern, dim3(grid), dim3(64 * WM * WN), lds, s, A, B, epi, M, N, K, plan);
}

template <int BM, int BN, int WM, int WN, int NS, int PER_CU, bool AKC, bool BKC, bool ROWSUM, class Epi>
static hipError_t launch3_inst(int kc, const G3Operand<AKC>& A, const G3Operand<BKC>& B, const Epi& epi, int M, int N, int K,
                               const G3Plan& plan, hipStream_t s) {
    if (!g3_lane_offsets(AKC, BM, A.ld) || !g3_lane_offsets(BKC, BN, B.ld)) {
        if constexpr (WM * WN > 4 && AKC && BKC) return hipErrorInvalidValue;   // (g3_forward_takes)
        else return launch3_form<BM, BN, WM, WN, NS, PER_CU, AKC, BKC, ROWSUM, true>(kc, A, B, epi, M, N, K, plan, s);
    }
    if constexpr (Epi::kFormed) return launch3_form<BM, BN, WM, WN, NS, PER_CU, AKC, BKC, ROWSUM, false>(kc, A, B, epi, M, N, K, plan, s);
    else
        return with_form(epi.form(), epi, [&](const auto& e) {
            return launch3_form<BM, BN, WM, WN, NS, PER_CU, AKC, BKC, ROWSUM, false>(kc, A, B, e, M, N, K, plan, s);
        });
}

template <bool AKC, bool BKC, bool ROWSUM, class Epi>
static hipError_t launch3(int kc, const G3Operand<AKC>& A, const G3Operand<BKC>& B, const Epi& epi, int M, int N, int K,
                          const G3Plan& plan, hipStream_t s) {
    return launch3_inst<256, 256, 2, 4, 2, 1, AKC, BKC, ROWSUM>(kc, A, B, epi, M, N, K, plan, s);
}

// ---- weight gradients of several layers in one persistent launch (G3Group) --------------------------------------------------
constexpr int kG3GroupStages = 3;
__global__ __launch_bounds__(256) void gemm3_kernel(G3Group work) {
    gemm3_walk<G3Group::kRows, G3Group::kCols, 64, 2, 2, kG3GroupStages, false, false, true>(work);
}
__global__ __launch_bounds__(256) void gemm3_kernel(G3GroupRagged work) {
    gemm3_walk<G3Group::kRows, G3Group::kCols, 64, 2, 2, kG3GroupStages, false, false, true>(work);
}

// Adds up the slices of the cut tiles, in slice order: workgroup (r, y) takes 32 rows of cut tile r, a thread 4 columns of 4 rows.
__global__ __launch_bounds__(256) void g3_group_sum_kernel(G3Group work) {
    constexpr int L = G3Group::kCols / 4, R = 256 / L;   // threads of a row, rows at a time
    const int r = blockIdx.x, tid = threadIdx.x;
    int m0, n0;
    const G3Job& j = work.job[work.place(work.whole + r, m0, n0)];
    const float* const p = work.part + (int64_t)r * work.slices * G3Group::kPart;
    const int n = n0 + tid % L * 4, row0 = blockIdx.y * (4 * R) + tid / L;
    if (n < j.N) {
        float4 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const float4*>(p + (row0 + R * i) * G3Group::kCols + tid % L * 4);
        for (int z = 1; z < work.slices; ++z) {
            const float* const q = p + (int64_t)z * G3Group::kPart;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 w = *reinterpret_cast<const float4*>(q + (row0 + R * i) * G3Group::kCols + tid % L * 4);
                v[i].x += w.x; v[i].y += w.y; v[i].z += w.z; v[i].w += w.w;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + row0 + R * i;
            if (m < j.M) *reinterpret_cast<float4*>(j.out + (int64_t)m * j.N + n) = v[i];
        }
    }
    if (n0 == 0 && blockIdx.y == 0 && m0 + tid < j.M) {
        float v = 0.0f;
        for (int z = 0; z < work.slices; ++z) v += p[(int64_t)z * G3Group::kPart + G3Group::kRows * G3Group::kCols + tid];
        j.out[(int64_t)j.M * j.N + m0 + tid] = v;
    }
}

// Estimates of weight gradients in us: 1.78 for a k-tile of a 256 x 256 tile (8192^3: 911 us for 512 of them in a row), 8 for a unit's prologue and epilogue, partial sums at 6 TB/s and a
// launch.  Estimated and measured: 4096 x 4096 over 1024 / 2048 / 4096 / 8192 rows 36 and 42 / 65 and 69 / 122 and 122 / 236 and 233, 3072 x 768 over 8192 57 and 58, 2304 x 768 50 and 48.
constexpr double kG3KtileUs = 1.78, kG3UnitUs = 8.0;
// The same of a 256 x 128 tile of a group, and for adding its accumulators to the totals: 12 layers of 768 features over 1024 / 8192 rows 86 and 82 / 448 and 455.  What the estimates choose was
// the quicker of one launch and several for 52 of 60 groups measured (one to four transformer blocks of 512 to 1280 features, one to twenty square layers of 768 to 4096, 1024 to 8192 rows); the other
// eight keep launches of their own where one would be 6 to 25 % quicker: one block of 1024 features 61 and 53 us over 1024 rows, 95 and 79 over 2048.
constexpr double kGroupKtileUs = 1.10, kGroupUnitUs = 9.0, kGroupTotalUs = 0.5;
static double partial_sums_us(double slices, double elems) { return slices > 1 ? 3.0 + (slices + 1.0) * elems * 4.0 / 6e6 : 0.0; }

struct G3GroupPlan {
    int whole, slices, k_per_slice, chain;
    double us;
};
// k-tiles that are summed in one go, of kt: about the square root of as many multiplies, with as many roundings in a chain as in the totals
static int g3_group_chain(int64_t kt) { return kt < 16 ? 2 : kt < 64 ? 4 : 8; }
static int64_t g3_group_tiles(int64_t M, int64_t N) { return (int64_t)cdiv(M, G3Group::kRows) * cdiv(N, G3Group::kCols); }
// `whole` tiles (whole rounds of the device) unsliced, the others in the number of slices that is quickest.
static G3GroupPlan g3_group_plan(int64_t tiles, int64_t K, int64_t ws_elems) {
    const int cus = compute_units();
    const int64_t kt = cdiv(K, 64), full = tiles / cus;
    const int chain = g3_group_chain(kt);
    const double ktile_us = kGroupKtileUs + kGroupTotalUs / chain;
    G3GroupPlan best{0, 0, 0, chain, 0.0};
    for (int64_t f = full > 0 ? full - 1 : 0; f <= full; ++f) {
        const int64_t whole = f * cus, cut = tiles - whole;
        for (int64_t want = 1; want <= 16; ++want) {
            if (want > 1 && (kt < want * 8 || cut == 0)) break;
            const int64_t per = cdiv(kt, want), slices = cdiv(kt, per), rounds = cdiv(cut * slices, cus);
            if (slices > 1 && cut * slices * G3Group::kPart > ws_elems) break;
            const double us = (double)(f * kt + rounds * per) * ktile_us + (double)(f + rounds) * kGroupUnitUs +
                              partial_sums_us((double)slices, (double)cut * G3Group::kRows * G3Group::kCols);
            if (best.slices == 0 || us < best.us) best = {(int)whole, (int)slices, (int)per * 64, chain, us};
        }
    }
    return best;
}

static double wgrad_alone_us(int64_t M, int64_t N, int64_t K) {
    const int s3 = g3_wgrad_slices(M, N, K);
    if (s3 == 0) return plan_for(M, N, K, true, 2, kByKDense).cost / 2400.0;
    const int64_t per = cdiv(K / 64, s3), rounds = cdiv(g3_tiles(M, N) * s3, compute_units());
    return (double)(rounds * per) * kG3KtileUs + (double)rounds * kG3UnitUs + partial_sums_us(s3, (double)M * N);
}

// (not where more than a quarter of the 256-wide tiles would be padding; the eight rows that a wave stores at once lie within 2^32 bytes up to 2^27 columns of fp32, with
// at least 192 rows 360 GB of masters, momentum, gradient and working copy)
constexpr int64_t kGroupMaxCols = int64_t(1) << 27;
static_assert((7 * kGroupMaxCols + 64) * 4 <= (int64_t(1) << 32), "offsets of a wave's stores");
bool dense_wgrad_groups(int dtype, int64_t rows, int Din, int Dout) {
    return dtype == kBF16 && rows >= 512 && rows < (int64_t(1) << 31) && Din % 8 == 0 && Dout % 8 == 0 && Din <= kGroupMaxCols &&
           (int64_t)cdiv(Din, 256) * 256 * 3 <= (int64_t)Din * 4 && (int64_t)cdiv(Dout, 256) * 256 * 3 <= (int64_t)Dout * 4;
}

constexpr int64_t kGroupMaxElems = (int64_t)1024 * G3Group::kPart;   // partial tiles of four rounds of the device

static_assert(kG3GroupMax == kWgradGroupMax, "a stage fills groups that one launch takes");
int64_t dense_wgrad_group_elems(int64_t rows, const int (*dims)[2], int n) {
    if (n < 1 || n > kG3GroupMax) return -1;
    int64_t tiles = 0;
    double alone = 0.0;
    for (int i = 0; i < n; ++i) {
        tiles += g3_group_tiles(dims[i][1], dims[i][0]);
        alone += wgrad_alone_us(dims[i][1], dims[i][0], rows);
    }
    const G3GroupPlan p = g3_group_plan(tiles, rows, kGroupMaxElems);
    if (p.us > 0.95 * alone) return -1;
    return p.slices > 1 ? (tiles - p.whole) * p.slices * G3Group::kPart : 0;
}

hipError_t dense_wgrad_group(int dtype, const DenseWgradJob* jobs, int n, int64_t rows, float* ws, int64_t ws_elems, hipStream_t s) {
    if (n < 1) return hipSuccess;
    if (dtype != kBF16 || n > kG3GroupMax) return hipErrorInvalidValue;
    G3GroupRagged g;
    int tiles = 0;
    bool whole_rows = rows % 64 == 0;
    for (int i = 0; i < n; ++i) {
        const DenseWgradJob& j = jobs[i];
        whole_rows = whole_rows && g3_lane_offsets(false, G3Group::kRows, j.Dout) && g3_lane_offsets(false, G3Group::kCols, j.Din);
        if (!dense_wgrad_groups(dtype, rows, j.Din, j.Dout) || !aligned16(j.dy) || !aligned16(j.x) || !aligned16(j.gw)) return hipErrorInvalidValue;
        const int tm = cdiv(j.Dout, G3Group::kRows), tn = cdiv(j.Din, G3Group::kCols), col_major = j.Din > j.Dout ? 1 : 0;
        g.job[i] = G3Job{(const bf16_t*)j.dy, (const bf16_t*)j.x, j.gw, j.Dout, j.Din, tiles, col_major, FastDiv(col_major ? tm : tn)};
        tiles += tm * tn;
    }
    const G3GroupPlan p = g3_group_plan(tiles, rows, ws && aligned16(ws) ? ws_elems : 0);
    const int cut = tiles - p.whole;
    g.jobs = n; g.k_total = (int)rows; g.tiles = tiles; g.whole = p.whole; g.k_per_slice = p.k_per_slice; g.part = ws;
    g.slices = p.slices; g.chain = p.chain;
    if (p.slices == 1) g.whole = tiles;   // (one slice is the whole of k)
    g.d_cut = FastDiv(cut > 0 ? cut : 1);
    constexpr int lds = gemm3_lds_bytes<G3Group::kRows, G3Group::kCols, 64, kG3GroupStages>(4);
    void (*const kern)(G3Group) = gemm3_kernel;
    void (*const ragged)(G3GroupRagged) = gemm3_kernel;
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    static hipError_t attr_r = hipFuncSetAttribute(reinterpret_cast<const void*>(ragged), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess || attr_r != hipSuccess) return attr != hipSuccess ? attr : attr_r;
    const int units = g.whole + (tiles - g.whole) * g.slices, slots = compute_units();
    const dim3 grid(units < slots ? units : slots);
    hipError_t e = whole_rows ? launch_timed(kcDenseWgrad, kern, grid, dim3(256), lds, s, (const G3Group&)g)
                                  : launch_timed(kcDenseWgrad, ragged, grid, dim3(256), lds, s, g);
    if (e != hipSuccess || p.slices == 1) return e;
    return launch_timed(kcSliceSum, g3_group_sum_kernel, dim3(cut, G3Group::kRows / 32), dim3(256), 0, s, (const G3Group&)g);
}

// ---------------------------------------------------------------------------------------- dense
// The dense contractions with the kernel class they are accounted under as a parameter: a 1x1 convolution with unit
// stride and no padding is the same contraction over its positions.
template <class Epi>
static hipError_t dense_forward_bf16(int kc, const bf16_t* x, const bf16_t* w, const Epi& epi, bool aligned, int B, int Din, int Dout, float* ws,
                                     hipStream_t s) {
    if (aligned && g3_forward_takes(B, Dout, Din) && aligned16(x) && aligned16(w)) {
        G3Operand<true> A{x, B, Din};
        G3Operand<true> Bv{w, Dout, Din};
        return launch3<true, true, false>(kc, A, Bv, epi, B, Dout, Din, g3_plan(B, Dout, Din, 1), s);
    }
    // (from 1024 on, where the persistent kernel was the quicker one when the line was drawn: 8192 x 768 over 512 / 768 / 1024 16.4 / 19.0 / 22.0 us and 15.7 / 19.7 / 22.9.
    // Forward passes alone on the device now, persistent and other kernels (us), over 512 / 768 / 1024 / 2048 / 4096: 8192 x 768 14.2 / 16.1 / 18.2 /
    // 29 / 51 and 17.3 / 20.5 / 23.2 / 40 / 73, 6144 x 768 11.9 / 14.1 / 17.1 / 26 / 45 and 15.0 / 18.4 / 22.2 / 38 / 70, 4096 x 1280
    // 12.9 / 15.8 / 17.5 / 27 / 47 and 15.0 / 19.0 / 22.3 / 39 / 70: 512 and 768 would be quicker there as well)
    if (aligned && Din >= 1024 && g3_narrow_ok(B, Dout, Din) && aligned16(x) && aligned16(w))
        return launch3_inst<256, 128, 2, 2, 3, 1, true, true, false>(kc, G3Operand<true>{x, B, Din}, G3Operand<true>{w, Dout, Din}, epi, B, Dout, Din,
                                                                     g3_plan(B, Dout, Din, 1, 256, 128), s);
    return dense_forward_t<bf16_t>(kc, x, w, epi, B, Din, Dout, ws, s);
}

static hipError_t dense_forward_as(int kc, int dtype, const void* x, const void* w, const float* bias, void* y, int B, int Din,
                                   int Dout, int relu, int out_f32, const void* res, void* zout, float* ws, hipStream_t s) {
    if (dtype != kBF16)
        return dense_forward_f32(kc, (const float*)x, (const float*)w, EpiBiasAct<float>{(float*)y, bias, Dout, relu, (const float*)res, (float*)zout},
                                 B, Din, Dout, ws, s);
    const bool aligned = aligned16(y) && aligned16(bias) && aligned16(res) && aligned16(zout);
    if (out_f32)
        return dense_forward_bf16(kc, (const bf16_t*)x, (const bf16_t*)w, EpiBiasAct<float>{(float*)y, bias, Dout, relu, nullptr, (float*)zout}, aligned, B, Din, Dout, ws, s);
    return dense_forward_bf16(kc, (const bf16_t*)x, (const bf16_t*)w, EpiBiasAct<bf16_t>{(bf16_t*)y, bias, Dout, relu, (const bf16_t*)res, (bf16_t*)zout},
                              aligned, B, Din, Dout, ws, s);
}

hipError_t dense_forward(int dtype, const void* x, const void* w, const float* bias, void* y, int B, int Din,
                         int Dout, int relu, int out_f32, const void* res, void* zout, float* ws, hipStream_t s) {
    return dense_forward_as(tmps::kcDenseFwd, dtype, x, w, bias, y, B, Din, Dout, relu, out_f32, res, zout, ws, s);
}

bool norm_dense_takes(int dtype, int64_t rows, int D, int Dout) {
    return dtype == kBF16 ? norm_dense_takes<bf16_t>(rows, D, Dout) : norm_dense_takes_f32(rows, D, Dout);
}
hipError_t norm_dense_forward(int dtype, const void* x, const float* gamma, const float* beta, void* y, float* stats, float eps, const void* w, const float* bias,
                              void* out, int rows, int D, int Dout, int act, int out_f32, const void* res, void* zout, hipStream_t s) {
    const bool vec = dtype != kBF16 || (aligned16(x) && aligned16(y) && aligned16(gamma) && aligned16(beta));
    if (!vec) {
        const hipError_t e = layernorm_forward(dtype, x, gamma, beta, y, stats, rows, D, eps, s);
        return e != hipSuccess ? e : dense_forward(dtype, y, w, bias, out, rows, D, Dout, act, out_f32, res, zout, nullptr, s);
    }
    if (dtype != kBF16)
        return norm_dense_f32((const float*)x, gamma, beta, (float*)y, stats, (const float*)w,
                              EpiBiasAct<float>{(float*)out, bias, Dout, act, (const float*)res, (float*)zout}, rows, Dout, D, eps, s);
    if (out_f32)
        return norm_dense_small<bf16_t>(kcDenseFwd, (const bf16_t*)x, gamma, beta, (bf16_t*)y, stats, (const bf16_t*)w,
                                        EpiBiasAct<float>{(float*)out, bias, Dout, act, nullptr, (float*)zout}, rows, Dout, D, eps, s);
    return norm_dense_small<bf16_t>(kcDenseFwd, (const bf16_t*)x, gamma, beta, (bf16_t*)y, stats, (const bf16_t*)w,
                                    EpiBiasAct<bf16_t>{(bf16_t*)out, bias, Dout, act, (const bf16_t*)res, (bf16_t*)zout}, rows, Dout, D, eps, s);
}

static hipError_t dense_dgrad_as(int kc, int dtype, const void* dy, const void* w, void* dx, const void* mask, int mask_mode,
                                 const void* add, int B, int Din, int Dout, float* ws, hipStream_t s) {
    // dx[m, n] = sum_k dy[m, k] * w[k, n]:  A = dy (k-contiguous), B(n, k) = w[k*Din + n] (row-contiguous)
    if (dtype == kBF16) {
        EpiMask<bf16_t, bf16_t> epi{(bf16_t*)dx, (const bf16_t*)mask, Din, mask_mode, (const bf16_t*)add};
        const bool fast = (Dout % 8 == 0) && (Din % 8 == 0) && aligned16(dy) && aligned16(w);
        if (fast && g3_forward_ok(B, Din, Dout) && aligned16(dx) && aligned16(mask) && aligned16(add)) {
            G3Operand<true> A{(const bf16_t*)dy, B, Dout};
            G3Operand<false> Bv{(const bf16_t*)w, Din, Din};
            return launch3<true, false, false>(kc, A, Bv, epi, B, Din, Dout, g3_plan(B, Din, Dout, 1), s);
        }
        const int s3 = (fast && ws && aligned16(ws) && aligned16(dx) && aligned16(mask) && aligned16(add) && epi.wide_ok())
                           ? g3_long_k_slices(B, Din, Dout) : 0;
        if (s3 > 1) {
            G3Operand<true> A{(const bf16_t*)dy, B, Dout};
            G3Operand<false> Bv{(const bf16_t*)w, Din, Din};
            const G3Plan plan = g3_plan(B, Din, Dout, s3);
            const EpiForm<EpiPartial, 0> part{EpiPartial{ws, Din, (int64_t)B * Din}};   // (fewer than 192 tiles: rows are far shorter than kFormMaxLd)
            hipError_t e = launch3<true, false, false>(kc, A, Bv, part, B, Din, Dout, plan, s);
            if (e != hipSuccess) return e;
            return launch_timed(kcSplitFinish, splitk_finish8_kernel<EpiMask<bf16_t, bf16_t>, SameRows>, dim3(cdiv((int64_t)B * Din / 8, 256)),
                                dim3(256), 0, s, (const float*)ws, epi, B, Din, plan.slices, SameRows{});
        }
        if (fast && g3_narrow_ok(B, Din, Dout) && aligned16(dx) && aligned16(mask) && aligned16(add)) {
            G3Operand<true> A{(const bf16_t*)dy, B, Dout};
            G3Operand<false> Bv{(const bf16_t*)w, Din, Din};
            return launch3_inst<256, 128, 2, 2, 3, 1, true, false, false>(kc, A, Bv, epi, B, Din, Dout, g3_plan(B, Din, Dout, 1, 256, 128), s);
        }
        return dense_dgrad_t<bf16_t>(kc, (const bf16_t*)dy, (const bf16_t*)w, epi, B, Din, Dout, ws, s);
    }
    return dense_dgrad_f32(kc, (const float*)dy, (const float*)w,
                           EpiMask<float, float>{(float*)dx, (const float*)mask, Din, mask_mode, (const float*)add}, B, Din, Dout, ws, s);
}

hipError_t dense_dgrad(int dtype, const void* dy, const void* w, void* dx, const void* mask, int mask_mode,
                       const void* add, int B, int Din, int Dout, float* ws, hipStream_t s) {
    return dense_dgrad_as(tmps::kcDenseDgrad, dtype, dy, w, dx, mask, mask_mode, add, B, Din, Dout, ws, s);
}

static hipError_t dense_wgrad_as(int kc, int dtype, const void* dy, const void* x, float* gw, int B, int Din, int Dout,
                                 const Partials& ws, hipStream_t s) {
    // gw[m, n] = sum_k dy[k, m] * x[k, n]: both operands row-contiguous, contraction over the batch
    if (dtype == kBF16) {
        const bool fast = (Dout % 8 == 0) && (Din % 8 == 0) && aligned16(dy) && aligned16(x);
        const int s3 = fast && aligned16(gw) ? g3_wgrad_slices(Dout, Din, B) : 0;
        if (s3 >= 1 && (s3 == 1 || (ws.ws && aligned16(ws.ws)))) {
            G3Operand<false> A{(const bf16_t*)dy, Dout, Dout};
            G3Operand<false> Bv{(const bf16_t*)x, Din, Din};
            const G3Plan plan = g3_plan(Dout, Din, B, s3);
            const int64_t count = (int64_t)Dout * Din + Dout;
            EpiWgrad epi{plan.slices > 1 ? ws.ws : gw, Din, (int64_t)Dout * Din, count};
            hipError_t e = launch3<false, false, true>(kc, A, Bv, epi, Dout, Din, B, plan, s);
            if (e != hipSuccess || plan.slices <= 1) return e;
            return ws.finish(Reduction{ws.ws, gw, count, plan.slices, false}, s);
        }
        return dense_wgrad_t<bf16_t>(kc, (const bf16_t*)dy, (const bf16_t*)x, gw, B, Din, Dout, ws, s);
    }
    return dense_wgrad_f32(kc, (const float*)dy, (const float*)x, gw, B, Din, Dout, ws, s);
}

hipError_t dense_wgrad(int dtype, const void* dy, const void* x, float* gw, int B, int Din, int Dout, const Partials& ws,
                       hipStream_t s) {
    return dense_wgrad_as(tmps::kcDenseWgrad, dtype, dy, x, gw, B, Din, Dout, ws, s);
}

// ---- both gradients of a dense layer in one launch: estimates in us ----
// Small kernel, four waves to a tile: half a microsecond for every tile of a compute unit's share, and the longer of its share of the multiplies
// and the longest tile alone, per k of a 16 x 16 or a 32 x 32 tile.  Fitted on 32 to 1024 rows, widths of 10 to 1000 (one launch, two; us):
// fp32 32 x 64 -> 128 2.5 and 4.4, 235 x 1000 -> 10 3.5 and 6.2, 64 x 1000 -> 1000 8.3 and 10.6, 512 x 768 -> 768 21.1 and 32.3,
// 235 x 1000 -> 1000 20.2 and 19.5; bf16 32 x 64 -> 128 2.3 and 4.3, 512 x 512 -> 512 5.7 and 8.0, 256 x 768 -> 768 7.3 and 9.5, 235 x 1000 -> 1000 11.8 and 11.4.
int small_backward_tile(int64_t M, int64_t N, int esize) { return (int64_t)cdiv(M, 16) * cdiv(N, 16) <= (esize == 4 ? 2 : 1) * kCUs ? 1 : 2; }
double small_backward_us(int64_t B, int64_t Din, int64_t Dout, int esize) {
    const int tx = small_backward_tile(B, Din, esize), tw = small_backward_tile(Dout, Din, esize);
    const double nx = (double)cdiv(B, 16 * tx) * cdiv(Din, 16 * tx), nw = (double)cdiv(Dout, 16 * tw) * cdiv(Din, 16 * tw);
    auto shared = [&](int t) { return esize == 4 ? (t == 1 ? 0.0027 : 0.0085) : (t == 1 ? 0.0011 : 0.0035); };
    auto alone = [&](int t) { return esize == 4 ? (t == 1 ? 0.0030 : 0.0080) : (t == 1 ? 0.0017 : 0.0037); };
    const double share = (nx * Dout * shared(tx) + nw * B * shared(tw)) / kCUs, cx = Dout * alone(tx), cw = B * alone(tw), chain = cx > cw ? cx : cw;
    return 2.05 + 0.5 * (nx + nw) / kCUs + (share > chain ? share : chain);
}
// Tiled kernel in bf16, 64 x 64 tiles: a k-tile takes 0.33 us, alone on its unit or sharing it, and the weight gradient is written at 6 TB/s
// (one launch and two): 64 x 1024 -> 1024 9.6 and 10.6, 256 x 1024 -> 1024 9.6 and 10.7, 512 x 1024 -> 1024 10.3 and 15.6, 1024 x 768 -> 768 11.8
// and 17.1, 256 x 2048 -> 2048 17.0 and 21.9, 256 x 1024 -> 2048 15.3 and 14.7, 512 x 2048 -> 2048 25.4 and 24.7.
double tiled_backward_us(int64_t B, int64_t Din, int64_t Dout) {
    const int64_t n = cdiv(Din, 64), tx = n * cdiv(B, 64), tw = n * cdiv(Dout, 64), kx = cdiv(Dout, 64), kw = cdiv(B, 64);
    const double share = (double)(tx * kx + tw * kw) / kCUs, chain = (double)(kx > kw ? kx : kw);
    return 3.7 + 0.335 * (share > chain ? share : chain) + (double)Din * Dout * 4.0 / 6e6;
}
// Two launches with 2 us between and around them; 0 where one of them is the persistent kernel's.
double two_backward_us(int64_t B, int64_t Din, int64_t Dout, int esize) {
    if (esize == 2 && (g3_forward_ok(B, Din, Dout) || g3_narrow_ok(B, Din, Dout) || g3_long_k_slices(B, Din, Dout) || g3_wgrad_slices(Dout, Din, B))) return 0.0;
    auto alone = [&](int64_t M, int64_t N, int64_t K, bool rowsum) {
        const Plan2 p = plan_for(M, N, K, rowsum, esize, kByKDense);
        return (small_is_better(M, N, K, esize, p) ? small_plan(M, N, K, esize).cost : p.cost) / 2400.0;
    };
    return alone(B, Din, Dout, false) + 2.0 + alone(Dout, Din, B, true) + (double)Din * Dout * 4.0 / 6e6;
}

// What the gradients of a dense layer run on: kTwo launches, or one of the small or of the tiled kernel.  The tiled kernel's takes up to 1024 rows and the
// small one's up to 5120 in bf16, for which the estimates hold.  Beyond, its weight gradients are sums over all rows in one workgroup, where the launches they
// replace have slices: in one launch and in two (kernels alone, us) 4096 x 1024 -> 512 34.4 and 25.3, 1920 x 1920 -> 384 23.2 and 20.8, 2326 x 560 -> 856 22.8 and 26.9, with
// errors of 2.7e-7, 1.9e-7 and 2.0e-7 (2-norm, against 64 bits) instead of 1.3e-7, 0.9e-7 and 1.0e-7; 8115 x 24 -> 1960, small, 40.3 and 23.6, 6328 x 64 -> 800 24.2 and 20.1.
int backward_kind(int64_t B, int64_t Din, int64_t Dout, int esize) {
    const double two = two_backward_us(B, Din, Dout, esize), small = esize == 4 || B <= 5120 ? small_backward_us(B, Din, Dout, esize) : 1e9;
    const double tiled = esize == 2 && Din % 8 == 0 && Dout % 8 == 0 && B <= 1024 ? tiled_backward_us(B, Din, Dout) / 0.95 : 1e9;
    if (small >= two && tiled >= two) return kTwo;
    return small <= tiled ? kOneSmall : kOneTiled;
}

// fp32: whether the two launches of both gradients run as one on two kernels' tiles (gemm_mixed_backward_kernel): the small kernel's 32 x 32 and the tiled
// kernel's 64 x 64, unsliced, so the results are the same bits.  Forward and backward pass and update of one layer, two launches and one (us): 235 x 1000 -> 1000
// 39.1 and 32.2, 256 x 1024 -> 1024 39.7 and 32.6.  Where the small kernel takes both this is sometimes quicker too (235 x 784 -> 1000 33.7 and 30.5, but 512 x 768 -> 768
// 44.1 and 46.7), with longer chains in the sums of the weight gradient: 2.0e-7 (2-norm) from those in 64 bits instead of 1.0e-7.
bool mixed_backward_takes(int64_t B, int64_t Din, int64_t Dout) {
    if (Din % 4 != 0 || Dout % 4 != 0 || backward_kind(B, Din, Dout, 4) != kTwo) return false;
    const Plan2 pw = plan_for(Dout, Din, B, true, 4, kByKDense);
    return small_is_better(B, Din, Dout, 4, plan_for(B, Din, Dout, false, 4, kByKDense)) && small_plan(B, Din, Dout, 4).tm == 2 &&
           !small_is_better(Dout, Din, B, 4, pw) && pw.kind == kTiled && pw.bm == 64 && pw.bn == 64 && pw.slices == 1;
}

hipError_t dense_backward(int dtype, const void* dy, const void* x, const void* w, float* gw, void* dx, const void* mask, int mask_mode,
                          const void* add, int B, int Din, int Dout, float* ws, const Partials& ws_w, hipStream_t s) {
    const int kind = backward_kind(B, Din, Dout, dtype == kBF16 ? 2 : 4);
    const EpiMask<bf16_t, bf16_t> ex{(bf16_t*)dx, (const bf16_t*)mask, Din, mask_mode, (const bf16_t*)add};
    if (dtype != kBF16 && kind == kTwo && mixed_backward_takes(B, Din, Dout) && aligned16(dy) && aligned16(x))
        return mixed_backward_f32(kcDenseBackward, (const float*)dy, (const float*)x, (const float*)w, gw,
                                  EpiMask<float, float>{(float*)dx, (const float*)mask, Din, mask_mode, (const float*)add}, B, Din, Dout, s);
    if (kind == kOneSmall) {
        if (dtype != kBF16)
            return small_backward_f32(kcDenseBackward, (const float*)dy, (const float*)x, (const float*)w, gw,
                                      EpiMask<float, float>{(float*)dx, (const float*)mask, Din, mask_mode, (const float*)add}, B, Din, Dout, s);
        return small_backward_t<bf16_t>(kcDenseBackward, (const bf16_t*)dy, (const bf16_t*)x, (const bf16_t*)w, gw, ex, B, Din, Dout, s);
    }
    if (kind == kOneTiled && aligned16(dy) && aligned16(x) && aligned16(w)) {
        typedef bf16_t T;
        const EpiWgrad ew{gw, Din, (int64_t)Dout * Din, 0};
        constexpr int lds_x = gemm2_lds_bytes<64, 64, DenseKC<T>, DenseRC<T>>(), lds_w = gemm2_lds_bytes<64, 64, DenseRC<T>, DenseRC<T>>();
        const int n = cdiv(Din, 64), split = n * cdiv(B, 64), tw = n * cdiv(Dout, 64);
        return launch_timed(kcDenseBackward, gemm2_backward_kernel<4, T>, dim3(split + tw), dim3(256), lds_x > lds_w ? lds_x : lds_w, s, (const T*)dy, (const T*)x,
                            (const T*)w, ex, ew, B, Din, Dout, split, FastDiv(n), FastDiv(split), FastDiv(tw), ex.wide_ok() && ew.wide_ok() ? 1 : 0);
    }
    const hipError_t e = dense_wgrad(dtype, dy, x, gw, B, Din, Dout, ws_w, s);
    return e != hipSuccess ? e : dense_dgrad(dtype, dy, w, dx, mask, mask_mode, add, B, Din, Dout, ws, s);
}

// ---------------------------------------------------------------------------------- convolution
hipError_t conv_forward(int dtype, const void* x, const void* w, const float* bias, void* y, const ConvShape& c,
                        int relu, float* ws, hipStream_t s) {
    if (dtype != kBF16)
        return conv_forward_f32((const float*)x, (const float*)w, EpiBiasAct<float>{(float*)y, bias, c.Cout, relu ? kActRelu : kActNone}, c, ws, s);
    if (pointwise(c))
        return dense_forward_as(kcConvFwd, dtype, x, w, bias, y, c.B * c.Ho * c.Wo, c.Cin, c.Cout, relu ? kActRelu : kActNone, 0, nullptr,
                                nullptr, ws, s);
    return conv_forward_t<bf16_t>((const bf16_t*)x, (const bf16_t*)w, EpiBiasAct<bf16_t>{(bf16_t*)y, bias, c.Cout, relu}, c, ws, s);
}

hipError_t conv_affine_forward(int dtype, const void* x, const void* w, const float* bias, void* z, const float* gain,
                               const float* shift, void* again, const void* res, void* yout, int relu, const ConvShape& c,
                               float* ws, hipStream_t s) {
    if (dtype != kBF16)
        return conv_affine_f32((const float*)x, (const float*)w,
                               EpiConvAffine<float>{(float*)z, bias, c.Cout, gain, shift, (float*)again, (const float*)res, (float*)yout, relu}, c, ws, s);
    const int M = c.B * c.Ho * c.Wo, K = c.R * c.S * c.Cin;
    const bf16_t *xb = (const bf16_t*)x, *wb = (const bf16_t*)w;
    const EpiConvAffine<bf16_t> epi{(bf16_t*)z, bias, c.Cout, gain, shift, (bf16_t*)again, (const bf16_t*)res, (bf16_t*)yout, relu};
    if (pointwise(c) && pointwise_forward_takes(M, c.Cin, c.Cout, false) && aligned16(x) && aligned16(w) && epi.wide_ok())
        return pointwise_forward(PointwiseForward{x, w, res, bias, gain, shift, z, yout, again, relu}, nullptr, M, c.Cin, c.Cout, s);
    if (pointwise(c) && c.Cin % 8 == 0 && aligned16(x) && aligned16(w)) {
        if (g3_forward_takes(M, c.Cout, K) && aligned16(z) && aligned16(bias) && aligned16(gain) && aligned16(shift) &&
            aligned16(again) && aligned16(res) && aligned16(yout))
            return launch3<true, true, false>(kcConvFwd, G3Operand<true>{xb, M, K}, G3Operand<true>{wb, c.Cout, K}, epi, M, c.Cout, K,
                                              g3_plan(M, c.Cout, K, 1), s);
        return run2(kcConvFwd, DenseKC<bf16_t>{xb, M, K, K}, DenseKC<bf16_t>{wb, c.Cout, K, K}, epi, M, c.Cout, K, ws, s);
    }
    return conv_forward_t<bf16_t>(xb, wb, epi, c, ws, s);
}

hipError_t conv_dgrad(int dtype, const void* dy, const void* w, void* dx, const void* mask, const void* add,
                      const ConvShape& c, float* ws, hipStream_t s) {
    if (dtype != kBF16)
        return conv_dgrad_f32((const float*)dy, (const float*)w, EpiMask<float, float>{(float*)dx, (const float*)mask, c.Cin, kActRelu, (const float*)add},
                              c, ws, s);
    if (pointwise(c)) return dense_dgrad_as(kcConvDgrad, dtype, dy, w, dx, mask, kActRelu, add, c.B * c.H * c.W, c.Cin, c.Cout, ws, s);
    return conv_dgrad_t<bf16_t>((const bf16_t*)dy, (const bf16_t*)w,
                                EpiMask<bf16_t, bf16_t>{(bf16_t*)dx, (const bf16_t*)mask, c.Cin, kActRelu, (const bf16_t*)add}, c, ws, s);
}

size_t conv_wgrad_workspace_elems(int dtype, const ConvShape& c) {
    const int64_t cols = (int64_t)c.R * c.S * c.Cin, K = (int64_t)c.B * c.Ho * c.Wo;
    const size_t n = gemm_workspace_elems(c.Cout, cols, K, kWsRowSums | (dtype == kBF16 ? 0 : kWsF32));
    if (dtype != kBF16) return n;
    const int slices = conv_first_kind(c, true) ? conv_first_wgrad_slices(c) : conv_wgrad_rows_plan(c, plan_for(c.Cout, (int)cols, K, true, 2, kByKConv)).slices;
    return slices > 1 ? std::max(n, (size_t)slices * (size_t)(c.Cout * cols + c.Cout)) : n;
}

hipError_t conv_wgrad(int dtype, const void* dy, const void* x, float* gw, const ConvShape& c, const Partials& ws, hipStream_t s) {
    if (dtype != kBF16) return conv_wgrad_f32((const float*)dy, (const float*)x, gw, c, ws, s);
    if (pointwise(c)) return dense_wgrad_as(kcConvWgrad, dtype, dy, x, gw, c.B * c.Ho * c.Wo, c.Cin, c.Cout, ws, s);
    return conv_wgrad_t<bf16_t>((const bf16_t*)dy, (const bf16_t*)x, gw, c, ws, s);
}

}  // namespace tmps

extern "C" int tmps_dense_gradients_joint(int dtype, int64_t rows, int din, int dout) {
    using namespace tmps;
    return rows > 0 && din > 0 && dout > 0 && !dense_wgrad_groups(dtype, rows, din, dout) &&
           (backward_kind(rows, din, dout, dtype == kBF16 ? 2 : 4) != kTwo || (dtype != kBF16 && mixed_backward_takes(rows, din, dout)));
}
