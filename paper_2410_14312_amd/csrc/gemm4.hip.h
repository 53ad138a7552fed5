// MFMA GEMM for gfx950 whose waves share a tile by k: C[m, n] = sum_k A(m, k) * B(n, k), bf16 or fp32 in, fp32 accumulate.
//
// A workgroup owns a 64 x 64 tile of C and a range of k; each of its four waves multiplies the WHOLE tile over a quarter of
// the range, from LDS stages of its own that it fills with asynchronous copies (global_load_lds), so the k-loop has no
// barrier and a wave waits for nothing but its own copies; the four partial tiles are added through LDS at the end, in
// the order of the waves, and the epilogue follows in the same launch.
// For outputs of few tiles.  There the tiled kernel (gemm2.hip.h) either walks all of k in one workgroup per compute unit,
// spending a k-tile (0.3 us) on LDS writes, the barrier, LDS reads and multiplies one after the other, or cuts k into
// slices and pays for a second launch and the partial sums' way through memory.  Here the waves are at different steps, a
// k-tile is read from LDS once instead of twice (a wave multiplies 64 x 64 instead of 32 x 32) and no register holds data
// on its way to LDS: 1024 x 768 x 3072 15.4 -> 12.2 us (some 80 bytes/ns into a compute unit: that bounds it), a split launch
// with its finishing kernel some 4 to 6 us less.  One workgroup per compute unit (128 KB of LDS), so the tiled kernel stays
// the better one where there are tiles for several rounds.
#pragma once
#include "gemm3.hip.h"

namespace tmps {

// LDS layout of a wave's 64-row operand tile, 8 KB in eight 1-KB copy groups; group g, lane l:
//   k-contiguous   [64 rows][8 chunks]: row 8 g + l / 8, position l % 8 holds chunk (l % 8) ^ (row % 8)
//   row-contiguous bf16 [64 k][8 chunks of 8 rows]: k = 8 g + l / 8, position l % 8 holds chunk (l % 8) ^ 4 ((k / 2) % 2)
//                  fp32 [32 k][16 chunks of 4 rows]: k = 4 g + l / 16, position l % 16 holds chunk (l % 16) ^ 8 (g % 2)
template <class Op> struct WaveTile {
    typedef typename Op::T T;
    static constexpr int V = ElemTile<T>::V;
    static constexpr bool KC = Op::kContig;
    typename Op::KS ks;
    typename Op::Ctx c[8];
    __device__ __forceinline__ void init(const Op& op, int row0, int k_begin, int lane) {
        op.init_thread(ks, k_begin, (lane & 7) ^ (lane >> 3));
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            if constexpr (KC) op.init(c[g], row0 + g * 8 + (lane >> 3), 0, k_begin);
            else if constexpr (sizeof(T) == 2) op.init(c[g], row0 + ((lane & 7) ^ (((lane >> 4) & 1) << 2)) * V, g * 8 + (lane >> 3), k_begin);
            else op.init(c[g], row0 + ((lane & 15) ^ ((g & 1) << 3)) * V, g * 4 + (lane >> 4), k_begin);
        }
    }
    __device__ __forceinline__ void issue(const Op& op, int g, lds_t tile, int k_end) { copy16_to_lds(op.addr(c[g], ks, k_end), tile + g * 1024); }
    // fragment f (of 4) of rows 32 i .. 32 i + 31
    static __device__ __forceinline__ typename Frag<T>::type read(lds_t tile, int i, int f, int lane) {
        typedef typename Frag<T>::type frag_t;
        const int half = lane >> 5;
        if constexpr (KC) {
            const int row = 32 * i + (lane & 31);
            return *lds_ptr<const frag_t>(tile + row * 128 + (((2 * f + half) ^ (lane & 7)) << 4));
        } else if constexpr (sizeof(T) == 2) {
            const int k = f * 16 + half * 8 + ((lane & 15) >> 2);
            const int row = 32 * i + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
            const int sw = ((k >> 1) & 1) << 2;   // (k + 4 has the same)
            const lds_t p = tile + k * 128 + ((((row >> 3) ^ sw) << 4) | ((row & 7) * 2));
            union { s16x4_t h[2]; bf16x8_t v; } u;
            u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(p));
            u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(p + 4 * 128));
            return u.v;
        } else {
            // k = 8 f + 4 half + e lies in group 2 f + half
            const int row = 32 * i + (lane & 31);
            const lds_t p = tile + (2 * f + half) * 1024 + ((((row >> 2) ^ (half << 3)) << 4) | ((row & 3) * 4));
            frag_t v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = *lds_ptr<const float>(p + e * 256);
            return v;
        }
    }
};

constexpr int kGemm4Stages = 2, kGemm4Lds = 4 * kGemm4Stages * 16384;

template <bool ROWSUM, class AOp, class BOp, class Epi>
__global__ __launch_bounds__(256, 1) void gemm4_kernel(AOp A, BOp B, Epi epi, int M, int N, int K, int k_per_slice, int order, int wide,
                                                        FastDiv d_plane, FastDiv d_minor) {
    typedef typename AOp::T T;
    typedef typename Frag<T>::type frag_t;
    constexpr int BK = ElemTile<T>::BK, NS = kGemm4Stages;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int tile_x = blockIdx.x, tile_y = blockIdx.y, z = blockIdx.z;
    xcd_tile(order, d_plane, d_minor, gridDim.x, gridDim.y, gridDim.z, tile_x, tile_y, z);
    const int m0 = tile_y * 64, n0 = tile_x * 64;
    op_begin_tile(A, m0, 0);
    op_begin_tile(B, m0, 0);
    const int z_begin = z * k_per_slice, z_end = min(op_k_total(A, K, 0), z_begin + k_per_slice);
    const int tiles = max(0, (z_end - z_begin + BK - 1) / BK), per_wave = (tiles + 3) >> 2;
    const int k_begin = z_begin + wave * per_wave * BK, k_end = min(z_end, k_begin + per_wave * BK);
    const int nk = max(0, (k_end - k_begin + BK - 1) / BK);

    WaveTile<AOp> wa;
    WaveTile<BOp> wb;
    wa.init(A, m0, k_begin, lane);
    wb.init(B, n0, k_begin, lane);
    const lds_t mine = smem + wave * (NS * 16384);
    auto issue = [&](int stage, int g) {   // copy group g of 16 of the next k-tile
        const lds_t st = mine + stage * 16384;
        if (g < 8) wa.issue(A, g, st, k_end);
        else wb.issue(B, g - 8, st + 8192, k_end);
    };
    auto step = [&]() {
        A.next(wa.ks);
        B.next(wb.ks);
    };
    f32x16_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    float rs[2] = {0.0f, 0.0f};
    const bool sum_rows = ROWSUM && tile_x == 0;
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nk) {
#pragma unroll
            for (int g = 0; g < 16; ++g) issue(s, g);
            step();
        }
    int stage = 0;
    for (int t = 0; t < nk; ++t) {
        // this k-tile is the oldest copy in flight
        if (t + 1 < nk) wait_vmcnt<(NS - 1) * 16>();
        else wait_vmcnt<0>();
        const lds_t st = mine + stage * 16384;
        frag_t af[4][2], bfr[4][2];
#pragma unroll
        for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                af[f][i] = WaveTile<AOp>::read(st, i, f, lane);
                bfr[f][i] = WaveTile<BOp>::read(st + 8192, i, f, lane);
            }
        // the stage is refilled once its fragments are in registers, the copies spread over the multiplies
        const bool fill = t + NS < nk;
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        asm volatile("" ::: "memory");
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            if (fill) {
#pragma unroll
                for (int g = 4 * f; g < 4 * f + 4; ++g) issue(stage, g);
            }
            if constexpr (sizeof(T) == 2) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[f][i], bfr[f][j], acc[i][j], 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[f][i][e], bfr[f][j][e], acc[i][j], 0, 0, 0);
            }
            if (ROWSUM && sum_rows) {
#pragma unroll
                for (int i = 0; i < 2; ++i) rs[i] = add_frag(rs[i], af[f][i]);
            }
        }
        if (fill) step();
        stage ^= 1;
    }

    // ---- the four partial tiles are added through LDS ----
    __syncthreads();   // every wave is past its last read: the stages may be overwritten
    float* const part = reinterpret_cast<float*>(smem_raw);   // [4][64][64]
    const int half = lane >> 5;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                part[(wave * 64 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * 64 + j * 32 + (lane & 31)] = acc[i][j][r];
    float* const sums = part + 4 * 4096;   // [4][64]
    if (ROWSUM && sum_rows) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float both = rs[i] + __shfl_xor(rs[i], 32, 64);
            if (lane < 32) sums[wave * 64 + i * 32 + lane] = both;
        }
    }
    const int64_t ld = epi.ld;
    if (wide) {
        // 8 consecutive columns of a row per lane, what the epilogue reads requested before the barrier
        const int n = n0 + (tid & 7) * 8;
        const typename Epi::Col8 pcol = epi.col8(n < N ? n : 0);
        typename Epi::Row8 prow[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int m = m0 + p * 32 + (tid >> 3);
            prow[p] = epi.row8((int64_t)op_out_row(A, m < M ? m : 0, 0) * ld + n, m < M && n < N);
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int row = p * 32 + (tid >> 3);
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float* q = part + (w * 64 + row) * 64 + (tid & 7) * 8;
                const float4 lo = *reinterpret_cast<const float4*>(q), hi = *reinterpret_cast<const float4*>(q + 4);
                v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
                v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
            }
            const int m = m0 + row;
            if (m < M && n < N) epi.at8(pcol, prow[p], (int64_t)op_out_row(A, m, 0) * ld + n, v, z);
        }
    } else {
        __syncthreads();
        const int n = n0 + (tid & 63);
        if (n < N) {
            const auto col = epi.column(n);
#pragma unroll 4
            for (int row = tid >> 6; row < 64; row += 4) {
                const int m = m0 + row;
                const float* q = part + row * 64 + (tid & 63);
                if (m < M) epi.at(col, (int64_t)op_out_row(A, m, 0) * ld + n, (q[0] + q[4096]) + (q[8192] + q[12288]), z);
            }
        }
    }
    if (ROWSUM && sum_rows && tid < 64 && m0 + tid < M)
        epi.rowsum(m0 + tid, (sums[tid] + sums[64 + tid]) + (sums[128 + tid] + sums[192 + tid]), z);
}

}  // namespace tmps
