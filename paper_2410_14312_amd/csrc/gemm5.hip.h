// MFMA GEMM for gfx950 of 128 x 128 tiles with asynchronous copies: C[m, n] = sum_k A(m, k) * B(n, k), bf16 in, fp32 accumulate,
// operands described by the loaders of gemm2.hip.h.
//
// Eight waves in two groups of four (2 x 2, 64 x 64 each); a k-tile is every wave's, each group multiplies half of it, and the groups'
// partial tiles are added through LDS at the end.  k-tiles go from memory to LDS without passing through registers
// (global_load_lds) into five stages: the fragments of the next k-tile are read while one is multiplied, one LDS read after each
// MFMA, and the copies of the k-tile five ahead go into the stage that this freed, so that a copy has four k-tiles' time to arrive.
// One workgroup to a unit (160 KB of LDS), for outputs of some 100 to 256 tiles, where the tiled kernel's smaller tiles read each operand more often.
// What bounds it: 32 KB copied for 0.28 us of multiplies; and of 15 us some 6 are the launch, the first copies and the epilogue.  With two stages of
// two k-tiles, which left a copy issued last no time at all, 1024 x 3072 x 768 forward took 16.8 us in a transformer's stage (15.6 now), 1024 x 2304 x 768
// 13.4 (11.9), the input gradient of 12544 x 256 x 256 17.6 (15.3).  Against the tiled kernel, before that: 1024 x 3072 x 768 forward 13.9 -> 11.9 us, input
// gradient 13.7 -> 11.0 us, weight gradient 17.6 -> 14.0 us; 4096 x 768 -> 3072 weight gradient 52 -> 39 us; a stride-2 3 x 3 convolution of 64
// images of 28 x 28 x 256 35 -> 26 us.
// By the device clock 1024 x 3072 x 768 forward is 1.0 us of indices, 0.8 until the first k-tile, 6.2 of 12 steps and 2.0 of results; dense epilogues in their
// forms (see EpiForm; here and in the kernel whose waves share k): GPT-2's second stage 2738 -> 2719 us, 1F1B 20026 -> 19915.
#pragma once
#include "gemm4.hip.h"

namespace tmps {

// A wave's share of the copies of a 128-row operand tile, and its reads.  LDS: two subtiles of 64 rows, 8 KB in eight 1-KB groups each:
//   k-contiguous   [64 rows][8 chunks]: position p of row r holds chunk p ^ ((r / 2) % 8): sixteen consecutive rows read at one
//                  chunk lie in different banks
//   row-contiguous as in gemm4.hip.h
template <class Op> struct Tile128 {
    static constexpr bool KC = Op::kContig;
    typename Op::KS ks;
    typename Op::Ctx c[2];
    // (wave w of eight copies groups w and w + 8 of 16, both even or both odd)
    __device__ __forceinline__ void init(const Op& op, int row0, int k_begin, int w, int lane) {
        op.init_thread(ks, k_begin, (lane & 7) ^ (lane >> 4) ^ ((w & 1) << 2));
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int g = w + 8 * i;
            if constexpr (KC) op.init(c[i], row0 + g * 8 + (lane >> 3), 0, k_begin);
            else op.init(c[i], row0 + (g >> 3) * 64 + ((lane & 7) ^ (((lane >> 4) & 1) << 2)) * 8, (g & 7) * 8 + (lane >> 3), k_begin);
        }
    }
    __device__ __forceinline__ void copy(const Op& op, int i, lds_t tile, int w, int k_end) {
        copy16_to_lds(op.addr(c[i], ks, k_end), tile + (w + 8 * i) * 1024);
    }
    // fragment f (of 4) of rows 32 i .. 32 i + 31 of a subtile
    static __device__ __forceinline__ bf16x8_t read(lds_t tile, int i, int f, int lane) {
        if constexpr (KC)
            return *lds_ptr<const bf16x8_t>(tile + (32 * i + (lane & 31)) * 128 + (((2 * f + (lane >> 5)) ^ ((lane >> 1) & 7)) << 4));
        else return WaveTile<Op>::read(tile, i, f, lane);
    }
};

constexpr int kGemm5Waves = 8, kGemm5Stages = 5, kGemm5Lds = kGemm5Stages * 32768;
static_assert(kGemm5Lds >= kGemm5Waves * 64 * 64 * 4, "the partial tiles are added in the stages' place");

template <bool ROWSUM, class AOp, class BOp, class Epi>
__global__ __launch_bounds__(64 * kGemm5Waves, 2) void gemm5_kernel(AOp A, BOp B, Epi epi, int M, int N, int K, int k_per_slice, int order,
                                                           FastDiv d_plane, FastDiv d_minor) {
    constexpr int NW = kGemm5Waves, NS = kGemm5Stages, KG = NW / 4, STAGE = 32768, NF = 4 / KG;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave >> 2, w = wave & 3, wm = w >> 1, wn = w & 1;

    int tile_x = blockIdx.x, tile_y = blockIdx.y, z = blockIdx.z;
    xcd_tile(order, d_plane, d_minor, gridDim.x, gridDim.y, gridDim.z, tile_x, tile_y, z);
    const int m0 = tile_y * 128, n0 = tile_x * 128;
    op_begin_tile(A, m0, 0);
    op_begin_tile(B, m0, 0);
    const int k_begin = z * k_per_slice, k_end = min(op_k_total(A, K, 0), k_begin + k_per_slice);
    const int steps = max(0, (k_end - k_begin + 63) >> 6);

    Tile128<AOp> ta;
    Tile128<BOp> tb;
    ta.init(A, m0, k_begin, wave, lane);
    tb.init(B, n0, k_begin, wave, lane);
    auto copy = [&](int stage, int i) {   // the wave's copy i of 4 of the next k-tile (beyond the range: zeros)
        const lds_t st = smem + stage * STAGE;
        if (i < 2) ta.copy(A, i, st, wave, k_end);
        else tb.copy(B, i - 2, st + 16384, wave, k_end);
    };
    auto next_tile = [&]() {
        A.next(ta.ks);
        B.next(tb.ks);
    };
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) copy(s, i);
        next_tile();
    }
    f32x16_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    float rs[2] = {0.0f, 0.0f};
    const bool sum_rows = ROWSUM && tile_x == 0;

    struct Frags { bf16x8_t a[NF][2], b[NF][2]; };   // the group's half of a k-tile: 16 k, 16 of the other's
    auto read_a = [&](Frags& q, int stage, int f, int i) { q.a[f][i] = Tile128<AOp>::read(smem + stage * STAGE + wm * 8192, i, f * KG + kg, lane); };
    auto read_b = [&](Frags& q, int stage, int f, int i) { q.b[f][i] = Tile128<BOp>::read(smem + stage * STAGE + 16384 + wn * 8192, i, f * KG + kg, lane); };
    // One barrier per step, before the reads of the next step's fragments: behind it that step's k-tile is there (everyone has
    // waited for its copies; those of the NS - 2 k-tiles after it stay under way) and the stage of the step being multiplied is
    // free (everyone has its fragments in registers).
    int stage = 0;   // of the step being multiplied: refilled meanwhile
    auto one_step = [&](const Frags& cur, Frags& next) {
        const int ahead = stage + 1 == NS ? 0 : stage + 1;
        wait_vmcnt<(NS - 2) * 4>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[f][i], cur.b[f][j], acc[i][j], 0, 0, 0);
                    if (i == j) read_a(next, ahead, f, i);
                    else read_b(next, ahead, f, j);
                    __builtin_amdgcn_sched_barrier(0);
                    if (j == 1) copy(stage, 2 * f + i);
                }
            if (ROWSUM && sum_rows && (f & 1) == wn) {   // (both waves of a row pair hold its fragments: they take turns)
#pragma unroll
                for (int i = 0; i < 2; ++i) rs[i] = add_frag(rs[i], cur.a[f][i]);
            }
        }
        next_tile();
        stage = ahead;
    };
    Frags f0, f1;
    wait_vmcnt<(NS - 1) * 4>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            read_a(f0, 0, f, i);
            read_b(f0, 0, f, i);
        }
    for (int step = 0; step < steps; step += 2) {
        one_step(f0, f1);
        if (step + 1 < steps) one_step(f1, f0);
    }
    wait_vmcnt<0>();   // (the copies past the end)

    // ---- the groups' partial tiles are added through LDS, 8 consecutive columns of a row per lane ----
    const int64_t ld = epi.ld;
    const int n = n0 + (tid & 15) * 8;
    const typename Epi::Col8 pcol = epi.col8(n < N ? n : 0);
    constexpr int PASS = 4 * NW, NP = 128 / PASS;   // rows of a pass
    constexpr int PRE = NP < 4 ? NP : 4;            // what the epilogue reads of so many passes is requested beforehand
    typename Epi::Row8 prow[PRE];
    auto request = [&](int p) {
        const int m = m0 + p * PASS + (tid >> 4);
        prow[p % PRE] = epi.row8((int64_t)op_out_row(A, m < M ? m : 0, 0) * ld + n, m < M && n < N);
    };
#pragma unroll
    for (int p = 0; p < PRE; ++p) request(p);
    __syncthreads();   // every wave is past its last read: the stages may be overwritten
    float* const part = reinterpret_cast<float*>(smem_raw);   // [KG][2 x 2 subtiles][64][64]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                part[(wave * 64 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * 64 + j * 32 + (lane & 31)] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int row = p * PASS + (tid >> 4), m = m0 + row;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const float* q = part + ((k * 4 + (row >> 6) * 2 + ((tid >> 3) & 1)) * 64 + (row & 63)) * 64 + (tid & 7) * 8;
            const float4 lo = *reinterpret_cast<const float4*>(q), hi = *reinterpret_cast<const float4*>(q + 4);
            v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
            v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
        }
        if (m < M && n < N) epi.at8(pcol, prow[p % PRE], (int64_t)op_out_row(A, m, 0) * ld + n, v, z);
        if (p + PRE < NP) request(p + PRE);
    }
    if (ROWSUM && tile_x == 0) {   // (uniform in the workgroup)
        __syncthreads();
        float* const sums = part;   // [KG][2][128]
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float both = rs[i] + __shfl_xor(rs[i], 32, 64);
            if (lane < 32) sums[(kg * 2 + wn) * 128 + wm * 64 + i * 32 + lane] = both;
        }
        __syncthreads();
        if (tid < 128 && m0 + tid < M) {
            float t = sums[tid];
#pragma unroll
            for (int k = 1; k < 2 * KG; ++k) t += sums[k * 128 + tid];
            epi.rowsum(m0 + tid, t, z);
        }
    }
}

}  // namespace tmps
