// Weight gradients of 3 x 3 convolutions with unit stride that keep the map size, bf16 in, fp32 accumulate:
//   dW[n, r, s, c] = sum over positions m of dY[m, n] * X[m + (r - 1) W + (s - 1), c]
// for positions m = (image, row, column) in memory order, where the tap lies on the map; and the sums of dY over m.
//
// As in conv_rows.hip.h a tap is a shift of the position index: 128 positions need ONE run of 128 + 2 W + 2 rows of X for all taps.
// A workgroup copies that run and the rows of dY to LDS once and multiplies them for three taps, where the tiled kernels copy each
// tap's rows anew and compute their addresses chunk by chunk.  Where a position's row lies for a tap (in the run, or a row of zeros where the tap falls
// off the map) is looked up in a table that 384 threads write per chunk: told from flags in registers it took seven vector instructions a multiply.
//
// 128 positions take 0.93 us, 0.37 of them multiplies: LDS serves the transposed reads at half its rate (5 for 6 multiplies, 0.6 us).  All nine
// taps in a workgroup (32 x 32 for a wave, ten reads for nine multiplies) took 2.2 us, and give a third of the workgroups for the same slices, whose
// partial sums cost what they write; fragments read in the step they are multiplied in, 1.05 us.  On the other kernels and here, with the slices'
// sum (us): 128 images of 2 x 2 x 512 13.8 and 10.6, of 4 x 4 x 512 29 and 22, of 8 x 8 x 256 30 and 26, of 16 x 16 x 128 31 and 28, of
// 32 x 32 x 64 40 and 28; 64 images of 56 x 56 x 64 53 and 34, 32 of 28 x 28 x 128 30 and 25, of 14 x 14 x 256 27 and 23, of 7 x 7 x 512 23 and 18.
// Errors (2-norm, against 64 bits), there and here: 128 images of 4 x 4 x 512 1.7e-7 and 1.2e-7, of 32 x 32 x 64 2.6e-7 and 1.5e-7, 64 of 56 x 56 x 64
// 2.2e-7 and 1.7e-7, of 14 x 14 x 512 2.7e-7 and 1.6e-7 (the number of slices sees to it: conv_wgrad_rows_plan).
#pragma once
#include "gemm4.hip.h"

namespace tmps {

struct ConvWgradRows {
    const bf16_t* dy;   // [M][N]
    const bf16_t* x;    // [M][C]
    int M, N, C, H, W;
    int run_groups;     // kilobytes of a run of 128 + 2 W + 2 rows
    int per_slice;      // positions of a slice, a multiple of 128
    FastDiv d_tiles, d_row, d_w, d_h;   // by tiles of a slice, by tiles of 64 rows of dW, by W, by H
};

// LDS of a chunk: rows of dY, of X, one of zeros (in a kilobyte), and where each position's row for a tap lies
constexpr int kWgradStages = 3, kWgradPlaces = 128 * 3 * 2;
static inline int conv_wgrad_rows_lds(int run_groups) { return kWgradStages * (16384 + run_groups * 1024 + 1024 + kWgradPlaces); }

// A workgroup forms 64 x 64 (n, c) for the three taps of a filter row.  Eight waves in four groups, each group 32 of a chunk's 128 positions, each wave
// 64 x 32 of the tile.
template <int NS>
__global__ __launch_bounds__(512, 2) void conv_wgrad_rows_kernel(ConvWgradRows cv, EpiWgrad epi) {
    constexpr int NW = 8, KG = 4, NF = 2;   // waves; groups; fragments of 16 positions of a group
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const int zeros = 16384 + cv.run_groups * 1024, table = zeros + 1024, STAGE = table + kWgradPlaces;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave >> 1, wc = wave & 1;
    int z, n0, c0, row;
    {   // (the workgroups of an XCD own a contiguous run of tiles)
        const int total = gridDim.x, lin = blockIdx.x, xcd = lin & 7, idx = lin >> 3, q = total >> 3, r = total & 7;
        uint32_t zz, t, tn, rest;
        cv.d_tiles.divmod(xcd * q + min(xcd, r) + idx, zz, t);
        cv.d_row.divmod(t, tn, rest);
        z = (int)zz;
        n0 = (int)tn * 64;
        c0 = (int)(rest / 3) * 64;
        row = (int)(rest % 3);
    }
    const int k0 = z * cv.per_slice, k1 = min(cv.M, k0 + cv.per_slice), chunks = (k1 - k0 + 127) >> 7;

    // Copies: 1-KB groups of 8 rows; position p of a row holds chunk p ^ (4 (row / 2 % 2)), as in gemm4.hip.h.
    const int sw = ((lane & 7) ^ (((lane >> 4) & 1) << 2)) * 8;
    auto copy = [&](int chunk, int stage) {
        const lds_t st = smem + stage * STAGE;
        const int m0 = k0 + chunk * 128 + (lane >> 3);
        for (int g = wave; g < 16; g += NW) {
            const int m = m0 + g * 8;
            copy16_to_lds(at_if(cv.dy, (int64_t)m * cv.N + n0 + sw, m < k1), st + g * 1024);
        }
        for (int g = wave; g < cv.run_groups; g += NW) {
            const int m = m0 + g * 8 - cv.W - 1;
            copy16_to_lds(at_if(cv.x, (int64_t)m * cv.C + c0 + sw, m >= 0 && m < cv.M), st + 16384 + g * 1024);
        }
    };
    // Where the row of X for a position and a tap lies in its chunk's LDS (16 bits): in the run, or the row of zeros where the tap falls off the map or
    // the position past the end.  A lane's positions of a chunk lie next to each other.
    auto put_places = [&](int chunk, int stage) {
        const int p = tid & 127, m = k0 + chunk * 128 + p;
        uint32_t q, w, img, h;
        cv.d_w.divmod(m, q, w);
        cv.d_h.divmod(q, img, h);
        const lds_t to = smem + stage * STAGE + table + ((p >> 5) * 8 + ((p >> 3) & 1) * 4 + (p & 3)) * 24 + (((p >> 4) & 1) * 2 + ((p >> 2) & 1)) * 2;
        const int s = tid >> 7;
        if (s < 3) {
            const int at = p + row * cv.W + s;
            const bool on = m < k1 && (unsigned)((int)h + row - 1) < (unsigned)cv.H && (unsigned)((int)w + s - 1) < (unsigned)cv.W;
            *lds_ptr<uint16_t>(to + s * 8) = (uint16_t)(on ? 16384 + at * 128 + (((at >> 1) & 1) << 6) : zeros);
        }
    };

    // Where this lane reads: fragment f holds positions 16 f + 8 half + 0 .. 7 of the group's, in two transposed reads of four.
    const int k = kg * (16 * NF) + half * 8 + ((lane & 15) >> 2), part = (((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
    const int aoff = k * 128 + (part ^ (((k >> 1) & 1) << 6)), bpart = (wc << 6) | part;
    const int my_table = table + ((kg * 2 + half) * 4 + ((lane & 15) >> 2)) * 24;

    f32x16_t acc[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][n][r] = 0.0f;
    float rs[2] = {0.0f, 0.0f};
    const bool sum_rows = c0 == 0 && row == 0;

    // (copies of this wave for a chunk: at least 4)
    const int mine = 2 + ((cv.run_groups - wave + NW - 1) >> 3);
    if (tid < 8 * NS) *lds_ptr<bf16x8_t>(smem + (tid >> 3) * STAGE + zeros + (tid & 7) * 16) = bf16x8_t{};
    auto put = [&](int chunk, int stage) {
        put_places(chunk, stage);   // (past the last chunk: the row of zeros, for reads that are not used)
        if (chunk < chunks) copy(chunk, stage);
    };
#pragma unroll
    for (int i = 0; i < NS; ++i) put(i, i);

    // A chunk's fragments are read while the one before is multiplied, and where they lie one chunk before that.  One barrier per chunk, before the
    // reads: behind it the next chunk is there, and the stage of the one being multiplied is free.
    typedef uint32_t places_t __attribute__((ext_vector_type(NF)));
    struct Frags { bf16x8_t a[NF][2], b[NF][3]; };
    places_t places[3];
    auto read_places = [&](int stage) {
#pragma unroll
        for (int t = 0; t < 3; ++t) places[t] = *lds_ptr<const places_t>(smem + stage * STAGE + my_table + t * 8);
    };
    auto read_a = [&](Frags& q, lds_t st, int f, int n) {
        union { s16x4_t h[2]; bf16x8_t v; } u;
#pragma unroll
        for (int j = 0; j < 2; ++j) u.h[j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(((st + aoff) ^ (n << 6)) + f * 2048 + j * 512));
        q.a[f][n] = u.v;
    };
    auto read_b = [&](Frags& q, lds_t st, int f, int t) {
        union { s16x4_t h[2]; bf16x8_t v; } u;
#pragma unroll
        for (int j = 0; j < 2; ++j) u.h[j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>((((places[t][f] >> (16 * j)) & 0xFFFF) ^ bpart) + st));
        q.b[f][t] = u.v;
    };
    auto arrived = [&](bool more) {   // all copies but those of one later chunk, if there is one
        if (!more) wait_vmcnt<0>();
        else if (mine >= 6) wait_vmcnt<6>();
        else if (mine == 5) wait_vmcnt<5>();
        else wait_vmcnt<4>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    int stage = 0;   // of the chunk being multiplied
    auto one_step = [&](int chunk, const Frags& cur, Frags& next) {
        const int s1 = stage + 1 == NS ? 0 : stage + 1, s2 = s1 + 1 == NS ? 0 : s1 + 1;
        arrived(chunk + 2 < chunks);
        const lds_t st = smem + s1 * STAGE;   // (past the last chunk: read and not used)
#pragma unroll
        for (int i = 0; i < 3 * NF; ++i) {
            const int f = i / 3, t = i % 3;
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                acc[t][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[f][n], cur.b[f][t], acc[t][n], 0, 0, 0);
                if (n == 0) read_b(next, st, f, t);
                else if (t < 2) read_a(next, st, f, t);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (sum_rows && wc == 0) {
#pragma unroll
            for (int n = 0; n < 2; ++n) {   // (a sum of the chunk's own first: a slice's takes one rounding for each chunk)
                float chunk_sum = 0.0f;
#pragma unroll
                for (int f = 0; f < NF; ++f) chunk_sum = add_frag(chunk_sum, cur.a[f][n]);
                rs[n] += chunk_sum;
            }
        }
        read_places(s2);
        put(chunk + NS, stage);
        stage = s1;
    };
    Frags f0, f1;
    static_assert(NS == 3, "the copies of one chunk may be under way behind those waited for");
    arrived(false);
    read_places(0);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
        for (int n = 0; n < 2; ++n) read_a(f0, smem, f, n);
#pragma unroll
        for (int t = 0; t < 3; ++t) read_b(f0, smem, f, t);
    }
    read_places(1);
    for (int chunk = 0; chunk < chunks; chunk += 2) {
        one_step(chunk, f0, f1);
        if (chunk + 1 < chunks) one_step(chunk + 1, f1, f0);
    }

    // ---- the groups' results are added through LDS, tap by tap, 8 consecutive columns of a row per lane ----
    float* const sums = reinterpret_cast<float*>(smem_raw);   // [KG][64][64]
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) sums[(kg * 64 + n * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * 64 + wc * 32 + (lane & 31)] = acc[t][n][r];
        __syncthreads();
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            const float* q = sums + (g * 64 + (tid >> 3)) * 64 + (tid & 7) * 8;
            const float4 lo = *reinterpret_cast<const float4*>(q), hi = *reinterpret_cast<const float4*>(q + 4);
            v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
            v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
        }
        epi.at8(EpiWgrad::Col8{}, EpiWgrad::Row8{}, (n0 + (tid >> 3)) * epi.ld + (row * 3 + t) * cv.C + c0 + (tid & 7) * 8, v, z);
    }
    if (sum_rows) {   // (uniform in the workgroup)
        __syncthreads();
        if (wc == 0) {
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const float both = rs[n] + __shfl_xor(rs[n], 32, 64);
                if (lane < 32) sums[kg * 64 + n * 32 + lane] = both;
            }
        }
        __syncthreads();
        if (tid < 64) {
            float v = sums[tid];
#pragma unroll
            for (int g = 1; g < KG; ++g) v += sums[g * 64 + tid];
            epi.rowsum(n0 + tid, v, z);
        }
    }
}

}  // namespace tmps
