// Convolutions over eight channels (an RGB image padded to a 16-byte pixel: the first layer of a network), bf16 in, fp32 accumulate: forward
// pass and weight gradient of 3 x 3 filters with stride 1 and 7 x 7 filters with stride 2.
//
// A pixel is one 16-byte chunk, and a chunk is what a lane of a matrix instruction takes of the contraction: a step of 16 k is two taps.  A
// workgroup owns 8 x 16 positions of the result and copies the pixels that they need over all taps to LDS once; every tap's operand is read there, at an
// offset that is known when the kernel is compiled.  Nothing is gathered and no filter tap is fetched twice, where the tiled kernel computes an address
// for each of the 49 chunks of a position and fetches them all through L2.  With stride 2 the even columns of the pixels lie in front of the odd
// ones, so that the sixteen columns of a tap are sixteen chunks in a row.
//
// 64 images of 224 x 224, 7 x 7: forward 118 -> 54 us, 27 of them what a copy of its operands takes; the rest are LDS reads, one for a multiply.  Weight
// gradient 154 -> 65: a tile takes a workgroup 2.4 us, 1.0 of them multiplies, 1.5 transposed reads (LDS serves them at half its rate, six for eight
// multiplies).  Errors of the weight gradients (2-norm, against 64 bits) on the tiled kernels and here: 64 images of 224 x 224 5.0 and 2.5e-7, 8 of
// them 2.0 and 1.2e-7, 3 x 3 over 128 images of 32 x 32 1.5 and 1.1e-7, 64 of 64 x 64 2.1 and 1.1e-7.
#pragma once
#include "gemm4.hip.h"

namespace tmps {

struct ConvFirst {
    const bf16_t* x;   // [B][H][W][8]
    const bf16_t* o;   // weights [N][R][S][8] (forward); the result's gradient [B][Ho][Wo][N] (weight gradient)
    int H, W, Ho, Wo, N, pad;
    int tiles, per;    // tiles of 8 x 16 positions; of a workgroup (weight gradient)
    FastDiv d_img, d_row;   // by the tiles of an image and of a row of tiles
};

template <int R, int S, int STRIDE> struct FirstTile {
    static constexpr int TAPS = R * S, ROWS = 7 * STRIDE + R;
    static constexpr int PLANE = (15 * STRIDE + S + STRIDE - 1) / STRIDE, PITCH = STRIDE * PLANE;   // columns of one parity; pixels of a row in LDS
    static constexpr int GROUPS = (ROWS * PITCH + 63) / 64, BYTES = GROUPS * 1024;                  // of 64 pixels, a copy instruction each
    // where the pixel of a tap lies behind that of the first one
    static constexpr int offset(int tap) { return ((tap / S) * PITCH + (tap % S % STRIDE) * PLANE + tap % S / STRIDE) * 16; }

    // The pixels of the tile at rows r0.., columns c0.. of image img; those outside the map are zeros.
    static __device__ __forceinline__ void copy(const ConvFirst& cv, int img, int r0, int c0, lds_t to, int wave, int waves, int lane) {
        const int top = r0 * STRIDE - cv.pad, left = c0 * STRIDE - cv.pad;
        for (int g = wave; g < GROUPS; g += waves) {
            const int px = g * 64 + lane, row = px / PITCH, rest = px % PITCH, odd = STRIDE == 2 && rest >= PLANE ? 1 : 0;
            const int h = top + row, w = left + (rest - odd * PLANE) * STRIDE + odd;
            const bool ok = row < ROWS && (unsigned)h < (unsigned)cv.H && (unsigned)w < (unsigned)cv.W;
            copy16_to_lds(at_if(cv.x, (((int64_t)img * cv.H + h) * cv.W + w) * 8, ok), to + g * 1024);
        }
    }
};
template <int R, int S, int STRIDE> constexpr int conv_first_lds() { return 2 * FirstTile<R, S, STRIDE>::BYTES + 16; }

// Forward pass.  Four waves, each four rows of the tile and 32 columns of the result, whose weights it holds in registers over all of its
// workgroup's tiles: LDS serves one read for every multiply, where it served three for two with the weights in LDS too.
// The positions are the columns of the matrix instruction, so that a lane ends with eight consecutive channels of one position once it
// has exchanged halves with the lane 32 on: no results go through LDS.
template <int R, int S, int STRIDE, class Epi>
__global__ __launch_bounds__(256, 2) void conv_first_kernel(ConvFirst cv, Epi epi) {
    typedef FirstTile<R, S, STRIDE> Tile;
    constexpr int STEPS = (Tile::TAPS + 1) / 2;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const lds_t zeros = smem + 2 * Tile::BYTES;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, pos = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), n0 = blockIdx.y * 64 + (wave & 1) * 32, row0 = (wave >> 1) * 4;
    int img, r0, c0;
    auto place = [&](int t) {
        uint32_t i, rest, r, c;
        cv.d_img.divmod((uint32_t)t, i, rest);
        cv.d_row.divmod(rest, r, c);
        img = (int)i;
        r0 = (int)r * 8;
        c0 = (int)c * 16;
    };
    int t = blockIdx.x;
    place(t);
    Tile::copy(cv, img, r0, c0, smem, wave, 4, lane);
    bf16x8_t w[STEPS];   // of channel n0 + lane % 32: taps 2 k and 2 k + 1
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        const int tap = 2 * k + half;
        w[k] = *reinterpret_cast<const bf16x8_t*>(at_if(cv.o, ((int64_t)(n0 + pos) * Tile::TAPS + tap) * 8, tap < Tile::TAPS && n0 + pos < cv.N));
    }
    if (tid == 0) *lds_ptr<bf16x8_t>(zeros) = bf16x8_t{};

    typename Epi::Col8 col[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int n = n0 + 8 * (2 * p + half);
        col[p] = epi.col8(n < cv.N ? n : 0);
    }
    const int first = ((row0 + (pos >> 4)) * STRIDE * Tile::PITCH + (pos & 15)) * 16;
    bool inside = false;   // the tile before this one lay on the map, so that the wave has stored four times at least
    for (int buf = 0;; buf ^= 1) {
        // (this tile's copies are older than the stores of the one before)
        if (inside) wait_vmcnt<4>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        int64_t m[2];
        bool on[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int h = r0 + row0 + 2 * j + (pos >> 4), c = c0 + (pos & 15);
            m[j] = ((int64_t)img * cv.Ho + h) * cv.Wo + c;
            on[j] = h < cv.Ho && c < cv.Wo;
        }
        inside = r0 + 8 <= cv.Ho && c0 + 16 <= cv.Wo && n0 + 32 <= cv.N;
        const int next = t + gridDim.x;
        if (next < cv.tiles) {
            place(next);
            Tile::copy(cv, img, r0, c0, smem + (buf ^ 1) * Tile::BYTES, wave, 4, lane);
        }
        if (n0 < cv.N) {
            f32x16_t acc[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
            const lds_t px = smem + buf * Tile::BYTES + first;
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                const int second = 2 * k + 1;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const lds_t at = px + j * (2 * STRIDE * Tile::PITCH * 16);
                    const lds_t from = second < Tile::TAPS ? at + (half ? Tile::offset(second) : Tile::offset(2 * k)) : half ? zeros : at + Tile::offset(2 * k);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[k], *lds_ptr<const bf16x8_t>(from), acc[j], 0, 0, 0);
                }
            }
            typename Epi::Row8 rows[2][2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int n = n0 + 8 * (2 * p + half);
                    rows[j][p] = epi.row8(m[j] * epi.ld + n, on[j] && n < cv.N);
                }
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    // A lane holds channels 8 q + 4 half .. + 3 of its position for q = 0 .. 3: of q = 2 p the lower lane takes the other's, of
                    // q = 2 p + 1 the upper one.
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[j][8 * p + e]), __float_as_uint(acc[j][8 * p + 4 + e]), false, false);
                        v[e] = __uint_as_float(s[0]);
                        v[4 + e] = __uint_as_float(s[1]);
                    }
                    const int n = n0 + 8 * (2 * p + half);
                    if (on[j] && n < cv.N) epi.at8(col[p], rows[j][p], m[j] * epi.ld + n, v, 0);
                }
        }
        if (next >= cv.tiles) break;
        t = next;
    }
}

// Weight gradient dW[n, tap, c] = sum over positions m of dY[m, n] X[pixel(m, tap), c], and the sums of dY over m.  The columns of the matrix
// instruction are the eight channels of four taps, its contraction sixteen columns of a row of the tile; both operands are read transposed.  Eight
// waves: SETS of them share the taps, four at a time in turn, the 8 / SETS groups the tile's rows.  A workgroup walks `per` tiles, three of them in
// LDS, and writes a partial result.
constexpr int kFirstStages = 3;
template <int R, int S, int STRIDE> constexpr int conv_first_wgrad_lds() {
    constexpr int main = kFirstStages * (16384 + FirstTile<R, S, STRIDE>::BYTES) + 16, sums = 8 * 64 * 32 * 4;
    return main > sums ? main : sums;
}
template <int R, int S, int STRIDE, int SETS>
__global__ __launch_bounds__(512, 2) void conv_first_wgrad_kernel(ConvFirst cv, EpiWgrad epi) {
    typedef FirstTile<R, S, STRIDE> Tile;
    constexpr int NW = 8, KG = NW / SETS, QUADS = (Tile::TAPS + 3) / 4, MINE = (QUADS + SETS - 1) / SETS, STAGE = 16384 + Tile::BYTES, NS = kFirstStages;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const lds_t zeros = smem + NS * STAGE;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave / SETS, set = wave % SETS;
    const int z = blockIdx.x, n0 = blockIdx.y * 64, t0 = z * cv.per, tiles = min(cv.tiles - t0, cv.per);
    auto place = [&](int t, int& img, int& r0, int& c0) {
        uint32_t i, rest, r, c;
        cv.d_img.divmod((uint32_t)(t0 + t), i, rest);
        cv.d_row.divmod(rest, r, c);
        img = (int)i;
        r0 = (int)r * 8;
        c0 = (int)c * 16;
    };
    // Copies: dY in 1-KB groups of 8 positions (half a row of the tile), position p of a row of 128 bytes holding chunk p ^ (4 (row / 2 % 2)), as in gemm4.hip.h.
    const int n = n0 + ((lane & 7) ^ (((lane >> 4) & 1) << 2)) * 8;
    auto copy = [&](int t, int stage) {
        int img, r0, c0;
        place(t, img, r0, c0);
        const lds_t st = smem + stage * STAGE;
#pragma unroll
        for (int g = wave; g < 16; g += NW) {
            const int h = r0 + (g >> 1), w = c0 + (g & 1) * 8 + (lane >> 3);
            copy16_to_lds(at_if(cv.o, (((int64_t)img * cv.Ho + h) * cv.Wo + w) * cv.N + n, h < cv.Ho && w < cv.Wo && n < cv.N), st + g * 1024);
        }
        Tile::copy(cv, img, r0, c0, st + 16384, wave, NW, lane);
    };
    const int mine = 2 + (Tile::GROUPS - wave + NW - 1) / NW;   // copies of this wave for a tile: 2, 3 or 4
    static_assert(Tile::GROUPS <= 2 * NW, "at most two groups of pixels to a wave");

    // Where this lane reads: a step's sixteen positions are columns 8 half + 0 .. 7 of a row, in two transposed reads of four.
    const int k = half * 8 + ((lane & 15) >> 2), part = (((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) * 16 + (lane & 1) * 8;
    const int aoff = k * 128 + (part ^ (((k >> 1) & 1) << 6));
    int boff[MINE];
#pragma unroll
    for (int q = 0; q < MINE; ++q) {
        const int tap = min((set + q * SETS) * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1), Tile::TAPS - 1);   // (columns past the last tap are not stored)
        const int r = tap / S, s = tap % S;
        boff[q] = 16384 + (r * Tile::PITCH + s % STRIDE * Tile::PLANE + s / STRIDE + k) * 16 + (lane & 1) * 8;
    }
    f32x16_t acc[MINE][2];
#pragma unroll
    for (int q = 0; q < MINE; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[q][i][r] = 0.0f;
    float rs[2] = {0.0f, 0.0f};
    if (tid == 0) *lds_ptr<bf16x8_t>(zeros) = bf16x8_t{};
    copy(0, 0);
    if (tiles > 1) copy(1, 1);
    int stage = 0;
    for (int t = 0; t < tiles; ++t) {
        if (t + 1 >= tiles) wait_vmcnt<0>();
        else if (mine == 4) wait_vmcnt<4>();
        else if (mine == 3) wait_vmcnt<3>();
        else wait_vmcnt<2>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // (everyone is past its last read of the tile before this one)
        if (t + 2 < tiles) copy(t + 2, stage >= 1 ? stage - 1 : NS - 1);
        int img, r0, c0;
        place(t, img, r0, c0);
        // (a position off the map has a gradient of zero; its pixels count as zeros too, so that no infinity among them makes a NaN of it)
        const int left = cv.Wo - c0 - k, below = cv.Ho - r0;
        const lds_t st = smem + stage * STAGE;
        float tile_rs[2] = {0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < 8 / KG; ++j) {
            const int row = kg + j * KG;
            const bool on[2] = {row < below && left > 0, row < below && left > 4};
            bf16x8_t a[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                union { s16x4_t h[2]; bf16x8_t v; } u;
#pragma unroll
                for (int e = 0; e < 2; ++e) u.h[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(((st + aoff) ^ (i << 6)) + row * 2048 + e * 512));
                a[i] = u.v;
            }
            const lds_t px = st + row * (STRIDE * Tile::PITCH * 16);
#pragma unroll
            for (int q = 0; q < MINE; ++q) {
                if (set + q * SETS >= QUADS) continue;
                union { s16x4_t h[2]; bf16x8_t v; } u;
#pragma unroll
                for (int e = 0; e < 2; ++e) u.h[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(on[e] ? px + boff[q] + e * 64 : zeros));
#pragma unroll
                for (int i = 0; i < 2; ++i) acc[q][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], u.v, acc[q][i], 0, 0, 0);
            }
            if (set == 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i) tile_rs[i] = add_frag(tile_rs[i], a[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) rs[i] += tile_rs[i];
        stage = stage + 1 == NS ? 0 : stage + 1;
    }

    // ---- the groups' sums are added through LDS, four taps of every set at a time ----
    float* const sums = reinterpret_cast<float*>(smem_raw);   // [NW][64][32]
#pragma unroll
    for (int q = 0; q < MINE; ++q) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) sums[(wave * 64 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * 32 + (lane & 31)] = acc[q][i][r];
        __syncthreads();
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const int row = tid >> 3, c = (tid & 7) * 4, col = (s + q * SETS) * 32 + c;
            float4 v = *reinterpret_cast<const float4*>(sums + (s * 64 + row) * 32 + c);
#pragma unroll
            for (int g = 1; g < KG; ++g) {
                const float4 w = *reinterpret_cast<const float4*>(sums + ((g * SETS + s) * 64 + row) * 32 + c);
                v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
            }
            if (n0 + row < cv.N && col < Tile::TAPS * 8) *reinterpret_cast<float4*>(epi.out + z * epi.slice_stride + (int64_t)(n0 + row) * epi.ld + col) = v;
        }
    }
    __syncthreads();
    if (set == 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const float both = rs[i] + __shfl_xor(rs[i], 32, 64);
            if (lane < 32) sums[kg * 64 + i * 32 + lane] = both;
        }
    }
    __syncthreads();
    if (tid < 64 && n0 + tid < cv.N) {
        float v = sums[tid];
#pragma unroll
        for (int g = 1; g < KG; ++g) v += sums[g * 64 + tid];
        epi.rowsum(n0 + tid, v, z);
    }
}

}  // namespace tmps
