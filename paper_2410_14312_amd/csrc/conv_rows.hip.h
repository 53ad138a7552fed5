// Convolutions with unit stride that keep the map size (forward pass and input gradient), bf16 in, fp32 accumulate:
//   C[m, n] = sum over taps (r, s) and channels c of X[m + (r - pad) W + (s - pad), c] * B(n, r, s, c)
// for positions m = (image, row, column) in memory order.  With maps of equal size a tap is a shift of the position index,
// so the rows of X that a tile of consecutive positions needs, over all taps, are ONE run of consecutive rows: tile +
// (R - 1) W + S - 1.  A workgroup copies that run to LDS once per 64 channels (whole rows, no address arithmetic) and reads every
// tap's operand from it at a shifted row; positions whose tap falls off the map read a row of zeros instead.
//
// The tiled kernel fetches each tap's rows anew and computes their addresses chunk by chunk: nine copies of X through L2 and
// LDS for a 3 x 3 filter and a k-tile of 1100 to 1800 cycles, three times what its multiplies take.  Here only the weights'
// tiles (64 channels x 64 or 32 columns per tap) are streamed.  Forward / input gradient, 3 x 3, on the tiled kernel and here (us): 64 images
// of 56 x 56 x 64 47 / 56 and 29 / 27, of 28 x 28 x 128 37 / 44 and 26 / 25, of 14 x 14 x 256 33 / 39 and 21 / 21, of 7 x 7 x 512
// 29 / 32 and 21 / 22; 128 images of 8 x 8 x 256 26 / 33 and 15 / 15, of 4 x 4 x 512 22 / 32 and 16 / 17, of 2 x 2 x 512 19 / 23 and 12 / 14.
//
// NW waves, WM of them along the 64 WM positions of a tile; the NW / WM groups take the taps in turn, each wave a tile of 64 x 32 TN
// over its group's taps; the groups' partial tiles are added through LDS at the end.  A step (one tap for every wave) takes
// 0.44 to 0.75 us where its multiplies take 0.25 (four waves on a unit) or 0.5 (eight): LDS serves 16 KB for every wave's 16 MFMAs, as long as these
// take, and receives the copies besides.  Contractions over 64 channels are bound by what is not overlapped around their few steps.
#pragma once
#include "gemm4.hip.h"

namespace tmps {

struct ConvRows {
    const bf16_t* x;    // [M][C] positions x channels: the operand that is shifted
    const bf16_t* w;    // weights [Cout][R][S][Cin]
    int M, N, C;        // positions, columns of the result, channels summed over (a multiple of 64)
    int H, W, S, RS, pad;
    int patch_rows;     // 64 WM + (R - 1) W + S - 1
    int patch_bytes;    // LDS of one run of rows (whole kilobytes)
    int two;            // two runs in LDS (more than 64 channels)
    FastDiv d_hw, d_w, d_s;
};

template <int NW, int WM, int TN> constexpr int conv_rows_stage_bytes() { return NW / WM * TN * 4096; }

// DGRAD: X is the gradient of the result, N = Cin, C = Cout, and B(n, r, s, c) = w[c][R - 1 - r][S - 1 - s][n]; else w[n][r][s][c].
template <int NW, int WM, int TN, int NS, bool DGRAD, class Epi>
__global__ __launch_bounds__(64 * NW, 2) void conv_rows_kernel(ConvRows cv, Epi epi, FastDiv d_tn) {
    constexpr int KG = NW / WM, BM = 64 * WM, BN = 32 * TN, CPW = 4 * TN / WM, STAGE = conv_rows_stage_bytes<NW, WM, TN>(), WTILE = STAGE / KG;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;
    const lds_t patches = smem + NS * STAGE, zeros = patches + cv.patch_rows * 128;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), kg = wave / WM, wm = wave % WM;
    int tile_m, tile_n;
    {   // (the workgroups of an XCD own a contiguous run of tiles, the column tiles of the same positions next to each other)
        const int total = gridDim.x, lin = blockIdx.x, xcd = lin & 7, idx = lin >> 3, q = total >> 3, r = total & 7;
        uint32_t a, b;
        d_tn.divmod(xcd * q + min(xcd, r) + idx, a, b);
        tile_m = (int)a;
        tile_n = (int)b;
    }
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    // (R S + 1 >= 2 KG: a run is copied during the last step of the one two before it, and first read two steps later)
    const int chunks = cv.C >> 6, taps = chunks * cv.RS, steps = (taps + KG - 1) / KG;

    // Copies of the run of rows: group g of 8 rows; position p of a row holds chunk p ^ ((row / 2) % 8): sixteen consecutive rows
    // read at one chunk then lie in different banks.
    const int pgroups = cv.patch_bytes >> 10;
    auto chunk_of = [&](int g) { return ((lane & 7) ^ (lane >> 4) ^ ((g & 1) << 2)) * 8; };
    const int sw = chunk_of(wave);   // (a wave's groups are all even or all odd)
    const int first = m0 - cv.pad * cv.W - cv.pad + (lane >> 3);
    auto copy_patch = [&](int chunk) {
        const bf16_t* src = cv.x + chunk * 64 + sw;
        const lds_t dst = patches + (chunk & 1) * cv.patch_bytes;   // (one chunk: buffer 0)
        for (int g = wave; g < pgroups; g += NW) {
            int row = first + g * 8;
            row = row < 0 ? 0 : row >= cv.M ? cv.M - 1 : row;   // (rows outside the tensor belong to no valid tap)
            // (the rows behind the run are zeros: the first of them, of run 0, is what invalid taps read)
            copy16_to_lds(at_if(src, (int64_t)row * cv.C, g * 8 + (lane >> 3) < cv.patch_rows), dst + g * 1024);
        }
    };
    // Copies of a tap's 64 x BN weights: CPW of 4 TN groups by each wave of the tap's own group, from offsets (bytes) behind the tap's first weight.
    const int my_taps = (taps - kg + KG - 1) / KG;   // (R S > KG: at least one)
    uint32_t woff[CPW];
#pragma unroll
    for (int g = 0; g < CPW; ++g) {
        const int grp = wm * CPW + g;
        if constexpr (DGRAD) {   // LDS [64 c][8 or 4 chunks of n]
            int n = n0 + (TN == 2 ? (lane & 7) ^ (((lane >> 4) & 1) << 2) : lane & 3) * 8;
            n = n + 8 <= cv.N ? n : cv.N - 8;
            woff[g] = (uint32_t)((TN == 2 ? grp * 8 + (lane >> 3) : grp * 16 + (lane >> 2)) * cv.RS * cv.N + n) * 2;
        } else {                 // LDS [BN n][8 chunks of c]
            int n = n0 + grp * 8 + (lane >> 3);
            n = n < cv.N ? n : cv.N - 1;
            woff[g] = (uint32_t)((n - n0) * cv.RS * cv.C + chunk_of(grp)) * 2;
        }
    }
    const bf16_t* wsrc = cv.w + (DGRAD ? (int64_t)(cv.RS - 1 - kg) * cv.N : (int64_t)n0 * cv.RS * cv.C + (int64_t)kg * cv.C);   // of the tap copied next
    const int64_t wstep = DGRAD ? -(int64_t)KG * cv.N : (int64_t)KG * cv.C;   // to the group's next tap, in the same 64 channels or in the next
    const int64_t wwrap = DGRAD ? (int64_t)(65 * cv.RS - KG) * cv.N : 64 - (int64_t)(cv.RS - KG) * cv.C;
    int ctap = kg, wleft = my_taps, fill = 0;    // (past the group's last tap its weights are copied again: the waits count copies)
    lds_t wdst = smem + kg * WTILE + wm * CPW * 1024;
    auto copy_weights = [&](int g) { copy16_to_lds(wsrc, woff[g], wdst + g * 1024); };
    auto next_weights = [&]() {
        ctap += KG;
        const bool wrap = ctap >= cv.RS;
        const int64_t by = wrap ? wwrap : wstep;
        ctap = wrap ? ctap - cv.RS : ctap;
        wsrc += --wleft > 0 ? by : 0;
        fill = fill + 1 == NS ? 0 : fill + 1;
        wdst = smem + fill * STAGE + kg * WTILE + wm * CPW * 1024;
    };

    copy_patch(0);
#pragma unroll
    for (int st = 0; st < NS; ++st) {
#pragma unroll
        for (int g = 0; g < CPW; ++g) copy_weights(g);
        next_weights();
    }

    // This lane's two rows: which taps lie on the map.
    uint32_t valid[2];
    int lrow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        lrow[i] = wm * 64 + i * 32 + (lane & 31);
        const int m = m0 + lrow[i];
        uint32_t img, rem, h, w;
        cv.d_hw.divmod(m < cv.M ? m : 0, img, rem);
        cv.d_w.divmod(rem, h, w);
        uint32_t v = 0;
        for (int t = 0; t < cv.RS; ++t) {
            uint32_t r, s;
            cv.d_s.divmod(t, r, s);
            const bool ok = m < cv.M && (unsigned)((int)h + (int)r - cv.pad) < (unsigned)cv.H && (unsigned)((int)w + (int)s - cv.pad) < (unsigned)cv.W;
            v |= (ok ? 1u : 0u) << t;
        }
        valid[i] = v;
    }

    f32x16_t acc[2][TN];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // A step's fragments are read while the step before is multiplied: one barrier per step, before the reads.  Behind it the step's
    // weights are there (everyone has waited for its copies) and the stage of the step being multiplied is free (everyone has
    // its fragments in registers).  Reads and copies are issued one after each multiply: all at once they would occupy the
    // wave until the LDS has served most of them, and the multiplies would come after that instead of meanwhile.
    // So are the addresses of the reads after those, and a copy of weights costs two scalar instructions (a base that all lanes share, one offset per
    // lane and group): computed behind the barrier, with nothing to multiply meanwhile, and with a 64-bit select for each copy, they took as long
    // as the multiplies (3 x 3 over 512 channels, forward / gradient, before and after, us: 128 images of 2 x 2 17.4 / 17.5 and 15.2 / 16.3, of
    // 4 x 4 19.2 / 19.0 and 17.5 / 18.1, 64 of 7 x 7 24.7 / 25.2 and 22.6 / 24.1; 256 channels, 64 images of 8 x 8 12.1 / 12.2 and 11.0 / 11.1).
    struct Frags { bf16x8_t a[4][2], b[4][TN]; };
    int tap = kg, run = 0, stage = 0;            // of the step whose addresses are computed next
    const int run_bytes = cv.two ? cv.patch_bytes : 0, inv_s = 65536 / cv.S + 1, row_step = cv.W - cv.S;   // (tap / S: at most 31 taps)
    lds_t pa[2], pb;
    constexpr int CP = TN * 64;                  // bytes of a channel's row of columns
    const int bl = DGRAD ? (half * 8 + ((lane & 15) >> 2)) * CP + ((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ (TN == 2 ? ((lane >> 3) & 1) << 2 : 0)) * 16 + (lane & 1) * 8
                         : (lane & 31) * 128 + ((half ^ ((lane >> 1) & 7)) << 4);
    // two parts, for between multiplies
    int shift;
    lds_t next_run, next_pb;
    uint32_t tap_bit;
    auto address_tap = [&]() {
        shift = tap + ((tap * inv_s) >> 16) * row_step;   // r W + s
        tap_bit = 1u << tap;
        next_run = patches + run;
        next_pb = smem + stage * STAGE + kg * WTILE + bl;
        tap += KG;
        const bool wrap = tap >= cv.RS;
        tap = wrap ? tap - cv.RS : tap;
        run = wrap ? run_bytes - run : run;
        stage = stage + 1 == NS ? 0 : stage + 1;
    };
    auto address_rows = [&]() {
        const int row = lrow[0] + shift;   // (the other one lies 32 rows on)
        const int at = row * 128 + next_run, sw = (half ^ ((row >> 1) & 7)) << 4;
        pa[0] = (valid[0] & tap_bit ? at : zeros) + sw;
        pa[1] = (valid[1] & tap_bit ? at + 4096 : zeros) + sw;
        pb = next_pb;
    };
    auto read_a = [&](Frags& q, int f, int i) { q.a[f][i] = *lds_ptr<const bf16x8_t>(pa[i] ^ (f << 5)); };
    auto read_b = [&](Frags& q, int f, int i) {
        if constexpr (DGRAD) {   // (rows 32 i .. of the 16 channels 16 f .., as in WaveTile)
            const lds_t p = (pb ^ (i << 6)) + f * 16 * CP;
            union { s16x4_t h[2]; bf16x8_t v; } u;
            u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(p));
            u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(p + 4 * CP));
            q.b[f][i] = u.v;
        } else q.b[f][i] = *lds_ptr<const bf16x8_t>((pb ^ (f << 5)) + 4096 * i);
    };
    int next_patch = 2;                          // the next run of rows to copy, into the buffer of run next_patch - 2 ...
    int last_use = (cv.RS - 1) / KG;             // ... whose last tap is in this step
    auto one_step = [&](int step, const Frags& cur, Frags& next) {
        wait_vmcnt<(NS - 2) * CPW>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (step == 0 && cv.two) copy_patch(1);
        if (step == last_use) {
            if (next_patch < chunks) copy_patch(next_patch);
            last_use = (next_patch * cv.RS - 1) / KG;
            ++next_patch;
        }
        if (step >= my_taps) return;   // (the last step, of a group without a tap in it)
#pragma unroll
        for (int f = 0; f < 4; ++f) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur.a[f][i], cur.b[f][j], acc[i][j], 0, 0, 0);
                    if (TN == 1 || i == j) read_a(next, f, i);
                    if (TN == 1 ? i == 0 : i != j) read_b(next, f, j);
                    if (f == 3 && i == 0 && j == TN - 1) address_tap();
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
            for (int g = f * CPW / 4; g < (f + 1) * CPW / 4; ++g) copy_weights(g);
        }
        address_rows();
        next_weights();
    };
    Frags f0, f1;
    address_tap();
    address_rows();
    wait_vmcnt<(NS - 1) * CPW>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            read_a(f0, f, i);
            if (i < TN) read_b(f0, f, i);
        }
    address_tap();
    address_rows();
    for (int step = 0; step < steps; step += 2) {
        one_step(step, f0, f1);
        if (step + 1 < steps) one_step(step + 1, f1, f0);
    }
    wait_vmcnt<0>();   // (the copies past the last tap)

    // ---- the groups' partial tiles are added through LDS, 8 consecutive columns of a row per lane ----
    const int64_t ld = epi.ld;
    constexpr int OCT = 4 * TN;   // lanes to a row
    const int n = n0 + tid % OCT * 8;
    const typename Epi::Col8 pcol = epi.col8(n < cv.N ? n : 0);
    constexpr int PASS = 64 * NW / OCT, NP = BM / PASS;   // rows of a pass
    typename Epi::Row8 prow[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int m = m0 + p * PASS + tid / OCT;
        prow[p] = epi.row8((int64_t)(m < cv.M ? m : 0) * ld + n, m < cv.M && n < cv.N);
    }
    __syncthreads();   // every wave is past its last read: the stages may be overwritten
    float* const part = reinterpret_cast<float*>(smem_raw);   // [NW][64][BN]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                part[(wave * 64 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * BN + j * 32 + (lane & 31)] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int row = p * PASS + tid / OCT, m = m0 + row;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const float* q = part + ((k * WM + (row >> 6)) * 64 + (row & 63)) * BN + tid % OCT * 8;
            const float4 lo = *reinterpret_cast<const float4*>(q), hi = *reinterpret_cast<const float4*>(q + 4);
            v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
            v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
        }
        if (m < cv.M && n < cv.N) epi.at8(pcol, prow[p], (int64_t)m * ld + n, v, 0);
    }
}

}  // namespace tmps
