// Persistent MFMA GEMM for gfx950 with asynchronous global -> LDS copies (bf16 in, fp32 accumulate), used
// by the dense contractions whose shapes allow it (K a multiple of 64 but in groups of weight gradients, row counts of row-contiguous
// operands a multiple of 8, 16-byte aligned operands).
//
//   C[m, n] = sum_k A(m, k) * B(n, k)
//
// An operand is k-contiguous (element (row, k) at p[row*ld + k]) or row-contiguous (p[k*ld + row]).
//
// Work decomposition: the output is cut into BM x BN tiles and k into `slices` equal ranges; a work unit
// is (tile, slice).  The grid has one workgroup per compute unit; workgroup b (renumbered so that the workgroups
// of an XCD are neighbours) processes units b, b + grid, b + 2 grid, ...  The k-loop is software-pipelined ACROSS units: the copies of the next
// NS-1 k-tiles are always in flight, also over a unit boundary, so a unit's first tiles arrive while the
// previous unit is still being multiplied and its results are being stored.  Short contractions (a dozen
// k-tiles per unit) therefore pay the memory latency once per workgroup, not once per tile.
//
// Copies: one wave instruction copies 64 x 16 bytes from per-lane global addresses to 1 KB of consecutive
// LDS (global_load_lds_dwordx4); nothing is staged in registers.  LDS tiles are unpadded; bank conflicts
// are avoided by permuting 16-byte chunks with an XOR of the row (k-contiguous tiles, [rows][64]) or of k
// (row-contiguous tiles, [64][rows]), which only changes WHICH global chunk a lane fetches.
// Fragments: k-contiguous tiles are read with 16-byte LDS reads, row-contiguous ones with the transpose
// read of gfx950.  Results are transposed through 4 KB of LDS that each wave has to itself, so that every lane stores 16 bytes and
// a store instruction covers whole 128-byte lines.  Copies and stores are counted by the same counter, in order: before a unit's first store the
// wave waits for its copies in flight, which have had the last multiplies to arrive in, and then need not wait again for NS - 1 k-tiles, in which
// the stores drain.
// What bounds it, by the device clock of each workgroup (us): a unit of 256 x 128 over 3072 (8192 x 768, 41 a launch) waits 1.9 for its first copies, 34.3 are the
// k-loop, 0.4 the wait for the last ones under way, 2.3 the results; over 768 (16 a launch) 1.7, 8.6, 0.4 and 2.3.  A unit of 256 x 256 over 768 (8192 x 3072, 50 a
// launch): 1.7, 18.5, 0.6 and 3.0, with GELU and its derivative 7.9, with GELU's mask 5.8 and 4.3 (the first unit's code is fetched), and between units 0.2.
// The results took 4.5 us (6.6 the first time) as long as they asked at each 8 elements what to do with them (see EpiForm): 8192 x 768
// over 2304 37.7 -> 35.0 us, 8192 x 3072 over 768 with GELU's mask in GPT-2's stage 66 -> 61.
#pragma once
#include <type_traits>
#include <utility>

#include "gemm2.hip.h"

namespace tmps {

// LDS is addressed by 32-bit byte addresses throughout this kernel (lds_t), turned into LDS pointers where a value is
// read or written: generic pointers into LDS make the compiler carry null checks and aperture tests around (and, in
// some arrangements of this kernel's control flow, fail in its instruction verifier).
typedef uint32_t lds_t;
template <class T> __device__ __forceinline__ __attribute__((address_space(3))) T* lds_ptr(lds_t a) {
    return (__attribute__((address_space(3))) T*)(uintptr_t)a;
}

template <bool KC> struct G3Operand {
    static constexpr bool kContig = KC;
    const bf16_t* p;
    int rows;    // valid rows (m or n extent)
    int64_t ld;  // elements between consecutive rows (KC) or consecutive k (RC)
};

// f(0), f(1), .. f(N - 1) with the index as a constant
template <class F, int... I> __device__ __forceinline__ void static_for_each(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

// wait until at most N vector-memory operations of this wave are outstanding
// (the trailing comment tells this wait from the ones the compiler inserts, for tests/test_gemm3_isa.py)
template <int N> __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0) ; tmps" ::"n"(N) : "memory");
}

// One wave instruction that copies 16 bytes per lane from `src` (per lane) to 1 KB of consecutive LDS at `dst` (the same
// for all lanes).  Written out as instructions rather than through the compiler's builtin: the compiler cannot tell
// which LDS reads a copy in flight may alias and makes the wave wait for ALL its outstanding copies before the next
// LDS read it sees, which serialises the copy pipeline; here the kernel's own counter waits and barriers order copies
// and reads (a stage is read only after the wait and barrier that follow its copies, and refilled only after the
// barrier that follows its last read).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is reserved: the compiler keeps nothing in it across statements
__device__ __forceinline__ void copy16_to_lds(const void* src, lds_t dst) {
    const uint32_t lds = __builtin_amdgcn_readfirstlane(dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}
// the same from `off` bytes (of each lane) behind a base that all lanes share to LDS `DIST` bytes behind `dst`
template <int DIST = 0> __device__ __forceinline__ void copy16_to_lds(const void* base, uint32_t off, lds_t dst) {
    const uint32_t lds = __builtin_amdgcn_readfirstlane(dst);
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base), "n"(DIST) : "memory", "m0", "scc");
}
#pragma clang diagnostic pop

// Makes the compiler treat every 32-bit word of `t` (values requested from memory earlier) as read here, on every
// path: a request whose result is never read stays "in flight" in the compiler's book-keeping, and the wait it then
// inserts wherever the register is next written — in the k-loop of the following unit — would drain the copy pipeline
// on every k-tile.
template <class T> __device__ __forceinline__ void settle(const T& t) {
    if constexpr (!std::is_empty<T>::value) {
        static_assert(sizeof(T) % 4 == 0, "whole registers");
        uint32_t w[sizeof(T) / 4];
        __builtin_memcpy(w, &t, sizeof(T));
#pragma unroll
        for (unsigned i = 0; i < sizeof(T) / 4; ++i) asm volatile("" ::"v"(w[i]));
    }
}

// LDS bytes of one launch: the stages, and 4 KB for each wave's results on their way out
constexpr int kG3StageOut = 4096;
template <int BM, int BN, int BK, int NS> constexpr int gemm3_lds_bytes(int waves) { return NS * (BM + BN) * BK * 2 + waves * kG3StageOut; }

// Whether the bytes from a tile's first element to any of its chunks fit 32 bits: `lines` rows of the tile (k-contiguous) or k of a k-tile (row-contiguous), `ld`
// elements apart, `across` elements each: up to 8.4 million elements apart for 256 rows, 34 million for 64 k.
constexpr bool g3_offsets_fit(int lines, int across, int64_t ld) { return ((int64_t)(lines - 1) * ld + across) * 2 <= (int64_t(1) << 32); }

// what a copy reads in place of elements that are not there
__device__ __attribute__((aligned(16))) static const uint32_t g3_zeros[4] = {0, 0, 0, 0};

// Per-wave copy state of one operand tile of ROWS rows x BK k (BK = 32 or 64): GROUPS 1-KB groups per k-tile.  A lane's address is a base that
// the wave shares, stepped by the scalar unit, and a 32-bit offset that stays as it is for a unit: a copy is then three instructions.  With an
// address of 64 bits in each lane, stepped after each copy, the vector unit's additions and moves took issue slots between the multiplies
// (see the k-loop).  WIDE instances keep such addresses: units whose last k-tile may end early, where zeros replace single lanes' sources, and operands whose rows
// (k-contiguous) or k (row-contiguous) lie so far apart that offsets inside a tile do not fit 32 bits (see offsets_fit).
template <int ROWS, int BK, int NW, bool KC, bool WIDE> struct G3Loader {
    static constexpr int GROUPS = ROWS * BK * 2 / 1024 / NW;
    static_assert(GROUPS >= 1 && GROUPS * NW * 1024 == ROWS * BK * 2, "the waves must share a tile evenly");
    static_assert(KC || (ROWS / 8 <= 64 && 64 % (ROWS / 8) == 0), "a 1 KB group of a row-contiguous tile covers whole k-rows");
    const bf16_t* base;
    uint32_t off[WIDE ? 1 : GROUPS];
    const bf16_t* ptr[WIDE ? GROUPS : 1];
    __device__ __forceinline__ void place(int g, int line, int64_t ld, int at) {
        if constexpr (WIDE) ptr[g] = base + (line * ld + at);
        else off[g] = ((uint32_t)line * (uint32_t)ld + at) * 2;
    }
    // (re)compute the lane addresses for the tile starting at row0, k range starting at k0
    __device__ __forceinline__ void seek(const G3Operand<KC>& op, int row0, int k0, int wave, int lane) {
        base = op.p + (KC ? (int64_t)row0 * op.ld + k0 : (int64_t)k0 * op.ld + row0);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int grp = wave + g * NW;
            if constexpr (KC) {
                // LDS tile [ROWS][BK]; a group is 1 KB of consecutive rows; the 16-byte chunk at (r, p) holds global
                // chunk p ^ s(r) of row r, s(r) = (r >> 1) & 7 for BK = 64 (8 chunks per row), (r >> 2) & 3 for BK = 32
                constexpr int CPR = BK / 8;   // chunks per row
                const int r = grp * (64 / CPR) + lane / CPR;
                const int c = (lane % CPR) ^ (BK == 64 ? ((r >> 1) & 7) : ((r >> 2) & 3));
                place(g, min(r, op.rows - 1 - row0), op.ld, c * 8);
            } else {
                // LDS tile [BK][ROWS]; the chunk at (k, p) holds rows 8 * (p ^ ((k & 3) << 2)) .. + 7 of k
                constexpr int CPR = ROWS / 8;  // chunks per k-row
                const int k = grp * (64 / CPR) + lane / CPR;
                const int c = (lane % CPR) ^ ((k & 3) << 2);
                place(g, k, op.ld, min(c * 8, op.rows - 8 - row0));
            }
        }
    }
    // copy one of this wave's groups of the current k-tile (every one exactly once, in any order) into the tile whose LDS starts `wave` KB before `dst`
    template <int G> __device__ __forceinline__ void issue_group(lds_t dst) const {
        if constexpr (WIDE) copy16_to_lds(ptr[G], dst + G * NW * 1024);
        else copy16_to_lds<G * NW * 1024>(base, off[G], dst);
    }
    // step to the next k-tile
    __device__ __forceinline__ void next(int64_t ld) {
        if constexpr (WIDE) {
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) ptr[g] += KC ? BK : BK * ld;
        } else base += KC ? BK : BK * ld;
    }
    // the current k-tile is a unit's last and has `left` k (fewer than BK): zeros take the place of those behind its end, which are not read
    __device__ __forceinline__ void cut(int wave, int lane, int left) {
        static_assert(!KC && WIDE, "k-rows are whole lanes of a row-contiguous tile only");
        constexpr int CPR = ROWS / 8;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
            if ((wave + g * NW) * (64 / CPR) + lane / CPR >= left) ptr[g] = reinterpret_cast<const bf16_t*>(g3_zeros);
    }
};

// Fragment reader of one operand for a wave whose first row in the tile is wrow0: T fragments of 32 rows.
template <int ROWS, int BK, int T, bool KC> struct G3Frags {
    static constexpr int KK = BK / 16;
    int at[KC ? KK : T];   // byte offsets in a tile that depend on the lane, of a multiply step (KC) or of a fragment
    __device__ __forceinline__ void init(int wrow0, int lane) {
        if constexpr (KC) {
            // s(row) of row = wrow0 + 32 i + lane % 32 depends on the lane only
            const int half = lane >> 5, swz = BK == 64 ? ((lane >> 1) & 7) : ((lane >> 2) & 3);
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) at[kk] = (wrow0 + (lane & 31)) * (BK * 2) + (((kk * 2 + half) ^ swz) << 4);
        } else {
            // transpose read: lane supplies 4 consecutive rows (8 bytes) at k = 16 kk + 8 half + (lane % 16) / 4,
            // rows rb + 16 ((lane / 16) % 2) + 4 (lane % 4); a second read 4 k further completes the 8 k of a lane
            const int kl = (lane >> 5) * 8 + ((lane & 15) >> 2);
            const int sw = ((lane >> 2) & 3) << 2;   // (k & 3) << 2
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const int col = wrow0 + 32 * i + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
                at[i] = kl * (ROWS * 2) + (((col >> 3) ^ sw) << 4) + (col & 7) * 2;
            }
        }
    }
    __device__ __forceinline__ bf16x8_t read(lds_t tile, int i, int kk) const {
        if constexpr (KC) {
            return *lds_ptr<const bf16x8_t>(tile + at[kk] + i * (32 * BK * 2));
        } else {
            const lds_t p = tile + at[i] + kk * 16 * (ROWS * 2);
            union { s16x4_t h[2]; bf16x8_t v; } u;
            u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(p));
            u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_ptr<s16x4_t>(p + 4 * (ROWS * 2)));
            return u.v;
        }
    }
};

// Work geometry, computed on the host.
struct G3Plan {
    int tiles_m, tiles_n, slices, k_per_slice;  // k_per_slice a multiple of the kernel's BK
    int units;                                  // tiles_m * tiles_n * slices
    int col_major;                              // consecutive units walk down a column of tiles (share B) instead of along a row (share A)
    FastDiv d_tn, d_tiles;                      // by tiles_n (tiles_m when col_major) and by tiles_m * tiles_n
    // gm > 0: the tiles of a slice are numbered block by block, a block being gm x gn tiles (gm * gn = 32, the
    // workgroups of one XCD in a round; gm divides tiles_m, gn divides tiles_n): the 32 tiles an XCD works on at a time
    // then share gm + gn operand panels instead of 1 + 32, and most LDS fills find their lines in the XCD's L2.
    int gm, gn;
    FastDiv d_blk, d_gn, d_nbn;                 // by 32, by gn, by tiles_n / gn
};

// One work unit as the kernel walks it: the first row and column of its tile, its k range and what its epilogue needs to know.
struct G3Unit {
    int m0, n0, k0, nk;   // nk: k-tiles of BK
    int last;             // k of the last one (kRagged: BK or fewer)
    int z, job, part_tile;   // k-slice; which contraction of a group and which of its cut tiles
    bool first_col;       // a tile of the first column of tiles
};

// The units of one contraction.
template <int BM, int BN, int BK, bool AKC, bool BKC, class Epi_, bool WIDE> struct G3One {
    typedef Epi_ Epi;
    static constexpr bool kTotals = false, kRagged = false, kWide = WIDE;
    G3Operand<AKC> A;
    G3Operand<BKC> B;
    Epi_ e;
    int rows, cols, k_total;
    G3Plan plan;
    __device__ __forceinline__ int units() const { return plan.units; }
    __device__ __forceinline__ G3Unit unit(int u) const {
        uint32_t zz, rem, m_, n_;
        plan.d_tiles.divmod((uint32_t)u, zz, rem);
        if (plan.gm) {
            uint32_t blk, w, bm, bn, i, j;
            plan.d_blk.divmod(rem, blk, w);
            plan.d_nbn.divmod(blk, bm, bn);
            plan.d_gn.divmod(w, i, j);
            m_ = bm * plan.gm + i;
            n_ = bn * plan.gn + j;
        } else if (plan.col_major) plan.d_tn.divmod(rem, n_, m_);
        else plan.d_tn.divmod(rem, m_, n_);
        const int z = (int)zz, k0 = z * plan.k_per_slice, k1 = min(k_total, k0 + plan.k_per_slice);
        return G3Unit{(int)m_ * BM, (int)n_ * BN, k0, (k1 - k0) / BK, BK, z, 0, 0, n_ == 0};
    }
    __device__ __forceinline__ const G3Operand<AKC>& a(const G3Unit&) const { return A; }
    __device__ __forceinline__ const G3Operand<BKC>& b(const G3Unit&) const { return B; }
    __device__ __forceinline__ const Epi_& epi(const G3Unit&) const { return e; }
    __device__ __forceinline__ int M(const G3Unit&) const { return rows; }
    __device__ __forceinline__ int N(const G3Unit&) const { return cols; }
};

// ROWSUM: units of the first tile column also sum A over k (bias gradient of a weight-gradient GEMM, whose
// A operand is dY, row-contiguous), from the fragments in registers; the sums go to epi.rowsum(m, v, slice).
template <int BM, int BN, int BK, int WM, int WN, int NS, bool AKC, bool BKC, bool ROWSUM, class Work>
__device__ __forceinline__ void gemm3_walk(const Work& work) {
    constexpr int NW = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int KK = BK / 16;
    constexpr int A_BYTES = BM * BK * 2, STAGE = (BM + BN) * BK * 2;
    typedef G3Loader<BM, BK, NW, AKC, Work::kWide> LoaderA;
    typedef G3Loader<BN, BK, NW, BKC, Work::kWide> LoaderB;
    constexpr int G = LoaderA::GROUPS + LoaderB::GROUPS;   // copy instructions per wave and k-tile
    static_assert((NS - 1) * G <= 63, "too many copies in flight for the vmcnt counter");
    static_assert(!ROWSUM || !AKC, "row sums are built for a row-contiguous A");
    static_assert(TN % 2 == 0, "results are staged 16 x 64 at a time");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
    const lds_t smem = (lds_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem_raw;

    const int tid = threadIdx.x, lane = tid & 63;
    // (the wave's index as a scalar: what derives from it — LDS addresses of its copies, its place in the tile — then
    // lives in scalar registers and is computed by the scalar unit)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int grid = gridDim.x;
    // Workgroups are handed to the 8 XCDs (each with its own L2) round-robin in launch order.  Renumber them so that
    // the workgroups of one XCD take CONSECUTIVE units of every round: consecutive units are tiles of one row and
    // slice, which share their A panel (and all of them the few B panels), so an XCD fetches a panel once instead
    // of every XCD fetching every panel.
    int vb = blockIdx.x;
    {
        const int xcd = vb & 7, idx = vb >> 3, q = grid >> 3, r = grid & 7;
        vb = xcd * q + min(xcd, r) + idx;
    }

    // ---- copy cursor: runs NS-1 k-tiles ahead of the multiply cursor ----
    LoaderA la;
    LoaderB lb;
    const int units = work.units();
    int iu = vb, ikt = 0, ink = 0, istage = 0, ilast = BK;
    int64_t ild_a = 0, ild_b = 0;   // leading dimensions of the cursor's operands
    int left = 0;                   // k-tiles that are still to be copied
    for (int u = vb; u < units; u += grid) left += work.unit(u).nk;
    auto seek_unit = [&]() {
        if (iu < units) {
            const G3Unit t = work.unit(iu);
            const auto& A = work.a(t);
            const auto& B = work.b(t);
            ink = t.nk;
            ilast = t.last;
            ild_a = A.ld;
            ild_b = B.ld;
            la.seek(A, t.m0, t.k0, wave, lane);
            lb.seek(B, t.n0, t.k0, wave, lane);
        }
        ikt = 0;
    };
    auto cut_last = [&]() {
        if constexpr (Work::kRagged) {
            if (ikt + 1 == ink && ilast < BK) {
                la.cut(wave, lane, ilast);
                lb.cut(wave, lane, ilast);
            }
        }
    };
    // copy group g (of G) of the cursor's k-tile into stage `istage`
    auto issue_group = [&](auto group) {
        constexpr int g = decltype(group)::value;
        const lds_t st = smem + istage * STAGE + wave * 1024;
        if constexpr (g < LoaderA::GROUPS) la.template issue_group<g>(st);
        else lb.template issue_group<g - LoaderA::GROUPS>(st + A_BYTES);
    };
    // all G groups of the cursor's k-tile are issued: step the cursor
    auto advance = [&]() {
        istage = istage + 1 == NS ? 0 : istage + 1;
        --left;
        la.next(ild_a);
        lb.next(ild_b);
        if (++ikt == ink) {
            iu += grid;
            seek_unit();
        }
        cut_last();
    };
    // copy the cursor's whole k-tile (if any is left); returns false when all is issued
    auto issue_next = [&]() -> bool {
        if (left <= 0) return false;
        static_for<G>([&](auto g) { issue_group(g); });
        advance();
        return true;
    };

    G3Frags<BM, BK, TM, AKC> fa;
    G3Frags<BN, BK, TN, BKC> fb;
    fa.init(wm * (BM / WM), lane);
    fb.init(wn * (BN / WN), lane);

    seek_unit();
    cut_last();
    int ahead = 0;   // k-tiles issued beyond the one being multiplied
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (issue_next()) ++ahead;
    if (ahead == 0) return;   // no unit for this workgroup (uniform)
    --ahead;
    // Fragments are fetched PD multiply steps (of 16 k) ahead of their use.  With two waves per SIMD one step is
    // enough: the other wave's multiplies cover a wave's LDS latency.  With one wave per SIMD (the 4-wave instances)
    // a fragment requested during a step of TM * TN multiplies has not arrived when the next step starts, so these
    // run two steps ahead, with four sets of fragment registers.
    constexpr int PD = NW <= 4 ? 2 : 1, NBUF = PD == 2 ? 4 : 2;
    static_assert(PD < KK && KK % NBUF == 0, "the fragment sets rotate once per k-tile");
    bf16x8_t af[NBUF][TM], bfr[NBUF][TN];
    // Weight gradients keep a unit's last k-tile apart and refill its stage behind the results: with two sets of sums the registers that it would take to walk on
    // are moved back and forth in every k-tile (ragged rows: 418 moves instead of 256; a stage of two blocks of 512 features over 3996 rows 1065 us instead of 1005).
    constexpr bool PEEL = ROWSUM;
    int cstage = 0;
    for (int cu = vb; cu < units; cu += grid) {
        const G3Unit cur = work.unit(cu);
        const int nk = cur.nk, m0 = cur.m0, n0 = cur.n0, z = cur.z;
        const auto& epi = work.epi(cur);
        const int M = work.M(cur), N = work.N(cur);
        f32x16_t acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
        // ROWSUM: in units of the first tile column the waves add up the A fragments they multiply with anyway (a lane
        // holds 8 consecutive k of one row: four two-element dot products with ones).  The WN waves of a wave row hold
        // the same fragments: wave column c takes the fragments i with i % WN == c, so that no wave falls behind.
        float rs[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) rs[i] = 0.0f;
        const bool sum_rows = ROWSUM && cur.first_col;
        // kTotals: every `chain` k-tiles an accumulator is added to a second sum and starts again at zero, so that no sum takes a rounding for every
        // multiply of a long contraction.  A row of accumulators at a time, in the first step of a k-tile, in front of its multiplies.
        constexpr bool TOT = Work::kTotals;
        f32x16_t tot[TOT ? TM : 1][TOT ? TN : 1];
        float rs_tot[TOT ? TM : 1];
        int chain = 1;
        if constexpr (TOT) {
            chain = work.chain;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                rs_tot[i] = 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) tot[i][j][r] = 0.0f;
            }
        }
        auto add_to_totals = [&](int i) {
            if constexpr (TOT) {
                rs_tot[i] += rs[i];
                rs[i] = 0.0f;
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; r += 4) {
                        // Written out so that the accumulators stay in accumulation registers: left to itself the compiler moves all of them
                        // back and forth in every k-tile.  (The multiplies that wrote them lie six multiplies back; a multiply that reads
                        // them may follow two instructions behind.)
                        float v[4], a[4] = {acc[i][j][r], acc[i][j][r + 1], acc[i][j][r + 2], acc[i][j][r + 3]};
                        asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7\n\t"
                                     "v_accvgpr_write_b32 %4, 0\n\tv_accvgpr_write_b32 %5, 0\n\tv_accvgpr_write_b32 %6, 0\n\tv_accvgpr_write_b32 %7, 0\n\t"
                                     "s_nop 1"
                                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "+a"(a[0]), "+a"(a[1]), "+a"(a[2]), "+a"(a[3]));
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            tot[i][j][r + q] += v[q];
                            acc[i][j][r + q] = a[q];
                        }
                    }
            }
        };

        // What the epilogue reads from memory (a bias per column, a residual source or a mask per element), block by
        // block of 32 rows x 64 columns of this wave's results (block b: rows 32 (b / (TN / 2)), columns 64 (b % (TN / 2))).  Places outside the
        // matrix read the last ones inside it: a load under a lane's condition is a branch each.
        constexpr int NB = TM * (TN / 2);
        const int64_t epi_ld = epi.ld;
        typename Work::Epi::Col8 pcol[TN / 2];
        typename Work::Epi::Row8 prow[NB][4];
        // (ln: the lane's index as the caller has it; see the epilogue)
        auto epi_n = [&](int jp, int ln) { return n0 + wn * (BN / WN) + jp * 64 + (ln & 7) * 8; };
        constexpr bool FORMED = Work::Epi::kFormed, ROWS = !std::is_empty<typename Work::Epi::Row8>::value;
        const int mw = m0 + wm * (BM / WM), mr = min(mw, M - 1);   // the wave's first row, and where its requests start
        auto epi_request = [&](int b, int ln) {
            const int i = b / (TN / 2), jp = b % (TN / 2), n = min(epi_n(jp, ln), N - 8);
            if (i == 0) pcol[jp] = epi.col8(n);
            if constexpr (ROWS) {
#pragma unroll
                for (int sp = 0; sp < 4; ++sp) {
                    const int r = min(i * 32 + sp * 8 + (ln >> 3), M - 1 - mr);
                    if constexpr (FORMED) prow[b][sp] = epi.row8f((int64_t)mr * epi_ld, __umul24((uint32_t)r, (uint32_t)epi_ld) + n);
                    else prow[b][sp] = epi.row8((int64_t)(mr + r) * epi_ld + n, true);
                }
            }
        };
        // With registers to spare (the 4-wave instances: 512 per lane) all of it is requested before the k-loop; the
        // 8-wave instances, which would spill, request a block's data while they work on the block before.  A wave waits for
        // its requests in issue order, stores included: waiting for data requested after a store means waiting for the
        // store to be acknowledged.
        constexpr bool EARLY = NW <= 4;
        // (a block at a time where the columns' data is more than a bias: 24 registers of gains, shifts and biases leave none for two blocks' rows; and where the
        // general epilogue has 8 registers of a row)
        constexpr bool AHEAD = !EARLY && sizeof(typename Work::Epi::Col8) <= 32 && (Work::Epi::kFormed || sizeof(typename Work::Epi::Row8) < 32);
        // k-tiles whose next one has landed: the copies that were waited for before the last unit's first store are those of NS k-tiles (one fewer with PEEL)
        const int quiet = cu == vb ? 0 : PEEL ? NS - 2 : NS - 1;
        if (cu == vb) {
            // The workgroup's first k-tile: wait for it and make it visible to all waves.  (Here, so that what stands above, which needs none of it, is
            // done while it is on its way.)
            if (ahead == NS - 1) wait_vmcnt<(NS - 1) * G>();
            else wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        // The unit's first fragments.  (Its first k-tile is there since the barrier of the last unit's last one; requested then already and kept, they would
        // take registers that the results need on their way out.  Without PEEL that k-tile requests them all the same, as every k-tile does the next one's, and they
        // are dropped: of a unit of 12 k-tiles 2 % of the LDS reads with eight waves and 4 % with four.)
        {
            const lds_t sa = smem + cstage * STAGE;
#pragma unroll
            for (int p = 0; p < PD; ++p) {
#pragma unroll
                for (int i = 0; i < TM; ++i) af[p][i] = fa.read(sa, i, p);
#pragma unroll
                for (int j = 0; j < TN; ++j) bfr[p][j] = fb.read(sa + A_BYTES, j, p);
            }
        }
        if constexpr (EARLY) {
#pragma unroll
            for (int b = 0; b < NB; ++b) epi_request(b, lane);
        }

        // One k-tile.  Invariant: the fragments of its first PD multiply steps are in registers or on their way (requested during the previous
        // k-tile's last PD steps); `ahead` younger k-tiles are in flight or have landed.  last: the unit's last one, if that is a form of its own (PEEL),
        // which requests no fragments for a next.
        //
        // fill: after the barrier its stage is free and refilled at once, the copies spread over the multiplies that follow the barrier, unless all is
        // copied.  The two forms are loops of their own, and the
        // one that is walked nearly always has no branch in it: with a wave or two to a SIMD every branch, every address that is put together and every
        // pointer that is stepped between two multiplies delays the next one.  256 x 128 tiles, four waves: 1830 cycles a k-tile with a test before
        // each copy and its address in 64-bit registers, 1500 as it is (multiplies 1024); 8192 x 768 over 3072 forward 51 -> 41 us, input gradient 52 -> 43, 8192^3 in 256 x 256
        // tiles 874 -> 807 us (with the exchanged operands and the third stage; on another machine 41, 40 and 850 now).
        auto k_tile = [&](int kt, auto fill, auto last) {
            constexpr bool FILL = decltype(fill)::value, LAST = decltype(last)::value;
            // (comments in the instruction stream, by which tests/test_gemm3_isa.py finds the three forms)
            if constexpr (FILL) asm volatile("; tmps k-tile begin");
            else if constexpr (LAST) asm volatile("; tmps last k-tile begin");
            else asm volatile("; tmps draining k-tile begin");
            const lds_t sa = smem + cstage * STAGE;
            const int nstage = cstage + 1 == NS ? 0 : cstage + 1;
            const lds_t sn = smem + nstage * STAGE;
            static_for<KK>([&](auto step) {
                constexpr int kk = decltype(step)::value;
                constexpr int nx = kk + PD;   // the step whose fragments are requested during this one
                if constexpr (nx == KK) {
                    // Every fragment of this k-tile has been requested.  The next k-tile is the oldest copy in
                    // flight: copies complete in issue order, so it has landed once at most (ahead - 1) * G younger
                    // copies are outstanding.  While the pipeline drains (ahead < NS - 1) wait for everything.
                    // A unit's first `quiet` k-tiles wait for nothing: what comes next was waited for in front of the last unit's first store.  The k-tile that is
                    // waited for first was copied behind those stores, so this wait is for them as well; they have had `quiet` k-tiles to drain in.
                    if (kt >= quiet) {
                        if (FILL || ahead == NS - 1) wait_vmcnt<(NS - 2) * G>();
                        else wait_vmcnt<0>();
                    }
                    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's reads of the current stage are done
                    __builtin_amdgcn_s_barrier();
                    // All waves are past their last read of the current stage, and the next k-tile is visible to all:
                    // its first fragments are fetched under the cover of the remaining multiply steps.
                }
                // This step in program order, kept by the scheduling barriers: before multiply g, the g-th share of
                // the fragment requests of step nx and, after the barrier, of the copies: a wave has one instruction
                // stream, and what it issues between two multiplies costs nothing while the matrix unit is busy.
                const lds_t ra = nx < KK ? sa : sn;
                constexpr int rk = nx < KK ? nx : nx - KK;
                constexpr int NM = TM * TN, NR = TM + TN, CPS = G / PD;
                static_assert(G % PD == 0, "the copies of a k-tile are spread evenly over the steps after the barrier");
                static_for<NM>([&](auto multiply) {
                    constexpr int g = decltype(multiply)::value;
#pragma unroll
                    for (int r = g * NR / NM; r < (g + 1) * NR / NM; ++r) {
                        if (LAST && nx >= KK) continue;
                        if (r < TM) af[nx % NBUF][r] = fa.read(ra, r, rk);
                        else bfr[nx % NBUF][r - TM] = fb.read(ra + A_BYTES, r - TM, rk);
                    }
                    if constexpr (FILL && nx >= KK) {
                        constexpr int c0 = g * CPS / NM, c1 = (g + 1) * CPS / NM;
                        static_for<c1 - c0>([&](auto c) { issue_group(std::integral_constant<int, (nx - KK) * CPS + c0 + decltype(c)::value>{}); });
                    }
                    if constexpr (TOT && kk == 0 && g % TN == 0) {
                        if (((kt - (g / TN) * chain / TM) & (chain - 1)) == 0) add_to_totals(g / TN);
                    }
                    // (B's fragment first: the block comes out transposed, four consecutive columns of a row in a lane's registers; see the results)
                    acc[g / TN][g % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk % NBUF][g % TN], af[kk % NBUF][g / TN], acc[g / TN][g % TN], 0, 0, 0);
                    if constexpr (ROWSUM && g % TN == 0) {
                        // Behind the fragment's first multiply, so that it is issued while that one runs; written as
                        // instructions because the compiler otherwise turns the branch into selects and moves the
                        // additions, which nothing in the loop depends on, below the multiplies of the k-tile.
                        if (sum_rows && (g / TN) % WN == wn) {
                            typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
                            const u32x4_t f = __builtin_bit_cast(u32x4_t, af[kk % NBUF][g / TN]);
#pragma unroll
                            for (int q = 0; q < 4; ++q)   // rs += f[q].lo * 1 + f[q].hi * 1 (0x3f80 = 1.0 in bf16)
                                asm volatile("v_dot2c_f32_bf16_e32 %0, 0x3f803f80, %1" : "+v"(rs[g / TN]) : "v"(f[q]));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            if constexpr (FILL) advance();
            else if (ahead > 0) --ahead;
            cstage = nstage;
            if constexpr (FILL) asm volatile("; tmps k-tile end");
            else if constexpr (LAST) asm volatile("; tmps last k-tile end");
            else asm volatile("; tmps draining k-tile end");
        };
        const int filled = min(PEEL ? nk - 1 : nk, left);
        int kt = 0;
        for (; kt < filled; ++kt) k_tile(kt, std::true_type{}, std::false_type{});
        for (; kt < (PEEL ? nk - 1 : nk); ++kt) k_tile(kt, std::false_type{}, std::false_type{});
        if constexpr (PEEL) k_tile(kt, std::false_type{}, std::true_type{});
        if constexpr (TOT) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                rs[i] += rs_tot[i];
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[i][j][r] += tot[i][j][r];
            }
        }

        // ---- results ----
        // Each wave passes its accumulators through 4 KB of LDS of its own, one half of a block at a time (16 rows x 64 columns of fp32), and leaves with 8
        // consecutive columns of one row per lane: a store instruction then writes 8 rows of 128 (bf16) or 256 (fp32) consecutive bytes.  A half's
        // 16-byte chunks lie at an XOR of their row, so that neither side's accesses meet in a bank.
        {
            // Everything the epilogue derives from the lane's index is derived here, from a copy of the index that the
            // compiler cannot trace back: otherwise it computes these offsets before the k-loop and, in the 8-wave
            // instances, whose loop leaves no register free, spills them around it — and every reload from scratch
            // memory is a wait for all of the wave's requests, result stores included.
            int ln = lane;
            asm volatile("" : "+v"(ln));
            // staged row r (of 16) takes 256 bytes; chunk c (4 columns) lies at c ^ r
            const lds_t stg = smem + NS * STAGE + wave * kG3StageOut;
            lds_t put = stg + (ln & 15) * 256 + (((ln >> 5) ^ (ln & 15)) << 4);
            lds_t get = stg + (ln >> 3) * 256 + (((2 * (ln & 7)) ^ (ln >> 3)) << 4);
            typedef float f32x4_t __attribute__((ext_vector_type(4)));
            // half h (16 rows) of block b through LDS.  (A wave's LDS instructions take effect in order.)
            auto stage = [&](int b, int h) {
                const int i = b / (TN / 2), jp = b % (TN / 2);
                // accumulator register r of a lane: row lane % 32, column 8 (r / 4) + 4 (lane / 32) + r % 4
                if (((ln >> 4) & 1) == h) {
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x16_t& v = acc[i][2 * jp + jj];
                            *lds_ptr<f32x4_t>(put ^ ((jj * 8 + q * 2) << 4)) = f32x4_t{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                        }
                }
                asm volatile("" ::: "memory");
            };
            auto fetch = [&](float (&v)[2][8]) {
#pragma unroll
                for (int sp = 0; sp < 2; ++sp) {
                    // staged row 8 sp + lane / 8, chunks 2 (lane % 8) and the next
                    const lds_t src = (get ^ (sp << 7)) + sp * 2048;
                    const f32x4_t lo = *lds_ptr<const f32x4_t>(src), hi = *lds_ptr<const f32x4_t>(src ^ 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[sp][e] = lo[e];
                        v[sp][4 + e] = hi[e];
                    }
                }
                asm volatile("" ::: "memory");
            };
            if constexpr (EARLY) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (b < TN / 2) settle(pcol[b]);
                    if constexpr (ROWS) {
#pragma unroll
                        for (int sp = 0; sp < 4; ++sp) settle(prow[b][sp]);
                    }
                }
            } else if constexpr (AHEAD) epi_request(0, ln);
            // The half in work and, where registers allow, the next one, on its way through LDS meanwhile (8-wave instances that ask for everything have none left).
            constexpr bool NEXT = EARLY || FORMED;
            float v[2][2][8];
            if constexpr (NEXT) {
                stage(0, 0);
                fetch(v[0]);
            }
            const uint32_t off = (uint32_t)(ln >> 3) * (uint32_t)epi_ld + (ln & 7) * 8;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int i = b / (TN / 2), jp = b % (TN / 2);
                const int n = epi_n(jp, ln);
                if constexpr (!EARLY) {
                    // the block's data before the next block's requests and its own first store
                    if constexpr (!AHEAD) epi_request(b, ln);
                    if (i == 0) settle(pcol[jp]);
                    if constexpr (ROWS) {
#pragma unroll
                        for (int sp = 0; sp < 4; ++sp) settle(prow[b][sp]);
                    }
                }
                if (b == 0) wait_vmcnt<0>();
                if constexpr (AHEAD) {
                    if (b + 1 < NB) epi_request(b + 1, ln);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if constexpr (!NEXT) {
                        stage(b, h);
                        fetch(v[h]);
                    } else if (2 * b + h + 1 < 2 * NB) {
                        stage(b + (h == 1), 1 - h);
                        fetch(v[1 - h]);
                    }
#pragma unroll
                    for (int sp = 0; sp < 2; ++sp) {
                        const int row = i * 32 + h * 16 + sp * 8;   // of the wave's
                        const int m = mw + row + (ln >> 3);
                        if (m < M && n < N) {   // N is a multiple of 8
                            if constexpr (FORMED) epi.at8f(pcol[jp], prow[b][2 * h + sp], (int64_t)(mw + row) * epi_ld + (n0 + wn * (BN / WN) + jp * 64), off, v[h][sp], z);
                            else epi.at8(pcol[jp], prow[b][2 * h + sp], (int64_t)m * epi_ld + n, v[h][sp], z);
                        }
                    }
                }
            }
        }
        if constexpr (ROWSUM) {
            if (sum_rows) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    if (i % WN != wn) continue;
                    // lanes l and l + 32 hold the two halves of every 16 k of row 32 i + l % 32
                    const float total = rs[i] + __shfl_xor(rs[i], 32, 64);
                    const int m = m0 + wm * (BM / WM) + i * 32 + (lane & 31);
                    if (lane < 32 && m < M) epi.rowsum(m, total, z);
                }
            }
        }
        if constexpr (PEEL) {
            if (issue_next()) ++ahead;
        }
    }
}

template <int BM, int BN, int BK, int WM, int WN, int NS, bool AKC, bool BKC, bool ROWSUM, bool WIDE, class Epi>
__global__ __launch_bounds__(64 * WM * WN) void gemm3_kernel(G3Operand<AKC> A, G3Operand<BKC> B, Epi epi, int M, int N,
                                                              int K, G3Plan plan) {
    const G3One<BM, BN, BK, AKC, BKC, Epi, WIDE> work{A, B, epi, M, N, K, plan};
    gemm3_walk<BM, BN, BK, WM, WN, NS, AKC, BKC, ROWSUM>(work);
}

// ---- several weight gradients in one launch ----------------------------------------------------------------------------
// The weight gradients of a stage's dense layers contract over the same rows and depend on nothing but stored activations and
// gradients, so they can be one launch at the end of the backward pass.  A single one has too few tiles for the device (36 of 256 x 256 for
// 3072 x 768) and runs in k-slices, whose fp32 partial sums cost as much as a third of its multiplies to write and add
// up.  Together their tiles are walked in whole rounds of the device with no slices at all; only the tiles beyond the last whole round are cut
// along k, into as many slices as fill a round, and summed by g3_group_sum_kernel.
//
// Precision: a sum that is added to once per multiply (16 rows) is, after n of them, 2^-24 sqrt(n / 6) (2-norm) from the sum in 64 bits: 5.7e-7 over
// 8192 rows in one chain.  The slices of the launches this one replaces were chains of some 1000 rows (1.5 to 2.1e-7), so it has a second set of sums
// (see kTotals): with chains of 2, 4 and 8 k-tiles below 1024, below 4096 and from 4096 rows on its errors are 0.7, 0.9, 1.0, 1.4, 1.5 and 1.6e-7 over 512,
// 1024, .. 16384 rows, those of the layers' own launches 0.9, 1.3, 1.3 to 1.9, 1.9 to 2.7, 1.5 to 2.1 and 2.1 to 3.0e-7.  Two sets fit where there is one
// wave to a SIMD: 256 x 128 tiles, four waves of 128 x 64, three stages (two: 8 % slower, the copies of a k-tile then have less than one to
// arrive in).  Against 256 x 256 tiles with eight waves and one set that is 6 % for the totals and 16 % for copies and transposed reads, which LDS serves for half as
// many multiplies: 12 layers of 768 features over 8192 rows 450 us instead of 356.  Totals in memory instead were estimated at the same.
//
// The four layers of a transformer block of 768 features over 8192 / 1024 rows, one block, two, three, four (us, launches of their own and one):
// 192 and 142, 394 and 309, 595 and 448, 792 and 590 / 55 and 31, 109 and 54, 161 and 78, 215 and 107; 20 of 1024 x 1024 over 1024 rows 218 and 82.
constexpr int kG3GroupMax = 32;   // contractions of a launch (kernel arguments hold 4 KB)
struct G3Job {
    const bf16_t* a;   // dY [K][M]
    const bf16_t* b;   // X [K][N]
    float* out;        // [M][N], then M row sums
    int M, N, first_tile, col_major;
    FastDiv d_minor;   // by the tiles along the direction walked first
};
struct G3Group {
    typedef EpiForm<EpiWgrad, 0> Epi;
    static constexpr bool kTotals = true, kRagged = false, kWide = false;
    static constexpr int kRows = 256, kCols = 128, kPart = kRows * kCols + kRows;   // a tile; floats of a partial one: results, then row sums
    G3Job job[kG3GroupMax];
    int jobs, k_total, tiles, whole;   // tiles of all jobs; the first `whole` of them are not sliced
    int slices, k_per_slice;           // of the others
    int chain;                         // k-tiles summed in one go, a power of two
    float* part;                       // [tiles - whole][slices][kPart]
    FastDiv d_cut;                     // by tiles - whole

    __device__ __forceinline__ int units() const { return whole + (tiles - whole) * slices; }
    // job and coordinates of a tile
    __device__ __forceinline__ int place(int t, int& m0, int& n0) const {
        int j = 0;
        while (j + 1 < jobs && t >= job[j + 1].first_tile) ++j;
        uint32_t major, minor;
        job[j].d_minor.divmod((uint32_t)(t - job[j].first_tile), major, minor);
        m0 = (int)(job[j].col_major ? minor : major) * kRows;
        n0 = (int)(job[j].col_major ? major : minor) * kCols;
        return j;
    }
    __device__ __forceinline__ G3Unit unit(int u) const {
        G3Unit g;
        int t = u;
        g.z = -1;   // (not sliced)
        g.k0 = 0;
        int k1 = k_total;
        if (u >= whole) {
            uint32_t z, r;
            d_cut.divmod((uint32_t)(u - whole), z, r);
            t = whole + (int)r;
            g.z = (int)z;
            g.k0 = g.z * k_per_slice;
            k1 = min(k_total, g.k0 + k_per_slice);
        }
        g.nk = (k1 - g.k0) >> 6;
        g.last = 64;
        g.job = place(t, g.m0, g.n0);
        g.first_col = g.n0 == 0;
        g.part_tile = t - whole;
        return g;
    }
    __device__ __forceinline__ G3Operand<false> a(const G3Unit& g) const { return G3Operand<false>{job[g.job].a, job[g.job].M, job[g.job].M}; }
    __device__ __forceinline__ G3Operand<false> b(const G3Unit& g) const { return G3Operand<false>{job[g.job].b, job[g.job].N, job[g.job].N}; }
    __device__ __forceinline__ int M(const G3Unit& g) const { return job[g.job].M; }
    __device__ __forceinline__ int N(const G3Unit& g) const { return job[g.job].N; }
    // (addressed as the whole matrix is: a partial tile's base lies as far in front of it as the tile's first element lies inside the matrix)
    __device__ __forceinline__ Epi epi(const G3Unit& g) const {
        const G3Job& j = job[g.job];
        if (g.z < 0) return Epi{EpiWgrad{j.out, j.N, (int64_t)j.M * j.N, 0}};
        const int64_t first = (int64_t)g.m0 * kCols + g.n0;
        return Epi{EpiWgrad{part + ((int64_t)g.part_tile * slices + g.z) * kPart - first, kCols, first + kRows * kCols - g.m0, 0}};
    }
};
// Over rows that are no multiple of 64: the last k-tile of the last slice is short.  An instance and a way to a unit of its own, so that its tests are paid only where rows
// need them (with a short last k-tile in the common unit() the whole rows' instance took 447 us for three GPT-2 blocks, 437 without).  In launches of their own such gradients ran on 64 x 64 tiles: eight of a stage with two blocks of 512
// features over 3996 rows 156 us, the stage 1127 us and 1087 with one launch; four blocks of 768 over two stages with 1266 rows, two mini-batches, 2570 and
// 2399; four blocks of 640 in 1F1B order, 1564 rows a pass, 9 % of a run; one mini-batch of three blocks of 768 over 524 rows 1.5 %.
// Errors of the gradients (2-norm, against 64 bits) of a block's layers in launches of their own and in one: 999 rows, 512 features 1.3 and 0.9e-7, 524 rows, 768 0.9 and
// 0.7e-7, 1564 rows, 640 1.6 and 1.0e-7, 3996 rows, 512 1.9 and 1.1e-7 (the layer of 512 into 512, which had more slices, 1.0 and 1.1e-7), 8100 rows, 768 3.2 and 1.5e-7.
// It also takes rows of any length (kWide).
struct G3GroupRagged : G3Group {
    static constexpr bool kRagged = true, kWide = true;
    __device__ __forceinline__ G3Unit unit(int u) const {
        G3Unit g = G3Group::unit(u);
        const int k = (g.z < 0 ? k_total : min(k_total, g.k0 + k_per_slice)) - g.k0;
        g.nk = (k + 63) >> 6;
        g.last = k - (g.nk - 1) * 64;
        return g;
    }
};

}  // namespace tmps
