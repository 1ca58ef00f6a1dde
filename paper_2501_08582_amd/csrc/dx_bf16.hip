// Backward data gradient with weight recompute, bf16 on gfx950.
//
//   dX[L x C] = dY[L x R] . W',   W' = select(M, W + s.B.A, 0)
//
// (dX step of the SP-LoRA backward list in Section 2.2; the merged weight is
// recomputed instead of stored, Algorithm 2 / Section 2.3.)  GEMM over K = R.
//
// Same structure as the forward: each of the 4 waves owns 64 input features
// (n) of the 256 x 256 tile and rebuilds W'[k][n] for its columns in
// registers, in the B-operand layout of the main MFMA (rank-r MFMA with its
// k rows taken in the order pi, see the forward kernel).  Differences:
//   * W is stored [k][n] (k = R), so the raw W values a lane needs -- eight
//     consecutive k of one column n -- come from two LDS transpose loads; the
//     W slab is four per-wave blocks (the 64 k rows of that wave's 64
//     columns, tr64 layout), each filled by its own wave's copies;
//   * the k-rows of the rank-r product are B[k][:], read from a B slab copied
//     contiguously into LDS each K-step; A[:, n] is resident in registers;
//   * the mask bits a lane needs run along k for a fixed n, so they are read
//     from the transposed bitmap M^T (built once per backward call).
// The schedule is the forward's: four sub-steps of 16 k per K-step, each
// MFMA slot carrying a fixed share of the next sub-step's operand reads and
// merge arithmetic, one barrier per K-step before the last sub-step, which
// interleaves the copies of stage kt+2 and the first sub-step of stage kt+1.
// For a power-of-two scale the merge is folded as in the forward: the
// resident A operand is pre-scaled by s, the rank-r MFMA accumulates onto W
// (read, for the next stage, as soon as the wave's own W copies landed), and
// a merge piece is the rounding and the select.
// Works on ranks that are multiples of 8 (the launcher pads other ranks with a
// zero-filled copy of B); ranks above 64 as half-feature tiles only.
#include "gemm_common.hpp"
#include "kernels.hpp"

#include <cmath>
#include <type_traits>

namespace lors {
namespace {

constexpr int NT = 256;
constexpr int BM = 256;  // tokens per tile
constexpr int BN = 256;  // input features per whole tile (64 per wave)
constexpr int BK = 64;   // output features (rows of W) per K-step
constexpr int GROUP_M = 4;
constexpr int kEarly = 12;  // copies of a stage issued right after the barrier; the rest a sub-step later

// B slab [k][rank]: 64 rows of PITCH = 32*RKP bytes (ranks padded to 16*RKP;
// RKP = RK rounded up to a power of two, so that a row holds a power of two of 16-byte
// chunks).  Chunk q of row k is stored at chunk q ^ bswz(k): the merge reads
// one chunk of 16 consecutive rows per 16 lanes, and with rows 32*RKP bytes
// apart those rows would fall on only 8 / RKP of the 16 bank groups; the XOR
// spreads them over all 16 (a 256-byte bank window holds 8 / RKP rows, and
// bswz takes 2*RKP distinct values over 16 consecutive rows).
// TM: tokens per tile, NF: 32-column blocks per wave -- BM and 2 for a whole
// tile; a thin tile of a short last wave has half the columns (NF = 1) and
// TM = 256, 128 or 64 tokens.
// W slab: 4 per-wave blocks of [64 k][32 NF n]; with NF = 2 a block has
// 128-byte rows in the tr64 layout, with NF = 1 64-byte rows unswizzled (the
// four rows a 32-lane transpose read covers are then 256 consecutive bytes,
// one per bank).
template <int RK, int TM, int NF>
struct Layout {
    static constexpr int FT = 128 * NF;            // input features per tile
    static constexpr int WROW = 64 * NF;           // bytes per row of a wave's W block
    static constexpr int WBW = BK * WROW;          // one wave's W block
    static constexpr int WB = 4 * WBW;             // W slab
    static constexpr int MB = FT * 2 * 4;          // M^T words [n][kb]
    static constexpr int DB = TM * kRow64;         // dY slab: TM rows of 64 k
    static constexpr int RKP = RK == 3 ? 4 : RK > 4 ? 8 : RK;
    static constexpr int PITCH = 32 * RKP;
    static constexpr int BB = BK * PITCH;          // B slab: 2 KiB per 16 ranks
    static constexpr int D = 0, W = DB, B = DB + WB, M = DB + WB + BB;
    static constexpr int STAGE = DB + WB + BB + MB;
    static constexpr int NBC = BB / 1024;          // 1 KiB copies per B slab
    static constexpr int NB = (NBC + 3) / 4;       // B-slab copies per wave
    static constexpr int PAD = NBC % 4 ? 1024 : 0; // target of the B slab's padding copies, where it has any
    static constexpr int S = stages_that_fit(STAGE, 256 + PAD);
    static constexpr int LUT = S * STAGE;          // select table: 16 x 8 B
    static constexpr int SINK = LUT + 256;
    static constexpr int TOTAL = SINK + PAD;
    static constexpr int ND = TM / 32;             // dY-slab copies per wave
    static constexpr int NWC = WBW / 1024;         // W-block copies per wave
    static constexpr int NMC = NF;                 // M^T copies per wave
    static constexpr int COPIES = ND + NWC + NB + NMC;  // copies per wave per stage
    static constexpr int EARLY = COPIES < kEarly ? COPIES : kEarly;
    static constexpr int FLY = (S - 2) * COPIES;  // copies of later stages in flight at a K-step's barrier
    static_assert(COPIES - EARLY <= 8, "the late copies fit the eight merge slots");
    static_assert(FLY + COPIES < 64, "vmcnt range");
    // physical chunk of logical chunk q in B-slab row k
    static __device__ __forceinline__ int bswz(int k, int q) { return q ^ ((k / (8 / RKP)) & (2 * RKP - 1)); }
};

#define SLOT_END() __builtin_amdgcn_sched_barrier(0)

// Copies as in the forward: token rows past L and columns past C are not
// read (their lanes copy the last row or column chunk that exists, and what
// they lead to is never stored), so any L and C take the copies of a uniform
// base plus fixed offsets.  KRAG: the last K-step reaches past R, or the
// offsets exceed 32 bits; every copy then checks its lanes and reads the zero
// page outside the tensors.
// r: the rank the kernel works on, a multiple of 8 (B's columns ra .. r-1
// are zero); ra: the rows of A that exist (A rows ra .. r-1 are read as zero).
// TM, NF < (BM, 2): a thin tile of TM tokens and 128 NF input features, as in
// the forward kernel.
template <int RK, bool KRAG, bool FOLD, int TM, int NF>
__global__ __launch_bounds__(NT, 1) void dx_kernel(
    const uint16_t* __restrict__ dY, const uint16_t* __restrict__ W,
    const uint32_t* __restrict__ Mt, const uint16_t* __restrict__ Bm,
    const uint16_t* __restrict__ Am, uint16_t* __restrict__ dX, int64_t L, int R, int C, int r,
    int ra, float s, int tiles_m, int tiles_n, float* __restrict__ z0, int64_t nz0,
    float* __restrict__ z1, int64_t nz1, int n_full, int split, float* __restrict__ part) {
    using Lay = Layout<RK, TM, NF>;
    constexpr int MBW = TM / 32;  // 32-token blocks per wave
    constexpr int SPAN = thin_span(TM);  // tokens of a logical tile
    static_assert(NF == 1 || RK <= 4, "ranks above 64: half-feature tiles");
    static_assert(Lay::TOTAL <= 160 * 1024, "LDS budget");
    static_assert(4 * TM * 64 * NF <= Lay::S * Lay::STAGE, "output staging fits the stage buffers");
    // the prologue parks the merge's A block in the last PARK stages
    constexpr int PROW = 2 * Lay::FT;
    constexpr int PARK = (16 * RK * PROW + Lay::STAGE - 1) / Lay::STAGE;
    static_assert(PARK < Lay::S, "A block fits beside stage 0");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[Lay::TOTAL];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31;
    const int h = lane >> 5;

    // z0, z1: dB and dA of the combined backward, cleared here for the fp32
    // atomics of the weight-gradient kernel that follows on the same stream
    // (one launch fewer; plain stores, grid-stride)
    if (z0 != nullptr) {
        const int64_t stride = (int64_t)gridDim.x * NT;
        for (int64_t t = (int64_t)blockIdx.x * NT + tid; t < nz0 + nz1; t += stride) {
            if (t < nz0) z0[t] = 0.f;
            else z1[t - nz0] = 0.f;
        }
    }

    // tile and K-steps: ids past n_full are pieces of split tiles (their
    // partial sums go to `part`, see the epilogue).  Thin tiles: the grid
    // covers logical tiles n_full .. n_full+split-1, each cut into SPAN/TM
    // token parts of each of its 2/NF feature parts (see thin_coords), with
    // every K-step.
    int tm, tn;
    int kbeg, nk;
    int64_t m0;
    int n0;
    if constexpr (TM == BM && NF == 2) {
        work_coords(blockIdx.x, tiles_m, tiles_n, GROUP_M, n_full, split, (R + BK - 1) / BK, tm, tn, kbeg, nk);
        m0 = (int64_t)tm * BM;
        n0 = tn * BN;
    } else {
        int u;
        thin_coords(blockIdx.x, tiles_m, tiles_n, GROUP_M, n_full, split, (SPAN / TM) * (2 / NF), tm, tn, u);
        kbeg = 0;
        nk = (R + BK - 1) / BK;
        m0 = (int64_t)tm * SPAN + (int64_t)(u % (SPAN / TM)) * TM;
        n0 = tn * BN + (u / (SPAN / TM)) * Lay::FT;
        if (m0 >= L || n0 >= C) return;  // a part of an edge tile that holds no output
    }
    // last row of the dY slab, last column chunk and last column that exist
    const int lastm = (int)min(L - 1 - m0, (int64_t)(TM - 1));
    const int lastc = C - 8 - n0, lastn = C - 1 - n0;
    const int kofs = kbeg * BK;
    const int wprT = (R + 31) >> 5;  // words per row of M^T
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem));
    const uint8_t* zsrc = (const uint8_t*)g_zero_page + 16 * lane;
    // B-slab copy q of this wave lands at slab byte 1024*(4q + wave) + 16*lane,
    // i.e. row brow[q], physical chunk p; it carries logical chunk
    // bswz(brow, p) -- ranks 8*that .. +7 of B row k0 + brow[q], zeros for
    // ranks at or past r
    int brow[Lay::NB], bcol[Lay::NB];
    bool bval[Lay::NB];
#pragma unroll
    for (int q = 0; q < Lay::NB; ++q) {
        const int blk = 4 * q + wave;
        const int off = 1024 * blk + 16 * lane;
        brow[q] = off / Lay::PITCH;
        const int lq = Lay::bswz(brow[q], (off % Lay::PITCH) / 16);
        bcol[q] = 16 * lq;
        bval[q] = blk < Lay::NBC && 8 * lq < r;
    }

    // M^T is a plain bitmap whatever the caller's layout.
    if (tid < 16) *(u32x2*)(smem + Lay::LUT + 8 * tid) = select_lut16_entry<false>((uint32_t)tid);

    // ---- slab copies.  Copies 0..ND-1: dY slab rows 8*(ND*wave + q) + lane/8
    // (64 k per row); copies ND..ND+NWC-1: this wave's W block, its 32 NF
    // columns (NF = 2: rows 8q + lane/8 in the tr64 layout; NF = 1: rows
    // 16q + lane/4, 16-byte chunk lane % 4); then the B slab and the M^T
    // words.
    uint32_t offD[Lay::ND], offW[Lay::NWC];
#pragma unroll
    for (int q = 0; q < Lay::ND; ++q) {
        const int rd = 8 * (Lay::ND * wave + q) + (lane >> 3);
        offD[q] = (uint32_t)((min(rd, lastm) * R + 8 * ((lane & 7) ^ ((rd >> 1) & 7))) * 2);
    }
#pragma unroll
    for (int q = 0; q < Lay::NWC; ++q) {
        if constexpr (NF == 2) {
            const int rw = 8 * q + (lane >> 3);
            offW[q] = (uint32_t)((rw * C + min(64 * wave + 8 * ((lane & 7) ^ tr64_swz(rw)), lastc)) * 2);
        } else {
            const int rw = 16 * q + (lane >> 2);
            offW[q] = (uint32_t)((rw * C + min(32 * wave + 8 * (lane & 3), lastc)) * 2);
        }
    }
    // M^T words of a K-step: with whole tiles the tile's columns hold them
    // as one contiguous run of 2 words per column (see mt_index), so copy q
    // of a wave moves 256 consecutive bytes of it
    uint32_t offM[Lay::NMC];
#pragma unroll
    for (int q = 0; q < Lay::NMC; ++q) {
        const int e = 64 * (Lay::NMC * wave + q) + lane;
        offM[q] = (uint32_t)((2 * min(e >> 1, lastn) + (e & 1)) * 4);
    }
    const uint16_t* Dt = uniform_ptr(dY + m0 * R);
    const uint16_t* Wn = uniform_ptr(W + n0);
    const uint32_t* Mn = uniform_ptr(Mt + 2 * (int64_t)n0);

    auto copy_j = [&](int j, int k0, uint32_t sb) {
        k0 += kofs;
        if (j < Lay::ND) {
            const int q = j, blk = Lay::ND * wave + q;
            const uint32_t dst = sb + Lay::D + 1024 * blk;
            if constexpr (!KRAG) {
                copy16s_to_lds(uniform_ptr(Dt + k0), offD[q], dst);
            } else {
                const int row = 8 * blk + (lane >> 3);
                const int lc = (lane & 7) ^ ((row >> 1) & 7);
                const bool ok = m0 + row < L && k0 + 8 * lc < R;
                copy16_to_lds(ok ? (const void*)(Dt + (int64_t)row * R + k0 + 8 * lc) : (const void*)zsrc, dst);
            }
        } else if (j < Lay::ND + Lay::NWC) {
            const int q = j - Lay::ND;
            const uint32_t dst = sb + Lay::W + Lay::WBW * wave + 1024 * q;
            if constexpr (!KRAG) {
                copy16s_to_lds(uniform_ptr(Wn + (int64_t)k0 * C), offW[q], dst);
            } else {
                const int row = NF == 2 ? 8 * q + (lane >> 3) : 16 * q + (lane >> 2);
                const int col = NF == 2 ? 64 * wave + 8 * ((lane & 7) ^ tr64_swz(row)) : 32 * wave + 8 * (lane & 3);
                const bool ok = k0 + row < R && n0 + col < C;
                copy16_to_lds(ok ? (const void*)(Wn + (int64_t)(k0 + row) * C + col) : (const void*)zsrc, dst);
            }
        } else if (j < Lay::ND + Lay::NWC + Lay::NB) {
            // the swizzled B slab of rows k0 .. k0+63; every wave issues NB
            // copies, those past the slab go to the sink
            const int q = j - Lay::ND - Lay::NWC, blk = 4 * q + wave;
            const bool real = blk < Lay::NBC;
            const bool ok = bval[q] && (!KRAG || k0 + brow[q] < R);
            const void* src = (const uint8_t*)Bm + ((int64_t)k0 + brow[q]) * (2 * (int64_t)r) + bcol[q];
            copy16_to_lds(ok ? src : (const void*)zsrc, real ? sb + Lay::B + 1024 * blk : lds0 + Lay::SINK);
        } else {
            const int q = j - Lay::ND - Lay::NWC - Lay::NB;
            const uint32_t dst = sb + Lay::M + 256 * (Lay::NMC * wave + q);
            if constexpr (!KRAG) {
                copy4s_to_lds(uniform_ptr(Mn + (int64_t)(k0 >> 5) * C), offM[q], dst);
            } else {
                const int e = 64 * (Lay::NMC * wave + q) + lane;
                const int n = e >> 1, gw = (k0 >> 5) + (e & 1);
                const bool ok = n0 + n < C && gw < wprT;
                copy4_to_lds(ok ? (const void*)(Mt + mt_index(n0 + n, gw, C, wprT)) : (const void*)zsrc, dst);
            }
        }
    };

    // Rows of the merge A operand: lane (rho = l32, h) reads B row pi(rho).
    const int rho = l32;
    const int pik = 16 * (rho >> 4) + 8 * ((rho >> 2) & 1) + 4 * ((rho >> 3) & 1) + (rho & 3);
    const int ncol0 = 32 * NF * wave + l32;
    // transpose-read offsets of the raw W fragments in this wave's W block,
    // sub-step 0 (sub-step c4 is 16 rows further): group g of 16 lanes reads
    // rows 8(g/2) + 4t + 0..3, columns 32nb + 16(g%2) + 0..15
    int offWt[NF][2];
    {
        const int g = lane >> 4, jj = lane & 15;
#pragma unroll
        for (int nb = 0; nb < NF; ++nb)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int row = 8 * (g >> 1) + 4 * t + (jj >> 2), col = 32 * nb + 16 * (g & 1) + 4 * (jj & 3);
                offWt[nb][t] = Lay::W + Lay::WBW * wave + (NF == 2 ? tr64_elem_off(row, col) : row * Lay::WROW + 2 * col);
            }
    }
    auto doff = [&](int mb, int c4) { return Lay::D + slab64_off(32 * mb + l32, 2 * c4 + h); };

    f32x16 acc[MBW][NF];
#pragma unroll
    for (int i = 0; i < MBW; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    bf16x8 da[MBW], db[MBW];  // dY fragments of alternate sub-steps
    u32x4 wa[NF], wb[NF];     // W' fragments of alternate sub-steps
    f32x16 T[NF];             // rank-r block of the current 32-wide k half
    uint32_t mw[NF][2];       // M^T words [nb][kb] of the current K-step
    u32x4 raw[NF], sel[NF];
    u32x4 rwa[NF], rwb[NF];   // folded merge: W of the two sub-steps of a k half
    bf16x8 bfr[RK];           // B[32kb + pi(rho)][16c + 8h .. +7]
    bf16x8 afr[NF][RK];       // A[16c + 8h .. +7][n] (scaled by s when the merge is folded)

    // MFMA slot i of a sub-step: token block i/2, feature block i%2; the fewer
    // MFMAs of a thin tile are spread over the 16 slots, so that the merge
    // pieces of the later slots have some to hide behind
    auto mm = [&](int i, const bf16x8 (&df)[MBW], const u32x4 (&wf)[NF]) {
        constexpr int kStep = 16 / (MBW * NF);
        const int mb = i / (kStep * NF), nb = NF == 2 ? i & 1 : 0;
        if (i % kStep == 0 && mb < MBW) acc[mb][nb] = mfma_32x32x16(df[mb], as_bf16x8(wf[nb]), acc[mb][nb]);
    };
    // ranks 16c + 8h .. +7 of B row 32kb + pik; the slab holds zeros for
    // ranks at or past r, so the read needs no per-lane test (a lane-dependent
    // branch would split the loop body and undo its per-slot schedule)
    auto read_bfr = [&](const uint8_t* sb, int kb) {
        const int k = 32 * kb + pik;
#pragma unroll
        for (int c = 0; c < RK; ++c)
            bfr[c] = *(const bf16x8*)(sb + Lay::B + k * Lay::PITCH + 16 * Lay::bswz(k, 2 * c + h));
    };
    auto read_mw = [&](const uint8_t* sb) {
#pragma unroll
        for (int nb = 0; nb < NF; ++nb) {
            const u32x2 v = *(const u32x2*)(sb + Lay::M + 8 * (ncol0 + 32 * nb));
            mw[nb][0] = v[0];
            mw[nb][1] = v[1];
        }
    };
    auto read_rs = [&](const uint8_t* sb, int c4) {
#pragma unroll
        for (int nb = 0; nb < NF; ++nb) {
            const u32x2 lo = lds_tr_read(sb + offWt[nb][0] + 16 * c4 * Lay::WROW);
            const u32x2 hi = lds_tr_read(sb + offWt[nb][1] + 16 * c4 * Lay::WROW);
            raw[nb][0] = lo[0];
            raw[nb][1] = lo[1];
            raw[nb][2] = hi[0];
            raw[nb][3] = hi[1];
            sel[nb] = read_sel16(smem + Lay::LUT, mw[nb][c4 >> 1], 8 * (2 * (c4 & 1) + h));
        }
    };
    auto read_d2 = [&](bf16x8 (&df)[MBW], const uint8_t* sb, int c4, int p) {
        if (2 * p < MBW) df[2 * p] = *(const bf16x8*)(sb + doff(2 * p, c4));
        if (2 * p + 1 < MBW) df[2 * p + 1] = *(const bf16x8*)(sb + doff(2 * p + 1, c4));
    };
    auto merge_piece = [&](u32x4 (&wf)[NF], int p, int cp) {
        const int nb = p >> 2, q = p & 3;
        if (nb < NF)
            wf[nb][q] = merge_pair(raw[nb][q], T[nb][8 * cp + 2 * q], T[nb][8 * cp + 2 * q + 1], s, sel[nb][q]);
    };
    // folded merge (see the forward kernel): raw W of sub-step c4, its select
    // masks, the unpack of a W pair into the rank-r accumulator, the merge
    auto read_raw = [&](u32x4 (&rw)[NF], const uint8_t* sb, int c4) {
#pragma unroll
        for (int nb = 0; nb < NF; ++nb) {
            const u32x2 lo = lds_tr_read(sb + offWt[nb][0] + 16 * c4 * Lay::WROW);
            const u32x2 hi = lds_tr_read(sb + offWt[nb][1] + 16 * c4 * Lay::WROW);
            rw[nb][0] = lo[0];
            rw[nb][1] = lo[1];
            rw[nb][2] = hi[0];
            rw[nb][3] = hi[1];
        }
    };
    auto read_sel = [&](int c4) {
#pragma unroll
        for (int nb = 0; nb < NF; ++nb) {
            sel[nb] = read_sel16(smem + Lay::LUT, mw[nb][c4 >> 1], 8 * (2 * (c4 & 1) + h));
        }
    };
    auto unpack = [&](const u32x4 (&rw)[NF], int cp, int p) {
        const int nb = p >> 2, q = p & 3;
        if (nb < NF) {
            T[nb][8 * cp + 2 * q] = __uint_as_float(rw[nb][q] << 16);
            T[nb][8 * cp + 2 * q + 1] = __uint_as_float(rw[nb][q] & 0xFFFF0000u);
        }
    };
    auto merge_fold = [&](u32x4 (&wf)[NF], int p, int cp) {
        const int nb = p >> 2, q = p & 3;
        if (nb < NF) wf[nb][q] = pack_bf16x2(T[nb][8 * cp + 2 * q], T[nb][8 * cp + 2 * q + 1]) & sel[nb][q];
    };
    // late_*: the copies EARLY.. of the stage in the other buffer, issued in
    // the merge slots of the first sub-step of a K-step (see the main loop)
    auto substep = [&](const bf16x8 (&dc)[MBW], const u32x4 (&wc)[NF], bf16x8 (&dn)[MBW], u32x4 (&wn)[NF],
                       const uint8_t* sb, int c4n, auto rank_tag, int late_k = 0, uint32_t late_sq = 0,
                       bool late_on = false) {
        constexpr bool RANK = decltype(rank_tag)::value;
        mm(0, dc, wc); read_rs(sb, c4n); SLOT_END();
        mm(1, dc, wc); if constexpr (RANK) read_bfr(sb, 1); SLOT_END();
        mm(2, dc, wc); read_d2(dn, sb, c4n, 0); SLOT_END();
        mm(3, dc, wc); read_d2(dn, sb, c4n, 1); SLOT_END();
        mm(4, dc, wc); read_d2(dn, sb, c4n, 2); SLOT_END();
        mm(5, dc, wc); read_d2(dn, sb, c4n, 3); SLOT_END();
        mm(6, dc, wc); SLOT_END();
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            mm(7 + p, dc, wc);
            merge_piece(wn, p, c4n & 1);
            if (late_on && Lay::EARLY + p < Lay::COPIES) copy_j(Lay::EARLY + p, late_k, late_sq);
            SLOT_END();
        }
        mm(15, dc, wc);
        if constexpr (RANK) rank_mfma2<RK>(T, bfr, afr);  // after the merge pieces read T
        SLOT_END();
    };
    // the sub-steps with the folded merge (schedule as in the forward)
    auto substep_fold = [&](const bf16x8 (&dc)[MBW], const u32x4 (&wc)[NF], bf16x8 (&dn)[MBW], u32x4 (&wn)[NF],
                            const uint8_t* sb, const uint8_t* snext, int c4n, int late_k = 0,
                            uint32_t late_sq = 0, bool late_on = false) {
        const int cp = c4n & 1;
        mm(0, dc, wc); read_sel(c4n); if (c4n == 1) read_raw(rwa, sb, 2); SLOT_END();
        mm(1, dc, wc); if (c4n == 1) { read_bfr(sb, 1); read_raw(rwb, sb, 3); } SLOT_END();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            mm(2 + i, dc, wc);
            read_d2(dn, sb, c4n, i);
            if (c4n == 1) { unpack(rwa, 0, 2 * i); unpack(rwa, 0, 2 * i + 1); }
            if (c4n == 3 && i == 3) {
                wait_vmcnt<Lay::NB + Lay::NMC + Lay::FLY>();  // this wave's W copies of the next stage
                read_raw(rwa, snext, 0);
                read_raw(rwb, snext, 1);
            }
            SLOT_END();
        }
        mm(6, dc, wc); SLOT_END();
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            mm(7 + p, dc, wc);
            merge_fold(wn, p, cp);
            if (c4n == 1) unpack(rwb, 1, p);
            if (c4n == 3) { unpack(rwb, 1, p); unpack(rwa, 0, p); }
            if (late_on && Lay::EARLY + p < Lay::COPIES) copy_j(Lay::EARLY + p, late_k, late_sq);
            SLOT_END();
        }
        mm(15, dc, wc);
        if (c4n == 1) rank_mfma2_acc<RK>(T, bfr, afr);  // after the merge pieces read T
        SLOT_END();
    };

    // ---- prologue.  The A block of the merge goes to the last PARK stages'
    // buffers while the stages before them are copied; once it and stage 0
    // landed, the A block is read into registers and those stages are copied
    // over it (the K-steps' barriers wait for them), so the two round trips to
    // memory overlap.
    // A[:, n0 .. n0+FT-1]: 16*RK rows of PROW bytes, chunks permuted as in tile_off
    constexpr int kPark = (Lay::S - PARK) * Lay::STAGE;
#pragma unroll
    for (int q = 0; q < 16 * RK * PROW / 4096; ++q) {
        const int blk = 4 * q + wave;
        const int row = 1024 / PROW * blk + lane / (PROW / 16);
        const int lc = swz_chunk(row, lane % (PROW / 16));
        const int gn = n0 + 8 * lc;
        copy16_to_lds((row < ra && gn < C) ? (const void*)(Am + (int64_t)row * C + gn) : (const void*)zsrc,
                      lds0 + kPark + 1024 * blk);
    }
#pragma unroll
    for (int i = 0; i < Lay::S - PARK; ++i)
#pragma unroll
        for (int j = 0; j < Lay::COPIES; ++j) copy_j(j, (i < nk ? i : nk - 1) * BK, lds0 + i * Lay::STAGE);
    stage_barrier<(Lay::S - PARK - 1) * Lay::COPIES>();
    // the merge's B operand A[16c + 8h + e][n] into registers via transpose
    // loads (lane and operand element as in tr_frag_off)
    auto park_off = [&](int row0, int col0, int t) {
        const int g = lane >> 4, j = lane & 15;
        const int row = row0 + 8 * (g >> 1) + 4 * t + (j >> 2), col = col0 + 16 * (g & 1) + 4 * (j & 3);
        return row * PROW + (swz_chunk(row, col >> 3) << 4) + ((col & 7) << 1);
    };
#pragma unroll
    for (int nb = 0; nb < NF; ++nb)
#pragma unroll
        for (int c = 0; c < RK; ++c)
            afr[nb][c] = frag_from_tr(lds_tr_read(smem + kPark + park_off(16 * c, 32 * NF * wave + 32 * nb, 0)),
                                      lds_tr_read(smem + kPark + park_off(16 * c, 32 * NF * wave + 32 * nb, 1)));
    if constexpr (FOLD) {  // s.A, exact for a power-of-two s
#pragma unroll
        for (int nb = 0; nb < NF; ++nb)
#pragma unroll
            for (int c = 0; c < RK; ++c) {
                u32x4 v = __builtin_bit_cast(u32x4, afr[nb][c]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] = pack_bf16x2(s * __uint_as_float(v[e] << 16), s * __uint_as_float(v[e] & 0xFFFF0000u));
                afr[nb][c] = as_bf16x8(v);
            }
    }
    lds_barrier();
#pragma unroll
    for (int i = Lay::S - PARK; i < Lay::S; ++i)
#pragma unroll
        for (int j = 0; j < Lay::COPIES; ++j) copy_j(j, (i < nk ? i : nk - 1) * BK, lds0 + i * Lay::STAGE);
    read_mw(smem);
    read_bfr(smem, 0);
    if constexpr (FOLD) {
        read_raw(rwa, smem, 0);
        read_raw(rwb, smem, 1);
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            unpack(rwa, 0, p);
            unpack(rwb, 1, p);
        }
        rank_mfma2_acc<RK>(T, bfr, afr);
        read_sel(0);
    } else {
        rank_mfma2<RK>(T, bfr, afr);
        read_rs(smem, 0);
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) read_d2(da, smem, 0, p);
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        if constexpr (FOLD) merge_fold(wa, p, 0);
        else merge_piece(wa, p, 0);
    }

    // ---- main loop (branch-free, see the forward kernel)
    for (int kt = 0, st = 0; kt < nk; ++kt) {
        constexpr int S = Lay::S;
        const int sx = st + 1 < S ? st + 1 : 0;  // buffers of K-steps kt+1 and kt-1
        const int sp = st > 0 ? st - 1 : S - 1;
        const uint8_t* sb = smem + st * Lay::STAGE;
        const uint8_t* sn = smem + sx * Lay::STAGE;
        // copies EARLY.. of stage kt+S-1 (buffer sp, free since the last
        // barrier); at kt = 0 the prologue issued all of them
        const int k1 = (kt + S - 1 < nk ? kt + S - 1 : nk - 1) * BK;
        if constexpr (FOLD) {
            substep_fold(da, wa, db, wb, sb, sn, 1, k1, lds0 + sp * Lay::STAGE, kt > 0);
            substep_fold(db, wb, da, wa, sb, sn, 2);
            substep_fold(da, wa, db, wb, sb, sn, 3);
        } else {
            substep(da, wa, db, wb, sb, 1, std::true_type{}, k1, lds0 + sp * Lay::STAGE, kt > 0);
            substep(db, wb, da, wa, sb, 2, std::false_type{});
            substep(da, wa, db, wb, sb, 3, std::false_type{});
        }
        stage_barrier<Lay::FLY>();  // the FLY copies issued last belong to later stages
        const int k2 = (kt + S < nk ? kt + S : nk - 1) * BK;
        const uint32_t sq = lds0 + st * Lay::STAGE;
        // one copy per MFMA slot: a copy issued behind an MFMA stalls the
        // wave while that MFMA runs, a second one would stall the next
        auto early = [&](int j) {
            if (j < Lay::EARLY) copy_j(j, k2, sq);
        };
        mm(0, db, wb); read_mw(sn); read_bfr(sn, 0); early(0); SLOT_END();
        mm(1, db, wb); early(1); SLOT_END();
        mm(2, db, wb); read_d2(da, sn, 0, 0); early(2); SLOT_END();
        mm(3, db, wb); read_d2(da, sn, 0, 1); early(3); SLOT_END();
        mm(4, db, wb);
        if constexpr (FOLD) read_sel(0);
        else read_rs(sn, 0);
        early(4); SLOT_END();
        mm(5, db, wb); read_d2(da, sn, 0, 2); early(5); SLOT_END();
        mm(6, db, wb); read_d2(da, sn, 0, 3);
        if constexpr (FOLD) rank_mfma2_acc<RK>(T, bfr, afr);
        else rank_mfma2<RK>(T, bfr, afr);
        early(6); SLOT_END();
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            mm(7 + p, db, wb);
            if constexpr (FOLD) merge_fold(wa, p, 0);
            else merge_piece(wa, p, 0);
            early(7 + p);
            SLOT_END();
        }
        mm(15, db, wb);
        SLOT_END();
        st = sx;
    }
    // ---- epilogue: round to bf16, stage the wave's TM x 32 NF block in LDS
    // (rows of 32 NF outputs), then 16-byte stores of whole rows.
    wait_vmcnt<0>();
    lds_barrier();  // every wave's copies landed and every read of the stages done
    if (TM == BM && NF == 2 && (int)blockIdx.x >= n_full) {
        // a piece of a split tile: its unrounded fp32 partial sums go to slice
        // blockIdx.x - n_full of `part` (256 tokens x 256 features); the
        // reduction launch adds the pieces in order and rounds once
        float* dst = part + (int64_t)((int)blockIdx.x - n_full) * (BM * BN);
#pragma unroll
        for (int nb = 0; nb < NF; ++nb)
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    dst[(32 * mb + 8 * (v >> 2) + 4 * h + (v & 3)) * BN + ncol0 + 32 * nb] = acc[mb][nb][v];
        return;
    }
    constexpr int OW = 32 * NF;   // outputs per staged row
    constexpr int CH = OW / 8;    // 16-byte chunks per row
    uint16_t* ol = (uint16_t*)(smem + wave * (TM * OW * 2));
#pragma unroll
    for (int nb = 0; nb < NF; ++nb)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                ol[(32 * mb + 8 * (v >> 2) + 4 * h + (v & 3)) * OW + 32 * nb + l32] = bf16_bits(acc[mb][nb][v]);
#pragma unroll 4
    for (int it = 0; it < TM * CH / 64; ++it) {
        const int row = (64 / CH) * it + lane / CH, ch = lane % CH;
        const u32x4 v = *(const u32x4*)(ol + row * OW + 8 * ch);
        const int64_t gm = m0 + row;
        const int gn = n0 + OW * wave + 8 * ch;
        if (gm < L && gn < C) *(u32x4*)(dX + gm * C + gn) = v;
    }
}

// s.A is exact in bf16 for a power-of-two s; the folded merge needs that
bool power_of_two(float s) {
    int e = 0;
    const float m = std::frexp(s, &e);
    return m == 0.5f || m == -0.5f;
}

// Whole tiles only, as in the forward (14336 x 4096, rank 64, 3333 tokens: 434
// against 422 us folded).
bool folds(const LayerArgs& a) { return dx_whole_tiles(a.L, a.R, a.C) && power_of_two(a.scale); }

// z0, z1: dB (R x rank) and dA (rank x C) to clear, or null
template <int RK, bool KRAG, bool FOLD, int TM, int NF>
void launch_tm(const LayerArgs& a, hipStream_t st, int ra, int grid, int tiles_m, int tiles_n, int n_full,
               int split, float* part, float* z0, int64_t nz0, float* z1, int64_t nz1) {
    hipLaunchKernelGGL((dx_kernel<RK, KRAG, FOLD, TM, NF>), dim3(grid), dim3(NT), 0, st, (const uint16_t*)a.dY,
                       (const uint16_t*)a.W, a.Mt, (const uint16_t*)a.B, (const uint16_t*)a.A, (uint16_t*)a.dX, a.L,
                       (int)a.R, (int)a.C, (int)a.r, ra, a.scale, tiles_m, tiles_n, z0, nz0, z1, nz1, n_full,
                       split, part);
}

#ifndef LORS_THIN_TILES

// a.r: the (padded) rank; ra: the rows of A that exist.  The first launch
// clears dB and dA when the caller asks for it (a.clear_grads).
template <int RK>
hipError_t launch_rk(const LayerArgs& a, hipStream_t st, int ra) {
    const int tiles_m = (int)((a.L + BM - 1) / BM);
    const int tiles_n = (int)((a.C + BN - 1) / BN);
    const int tiles = tiles_m * tiles_n;
    const bool krag = !dx_fixed_copies(a.R, a.C);
    const bool fold = folds(a);
    // A short last wave is cut over K when the caller gave room for the
    // pieces' partial sums (shapes without whole tiles); otherwise it runs as
    // thin tiles (the same bits as whole ones, no workspace).  Thin / split,
    // backward at rank 64 (us): 65792 x 2048, 200 tokens (8 tiles in 8 pieces)
    // 1100 / 545; 4096 x 11008, 1531 tokens (2 in 8) 406 / 378.
    TailSplit sp{tiles, 1, tiles};
    if (a.split_ws != nullptr && !dx_whole_tiles(a.L, a.R, a.C))
        sp = tail_split(tiles, (a.R + BK - 1) / BK, a.split_budget);
    const ThinPlan tp = sp.split == 1 ? thin_plan(a.L, a.C) : ThinPlan{tiles, 0, 0};
    float* part = sp.split > 1 ? (float*)a.split_ws : nullptr;
    // with thin tiles the whole-tile grid is exactly the first n_full tiles
    // (work_coords regroups ids over the tiles it is told the grid holds)
    const int grid = tp.tm > 0 ? tp.n_full : sp.grid;
    const int n_full = tp.tm > 0 ? tp.n_full : sp.n_full;
    // clear: dB (R x rank) and dA (rank x C) of the caller's problem, by the
    // first launch of this call
    const bool clear_here = a.clear_grads && grid > 0;
    float* z0 = clear_here ? a.dB : nullptr;
    float* z1 = clear_here ? a.dA : nullptr;
    const int64_t nz0 = clear_here ? a.R * a.r_grad : 0, nz1 = clear_here ? a.r_grad * a.C : 0;
    if (grid > 0) {
        if (krag)
            launch_tm<RK, true, false, BM, 2>(a, st, ra, grid, tiles_m, tiles_n, n_full, sp.split, part, z0,
                                                  nz0, z1, nz1);
        else if (fold)
            launch_tm<RK, false, true, BM, 2>(a, st, ra, grid, tiles_m, tiles_n, n_full, sp.split, part, z0,
                                                  nz0, z1, nz1);
        else
            launch_tm<RK, false, false, BM, 2>(a, st, ra, grid, tiles_m, tiles_n, n_full, sp.split, part,
                                                   z0, nz0, z1, nz1);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && tp.tm > 0)
        e = launch_dx_thin_bf16(a, st, ra, tp.n_full, tp.tail, tp.tm, a.clear_grads && !clear_here);
    if (e == hipSuccess && sp.split > 1)
        e = launch_split_reduce_bf16(part, sp.n_full, sp.split, tiles_m, tiles_n, GROUP_M, a.L, (int)a.C, nullptr,
                                     a.dX, st);
    return e;
}

#else  // LORS_THIN_TILES

// thin tiles of one feature half (NF = 1) and TM tokens: 2 SPAN / TM per tile
template <int RK, bool KRAG, bool FOLD, int TM>
hipError_t launch_thin_tm(const LayerArgs& a, hipStream_t st, int ra, int first, int tail, bool clear) {
    const int tiles_m = (int)((a.L + thin_span(TM) - 1) / thin_span(TM));
    const int tiles_n = (int)((a.C + BN - 1) / BN);
    float* z0 = clear ? a.dB : nullptr;
    float* z1 = clear ? a.dA : nullptr;
    const int64_t nz0 = clear ? a.R * a.r_grad : 0, nz1 = clear ? a.r_grad * a.C : 0;
    launch_tm<RK, KRAG, FOLD, TM, 1>(a, st, ra, tail * (2 * thin_span(TM) / TM), tiles_m, tiles_n, first, tail, nullptr,
                                          z0, nz0, z1, nz1);
    return hipGetLastError();
}

template <int RK, bool KRAG, bool FOLD>
hipError_t launch_thin_q(const LayerArgs& a, hipStream_t st, int ra, int first, int tail, int tm,
                         bool clear) {
    switch (tm) {
        case 64: return launch_thin_tm<RK, KRAG, FOLD, 64>(a, st, ra, first, tail, clear);
        case 128: return launch_thin_tm<RK, KRAG, FOLD, 128>(a, st, ra, first, tail, clear);
        case 192: return launch_thin_tm<RK, KRAG, FOLD, 192>(a, st, ra, first, tail, clear);
        case 256: return launch_thin_tm<RK, KRAG, FOLD, 256>(a, st, ra, first, tail, clear);
        default: return hipErrorInvalidValue;
    }
}

template <int RK>
hipError_t launch_thin_rk(const LayerArgs& a, hipStream_t st, int ra, int first, int tail, int tm,
                          bool clear) {
    if (!dx_fixed_copies(a.R, a.C)) return launch_thin_q<RK, true, false>(a, st, ra, first, tail, tm, clear);
    return folds(a) ? launch_thin_q<RK, false, true>(a, st, ra, first, tail, tm, clear)
                    : launch_thin_q<RK, false, false>(a, st, ra, first, tail, tm, clear);
}

#endif  // LORS_THIN_TILES

}  // namespace

#ifdef LORS_THIN_TILES

hipError_t launch_dx_thin_bf16(const LayerArgs& a, hipStream_t st, int ra, int first, int tail, int tm, bool clear) {
    if (tail <= 0) return hipSuccess;
    // a.r: a multiple of 8 (see launch_dx_bf16)
    if (a.r < 8 || a.r % 8 != 0) return hipErrorInvalidValue;
    switch ((a.r + 15) / 16) {
        case 1: return launch_thin_rk<1>(a, st, ra, first, tail, tm, clear);
        case 2: return launch_thin_rk<2>(a, st, ra, first, tail, tm, clear);
        case 3: return launch_thin_rk<3>(a, st, ra, first, tail, tm, clear);
        case 4: return launch_thin_rk<4>(a, st, ra, first, tail, tm, clear);
        case 5: return launch_thin_rk<5>(a, st, ra, first, tail, tm, clear);
        case 6: return launch_thin_rk<6>(a, st, ra, first, tail, tm, clear);
        case 7: return launch_thin_rk<7>(a, st, ra, first, tail, tm, clear);
        case 8: return launch_thin_rk<8>(a, st, ra, first, tail, tm, clear);
        default: return hipErrorInvalidValue;
    }
}

#else

hipError_t launch_dx_bf16(const LayerArgs& a, hipStream_t st) {
    if (a.L == 0 || a.dX == nullptr) return hipSuccess;
    if (a.Mt == nullptr || a.r < 1 || a.r > 128) return hipErrorInvalidValue;
    // The B slab is copied in whole 16-byte chunks of its rows.  A rank that
    // is not a multiple of 8 works on a copy of B whose rows are padded with
    // zero columns to rp = roundup8(r); the missing A rows are read as zero.
    LayerArgs ap = a;
    const int ra = (int)a.r;
    const int rp = (ra + 7) / 8 * 8;
    if (rp != ra) {
        if (a.b_pad == nullptr) return hipErrorInvalidValue;
        const hipError_t e = launch_pad_cols_bf16(a.B, a.R, a.r, rp, a.b_pad, st);
        if (e != hipSuccess) return e;
        ap.B = a.b_pad;
        ap.r = rp;
    }
    switch ((rp + 15) / 16) {
        case 1: return launch_rk<1>(ap, st, ra);
        case 2: return launch_rk<2>(ap, st, ra);
        case 3: return launch_rk<3>(ap, st, ra);
        case 4: return launch_rk<4>(ap, st, ra);
        default: break;
    }
    // ranks above 64: half-feature thin tiles only (see the forward)
    ThinPlan run[2];
    const int n = thin_only_plan(a.L, a.C, run);
    hipError_t e = hipSuccess;
    for (int i = 0; i < n && e == hipSuccess; ++i)
        e = launch_dx_thin_bf16(ap, st, ra, run[i].n_full, run[i].tail, run[i].tm, a.clear_grads && i == 0);
    return e;
}

#endif  // LORS_THIN_TILES

}  // namespace lors
