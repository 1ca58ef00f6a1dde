// Forward for few tokens (decoding, short prompts), bf16 on gfx950.
//
//   Y[L x R] = X[L x C] . W'^T,   W' = select(M, W + s.B.A, 0)
//
// With a handful of tokens the layer is one read of W, so the work is cut for
// the memory system and not for the matrix cores: a workgroup owns NB blocks of
// FT = 16 or 32 output features and MB blocks of FT tokens, and its waves share the
// contraction (64-k block j belongs to wave j mod NW), so that a few thousand
// features already put thousands of waves, each with several loads in flight,
// on the chip.  Nothing is shared inside the K-loop and it has no barrier:
// every operand goes from global memory into registers, SLOTS - 1 blocks
// ahead.  W rows, mask words and X rows are read in the MFMA operand layout
// directly (the lanes and loads of a block cover each row's 128-byte line); the
// A slab of the block, whose operand is transposed, passes through a
// wave-private LDS buffer.  W' is formed as in fwd_kernel: rank-r MFMAs whose
// rows are the k of the main operand in register order, one rounding, select
// masks from the 16-entry table.  At the end the waves' fp32 partial sums are
// added through LDS in wave order, so results are bitwise reproducible.
#include "gemm_common.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace lors {
namespace {

constexpr int BK = 64;  // input features per block

// Eight outputs (+ bias) of token gm, features gn .. gn+7, if they exist.
__device__ __forceinline__ void store8(const float (&sum)[8], int gm, int gn, int L, int R, const uint16_t* bias,
                                       uint16_t* Y) {
    if (gm >= L || gn >= R) return;
    const u32x4 bv = bias != nullptr ? *(const u32x4*)(bias + gn) : zero_u32x4();
    u32x4 o;
#pragma unroll
    for (int p = 0; p < 4; ++p)
        o[p] = pack_bf16x2(sum[2 * p] + __uint_as_float(bv[p] << 16),
                           sum[2 * p + 1] + __uint_as_float(bv[p] & 0xFFFF0000u));
    *(u32x4*)(Y + (int64_t)gm * R + gn) = o;
}

template <int FT, int RK, int MB, int NB>
struct Cfg {
    static constexpr int G = 64 / FT;           // lane groups: lane l holds column l % FT, k 8(l/FT) .. +7
    static constexpr int WV = 8 / G;            // operand vectors of a block: vector c holds k 8Gc ..
    static constexpr int RM = FT == 32 ? 16 : 32;        // ranks per rank MFMA
    static constexpr int RC = (16 * RK + RM - 1) / RM;   // rank MFMAs per block of rows
    static constexpr int NV = FT * FT / 64;     // accumulator elements per lane
    static constexpr int AW = RM * RC * kRow64; // one wave's A slab
    // Registers: a block in flight, and about what the rest of a wave needs.
    // FT = 16 (few workgroups) takes as many waves as hold two blocks each,
    // and a third block where it fits; FT = 32 two blocks, so that with NB = 1 two
    // workgroups share a CU where the registers allow (14336 x 4096, 32 tokens:
    // 44 us, against 49 with three blocks in flight and one workgroup).
    static constexpr bool XA = FT == 16 && MB <= 2;  // X is fetched ahead too (else inside its block: it is in L2)
    static constexpr int BLOCK = NB * (4 * WV + 2) + 8 * RK + (XA ? 4 * WV * MB : 0);
    static constexpr int OTHER = 56 + 4 * RC * NB + 2 * RK + NV * (MB * NB + 1) + (XA ? 0 : 4 * WV * MB);
    static constexpr int NW = FT == 16 && 2 * BLOCK + OTHER <= 128 ? 16 : 2 * BLOCK + OTHER <= 256 ? 8 : 4;
    static constexpr int SLOTS = FT == 16 && 3 * BLOCK + OTHER <= 2048 / NW ? 3 : 2;
    static constexpr int EU = FT == 32 && RK == 1 && MB == 1 && NB == 1 ? 4 : NW / 4;  // waves per SIMD
    static constexpr int RED = NW * NB * MB * NV * 64 * 4;    // the waves' partial sums (after the loop)
    static constexpr int LUT = NW * AW > RED ? NW * AW : RED;
    static constexpr int TOTAL = LUT + 128;
};

// KRAG: C is no multiple of 64; chunks past C are read from the row's first
// chunk and dropped by zero W' and zero X.
// (Its bounds checks take registers that EU = 4 does not leave: 8 spilled, 8192 x
// 4104, rank 16, 1 token 19.2 us against 15.6 without that bound.)
template <int FT, int RK, bool KRAG, int MB, int NB>
__global__ __launch_bounds__((64 * Cfg<FT, RK, MB, NB>::NW),
                             (KRAG ? Cfg<FT, RK, MB, NB>::NW / 4 : Cfg<FT, RK, MB, NB>::EU)) void fwd_few_kernel(
    const uint16_t* __restrict__ X, const uint16_t* __restrict__ W, const uint32_t* __restrict__ Mp,
    const uint16_t* __restrict__ Bm, const uint16_t* __restrict__ Am, const uint16_t* __restrict__ bias,
    uint16_t* __restrict__ Y, int L, int R, int C, int r, float s, int two_four) {
    using T = Cfg<FT, RK, MB, NB>;
    constexpr int NW = T::NW, G = T::G, WV = T::WV, RC = T::RC, NV = T::NV, SLOTS = T::SLOTS;
    static_assert(T::TOTAL <= kLdsBytes, "LDS budget");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[T::TOTAL];

    const int tid = threadIdx.x, lane = tid & 63, l = lane & (FT - 1), g = lane / FT;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * FT * NB, m0 = blockIdx.y * FT * MB;
    const int wpr = (C + 31) >> 5;
    const int nblk = (C + BK - 1) / BK;
    uint8_t* as = smem + wave * T::AW;

    // rows past R, L and r repeat the last one that exists (outputs of the
    // former are not stored, ranks past r are zero in both rank operands)
    int nl[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) nl[nb] = min(FT * nb + l, R - 1 - n0);
    const uint16_t* Wt = W + (int64_t)n0 * C;
    const uint32_t* Mt = Mp + (int64_t)n0 * wpr;
    const uint16_t* Xt = X + (int64_t)m0 * C;
    uint32_t offW[NB], offM[NB], offX[MB], offA[2 * RK];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        offW[nb] = (uint32_t)(nl[nb] * C + 8 * g);
        offM[nb] = (uint32_t)(nl[nb] * wpr);
    }
#pragma unroll
    for (int b = 0; b < MB; ++b) offX[b] = (uint32_t)(min(FT * b + l, L - 1 - m0) * C + 8 * g);
    const int arow = lane >> 3, achunk = lane & 7;
#pragma unroll
    for (int q = 0; q < 2 * RK; ++q) offA[q] = (uint32_t)(min(8 * q + arow, r - 1) * C + 8 * achunk);

    struct Block {
        u32x4 w[NB][WV], a[2 * RK], x[MB][WV];
        uint32_t m[NB][2];
    };
    auto load_x = [&](Block& t, int k0) {
#pragma unroll
        for (int c = 0; c < WV; ++c)
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                const bool in = !KRAG || k0 + 8 * G * c + 8 * g < C;
                t.x[b][c] = *(const u32x4*)(Xt + (in ? offX[b] + k0 + 8 * G * c : offX[b] - 8 * g));
                if (!in) t.x[b][c] = zero_u32x4();
            }
    };
    auto load = [&](Block& t, int blk) {
        const int k0 = blk * BK;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
            for (int c = 0; c < WV; ++c) {
                const bool in = !KRAG || k0 + 8 * G * c + 8 * g < C;
                t.w[nb][c] = *(const u32x4*)(Wt + (in ? offW[nb] + k0 + 8 * G * c : offW[nb] - 8 * g));
            }
            t.m[nb][0] = Mt[offM[nb] + 2 * blk];
            t.m[nb][1] = Mt[offM[nb] + (KRAG ? min(2 * blk + 1, wpr - 1) : 2 * blk + 1)];
        }
#pragma unroll
        for (int q = 0; q < 2 * RK; ++q) {
            const bool in = !KRAG || k0 + 8 * achunk < C;
            t.a[q] = *(const u32x4*)(Am + (in ? offA[q] + k0 : offA[q] - 8 * achunk));
        }
        if constexpr (T::XA) load_x(t, k0);
    };
    Block ring[SLOTS];
#pragma unroll
    for (int i = 0; i < SLOTS - 1; ++i)
        if (wave + i * NW < nblk) load(ring[i], wave + i * NW);

    if (tid < 16) *(u32x2*)(smem + T::LUT + 8 * tid) = two_four ? select_lut16_entry<true>((uint32_t)tid)
                                                            : select_lut16_entry<false>((uint32_t)tid);
    for (int e = lane; e < T::AW / 16; e += 64) *(u32x4*)(as + 16 * e) = zero_u32x4();  // ranks past r stay zero
    bf16x8 bfr[NB][RC];  // B[n][RM c + 8g .. +7]
    const bool b_vec = (r & 7) == 0;
#pragma unroll
    for (int i = 0; i < NB * RC; ++i) {
        const int nb = i / RC, c = i % RC;
        u32x4 v = zero_u32x4();
        const int j0 = T::RM * c + 8 * g;
        const uint16_t* src = Bm + (int64_t)(n0 + nl[nb]) * r + j0;
        if (b_vec) {
            if (j0 < r) v = *(const u32x4*)src;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e >> 1] |= (j0 + e < r ? (uint32_t)src[e] : 0u) << ((e & 1) * 16);
        }
        bfr[nb][c] = as_bf16x8(v);
    }

    // The A^T operand by transpose loads (16 lanes read 4 ranks x 16 k): rank
    // row and k column of this lane's address, for the MFMA's rank chunk 0.
    // FT = 32: MFMA t covers k 32t .. +31 in the order pi of fwd_kernel.
    // FT = 16: rows i of MFMA t are the k 8(i/4) + 4(t%2) + i%4 of k 32(t/2) ..
    constexpr int NT = FT == 32 ? 2 : 4;
    int offAt[NT][2];
    {
        const int g16 = lane >> 4, jj = lane & 15;
        const int sig = ((jj & 3) == 1) ? 2 : ((jj & 3) == 2) ? 1 : (jj & 3);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                offAt[t][u] = FT == 32 ? tr64_elem_off(8 * (g16 >> 1) + 4 * u + (jj >> 2), 32 * t + 16 * (g16 & 1) + 4 * sig)
                                       : tr64_elem_off(8 * g16 + 4 * u + (jj >> 2), 32 * (t >> 1) + 8 * (jj & 3) + 4 * (t & 1));
    }
    using Acc = std::conditional_t<FT == 32, f32x16, f32x4>;
    auto mfma = [](bf16x8 a, bf16x8 b, Acc c) {
        if constexpr (FT == 32) return mfma_32x32x16(a, b, c);
        else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    };
    Acc acc[NB][MB];
#pragma unroll
    for (int i = 0; i < NB * MB; ++i)
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[i / MB][i % MB][v] = 0.f;
    lds_barrier();  // the select table

    for (int base = wave; base < nblk; base += SLOTS * NW) {
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const int blk = base + i * NW;
            if (blk >= nblk) break;
            Block& cur = ring[i];
            if constexpr (!T::XA) load_x(cur, blk * BK);
#pragma unroll
            for (int q = 0; q < 2 * RK; ++q)
                if (8 * q + arow < r)
                    *(u32x4*)(as + (8 * q + arow) * kRow64 + 16 * (achunk ^ tr64_swz(arow))) = cur.a[q];
            const int ahead = blk + (SLOTS - 1) * NW;
            if (ahead < nblk) load(ring[(i + SLOTS - 1) % SLOTS], ahead);
            asm volatile("" ::: "memory");  // one wave's LDS operations complete in order
#pragma unroll
            for (int i2 = 0; i2 < 2 * NB; ++i2) {
                const int kb = i2 / NB, nb = i2 % NB;
                // rank products of k 32kb .. +31, in the register order of the main operand
                float tt[NV == 16 ? 16 : 8];
#pragma unroll
                for (int t = kb * NT / 2; t < (kb + 1) * NT / 2; ++t) {
                    Acc p;
#pragma unroll
                    for (int v = 0; v < NV; ++v) p[v] = 0.f;
#pragma unroll
                    for (int c = 0; c < RC; ++c)
                        p = mfma(frag_from_tr(lds_tr_read(as + offAt[t][0] + T::RM * kRow64 * c),
                                              lds_tr_read(as + offAt[t][1] + T::RM * kRow64 * c)),
                                 bfr[nb][c], p);
#pragma unroll
                    for (int v = 0; v < NV; ++v) tt[(FT == 32 ? 0 : 4 * (t & 1)) + v] = p[v];
                }
#pragma unroll
                for (int cp = 0; cp < WV / 2; ++cp) {
                    const int c = kb * WV / 2 + cp;
                    const u32x4 sel = read_sel16(smem + T::LUT, cur.m[nb][kb], 8 * (G * cp + g));
                    const bool in = !KRAG || blk * BK + 8 * G * c + 8 * g < C;
                    u32x4 wf;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        wf[q] = merge_pair(cur.w[nb][c][q], tt[8 * cp + 2 * q], tt[8 * cp + 2 * q + 1], s, sel[q]);
                        if (!in) wf[q] = 0u;
                    }
#pragma unroll
                    for (int b = 0; b < MB; ++b) acc[nb][b] = mfma(as_bf16x8(cur.x[b][c]), as_bf16x8(wf), acc[nb][b]);
                }
            }
            asm volatile("" ::: "memory");
        }
    }

    // ---- the waves' partial sums through LDS, in wave order: one item is a
    // token row and eight features
    __syncthreads();
    float* red = (float*)smem;
    constexpr int NI = NB * MB;  // accumulator tiles of a wave: feature block i / MB, token block i % MB
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int v = 0; v < NV; ++v) red[((wave * NI + i) * NV + v) * 64 + lane] = acc[i / MB][i % MB][v];
    __syncthreads();
    for (int it = tid; it < NI * FT * FT / 8; it += 64 * NW) {
        const int f8 = it % (FT / 8), row = it / (FT / 8) % FT, i = it / (FT * FT / 8);
        // accumulator element v of lane group gg is token row 4G(v/4) + 4gg + v%4
        const int v = 4 * (row / (4 * G)) + (row & 3), gg = (row >> 2) % G;
        float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int w = 0; w < NW; ++w) {
            const f32x4* p = (const f32x4*)(red + ((w * NI + i) * NV + v) * 64 + FT * gg + 8 * f8);
            const f32x4 lo = p[0], hi = p[1];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sum[e] += lo[e];
                sum[4 + e] += hi[e];
            }
        }
        store8(sum, m0 + FT * (i % MB) + row, n0 + FT * (i / MB) + 8 * f8, L, R, bias, Y);
    }
}

template <int FT, int RK, int MB, int NB = 1>
hipError_t launch(const LayerArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)((a.R + FT * NB - 1) / (FT * NB)), (unsigned)((a.L + FT * MB - 1) / (FT * MB)));
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * Cfg<FT, RK, MB, NB>::NW), 0, st, (const uint16_t*)a.X, (const uint16_t*)a.W, a.M,
                           (const uint16_t*)a.B, (const uint16_t*)a.A, (const uint16_t*)a.bias, (uint16_t*)a.Y,
                           (int)a.L, (int)a.R, (int)a.C, (int)a.r, a.scale, (int)a.two_four);
    };
    if (a.C % BK != 0) run(fwd_few_kernel<FT, RK, true, MB, NB>);
    else run(fwd_few_kernel<FT, RK, false, MB, NB>);
    return hipGetLastError();
}

template <int RK>
hipError_t launch_rk(const LayerArgs& a, hipStream_t st) {
    // 16 features per workgroup while that leaves at most one per CU, with
    // the smallest token block that takes all tokens
    const int64_t g16 = (a.R + 15) / 16, cus = device_cus();
    if (a.L <= 16 && g16 <= cus) return launch<16, RK, 1>(a, st);
    if (a.L <= 32 && g16 <= cus) return launch<16, RK, 2>(a, st);
    if (g16 * ((a.L + 63) / 64) <= cus) return launch<16, RK, 4>(a, st);
    // two 32-feature blocks per wave once one block each is more than a
    // workgroup per CU: X and A are read half as often (14336 x 4096, rank 16,
    // 32 tokens: 40.7 us against 47.1; 8192 x 4096, where it leaves half of the
    // CUs idle, 33.1 against 22.6); above rank 32 the registers do not hold it
    if constexpr (RK <= 2)
        if (a.L <= 32 && g16 > 2 * cus) return launch<32, RK, 1, 2>(a, st);
    return a.L <= 32 ? launch<32, RK, 1>(a, st) : launch<32, RK, 2>(a, st);
}

}  // namespace

hipError_t launch_fwd_few_bf16(const LayerArgs& a, hipStream_t st) {
    switch ((a.r + 15) / 16) {
        case 1: return launch_rk<1>(a, st);
        case 2: return launch_rk<2>(a, st);
        case 3: return launch_rk<3>(a, st);
        case 4: return launch_rk<4>(a, st);
        case 5:
        case 6: return launch_rk<6>(a, st);
        case 7:
        case 8: return launch_rk<8>(a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lors
