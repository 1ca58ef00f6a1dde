// fp32 kernels of the sparsity-preserved LoRA linear (debug/reference dtype).
//
// Every product runs on the fp32 MFMA (32x32x2, fp32 operands and
// accumulation, no reduced-precision mode).  A workgroup owns one 32 x 32
// output tile and its 8 waves share the contraction in blocks of 32, so that a
// 256 x 256 layer at 128 tokens still has 32 to 64 workgroups of short K-loops;
// operands go from global memory straight into the MFMA layout (lane l: row or
// column l % 32, k 8j + 4(l/32) + 0..3 of a block, four k of one lane forming
// one 16-byte load where k is contiguous), and the waves' partial tiles are
// added through LDS in wave order.  W' is rebuilt block by block in registers:
// the rank-r product of a 32 (k) x 32 (n) block comes out of the MFMA in
// exactly that layout.  These layers are bound by latency: 256 x 256, 128
// tokens, rank 8 takes 6.6 / 6.3 / 5.7 us (forward, dX, weight gradient), against
// 72 / 76 / 35 for 64 x 64 tiles whose threads formed every W' element's
// rank-r sum and the products on the vector units; 4096 x 4096, 2048 tokens,
// rank 16, where the operands come from L2: 1.36 ms forward (50 TFLOP/s)
// against 6.28, 2.94 ms backward against 8.06.
#include "device_common.hpp"
#include "kernels.hpp"

#include <type_traits>

namespace lors {
namespace {

constexpr int T = 32;   // tile edge and k block
constexpr int NW = 8;   // waves
constexpr int NT = 64 * NW;

__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
}
__device__ __forceinline__ f32x4 load4(const float* p, bool in) {
    return in ? *(const f32x4*)p : f32x4{0.f, 0.f, 0.f, 0.f};
}
// keep bits of the four columns of nibble q of a packed mask word
__device__ __forceinline__ uint32_t keep_nibble(uint32_t word, int q, bool two_four) {
    return two_four ? keep4<true>(word, 4 * q) : keep4<false>(word, 4 * q);
}
// The waves' partial tiles, summed in wave order: element v of lane is row
// 8(v/4) + 4(lane/32) + v%4, column lane % 32.
__device__ __forceinline__ void put_partial(float* red, int wave, int lane, const f32x16& acc) {
#pragma unroll
    for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[v];
}
// four columns 4c4 .. +3 of row `row`
__device__ __forceinline__ f32x4 sum_partials(const float* red, int row, int c4) {
    const int v = 4 * (row >> 3) + (row & 3), h = (row >> 2) & 1;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) s += *(const f32x4*)(red + (w * 16 + v) * 64 + 32 * h + 4 * c4);
    return s;
}

// Y[L x R] = X . W'^T (+bias), K = C.  RP: rank pairs (2 RP >= r).
template <int RP>
__global__ __launch_bounds__(NT) void fwd_f32(const float* __restrict__ X, const float* __restrict__ W,
                                              const uint32_t* __restrict__ Mp, const float* __restrict__ Bm,
                                              const float* __restrict__ Am, const float* __restrict__ bias,
                                              float* __restrict__ Y, int64_t L, int R, int C, int r, float s,
                                              int two_four, int x0, int y0) {
    __shared__ __attribute__((aligned(16))) float red[NW * 16 * 64];
    constexpr int TC = RP < 16 ? RP : 16;  // rank pairs whose operands are fetched at a time
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l = lane & 31, h = lane >> 5;
    const int64_t m0 = (int64_t)(y0 + blockIdx.y) * T;
    const int n0 = (x0 + blockIdx.x) * T, wpr = (C + 31) >> 5;
    // rows past L and R repeat the last one (their outputs are not stored)
    const int n = n0 + l < R ? n0 + l : R - 1;
    const int64_t m = m0 + l < L ? m0 + l : L - 1;
    const float* wrow = W + (int64_t)n * C;
    const float* xrow = X + m * C;
    float b[RP];
#pragma unroll
    for (int t = 0; t < RP; ++t) b[t] = 2 * t + h < r ? Bm[(int64_t)n * r + 2 * t + h] : 0.f;
    f32x16 acc = zero16();
    for (int blk = wave; blk < wpr; blk += NW) {
        const int k0 = T * blk;
        f32x4 w[4], x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + 8 * j + 4 * h;
            w[j] = load4(wrow + k, k < C);
            x[j] = load4(xrow + k, k < C);
        }
        const uint32_t word = Mp[(int64_t)n * wpr + blk];
        f32x16 ba = zero16();
#pragma unroll
        for (int t0 = 0; t0 < RP; t0 += TC) {
            float a[TC];
#pragma unroll
            for (int t = 0; t < TC; ++t) {
                const int j = 2 * (t0 + t) + h;
                a[t] = j < r && k0 + l < C ? Am[(int64_t)j * C + k0 + l] : 0.f;
            }
#pragma unroll
            for (int t = 0; t < TC; ++t) ba = mfma2(a[t], b[t0 + t], ba);
            if (RP > TC) __builtin_amdgcn_sched_barrier(0);  // one chunk's loads in flight
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // nothing is kept past C, where a 2:4 word's codes (0) name position 0
            const uint32_t keep = k0 + 8 * j + 4 * h < C ? keep_nibble(word, 2 * j + h, two_four) : 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = mfma2(x[j][e], (keep >> e) & 1u ? fmaf(s, ba[4 * j + e], w[j][e]) : 0.f, acc);
        }
    }
    put_partial(red, wave, lane, acc);
    __syncthreads();
    if (tid < T * T / 4) {
        const int row = tid >> 3, gn = n0 + 4 * (tid & 7);
        if (m0 + row < L && gn < R) {
            f32x4 y = sum_partials(red, row, tid & 7);
            if (bias) y += *(const f32x4*)(bias + gn);
            *(f32x4*)(Y + (m0 + row) * R + gn) = y;
        }
    }
}

// dX[L x C] = dY . W', K = R.
template <int RP>
__global__ __launch_bounds__(NT) void dx_f32(const float* __restrict__ dY, const float* __restrict__ W,
                                             const uint32_t* __restrict__ Mp, const float* __restrict__ Bm,
                                             const float* __restrict__ Am, float* __restrict__ dX, int64_t L, int R,
                                             int C, int r, float s, int two_four, int x0, int y0) {
    __shared__ __attribute__((aligned(16))) float red[NW * 16 * 64];
    constexpr int TC = RP < 16 ? RP : 16;  // rank pairs whose operands are fetched at a time
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l = lane & 31, h = lane >> 5;
    const int64_t m0 = (int64_t)(y0 + blockIdx.y) * T;
    const int n0 = (x0 + blockIdx.x) * T, wpr = (C + 31) >> 5, jw = n0 >> 5;
    const int n = n0 + l < C ? n0 + l : C - 1;
    const int64_t m = m0 + l < L ? m0 + l : L - 1;
    const float* drow = dY + m * R;
    float a[RP];
#pragma unroll
    for (int t = 0; t < RP; ++t) a[t] = 2 * t + h < r ? Am[(int64_t)(2 * t + h) * C + n] : 0.f;
    f32x16 acc = zero16();
    const int nblk = (R + T - 1) / T;
    for (int blk = wave; blk < nblk; blk += NW) {
        const int k0 = T * blk;
        f32x4 d[4];
        float w[16];
        uint32_t word[16];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[j] = load4(drow + k0 + 8 * j + 4 * h, k0 + 8 * j + 4 * h < R);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + 8 * j + 4 * h + e;
                w[4 * j + e] = k < R ? W[(int64_t)k * C + n] : 0.f;
                word[4 * j + e] = k < R ? Mp[(int64_t)k * wpr + jw] : 0u;
            }
        }
        f32x16 ba = zero16();
#pragma unroll
        for (int t0 = 0; t0 < RP; t0 += TC) {
            float b[TC];
#pragma unroll
            for (int t = 0; t < TC; ++t) {
                const int j = 2 * (t0 + t) + h;
                b[t] = j < r && k0 + l < R ? Bm[(int64_t)(k0 + l) * r + j] : 0.f;
            }
#pragma unroll
            for (int t = 0; t < TC; ++t) ba = mfma2(b[t], a[t0 + t], ba);
            if (RP > TC) __builtin_amdgcn_sched_barrier(0);  // one chunk's loads in flight
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            // (nothing is kept past R, whose 2:4 words read as 0)
            const uint32_t keep = k0 + 8 * (v >> 2) + 4 * h < R ? keep_nibble(word[v], l >> 2, two_four) >> (l & 3) : 0u;
            acc = mfma2(d[v >> 2][v & 3], keep & 1u ? fmaf(s, ba[v], w[v]) : 0.f, acc);
        }
    }
    put_partial(red, wave, lane, acc);
    __syncthreads();
    if (tid < T * T / 4) {
        const int row = tid >> 3, gn = n0 + 4 * (tid & 7);
        if (m0 + row < L && gn < C) *(f32x4*)(dX + (m0 + row) * C + gn) = sum_partials(red, row, tid & 7);
    }
}

// G tile = select(M, dY^T X, 0) over K = L into LDS, then fp32 atomics of the
// tile's contributions to dB = s G A^T and dA = s B^T G, one 32-rank block of
// either per wave.
__global__ __launch_bounds__(NT) void g_f32(const float* __restrict__ dY, const float* __restrict__ X,
                                            const uint32_t* __restrict__ Mp, const float* __restrict__ Bm,
                                            const float* __restrict__ Am, float* __restrict__ dB,
                                            float* __restrict__ dA, int64_t L, int R, int C, int r, float s,
                                            int two_four, int x0, int y0) {
    __shared__ __attribute__((aligned(16))) float red[NW * 16 * 64];
    __shared__ float G[T][T + 1];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l = lane & 31, h = lane >> 5;
    const int i0 = (y0 + blockIdx.y) * T, j0 = (x0 + blockIdx.x) * T, wpr = (C + 31) >> 5;
    const bool in_i = i0 + l < R, in_j = j0 + l < C;
    f32x16 acc = zero16();
    for (int64_t t0 = (int64_t)T * wave; t0 < L; t0 += T * NW) {
        float d[16], x[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t t = t0 + 8 * (v >> 2) + 4 * h + (v & 3);
            d[v] = in_i && t < L ? dY[t * R + i0 + l] : 0.f;
            x[v] = in_j && t < L ? X[t * C + j0 + l] : 0.f;
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc = mfma2(d[v], x[v], acc);
    }
    put_partial(red, wave, lane, acc);
    __syncthreads();
    if (tid < T * T / 4) {
        const int row = tid >> 3, c4 = tid & 7;
        uint32_t keep = 0;
        if (i0 + row < R && j0 + 4 * c4 < C)
            keep = keep_nibble(Mp[(int64_t)(i0 + row) * wpr + (j0 >> 5)], c4, two_four);
        const f32x4 g = sum_partials(red, row, c4);
#pragma unroll
        for (int e = 0; e < 4; ++e) G[row][4 * c4 + e] = (keep >> e) & 1u ? g[e] : 0.f;
    }
    __syncthreads();
    const int nrb = (r + T - 1) / T;
    for (int task = wave; task < 2 * nrb; task += NW) {
        const int jr0 = T * (task >> 1);
        f32x16 p = zero16();
        if ((task & 1) == 0) {  // dB: rows i, columns = ranks, k = columns j of the tile
            const bool in = jr0 + l < r;
            const float* arow = Am + (int64_t)(jr0 + l) * C + j0;
            f32x4 a[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] = load4(arow + 8 * j + 4 * h, in && j0 + 8 * j + 4 * h < C);
#pragma unroll
            for (int v = 0; v < 16; ++v) p = mfma2(G[l][8 * (v >> 2) + 4 * h + (v & 3)], a[v >> 2][v & 3], p);
            if (in)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = i0 + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (i < R) atomicAdd(dB + (int64_t)i * r + jr0 + l, s * p[v]);
                }
        } else {  // dA: rows = ranks, columns j, k = rows i of the tile
            float b[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = i0 + 8 * (v >> 2) + 4 * h + (v & 3);
                b[v] = i < R && jr0 + l < r ? Bm[(int64_t)i * r + jr0 + l] : 0.f;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) p = mfma2(b[v], G[8 * (v >> 2) + 4 * h + (v & 3)][l], p);
            if (in_j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int jr = jr0 + 8 * (v >> 2) + 4 * h + (v & 3);
                    if (jr < r) atomicAdd(dA + (int64_t)jr * C + j0 + l, s * p[v]);
                }
        }
    }
}

// runs f with the rank-pair count of the smallest bucket that holds r
template <class F>
void with_rank_pairs(int64_t r, F f) {
    if (r <= 8) f(std::integral_constant<int, 4>{});
    else if (r <= 16) f(std::integral_constant<int, 8>{});
    else if (r <= 32) f(std::integral_constant<int, 16>{});
    else if (r <= 64) f(std::integral_constant<int, 32>{});
    else f(std::integral_constant<int, 64>{});
}

// runs f(grid, x0, y0) over the tiles of a cols x rows output, in several
// launches where they exceed a grid's extents (2^32 threads by 65535 blocks)
template <class F>
hipError_t over_tiles(int64_t cols, int64_t rows, F f) {
    const int64_t nx = (cols + T - 1) / T, ny = (rows + T - 1) / T, mx = 1 << 22, my = 65535;
    for (int64_t y0 = 0; y0 < ny; y0 += my)
        for (int64_t x0 = 0; x0 < nx; x0 += mx) {
            const int64_t gx = nx - x0 < mx ? nx - x0 : mx, gy = ny - y0 < my ? ny - y0 : my;
            f(dim3((unsigned)gx, (unsigned)gy), (int)x0, (int)y0);
        }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_f32(const LayerArgs& a, hipStream_t st) {
    if (a.L == 0) return hipSuccess;
    return over_tiles(a.R, a.L, [&](dim3 grid, int x0, int y0) {
        with_rank_pairs(a.r, [&](auto rp) {
            hipLaunchKernelGGL(fwd_f32<decltype(rp)::value>, grid, dim3(NT), 0, st, (const float*)a.X,
                               (const float*)a.W, a.M, (const float*)a.B, (const float*)a.A, (const float*)a.bias,
                               (float*)a.Y, a.L, (int)a.R, (int)a.C, (int)a.r, a.scale, (int)a.two_four, x0, y0);
        });
    });
}

hipError_t launch_dx_f32(const LayerArgs& a, hipStream_t st) {
    if (a.L == 0 || a.dX == nullptr) return hipSuccess;
    return over_tiles(a.C, a.L, [&](dim3 grid, int x0, int y0) {
        with_rank_pairs(a.r, [&](auto rp) {
            hipLaunchKernelGGL(dx_f32<decltype(rp)::value>, grid, dim3(NT), 0, st, (const float*)a.dY,
                               (const float*)a.W, a.M, (const float*)a.B, (const float*)a.A, (float*)a.dX, a.L,
                               (int)a.R, (int)a.C, (int)a.r, a.scale, (int)a.two_four, x0, y0);
        });
    });
}

hipError_t launch_g_f32(const LayerArgs& a, hipStream_t st) {
    if (a.L == 0) return hipSuccess;
    return over_tiles(a.C, a.R, [&](dim3 grid, int x0, int y0) {
        hipLaunchKernelGGL(g_f32, grid, dim3(NT), 0, st, (const float*)a.dY, (const float*)a.X, a.M,
                           (const float*)a.B, (const float*)a.A, a.dB, a.dA, a.L, (int)a.R, (int)a.C, (int)a.r,
                           a.scale, (int)a.two_four, x0, y0);
    });
}

}  // namespace lors
