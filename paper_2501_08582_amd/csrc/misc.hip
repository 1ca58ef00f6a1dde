// Mask packing (dense 0/1 or weight != 0 -> 1 bit per element), unpacking,
// output clearing, the bias gradient, and the split of a short last wave of
// tiles over K (the rule and the reduction of the pieces' partial sums).
//
// Packed layouts (the paper keeps the mask as a dense boolean; the packing is
// this library's own):
//   bitmap: element (i, j) is bit j % 32 of word i*ceil(C/32) + j/32
//   2:4:    group g of row i keeps p0 < p1; nibble p0 | p1 << 2 at bits
//           4*(g % 8) of word i*ceil(C/32) + g/8
#include <atomic>

#include "device_common.hpp"
#include "kernels.hpp"

namespace lors {
namespace {

constexpr int NT = 256;
constexpr unsigned long long kNoBad = ~0ull;

// Sources of "kept" flags: a dense uint8 mask or a weight matrix (kept = value
// != 0, with -0 counting as zero).  E elements are one 16-byte vector.
struct DenseSrc {
    static constexpr int E = 16;
    const uint8_t* p;
    __device__ bool kept(int64_t e) const { return p[e] != 0; }
    __device__ uint32_t flags(u32x4 v) const {
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) bits |= (((v[e >> 2] >> (8 * (e & 3))) & 0xFFu) != 0u ? 1u : 0u) << e;
        return bits;
    }
};
struct Bf16WeightSrc {
    static constexpr int E = 8;
    const uint16_t* p;
    __device__ bool kept(int64_t e) const { return (p[e] & 0x7FFFu) != 0u; }
    __device__ uint32_t flags(u32x4 v) const {
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) bits |= ((v[e >> 1] & (e & 1 ? 0x7FFF0000u : 0x7FFFu)) != 0u ? 1u : 0u) << e;
        return bits;
    }
};
struct F32WeightSrc {
    static constexpr int E = 4;
    const float* p;
    __device__ bool kept(int64_t e) const { return p[e] != 0.f; }
    __device__ uint32_t flags(u32x4 v) const {
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) bits |= (__uint_as_float(v[e]) != 0.f ? 1u : 0u) << e;
        return bits;
    }
};

// The packed word of 32 keep flags f, of which the first `groups` groups of 4
// exist; for 2:4, an invalid group (number g0 + n) is reported to first_bad.
template <bool TWO_FOUR>
__device__ __forceinline__ uint32_t pack_word(uint32_t f, int groups, int64_t g0,
                                              unsigned long long* __restrict__ first_bad) {
    if constexpr (!TWO_FOUR) return f;
    uint32_t word = 0;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        if (n >= groups) break;
        const uint32_t nib = (f >> (4 * n)) & 0xFu;
        if (__popc(nib) != 2) {
            atomicMin(first_bad, (unsigned long long)(g0 + n));
            continue;
        }
        const uint32_t p0 = __ffs(nib) - 1;
        const uint32_t p1 = 31 - __clz(nib);
        word |= (p0 | (p1 << 2)) << (4 * n);
    }
    return word;
}

// OR of v over the P consecutive lanes (P = 2, 4 or 8) of an aligned group.
template <int P>
__device__ __forceinline__ uint32_t or_lanes(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);                          // lane ^ 1
    if constexpr (P >= 4) v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // lane ^ 2
    if constexpr (P >= 8) v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);  // the other quad
    return v;
}

// Rows of whole words (C % 32 == 0): the matrix is one run of words.  Bound by
// the read of the source, so every load is a coalesced 16-byte vector: a wave
// reads 64 P vectors (P = 32/E lanes to a word), P of them per lane and all
// requested before the first is used; the lanes of a word OR their flags, and
// lane p of a word keeps the one of load p.  14336 x 4096 bf16: 128 us with one
// thread per word and a load per element, 24.3 us so (5.1 TB/s).
template <class Src, bool TWO_FOUR>
__global__ __launch_bounds__(NT) void pack_rows_kernel(Src src, int64_t words, uint32_t* __restrict__ out,
                                                       unsigned long long* __restrict__ first_bad) {
    constexpr int E = Src::E, P = 32 / E;
    const int lane = threadIdx.x & 63, part = lane % P;
    const int64_t w0 = ((int64_t)blockIdx.x * (NT / 64) + (threadIdx.x >> 6)) * 64;  // 64 words per wave
    u32x4 v[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int64_t w = w0 + (64 / P) * i + lane / P;
        v[i] = w < words ? *((const u32x4*)src.p + w * P + part) : zero_u32x4();
    }
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const uint32_t word = or_lanes<P>(src.flags(v[i]) << (E * part));
        if (part == i) mine = word;
    }
    const int64_t w = w0 + (64 / P) * part + lane / P;
    if (w < words) out[w] = pack_word<TWO_FOUR>(mine, 8, 8 * w, first_bad);
}

// Any C: one thread per word, in 16-byte vectors where the word is whole and
// its row starts on one.  Byte masks of 4096 x 14352 (every row does) and 4096
// x 14332 (one in four): 119 us by elements alone, 16.6 and 86 us so.
template <class Src, bool TWO_FOUR>
__global__ __launch_bounds__(NT) void pack_words_kernel(Src src, int64_t R, int C, int wpr, uint32_t* __restrict__ out,
                                                        unsigned long long* __restrict__ first_bad) {
    const int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (t >= R * wpr) return;
    const int64_t i = t / wpr;
    const int c0 = (int)(t - i * wpr) * 32;
    constexpr int E = Src::E;
    const auto* at = src.p + i * C + c0;
    uint32_t f = 0;
    if (c0 + 32 <= C && ((uintptr_t)at & 15) == 0) {
#pragma unroll
        for (int q = 0; q < 32 / E; ++q) f |= src.flags(((const u32x4*)at)[q]) << (E * q);
    } else {
        for (int e = 0; e < 32 && c0 + e < C; ++e) f |= (src.kept(i * C + c0 + e) ? 1u : 0u) << e;
    }
    out[t] = pack_word<TWO_FOUR>(f, C / 4 - c0 / 4, i * (C / 4) + c0 / 4, first_bad);
}

__global__ void set_u64_kernel(unsigned long long* p, unsigned long long v) { *p = v; }

template <bool TWO_FOUR>
__global__ __launch_bounds__(NT) void unpack_kernel(const uint32_t* __restrict__ in, int64_t R, int C,
                                                    int wpr, uint8_t* __restrict__ dense) {
    const int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (t >= R * wpr) return;
    const int64_t i = t / wpr;
    const int w = (int)(t - i * wpr);
    const uint32_t word = in[t];
    uint8_t* row = dense + i * C;
    const int c0 = w * 32;
    for (int e = 0; e < 32 && c0 + e < C; ++e) row[c0 + e] = (uint8_t)keep1<TWO_FOUR>(word, (uint32_t)e);
}

// Keep bits of a word of eight 2:4 codes p0 | p1 << 2: in every nibble, bit k
// is set where both bits of p0, or both of p1, equal those of k.
__device__ __forceinline__ uint32_t expand_codes(uint32_t w) {
    auto spread = [](uint32_t v) {  // bit 0 of each nibble to its four bits
        v &= 0x11111111u;
        return (v << 4) - v;
    };
    const uint32_t p0 = (spread(w) ^ 0x55555555u) & (spread(w >> 1) ^ 0x33333333u);
    const uint32_t p1 = (spread(w >> 2) ^ 0x55555555u) & (spread(w >> 3) ^ 0x33333333u);
    return p0 | p1;
}

// 32 x 32 bit transpose over 32 lanes: lane i gives row i, lane c gets column
// c.  Step j exchanges, between lanes l and l ^ j, the bits whose index
// differs from the lane's in bit j.
__device__ __forceinline__ uint32_t transpose32(uint32_t x, int lane) {
    auto step = [&](uint32_t y, int j, uint32_t m) {  // y: x of lane ^ j; m: bits b with (b & j) == 0
        const uint32_t keep = lane & j ? ~m : m;
        const uint32_t moved = __builtin_amdgcn_alignbit(y, y, lane & j ? j : 32 - j);
        x = (x & keep) | (moved & ~keep);
    };
    step((uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (16 << 10) | 31), 16, 0x0000FFFFu);
    step((uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (8 << 10) | 31), 8, 0x00FF00FFu);
    step((uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (4 << 10) | 31), 4, 0x0F0F0F0Fu);
    step((uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true), 2, 0x33333333u);
    step((uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true), 1, 0x55555555u);
    return x;
}

// Transposed bitmap (K-step-major, see mt_index).  A wave takes 64 rows (lane =
// row, one aligned pair of output words) of four words; its workgroup's four
// waves share the rows' 64-byte segments.  After the bit transpose of its half,
// lane c holds the word of column c for rows 0 .. 31 (lane 32 + c: 32 .. 63),
// so a word's store is one 256-byte run.  The 32-step ballot form this
// replaces was bound by its vector instructions: 16 us at 13824 x 5120,
// 8.6 so (2.1 TB/s).
constexpr int TRQ = 4;  // words per wave
template <bool TWO_FOUR>
__global__ __launch_bounds__(NT) void transpose_kernel(const uint32_t* __restrict__ in, int64_t R, int C, int wpr,
                                                       int wprT, int col_groups, uint32_t* __restrict__ out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t rg = blockIdx.x / col_groups;
    const int jw0 = ((int)(blockIdx.x - rg * col_groups) * (NT / 64) + wave) * TRQ;
    const int64_t row = 64 * rg + lane;
    uint32_t w[TRQ];
#pragma unroll
    for (int q = 0; q < TRQ; ++q) w[q] = row < R && jw0 + q < wpr ? in[row * wpr + jw0 + q] : 0u;
    const int iw = (int)(2 * rg) + (lane >> 5);
#pragma unroll
    for (int q = 0; q < TRQ; ++q) {
        if constexpr (TWO_FOUR) {
            // groups past C/4 and rows past R hold no codes: clear their expansion
            const int cols = row < R ? C - 32 * (jw0 + q) : 0;
            w[q] = expand_codes(w[q]) & (cols >= 32 ? ~0u : cols > 0 ? (1u << cols) - 1u : 0u);
        }
        const uint32_t t = transpose32(w[q], lane);
        const int64_t col = (int64_t)32 * (jw0 + q) + (lane & 31);
        if (col < C && iw < wprT) out[mt_index(col, iw, C, wprT)] = t;
    }
}

__global__ __launch_bounds__(NT) void zero_kernel(float* __restrict__ p, int64_t n) {
    for (int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x; t < n; t += (int64_t)gridDim.x * NT) p[t] = 0.f;
}

__global__ __launch_bounds__(NT) void zero2_kernel(float* __restrict__ a, int64_t na, float* __restrict__ b,
                                                   int64_t nb) {
    const int64_t stride = (int64_t)gridDim.x * NT;
    for (int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x; t < na + nb; t += stride) {
        if (t < na) a[t] = 0.f;
        else b[t - na] = 0.f;
    }
}

// The two arrays as runs of 4-element vectors (their last one may be short).
__global__ __launch_bounds__(NT) void round_bf16_kernel(const float* __restrict__ a, int64_t na,
                                                        uint16_t* __restrict__ ao, const float* __restrict__ b,
                                                        int64_t nb, uint16_t* __restrict__ bo) {
    const int64_t va = (na + 3) / 4, vb = (nb + 3) / 4, stride = (int64_t)gridDim.x * NT;
    for (int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x; t < va + vb; t += stride) {
        const bool first = t < va;
        const int64_t e = 4 * (first ? t : t - va), left = (first ? na : nb) - e;
        const float* p = (first ? a : b) + e;
        uint16_t* o = (first ? ao : bo) + e;
        if (left >= 4) {
            const f32x4 v = *(const f32x4*)p;
            *(u32x2*)o = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        } else {
            for (int i = 0; i < left; ++i) o[i] = bf16_bits(p[i]);
        }
    }
}

// out[R x rp] = B[R x r] with columns r .. rp-1 zero (bf16 bit patterns).
__global__ __launch_bounds__(NT) void pad_cols_kernel(const uint16_t* __restrict__ B, int64_t R, int r, int rp,
                                                      uint16_t* __restrict__ out) {
    const int64_t n = R * rp, stride = (int64_t)gridDim.x * NT;
    for (int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x; t < n; t += stride) {
        const int64_t i = t / rp;
        const int j = (int)(t - i * rp);
        out[t] = j < r ? B[i * r + j] : (uint16_t)0;
    }
}

// dbias[R] = column sums of dY[L x R].  One read of dY: a lane owns one
// 16-byte vector of columns (R is a multiple of its V elements), the four
// waves take every fourth row of the workgroup's slice, eight loads ahead, and
// add up through LDS; the slices are combined with fp32 atomics (dbias zeroed
// first).  2048 x 4096 bf16: 60 us with one column per thread, 4.8 us so.
template <bool BF16>
__global__ __launch_bounds__(NT) void dbias_kernel(const void* __restrict__ dY, int64_t L, int R,
                                                   int64_t rows_per_block, float* __restrict__ dbias) {
    constexpr int V = BF16 ? 8 : 4;
    __shared__ float part[NT / 64][64 * V];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t col = ((int64_t)blockIdx.x * 64 + lane) * V;
    const int64_t l0 = (int64_t)blockIdx.y * rows_per_block;
    const int64_t l1 = l0 + rows_per_block < L ? l0 + rows_per_block : L;
    float acc[V] = {};
    if (col < R) {
        const uint8_t* p = (const uint8_t*)dY + col * (16 / V);
        const int64_t pitch = (int64_t)R * (16 / V);
#pragma unroll 8
        for (int64_t l = l0 + wave; l < l1; l += NT / 64) {
            const u32x4 v = *(const u32x4*)(p + l * pitch);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                if constexpr (BF16) acc[e] += __uint_as_float(e & 1 ? v[e >> 1] & 0xFFFF0000u : v[e >> 1] << 16);
                else acc[e] += __uint_as_float(v[e]);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) part[wave][64 * e + lane] = acc[e];
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * V; i += NT) {
        const int64_t c = (int64_t)blockIdx.x * 64 * V + i;
        const int at = 64 * (i % V) + i / V;
        if (c < R) atomicAdd(dbias + c, (part[0][at] + part[1][at]) + (part[2][at] + part[3][at]));
    }
}

template <class Src>
hipError_t launch_pack(Src src, int64_t R, int64_t C, bool two_four, uint32_t* packed,
                       int64_t* first_bad, hipStream_t st) {
    const int wpr = (int)((C + 31) / 32);
    const int64_t n = R * wpr;
    auto* fb = (unsigned long long*)first_bad;
    // -1 (all bits set): no invalid group
    if (fb) hipLaunchKernelGGL(set_u64_kernel, dim3(1), dim3(1), 0, st, fb, kNoBad);
    if (n > 0 && C % 32 == 0) {
        const unsigned blocks = (unsigned)((n + NT - 1) / NT);
        if (two_four)
            hipLaunchKernelGGL((pack_rows_kernel<Src, true>), dim3(blocks), dim3(NT), 0, st, src, n, packed, fb);
        else
            hipLaunchKernelGGL((pack_rows_kernel<Src, false>), dim3(blocks), dim3(NT), 0, st, src, n, packed, fb);
    } else if (n > 0) {
        const unsigned blocks = (unsigned)((n + NT - 1) / NT);
        if (two_four)
            hipLaunchKernelGGL((pack_words_kernel<Src, true>), dim3(blocks), dim3(NT), 0, st, src, R, (int)C, wpr,
                               packed, fb);
        else
            hipLaunchKernelGGL((pack_words_kernel<Src, false>), dim3(blocks), dim3(NT), 0, st, src, R, (int)C, wpr,
                               packed, fb);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_mask_pack(const uint8_t* dense, int64_t R, int64_t C, bool two_four,
                            uint32_t* packed, int64_t* first_bad, hipStream_t st) {
    return launch_pack(DenseSrc{dense}, R, C, two_four, packed, first_bad, st);
}

hipError_t launch_mask_from_weight(const void* W, bool w_is_bf16, int64_t R, int64_t C, bool two_four,
                                   uint32_t* packed, int64_t* first_bad, hipStream_t st) {
    if (w_is_bf16) return launch_pack(Bf16WeightSrc{(const uint16_t*)W}, R, C, two_four, packed, first_bad, st);
    return launch_pack(F32WeightSrc{(const float*)W}, R, C, two_four, packed, first_bad, st);
}

hipError_t launch_mask_unpack(const uint32_t* packed, int64_t R, int64_t C, bool two_four, uint8_t* dense,
                              hipStream_t st) {
    const int wpr = (int)((C + 31) / 32);
    const int64_t n = R * wpr;
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((n + NT - 1) / NT);
    if (two_four)
        hipLaunchKernelGGL(unpack_kernel<true>, dim3(blocks), dim3(NT), 0, st, packed, R, (int)C, wpr, dense);
    else
        hipLaunchKernelGGL(unpack_kernel<false>, dim3(blocks), dim3(NT), 0, st, packed, R, (int)C, wpr, dense);
    return hipGetLastError();
}

hipError_t launch_mask_transpose(const uint32_t* packed, int64_t R, int64_t C, bool two_four, uint32_t* mt,
                                 hipStream_t st) {
    const int wpr = (int)((C + 31) / 32);
    const int wprT = (int)((R + 31) / 32);
    const int col_groups = (wpr + TRQ * (NT / 64) - 1) / (TRQ * (NT / 64));
    const int64_t blocks = (int64_t)((wprT + 1) / 2) * col_groups;
    if (blocks == 0) return hipSuccess;
    if (two_four)
        hipLaunchKernelGGL(transpose_kernel<true>, dim3((unsigned)blocks), dim3(NT), 0, st, packed, R, (int)C, wpr,
                           wprT, col_groups, mt);
    else
        hipLaunchKernelGGL(transpose_kernel<false>, dim3((unsigned)blocks), dim3(NT), 0, st, packed, R, (int)C, wpr,
                           wprT, col_groups, mt);
    return hipGetLastError();
}

hipError_t launch_zero_f32(float* p, int64_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const int64_t want = (n + NT - 1) / NT;
    const unsigned blocks = (unsigned)(want < 4096 ? want : 4096);
    hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(NT), 0, st, p, n);
    return hipGetLastError();
}

// Workgroup (q, rb): rows 4*rb .. 4*rb+3 of split tile q (logical tile
// n_full + q); thread t covers 4 columns of one of those rows.
__global__ __launch_bounds__(NT) void split_reduce_kernel(const float* __restrict__ part, int n_full, int split,
                                                          int tiles_m, int tiles_n, int group_m, int64_t rows,
                                                          int cols, const uint16_t* __restrict__ bias,
                                                          uint16_t* __restrict__ out) {
    const int q = blockIdx.x >> 6, rb = blockIdx.x & 63;
    int tm, tn;
    group_coords(n_full + q, tiles_m, tiles_n, group_m, tm, tn);
    const int tr = 4 * rb + (threadIdx.x >> 6), tc = 4 * (threadIdx.x & 63);
    const int64_t gm = (int64_t)tm * 256 + tr;
    const int gn = tn * 256 + tc;
    if (gm >= rows || gn >= cols) return;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < split; ++p)
        sum += *(const f32x4*)(part + ((int64_t)q * split + p) * 65536 + tr * 256 + tc);
    uint16_t* o = out + gm * cols + gn;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (gn + e < cols) {
            const float b = bias != nullptr ? bf16_bits_to_f32(bias[gn + e]) : 0.f;
            o[e] = bf16_bits(sum[e] + b);
        }
    }
}

hipError_t launch_split_reduce_bf16(const float* part, int n_full, int split, int tiles_m, int tiles_n,
                                    int group_m, int64_t rows, int cols, const void* bias, void* out,
                                    hipStream_t st) {
    const int tail = tiles_m * tiles_n - n_full;
    if (tail <= 0 || split < 2) return hipSuccess;
    hipLaunchKernelGGL(split_reduce_kernel, dim3(tail * 64), dim3(NT), 0, st, part, n_full, split, tiles_m, tiles_n,
                       group_m, rows, cols, (const uint16_t*)bias, (uint16_t*)out);
    return hipGetLastError();
}

// compute units of the current device, read once per device (calls from
// several host threads may both read it; they store the same value)
int device_cus() {
    static std::atomic<int> cus_of[64];
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64) {
        int n = cus_of[dev].load(std::memory_order_relaxed);
        if (n == 0 && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cus_of[dev].store(n, std::memory_order_relaxed);
        if (n > 0) cus = n;
    }
    return cus;
}

bool fwd_few_tokens(int64_t L, int64_t R, int64_t C) {
    return C <= (1 << 24) && (L <= 32 || ((R + 31) / 32) * ((L + 63) / 64) <= device_cus());
}

TailSplit tail_split(int64_t tiles, int64_t nk, int64_t max_part_bytes) {
    const int cus = device_cus();
    TailSplit t{(int)tiles, 1, (int)tiles};
    const int64_t tail = tiles % cus;
    if (tail == 0 || 2 * tail > cus) return t;
    int64_t s = cus / tail;
    if (s > 8) s = 8;
    if (s > nk / 4) s = nk / 4;
    if (max_part_bytes != kNoPartials) {
        const int64_t fit = max_part_bytes / (tail * kPieceBytes);
        if (s > fit) s = fit;
    }
    if (s < 2) return t;
    t.n_full = (int)(tiles - tail);
    t.split = (int)s;
    t.grid = (int)(t.n_full + tail * s);
    return t;
}

// the thin tiles of a grid that is one short wave
static ThinPlan thin_grid(int64_t L, int64_t N, int cus) {
    int best = 256;
    double least = 0;
    for (int tm = 256; tm >= 64; tm -= 64) {
        const int64_t wgs = ((L + tm - 1) / tm) * ((N + 127) / 128);
        const double cost = (double)((wgs + cus - 1) / cus) * (0.45 + 0.0042 * tm);
        if (tm == 256 || cost < least) {
            least = cost;
            best = tm;
        }
    }
    const int64_t span = thin_span(best);
    return ThinPlan{0, (int)(((L + span - 1) / span) * ((N + 255) / 256)), best};
}

static int64_t tiles256(int64_t L, int64_t N) { return ((L + 255) / 256) * ((N + 255) / 256); }

ThinPlan thin_plan(int64_t L, int64_t N) {
    const int cus = device_cus();
    const int64_t tiles = tiles256(L, N), tail = tiles % cus;
    if (tail == 0 || 2 * tail > cus) return ThinPlan{(int)tiles, 0, 0};
    if (tail == tiles) return thin_grid(L, N, cus);
    return ThinPlan{(int)(tiles - tail), (int)tail, 8 * tail <= cus ? 64 : 4 * tail <= cus ? 128 : 256};
}

int thin_only_plan(int64_t L, int64_t N, ThinPlan run[2]) {
    const int cus = device_cus();
    const int64_t tiles = tiles256(L, N);
    if (2 * tiles <= cus) {
        run[0] = thin_grid(L, N, cus);
        return 1;
    }
    const int64_t rest = (2 * tiles % cus + 1) / 2;  // tiles of the last wave of feature halves
    const bool cut = rest > 0 && 4 * rest <= cus;
    run[0] = ThinPlan{0, (int)(cut ? tiles - rest : tiles), 256};
    run[1] = ThinPlan{(int)(tiles - rest), (int)rest, 8 * rest <= cus ? 64 : 128};
    return cut ? 2 : 1;
}

hipError_t launch_zero2_f32(float* a, int64_t na, float* b, int64_t nb, hipStream_t st) {
    const int64_t n = na + nb;
    if (n == 0) return hipSuccess;
    const int64_t want = (n + NT - 1) / NT;
    const unsigned blocks = (unsigned)(want < 2048 ? want : 2048);
    hipLaunchKernelGGL(zero2_kernel, dim3(blocks), dim3(NT), 0, st, a, na, b, nb);
    return hipGetLastError();
}

hipError_t launch_round_bf16(const float* a, int64_t na, void* a_out, const float* b, int64_t nb, void* b_out,
                             hipStream_t st) {
    const int64_t n = (na + 3) / 4 + (nb + 3) / 4;
    if (n == 0) return hipSuccess;
    const int64_t want = (n + NT - 1) / NT;
    const unsigned blocks = (unsigned)(want < 2048 ? want : 2048);
    hipLaunchKernelGGL(round_bf16_kernel, dim3(blocks), dim3(NT), 0, st, a, na, (uint16_t*)a_out, b, nb,
                       (uint16_t*)b_out);
    return hipGetLastError();
}

hipError_t launch_pad_cols_bf16(const void* B, int64_t R, int64_t r, int64_t rp, void* out, hipStream_t st) {
    const int64_t n = R * rp;
    if (n == 0) return hipSuccess;
    const int64_t want = (n + NT - 1) / NT;
    const unsigned blocks = (unsigned)(want < 2048 ? want : 2048);
    hipLaunchKernelGGL(pad_cols_kernel, dim3(blocks), dim3(NT), 0, st, (const uint16_t*)B, R, (int)r, (int)rp,
                       (uint16_t*)out);
    return hipGetLastError();
}

static hipError_t launch_dbias(const LayerArgs& a, hipStream_t st, bool bf16) {
    if (a.dbias == nullptr) return hipSuccess;
    hipError_t e = launch_zero_f32(a.dbias, a.R, st);
    if (e != hipSuccess || a.L == 0) return e;
    // slices of 64 rows, longer ones where they would be more than 4096
    int64_t ychunks = (a.L + 63) / 64;
    if (ychunks > 4096) ychunks = 4096;
    const int64_t rows = (a.L + ychunks - 1) / ychunks;
    const int64_t cols = 64 * (bf16 ? 8 : 4);
    dim3 grid((unsigned)((a.R + cols - 1) / cols), (unsigned)ychunks), block(NT);
    if (bf16)
        hipLaunchKernelGGL(dbias_kernel<true>, grid, block, 0, st, a.dY, a.L, (int)a.R, rows, a.dbias);
    else
        hipLaunchKernelGGL(dbias_kernel<false>, grid, block, 0, st, a.dY, a.L, (int)a.R, rows, a.dbias);
    return hipGetLastError();
}

hipError_t launch_dbias_bf16(const LayerArgs& a, hipStream_t st) { return launch_dbias(a, st, true); }
hipError_t launch_dbias_f32(const LayerArgs& a, hipStream_t st) { return launch_dbias(a, st, false); }

}  // namespace lors
